"""16-bit tree attention of rows whose whole weight is on one key: the result is that key's V.

Query n is 32 times the key that it looks for: its score is 32 |k|^2 / sqrt(Dh), some hundreds, and every other one's below it by more
than 40, so that all other probabilities together are under 2^-40.  The largest one is then exactly one in the sum and in the product (it is
rounded to half there), whatever the size of the scores, and so is the weight of the wave and of the workgroup that hold it; a
softmax whose largest probability is off by the rounding of a scaled maximum misses V by up to 1e-5 of it."""
import pytest
import torch

from synth import random_tree
from helpers import make_weights, small_shape
from gpu_util import gpu_session

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("Dh,H,B,T,L", [
    (128, 4, 1, 64, 3900),        # two query tiles to a wave, keys split over workgroups
    (128, 52, 2, 40, 1700),
    (64, 64, 5, 65, 300),         # four waves, no split
    (128, 4, 2, 128, 900),        # short contexts
    (128, 8, 1, 12, 2500),        # one query tile, keys split over workgroups
])
def test_one_key_takes_it_all(Dh, H, B, T, L):
    parent = random_tree(T, 4, 6)
    cfg = small_shape(d=H * Dh, NL=1, H=H, Dh=Dh, F=128, V=64, K=0, T=T, dtype="bf16")
    sess = gpu_session(cfg, parent, B, L + T, make_weights(cfg), page_perm_seed=3)
    g = torch.Generator(device=DEV).manual_seed(T + Dh)
    kv = torch.randn(B, L + T, 2, H, Dh, generator=g, device=DEV).half().float()
    at = torch.randint(0, L, (B, T), generator=g, device=DEV)
    rows = torch.arange(B, device=DEV)[:, None]
    q = (32 * kv[rows, at, 0]).contiguous()
    for b in range(B):
        s = torch.matmul(q[b].permute(1, 0, 2).double(), kv[b, :, 0].permute(1, 2, 0).double().contiguous()) / Dh ** 0.5
        top = s.topk(2, -1).values
        assert float((top[..., 0] - top[..., 1]).min()) > 40
    sess.main.kv_write(B, 0, sess.kv, 0, L + T, kv)
    sess.seq_len.fill_(L)
    sess.kv.seq_len_hint = L
    out = torch.zeros(B, T, H, Dh, device=DEV)
    print("case", Dh, H, B, T, L, flush=True)
    sess.main.tree_attention(B, 0, sess.ws, q, sess.seq_len, sess.kv, out)
    torch.cuda.synchronize()
    assert sess.main.read_flags() == 0
    # to two units in the last place: matrix instructions need not round to nearest what the other keys' terms leave
    want = kv[rows, at, 1]
    worst = float(((out - want).abs() / want.abs().clamp_min(1e-7)).max())
    assert worst <= 2.0 ** -22, worst
