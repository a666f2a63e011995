"""16-bit tree attention on both sides of the lines between its kernels: up to 40 tiles of 32 keys (short contexts); up to 52 with 33 to
64 queries and half of the chip without a workgroup of eight waves (a wave per query tile); more tiles, then workgroups of four waves
and of eight; rows longer than the host's hint."""
import pytest
import torch

from synth import random_tree
from helpers import make_weights, small_shape
from gpu_util import gpu_session
from test_gpu_attn_pair import _reference

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("Dh,H,T,totals", [
    (128, 3, 32, (1280, 1281)),
    (128, 3, 33, (1280, 1281, 1664, 1665)),
    (64, 4, 128, (1280, 1281)),
    (128, 32, 64, (1281, 1537, 1664, 1665, 2048, 2049)),        # eight waves: 96 workgroups, 128 from 1537 keys on, 160 from 2049
    (128, 40, 50, (1536, 1537)),                                # 120, 160
    (64, 16, 50, (1281, 1664, 1665)),                           # 48, 64
    (64, 32, 64, (1281,)),                                      # 96
])
def test_lines_between_the_kernels(Dh, H, T, totals):
    parent = random_tree(T, 4, 6)
    most = max(totals)
    cfg = small_shape(d=H * Dh, NL=1, H=H, Dh=Dh, F=128, V=64, K=0, T=T, dtype="bf16")
    sess = gpu_session(cfg, parent, 1, most, make_weights(cfg), page_perm_seed=3)
    g = torch.Generator(device=DEV).manual_seed(T + Dh)
    kv = torch.randn(1, most, 2, H, Dh, generator=g, device=DEV).half().float()
    q = (torch.randn(1, T, H, Dh, generator=g, device=DEV) * 2).half().float()
    own = torch.zeros(T, T, dtype=torch.bool, device=DEV)
    for n in range(T):
        if n:
            own[n] = own[parent[n]]
        own[n, n] = True
    out = torch.zeros(1, T, H, Dh, device=DEV)
    nan = torch.full_like(kv, float("nan"))
    for total, hint in [(n, n) for n in totals] + [(most, totals[0])]:
        print("case", Dh, H, T, total, hint, flush=True)
        sess.main.kv_write(1, 0, sess.kv, 0, most, nan)                  # whatever lies behind the row must not matter
        sess.main.kv_write(1, 0, sess.kv, 0, total, kv[:, :total].contiguous())
        L = total - T
        sess.seq_len.fill_(L)
        sess.kv.seq_len_hint = hint - T
        sess.main.tree_attention(1, 0, sess.ws, q, sess.seq_len, sess.kv, out)
        torch.cuda.synchronize()
        seen = torch.cat([torch.ones(T, L, dtype=torch.bool, device=DEV), own], 1)
        for h in sorted({0, H // 2, H - 1}):
            ref = _reference(q[0, :, h], kv[0, :total, 0, h], kv[0, :total, 1, h], seen)
            # as in test_gpu_attn_pair: half probabilities and |v| under 6
            assert float((out[0, :, h].double() - ref).abs().max()) <= 6 * 2.0 ** -11, (total, h)
    assert sess.main.read_flags() == 0
