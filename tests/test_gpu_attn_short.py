"""16-bit tree attention of short contexts (one workgroup per 32-query tile and share of the head's dims): every share, both
head sizes, rows that end anywhere in a 32-key tile, no cached token at all, and a row longer than the host's hint."""
import numpy as np
import pytest
import torch

from oracle import hydra_oracle as O
from synth import random_tree
from helpers import make_weights, small_shape
from gpu_util import gpu_session, max_rel, to_np

pytestmark = pytest.mark.gpu
TOL = 2e-2                      # the bar of the 16-bit family


# heads, rows and nodes decide how many ways the dims are shared: 256 workgroups at most
@pytest.mark.parametrize("Dh,H,B,T,share", [(128, 2, 2, 40, 4), (128, 24, 3, 32, 2), (128, 24, 3, 33, 1), (64, 4, 2, 40, 2), (64, 48, 3, 7, 1), (128, 2, 1, 128, 4), (128, 5, 2, 1, 4)])
def test_short_contexts(Dh, H, B, T, share):
    groups = -(-T // 32) * H * B
    assert groups * share <= 256 and (share == Dh // 32 or groups * share * 2 > 256)
    tree = O.Tree(random_tree(T, 3, 4) if T > 1 else [-1])
    lens = (0, 1, 15, 33, 255 - T % 32, 700)
    longest = 1500                                   # 48 tiles of 32 keys: six per wave
    cfg = small_shape(d=H * Dh, NL=1, H=H, Dh=Dh, F=128, V=64, K=0, T=T, dtype="bf16")
    sess = gpu_session(cfg, tree.parent, B, longest + T, make_weights(cfg), page_perm_seed=5)
    rng = np.random.default_rng(T + Dh)
    half = lambda a: a.astype(np.float16).astype(np.float64)
    q = half(rng.standard_normal((B, T, H, Dh)) * 1.5)
    keys, vals = half(rng.standard_normal((B, longest + T, H, Dh)) * 1.5), half(rng.standard_normal((B, longest + T, H, Dh)))
    # whatever lies behind the row must not matter: not a number in every slot that is not written
    nan = torch.full((B, longest + T, 2, H, Dh), float("nan"), device="cuda:0")
    qd, out = torch.tensor(q, dtype=torch.float32, device="cuda:0").contiguous(), torch.zeros(B, T, H, Dh, device="cuda:0")
    heads = sorted({0, 1, H // 2, H - 1})
    for L, hint in [(n, n) for n in lens] + [(longest, 100)]:
        print("case", Dh, H, B, T, L, flush=True)
        sess.main.kv_write(B, 0, sess.kv, 0, longest + T, nan)
        sess.main.kv_write(B, 0, sess.kv, 0, L + T, torch.tensor(np.stack([keys, vals], axis=2)[:, :L + T], dtype=torch.float32, device="cuda:0").contiguous())
        sess.seq_len.fill_(L)
        sess.kv.seq_len_hint = hint
        sess.main.tree_attention(B, 0, sess.ws, qd, sess.seq_len, sess.kv, out)
        torch.cuda.synchronize()
        got = to_np(out)
        for b in range(B):
            for h in heads:
                ref = O.tree_attention(q[b, :, h], keys[b, :L + T, h], vals[b, :L + T, h], L, tree)
                assert max_rel(got[b, :, h], ref) <= TOL, (b, h, L)
    assert sess.main.read_flags() == 0
