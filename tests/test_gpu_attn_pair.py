"""16-bit tree attention with two query tiles to a wave: four and eight waves, keys split over workgroups, a last query tile
without a partner, rows that end anywhere in a 32-key tile, and more tiles per wave than page ids are held at a time."""
import math

import pytest
import torch

from synth import random_tree
from helpers import make_weights, small_shape
from gpu_util import gpu_session

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _reference(q, keys, vals, seen):
    """float64 softmax attention of one head: q [T, Dh], keys and vals [n, Dh], seen [T, n]"""
    s = (q.double() @ keys.double().T.contiguous()) / math.sqrt(q.shape[1])
    return torch.softmax(s.masked_fill(~seen, -math.inf), -1) @ vals.double()


@pytest.mark.parametrize("Dh,H,B,T,waves,lens", [
    (128, 24, 11, 33, 4, (0, 1, 15, 31, 32, 33, 100, 127, 128, 200, 255)),     # more groups than CUs
    (64, 64, 5, 65, 4, (0, 16, 47, 300, 2200)),                                # two groups of query tiles, the second without a partner
    (128, 52, 1, 40, 8, (2100,)),                                              # keys split over workgroups
    (128, 4, 2, 40, 4, (1700, 1441)),                                          # ... of four waves: with eight half of the chip would idle
    (64, 6, 1, 128, 8, (3000,)),
    (64, 64, 2, 34, 8, (8300, 5)),                                             # 33 tiles for the first waves, none for the others of row 1
])
def test_two_query_tiles_per_wave(Dh, H, B, T, waves, lens):
    qgroups, L = (-(-T // 32) + 1) // 2, max(lens)
    tiles = -(-(L + T) // 32)
    eight = H * B * qgroups * -(-tiles // 16)
    assert (4 if H * B * qgroups > 256 or (T <= 64 and Dh == 128 and eight < 128) else 8) == waves
    assert tiles > 40 or -(-T // 32) * H * B > 256                             # else the kernel of short contexts takes it
    assert T > 64 or tiles > 52 or eight > Dh                                  # or the one with a wave per query tile
    parent = random_tree(T, 4, 6)
    cfg = small_shape(d=H * Dh, NL=1, H=H, Dh=Dh, F=128, V=64, K=0, T=T, dtype="bf16")
    sess = gpu_session(cfg, parent, B, L + T, make_weights(cfg), page_perm_seed=3)
    g = torch.Generator(device=DEV).manual_seed(T + Dh)
    kv = torch.randn(B, L + T, 2, H, Dh, generator=g, device=DEV).half().float()
    q = (torch.randn(B, T, H, Dh, generator=g, device=DEV) * 2).half().float()
    written = kv.clone()
    for b in range(B):
        written[b, lens[b] + T:] = float("nan")      # whatever lies behind a row must not matter
    sess.main.kv_write(B, 0, sess.kv, 0, L + T, written)
    sess.seq_len.copy_(torch.tensor(lens, dtype=torch.int32))
    sess.kv.seq_len_hint = L
    out = torch.zeros(B, T, H, Dh, device=DEV)
    print("case", Dh, H, B, T, lens, flush=True)
    sess.main.tree_attention(B, 0, sess.ws, q, sess.seq_len, sess.kv, out)
    torch.cuda.synchronize()
    own = torch.zeros(T, T, dtype=torch.bool, device=DEV)
    for n in range(T):
        if n:
            own[n] = own[parent[n]]
        own[n, n] = True
    for b in range(B):
        seen = torch.cat([torch.ones(T, lens[b], dtype=torch.bool, device=DEV), own], 1)
        for h in sorted({0, 1, H // 2, H - 1}):
            ref = _reference(q[b, :, h], kv[b, :lens[b] + T, 0, h], kv[b, :lens[b] + T, 1, h], seen)
            # q, K and V are exact in half; a probability is rounded to half (2^-12 of itself at most) and the sum of p |v| over p
            # stays below the largest |v|, under 6 for these values
            assert float((out[b, :, h].double() - ref).abs().max()) <= 6 * 2.0 ** -11, (b, h)
    assert sess.main.read_flags() == 0
