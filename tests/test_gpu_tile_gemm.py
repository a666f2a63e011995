"""The many-rows GEMM with both operands in LDS: every tile shape, with K whole and split over workgroups, at row counts and
widths that end inside a tile, against the oracle's verification forward."""
import os
import re
import subprocess

import numpy as np
import pytest
import torch

from oracle import hydra_oracle as O
from synth import random_tree, uniform_tokens
from helpers import make_weights, oracle_model, small_shape
from gpu_util import gpu_session, max_rel, to_np
from paper_2402_05109_amd import binding as hb
from paper_2402_05109_amd import build as build_lib

CFG = small_shape(d=512, NL=1, H=4, Dh=128, F=896, V=1003, K=0).with_(dtype="bf16")
# 40, 120, 88 and (ragged) 32 bands; 80 and 88 k-steps, of which four splits leave the 20 that the deepest ring (two times ten
# slots) asks for and three splits a shorter last one
WIDE = small_shape(d=1280, NL=1, H=10, Dh=128, F=1408, V=1003, K=0).with_(dtype="bf16")
_weights, _ref = {}, {}


def _made(cfg):
    if cfg.d not in _weights:
        _weights[cfg.d] = make_weights(cfg, gain_std=0.1, std=0.04 * (512 / cfg.d) ** 0.5)
    return _weights[cfg.d]


def _reference(T, B):
    """Oracle hidden and logits of every row of the wide shape, computed once per shape."""
    if (T, B) not in _ref:
        m = oracle_model(WIDE, _made(WIDE))
        parent = random_tree(T, 5, 7)
        toks = torch.stack([uniform_tokens(31, b, T, WIDE.V) for b in range(B)]).to(torch.int32)
        out = [O.tree_verify(m, O.FlatCache(m, T), 0, O.Tree(parent), toks[b].tolist())[:2] for b in range(B)]
        _ref[T, B] = (_made(WIDE), parent, toks, np.stack([o[0] for o in out]), np.stack([o[1] for o in out]))
    return _ref[T, B]


@pytest.mark.gpu
@pytest.mark.parametrize("tile,T,B,splits", [(tile, T, B, splits) for tile in range(1, 8)
                                             for T, B, splits in ((65, 1, 1), (128, 1, 3), (43, 3, 1), (37, 7, 2), (100, 3, 4))      # 65, 128, 129, 259, 300 rows
                                             if tile > 4 or T * B > 128])            # tiles of 256 rows are not planned for up to 128 rows
def test_every_tile_matches_the_oracle(tile, T, B, splits, monkeypatch):
    """16-bit parity bar of the repository (2e-2 relative); a wrong tile, k-step or row shows as an error of order 1.  Every
    product of the call runs on the tile and with the K splits named here (q|k|v, O, down and LM head; gate/up and, with one
    split, the residual epilogues have K whole) or the call is refused: see test_a_tile_that_cannot_be_had_is_refused."""
    monkeypatch.setenv("HYDRA_PLAN_TILE", "1")
    monkeypatch.setenv("HYDRA_PLAN_TILE_ID", str(tile))
    monkeypatch.setenv("HYDRA_PLAN_TILE_SPLITS", str(splits))
    monkeypatch.setenv("HYDRA_PLAN_QKV_UNFUSED", "1")
    W, parent, toks, hid, lg = _reference(T, B)
    sess = gpu_session(WIDE, parent, B, 32, W, page_perm_seed=5, want_logits=True)
    o = sess.out()
    o.tree_tokens.copy_(toks)
    sess.verify()
    first = [x.clone() for x in (o.hidden, o.logits, o.argmax)]
    sess.verify()
    torch.cuda.synchronize()
    assert sess.main.read_flags() == 0
    assert all(torch.equal(a, b) for a, b in zip(first, (o.hidden, o.logits, o.argmax)))      # fixed summation order
    assert max_rel(to_np(o.hidden).reshape(-1, WIDE.d), hid.reshape(-1, WIDE.d)) <= 2e-2
    assert max_rel(to_np(o.logits).reshape(-1, WIDE.V), lg.reshape(-1, WIDE.V)) <= 2e-2


@pytest.mark.gpu
@pytest.mark.parametrize("tile,T,B,splits", [(7, 100, 3, 5), (6, 100, 3, 6), (1, 128, 1, 1), (5, 65, 1, 9)])
def test_a_tile_that_cannot_be_had_is_refused(tile, T, B, splits, monkeypatch):
    """More splits than the ring leaves k-steps for or than are planned, or 256 rows for 128: the forced plan does not give way
    to another one, so the test above cannot pass on kernels that it does not name."""
    monkeypatch.setenv("HYDRA_PLAN_TILE", "1")
    monkeypatch.setenv("HYDRA_PLAN_TILE_ID", str(tile))
    monkeypatch.setenv("HYDRA_PLAN_TILE_SPLITS", str(splits))
    monkeypatch.setenv("HYDRA_PLAN_QKV_UNFUSED", "1")
    sess = gpu_session(WIDE, random_tree(T, 5, 7), B, 32, _made(WIDE))
    with pytest.raises(hb.HydraError) as e:
        sess.verify()
    assert e.value.code == hb.E_UNSUPPORTED


@pytest.mark.gpu
@pytest.mark.parametrize("start", [0, 1, 15, 16, 30])
@pytest.mark.parametrize("T", [66, 80])
def test_rotary_append_by_pages(start, T, monkeypatch):
    """Cache append as a kernel of its own: tokens that begin and end inside a page leave the page's other tokens alone and
    whole pages are written whole; compared with the fused q|k|v kernel on the same inputs."""
    W, parent = _made(CFG), random_tree(T, 5, 7)
    got = {}
    for mode in ("0", "1"):
        monkeypatch.setenv("HYDRA_PLAN_QKV_UNFUSED", mode)
        sess = gpu_session(CFG, parent, 2, 64, W, page_perm_seed=5)
        n = start + T + 13
        plain = torch.arange(2 * n * 2 * 512, dtype=torch.float32, device="cuda:0").remainder(1021).reshape(2, n, 2, 4, 128).contiguous() / 64
        sess.main.kv_write(2, 0, sess.kv, 0, n, plain)
        sess.seq_len.copy_(torch.tensor([start, start // 2], dtype=torch.int32)); sess.host_len = start
        sess.out().tree_tokens.copy_(torch.stack([uniform_tokens(3, b, T, CFG.V) for b in range(2)]).to(torch.int32))
        sess.verify()
        after = torch.empty_like(plain)
        sess.main.kv_read(2, 0, sess.kv, 0, n, after)
        torch.cuda.synchronize()
        for b, s in enumerate((start, start // 2)):
            assert torch.equal(after[b, :s], plain[b, :s]) and torch.equal(after[b, s + T:], plain[b, s + T:])
        got[mode] = after
    # two summation orders of the same fp32 products, rounded to half: at most one half-precision step apart
    a, b = got["0"], got["1"]
    assert float((a - b).abs().max() / a.abs().max()) <= 2.0 ** -10


@pytest.fixture(scope="module")
def compiled(tmp_path_factory):
    """(assembly of the tile kernels, the compiler's resource remarks)"""
    out = str(tmp_path_factory.mktemp("asm") / "tile.s")
    cmd = [build_lib._hipcc(), *build_lib.FLAGS, "-S", os.path.join(build_lib.CSRC, "bf16_gemm_tile.hip"), "-o", out, "--cuda-device-only",
           "-Rpass-analysis=kernel-resource-usage"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    with open(out) as f:
        return f.read(), r.stderr


def test_tile_kernels_keep_everything_in_registers(compiled):
    scratch = [int(x) for x in re.findall(r"ScratchSize \[bytes/lane\]: (\d+)", compiled[1])]
    assert len(scratch) >= 21 and not any(scratch)


def test_tile_kernels_end_their_reads_before_a_slot_is_refilled(compiled):
    """The barrier inside the loop over the slots lets other waves overwrite the slot before the current one: a wave must not
    arrive with reads of it under way, wherever the compiler has put the instructions that use them."""
    kernels = [k for k in re.split(r"\n(?=_ZN5hydra16gemm_tile_kernel\S+:)", compiled[0])[1:]]
    assert len(kernels) == 21
    for k in kernels:
        body = [x.strip() for x in k.split(".Lfunc_end")[0].splitlines()]
        code = [x for x in body if x and not x.startswith((";", "."))]
        waits = [code[i - 1] for i, x in enumerate(code) if x == "s_barrier"]
        ring = [w for w in waits if re.fullmatch(r"s_waitcnt vmcnt\(\d+\) lgkmcnt\(\d+\)", w) and "lgkmcnt(0)" not in w]
        assert len(ring) == 2, (k.split(":")[0], waits)              # waves with rows of their own, and waves that only fetch
