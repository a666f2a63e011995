"""The 128 x 128 tile of several row groups, whose two wave groups take alternate k-steps: no spilled registers, and row counts and
depths at its edges (an odd and an even number of slots, a last row group with one, two and four row blocks) against the oracle."""
import os
import re
import subprocess

import pytest
import torch

from oracle import hydra_oracle as O
from synth import random_tree, uniform_tokens
from helpers import make_weights, oracle_model, small_shape
from gpu_util import gpu_session, max_rel, to_np
from paper_2402_05109_amd import build as build_lib

TILE_128x128 = 6


@pytest.mark.gpu
@pytest.mark.parametrize("d,F,T,B,splits", [(512, 896, 65, 2, 1), (768, 1024, 85, 2, 1), (1280, 1408, 96, 2, 2), (640, 640, 128, 3, 1), (1280, 1408, 43, 6, 4)])
def test_row_groups(d, F, T, B, splits, monkeypatch):
    """16-bit parity bar (2e-2 relative); a k-step that one group leaves out or both take shows as an error of order 1."""
    monkeypatch.setenv("HYDRA_PLAN_TILE", "1")
    monkeypatch.setenv("HYDRA_PLAN_TILE_ID", str(TILE_128x128))
    monkeypatch.setenv("HYDRA_PLAN_TILE_SPLITS", str(splits))
    monkeypatch.setenv("HYDRA_PLAN_QKV_UNFUSED", "1")
    cfg = small_shape(d=d, NL=1, H=d // 128, Dh=128, F=F, V=1003, K=0, T=T, dtype="bf16")
    W = make_weights(cfg, gain_std=0.1, std=0.04 * (512 / d) ** 0.5)
    parent = random_tree(T, 5, 7)
    toks = torch.stack([uniform_tokens(31, b, T, cfg.V) for b in range(B)]).to(torch.int32)
    sess = gpu_session(cfg, parent, B, 32, W, page_perm_seed=5, want_logits=True)
    o = sess.out()
    o.tree_tokens.copy_(toks)
    sess.verify()
    first = [x.clone() for x in (o.hidden, o.logits)]
    sess.verify()
    torch.cuda.synchronize()
    assert sess.main.read_flags() == 0
    assert all(torch.equal(a, b) for a, b in zip(first, (o.hidden, o.logits)))
    m = oracle_model(cfg, W)
    for b in range(B):
        hid, lg = O.tree_verify(m, O.FlatCache(m, T), 0, O.Tree(parent), toks[b].tolist())[:2]
        assert max_rel(to_np(o.hidden[b]), hid) <= 2e-2 and max_rel(to_np(o.logits[b]), lg) <= 2e-2


@pytest.mark.gpu
@pytest.mark.parametrize("T,B", [(112, 2), (96, 3), (120, 4)])
def test_row_groups_that_the_rule_chooses(T, B):
    """2048 x 5504 without a named tile: two row groups (the kernel of eight waves side by side), three (192 workgroups of the halves), and
    four with a workgroup on every CU."""
    cfg = small_shape(d=2048, NL=1, H=16, Dh=128, F=5504, V=1003, K=0, T=T, dtype="bf16")
    W = make_weights(cfg, gain_std=0.1, std=0.02)
    parent = random_tree(T, 5, 7)
    toks = torch.stack([uniform_tokens(31, b, T, cfg.V) for b in range(B)]).to(torch.int32)
    sess = gpu_session(cfg, parent, B, 32, W, page_perm_seed=5, want_logits=True)
    o = sess.out()
    o.tree_tokens.copy_(toks)
    sess.verify()
    torch.cuda.synchronize()
    assert sess.main.read_flags() == 0
    m = oracle_model(cfg, W)
    for b in sorted({0, B - 1}):
        hid, lg = O.tree_verify(m, O.FlatCache(m, T), 0, O.Tree(parent), toks[b].tolist())[:2]
        assert max_rel(to_np(o.hidden[b]), hid) <= 2e-2 and max_rel(to_np(o.logits[b]), lg) <= 2e-2


def test_kernels_keep_everything_in_registers():
    cmd = [build_lib._hipcc(), *build_lib.FLAGS, "-c", os.path.join(build_lib.CSRC, "bf16_gemm_halves.hip"), "-o", os.devnull, "--cuda-device-only",
           "-Rpass-analysis=kernel-resource-usage"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    assert [int(x) for x in re.findall(r"ScratchSize \[bytes/lane\]: (\d+)", r.stderr)] == [0, 0, 0]
