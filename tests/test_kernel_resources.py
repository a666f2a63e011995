"""Compiler resource report of the hot kernels (no GPU needed: hipcc cross-compiles gfx950).

A streaming kernel whose accumulators or prefetch registers end up in scratch memory still computes the right
result, only several times slower, so parity tests cannot see it.  This test reads hipcc's per-kernel resource
remarks: no instantiation of the weight-streaming GEMM, of the attention kernels or of the fp32 family's products may use
scratch memory at all; the persistent layer kernel spills the few registers stated at its test."""
from __future__ import annotations

import os
import re
import subprocess

import pytest

from paper_2402_05109_amd import build as B


def _resource_report(source: str):
    """{kernel symbol: {"scratch": bytes per lane, "spill": spilled VGPRs, "vgprs": n}} for one source file"""
    cmd = [B._hipcc(), *B.FLAGS, "-c", os.path.join(B.CSRC, source), "-o", os.devnull,
           "--cuda-device-only", "-Rpass-analysis=kernel-resource-usage"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    out, cur = {}, None
    for line in r.stderr.splitlines():
        m = re.search(r"Function Name: (\S+)", line)
        if m:
            cur = out.setdefault(m.group(1), {})
            continue
        if cur is None:
            continue
        for key, pat in (("scratch", r"ScratchSize \[bytes/lane\]: (\d+)"), ("spill", r"VGPRs Spill: (\d+)"),
                         ("vgprs", r" VGPRs: (\d+)")):
            m = re.search(pat, line)
            if m:
                cur[key] = int(m.group(1))
    return out


def test_streaming_gemm_keeps_everything_in_registers():
    rep = {k: v for k, v in _resource_report("bf16_gemm.hip").items() if "gemm_bf16_kernel" in k or "gemm_bf16_sharedx_kernel" in k}
    assert len(rep) >= 50, "the GEMM instantiations were not found in the compiler's report"
    assert any("sharedx" in k for k in rep)
    bad = {k: v for k, v in rep.items() if v.get("scratch", 0) != 0 or v.get("spill", 0) != 0}
    assert not bad, f"GEMM instantiations using scratch memory: {bad}"


@pytest.mark.parametrize("source, families", [
    # QW 1 and 2, packed output or not, 64 and 128 dims; short: shares of the head's dims and streaming; pair: waves and streaming
    ("bf16_attn.hip", {"attn_bf16_kernel": 8, "attn_short_kernel": 14, "attn_pair_kernel": 8, "attn_merge_kernel": 4}),
    # five epilogues, with a norm in front or not, rows of whole 16 bytes or not; attention: 64 and 128 dims
    ("f32_family.hip", {"gemm_f32_kernel": 9, "attn_f32_kernel": 2}),
])
def test_attention_and_fp32_products_keep_everything_in_registers(source, families):
    rep = _resource_report(source)
    for family, n in families.items():
        found = {k: v for k, v in rep.items() if family in k}
        assert len(found) == n, f"{family}: {sorted(found)}"
        bad = {k: v for k, v in found.items() if v["scratch"] != 0 or v["spill"] != 0}
        assert not bad, f"instantiations using scratch memory: {bad}"


def test_layer_kernel_keeps_its_streams_in_registers():
    """The persistent layer kernel: with 64-wide heads it must not use scratch memory at all; with 128-wide heads the
    compiler spills three registers (16 bytes of scratch per lane) around the attention step, which needs all 256 as a
    kernel of its own.  Spills of the weight-streaming loops would be tens to hundreds."""
    rep = {k: v for k, v in _resource_report("bf16_layers.hip").items() if "layers_kernel" in k}
    assert len(rep) == 4
    for k, v in rep.items():
        limit = 0 if "ELi64EEE" in k else 4
        assert v["spill"] <= limit and v["scratch"] <= 4 * limit, f"{k}: {v}"


def test_typical_acceptance_keeps_its_row_in_registers():
    """One workgroup of 1024 threads holds a row of logits: 128 registers per lane, none of them spilled."""
    rep = {k: v for k, v in _resource_report("draft_accept.hip").items() if "typical_stats" in k or "typical_select" in k}
    assert len(rep) == 2
    bad = {k: v for k, v in rep.items() if v.get("scratch", 0) != 0 or v.get("spill", 0) != 0}
    assert not bad, f"typical acceptance using scratch memory: {bad}"
