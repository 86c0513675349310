"""Build-time guard for the hot kernels: no private memory.  The GEMM kernels keep their accumulator tiles in
registers; a change that makes the compiler index them dynamically moves them to scratch memory and costs
tens of per cent without failing any parity test.  The hand-scheduled loops must also name only registers
inside the budget their occupancy leaves (the compiler warns otherwise).  hipcc reports the per-kernel resources while cross-compiling
(no GPU needed)."""
import os
import re
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)


def _resources(src):
    from paper_2101_05615_amd import build
    flags = [f for f in build.FLAGS if f not in ("-shared",)]
    cmd = ["hipcc"] + flags + ["--cuda-device-only", "-c", "-Rpass-analysis=kernel-resource-usage",
                               os.path.join(build.CSRC, src), "-o", os.devnull]
    err = subprocess.run(cmd, check=True, capture_output=True, text=True).stderr
    # the hand-scheduled loops name fixed registers; all of them must lie inside the kernel's register budget
    assert "reserved registers" not in err, [l for l in err.splitlines() if "reserved registers" in l][:2]
    out, name = {}, None
    for line in err.splitlines():
        m = re.search(r"Function Name: (\S+)", line)
        if m:
            name = m.group(1)
            out[name] = {}
        for key in ("ScratchSize [bytes/lane]", "VGPRs Spill", "SGPRs Spill", "Occupancy [waves/SIMD]"):
            m = re.search(re.escape(key) + r": (\d+)", line)
            if m and name:
                out[name][key] = int(m.group(1))
    return out


@pytest.mark.timeout(600)
def test_gemm_kernels_use_no_scratch_memory_and_spill_nothing():
    with ThreadPoolExecutor(3) as ex:
        tile, skinny, patch = ex.map(_resources, ["gemm_tile.hip", "gemm_skinny.hip", "conv_patch.hip"])
    assert len(tile) >= 30 and len(skinny) >= 30 and len(patch) >= 40, "the resource report was not parsed"
    # the patch kernels' launcher counts on these waves per SIMD when it decides how many workgroups share a CU
    for name, r in patch.items():
        m = re.search(r"ILi(\d+)ELi(\d+)ELi(\d+)ELi(\d+)E", name)
        wm, wn, mb, nbw = (int(x) for x in m.groups())
        need = 2 if mb * nbw >= 8 else (7 if mb * nbw == 2 and wm * wn == 8 else 4)
        assert r["Occupancy [waves/SIMD]"] >= need, f"{name}: {r}"
    for name, r in {**tile, **skinny, **patch}.items():
        assert r.get("ScratchSize [bytes/lane]") == 0, f"{name} uses scratch memory: {r}"
        assert r.get("VGPRs Spill") == 0 and r.get("SGPRs Spill") == 0, f"{name} spills registers: {r}"


@pytest.mark.timeout(600)
def test_convolution_kernels_in_lds():
    """The few-channel and the group convolution: no scratch memory and no spilled vector registers, and the waves per SIMD
    that their launchers count on."""
    with ThreadPoolExecutor(2) as ex:
        runs, group = ex.map(_resources, ["conv_runs.hip", "conv_group.hip"])
    same = {n: r for n, r in group.items() if "qg_conv_same_mfma_kernel" in n}
    assert len(runs) >= 20 and len(same) >= 30, "the resource report was not parsed"
    for name, r in runs.items():
        assert r["ScratchSize [bytes/lane]"] == 0 and r["VGPRs Spill"] == 0, f"{name}: {r}"
        assert r["SGPRs Spill"] <= 2, f"{name}: {r}"   # (the form for any number of steps keeps two in a vector register)
        assert r["Occupancy [waves/SIMD]"] >= 4, f"{name}: {r}"   # two workgroups of eight waves per CU
    for name, r in same.items():
        assert r["ScratchSize [bytes/lane]"] == 0 and r["VGPRs Spill"] == 0 and r["SGPRs Spill"] == 0, f"{name}: {r}"
        m = re.search(r"ILi\d+ELi\d+ELi\d+ELb([01])ELb[01]ELi(n?\d+)ELb[01]E", name)
        compact, zero_points = not m.group(2).startswith("n"), m.group(1) == "1"
        assert r["Occupancy [waves/SIMD]"] >= (7 if compact and not zero_points else 4), f"{name}: {r}"
    # taps from memory: the form of 128 channels without zero points keeps three dwords per lane in scratch memory
    for name, r in group.items():
        if name not in same:
            assert r["ScratchSize [bytes/lane]"] <= (12 if "group_mfma_kernelILi3ELi3ELi4ELb0ELb0E" in name else 0), f"{name}: {r}"
