"""Compiled code of the GEMM, elementwise and probe kernels (CPU, hipcc only). No
instantiation spills VGPRs. A spill in an 8-wave GEMM tile lands in its K loop
(scratch traffic on every stage); the residual-epilogue instantiations once
spilled 40-103 registers that way."""
import os
import re
import shutil
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)


@pytest.mark.skipif(not os.path.exists("/opt/rocm/bin/hipcc") and shutil.which("hipcc") is None, reason="no hipcc")
@pytest.mark.parametrize("src", ["k_gemm.hip", "k_elementwise.hip", "k_probe.hip"])
def test_no_vgpr_spills(src, tmp_path):
    from paper_2503_22562_amd import build as B
    cmd = [B.HIPCC, *B.COMMON, *B.HIP_FLAGS, *B.EXTRA_FLAGS.get(src, []), "--cuda-device-only",
           "-Rpass-analysis=kernel-resource-usage", "-c", os.path.join(B.CSRC, src), "-o", str(tmp_path / "k.o")]
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stderr[-2000:]
    names = re.findall(r"Function Name: (\S+)", r.stderr)
    spills = [int(v) for v in re.findall(r"VGPRs Spill: (\d+)", r.stderr)]
    assert names and len(names) == len(spills)
    bad = [(n, s) for n, s in zip(names, spills) if s]
    assert not bad, bad


@pytest.mark.skipif(not os.path.exists("/opt/rocm/bin/hipcc") and shutil.which("hipcc") is None, reason="no hipcc")
def test_epilogue_strips_are_ordered_within_the_wave(tmp_path):
    """The pipelined GEMM's epilogues exchange blocks between a wave's lanes
    through LDS: wherever its code turns from LDS stores to loads or back after
    the K loop, a wave barrier (a mark for the compiler, no instruction) stands between."""
    from paper_2503_22562_amd import build as B
    out = tmp_path / "k.s"
    cmd = [B.HIPCC, *B.COMMON, *B.HIP_FLAGS, *B.EXTRA_FLAGS["k_gemm.hip"], "--cuda-device-only", "-S",
           os.path.join(B.CSRC, "k_gemm.hip"), "-o", str(out)]
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stderr[-2000:]
    bodies = re.findall(r"^(\S*gemm_pipe_kernel\S*):.*?\n(.*?)\n\.Lfunc_end", out.read_text(), re.M | re.S)
    assert bodies
    staged, bad = 0, []
    for name, body in bodies:
        kind, marked = None, False
        for line in body.splitlines():
            op = line.strip()
            if "wave barrier" in op:
                marked = True
            elif op.startswith(("s_barrier", ".LBB")):
                kind = None  # ordered by the barrier, or another block: its own start is not known
            elif op.startswith(("ds_write", "ds_read")):
                k = op[:6]
                if kind and k != kind:
                    staged += 1
                    if not marked:
                        bad.append((name, op))
                kind, marked = k, False
    assert staged and not bad, bad[:5]
