"""Host stepping of the row-band sweep that interpolates the coarse correction
into its input: tests/band_prolong_emu.cpp runs the kernel's own per-thread code
against the separate interpolation and two colour passes, bit for bit (no
contraction on the host; every weight is a power of two), with z coarsened and
kept, both colour orders, march directions and prefetch depths, and every access
checked against its buffer.
"""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_0904_4887_amd", "csrc")


def test_prolonging_sweep_steps_match_separate_passes(tmp_path):
    cxx = next((c for c in ("/opt/rocm/llvm/bin/clang++", shutil.which("clang++")) if c and os.path.exists(c)), None)
    if cxx is None:
        pytest.skip("no clang++ (the per-thread code uses clang vector types)")
    exe = str(tmp_path / "emu")
    r = subprocess.run([cxx, "-O1", "-std=c++17", "-ffp-contract=off", "-I", CSRC,
                        os.path.join(HERE, "band_prolong_emu.cpp"), "-o", exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and r.stdout.rstrip().endswith("OK (0 failing cases)"), r.stdout[-2000:] + r.stderr[-2000:]
