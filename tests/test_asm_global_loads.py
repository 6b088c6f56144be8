"""No kernel of the matrix products reaches device memory by flat instructions: these count with the LDS reads, whose hand-written
waits would then wait for the operands of stages to come."""
import os
import shutil
import subprocess

import pytest

import asm_check

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_ring_kernels_have_no_flat_accesses(tmp_path):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not (os.path.exists(hipcc) or shutil.which(hipcc)):
        pytest.skip("no hipcc")
    from paper_1710_03740_amd import build as mpt_build
    out = tmp_path / "gemm_ring.s"
    csrc = os.path.join(ROOT, "paper_1710_03740_amd", "csrc")
    cmd = [hipcc] + [f for f in mpt_build.HIP_FLAGS if f != "-fPIC"] + ["-x", "hip", "-S", "--cuda-device-only", "-o", str(out), os.path.join(csrc, "gemm_ring.hip")]
    subprocess.run(cmd, check=True, stdout=subprocess.PIPE, stderr=subprocess.STDOUT)
    n = 0
    for name, lines in asm_check.kernels(out.read_text(), r"k_gemm_(ring|any)"):
        assert not [l for l in lines if l.strip().startswith("flat_")], name
        n += 1
    assert n >= 15
