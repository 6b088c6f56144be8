"""k_conv_patch, compiled for gfx950, never touches a register that an LDS read in flight will still write, and reaches device memory by
no flat instruction (see asm_check.py)."""
import os
import shutil
import subprocess

import pytest

import asm_check

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_patch_kernels_keep_in_flight_read_registers_untouched(tmp_path):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not (os.path.exists(hipcc) or shutil.which(hipcc)):
        pytest.skip("no hipcc")
    from paper_1710_03740_amd import build as mpt_build
    out = tmp_path / "gemm_ring.s"
    csrc = os.path.join(ROOT, "paper_1710_03740_amd", "csrc")
    cmd = [hipcc] + [f for f in mpt_build.HIP_FLAGS if f != "-fPIC"] + ["-x", "hip", "-S", "--cuda-device-only", "-o", str(out), os.path.join(csrc, "gemm_ring.hip")]
    subprocess.run(cmd, check=True, stdout=subprocess.PIPE, stderr=subprocess.STDOUT)
    n = 0
    for name, lines in asm_check.kernels(out.read_text(), r"k_conv_patch"):
        found = asm_check.check_kernel(lines)
        assert not found, "%s: %s" % (name, found[:5])
        code = [l.split(";")[0].strip() for l in lines]
        assert not [l for l in code if l.startswith(("flat_", "scratch_"))], name
        assert sum("v_mfma" in l for l in code) >= 144
        # the wait at the end of a trip leaves its stores in flight and nothing else: there are as many as it counts
        assert sum(l.startswith("global_store") for l in code) == 8 and any("vmcnt(8)" in l for l in code)
        n += 1
    assert n == 4
