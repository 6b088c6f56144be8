"""No kernel of the matrix products reaches device memory by flat instructions: these count with the LDS reads, whose hand-written
waits would then wait for the operands of stages to come.  And no load of rows at any address claims more alignment than their elements have."""
import os
import re
import shutil
import subprocess

import pytest

import asm_check

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def compiled(out, *form):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not (os.path.exists(hipcc) or shutil.which(hipcc)):
        pytest.skip("no hipcc")
    from paper_1710_03740_amd import build as mpt_build
    csrc = os.path.join(ROOT, "paper_1710_03740_amd", "csrc")
    cmd = [hipcc] + [f for f in mpt_build.HIP_FLAGS if f != "-fPIC"] + ["-x", "hip", *form, "--cuda-device-only", "-o", str(out), os.path.join(csrc, "gemm_ring.hip")]
    subprocess.run(cmd, check=True, stdout=subprocess.PIPE, stderr=subprocess.STDOUT)
    return out.read_text()


def test_ring_kernels_have_no_flat_accesses(tmp_path):
    n = 0
    for name, lines in asm_check.kernels(compiled(tmp_path / "gemm_ring.s", "-S"), r"k_gemm_(ring|any|pieces)"):
        assert not [l for l in lines if l.strip().startswith("flat_")], name
        n += 1
    assert n >= 15


def test_loads_of_rows_at_any_address_claim_the_alignment_of_their_elements(tmp_path):
    """In the compiler's intermediate form, where a load states its alignment: operands are FP16 at any address, outputs FP16 or FP32."""
    text, kernels, beside = compiled(tmp_path / "gemm_ring.ll", "-S", "-emit-llvm"), 0, 0
    for m in re.finditer(r"^define [^\n]*?@(\w*k_gemm_(?:any|pieces)\w*)\(.*?^}", text, re.M | re.S):
        name = m.group(1)
        kernels += "k_gemm_any" in name
        beside += "k_gemm_pieces" in name
        loads = re.findall(r"= load (<\d+ x \w+>), ptr addrspace\(1\) .*?align (\d+)", m.group(0))
        for ty, align in loads:
            assert int(align) <= (4 if "float" in ty else 2), "%s: load %s, align %s" % (name, ty, align)
        # four pieces of a stage and the first two stages ahead of the loop, half of them where eight wavefronts share a 64 x 64 tile; pieces side by side that go to
        # LDS directly have the mask's and the old values' loads only
        assert len(loads) >= (2 if "RingMat" in name else 8 if "ELi32ELi16E" in name else 16), name
    assert kernels >= 40 and beside >= 18
