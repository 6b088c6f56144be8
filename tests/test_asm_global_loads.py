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
    text, kernels, beside, wide = compiled(tmp_path / "gemm_ring.ll", "-S", "-emit-llvm"), 0, 0, 0
    for m in re.finditer(r"^define [^\n]*?@(\w*k_gemm_(?:any|pieces)\w*)\(.*?^}", text, re.M | re.S):
        kernels += "k_gemm_any" in m.group(1)
        beside += "k_gemm_pieces" in m.group(1)
        for ty, align in re.findall(r"= load (<\d+ x \w+>), ptr addrspace\(1\) .*?align (\d+)", m.group(0)):
            wide += 1
            assert int(align) <= (4 if "float" in ty else 2), "%s: load %s, align %s" % (m.group(1), ty, align)
    # k_gemm_any: 3 operand layouts; 64 x 64 tiles, with and without cuts, and 128 x 128; four wavefronts or eight, of which each has half the loads; any extents (four
    # wavefronts); edges read over in the 2 layouts that have them; 6 with operands apart.  k_gemm_pieces: 3 layouts, four or eight wavefronts, pieces, ordinary extents or any
    assert kernels == 18 + 9 + 12 + 6 and beside == 18 and wide >= 8 * (kernels + beside)
