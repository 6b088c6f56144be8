"""The softmax of rows held in registers works the label's element of the gradient out once per chunk, not at each of its eight places."""
import os
import shutil
import subprocess

import pytest

import asm_check

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_the_label_is_worked_out_once_and_nothing_spills(tmp_path):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not (os.path.exists(hipcc) or shutil.which(hipcc)):
        pytest.skip("no hipcc")
    from paper_1710_03740_amd import build as mpt_build
    out = tmp_path / "elementwise.s"
    csrc = os.path.join(ROOT, "paper_1710_03740_amd", "csrc")
    cmd = [hipcc] + [f for f in mpt_build.HIP_FLAGS if f != "-fPIC"] + ["-x", "hip", "-S", "--cuda-device-only", "-o", str(out), os.path.join(csrc, "elementwise.hip")]
    subprocess.run(cmd, check=True, stdout=subprocess.PIPE, stderr=subprocess.STDOUT)
    n = 0
    for name, lines in asm_check.kernels(out.read_text(), r"k_softmax_xent_(rows|small)"):
        code = [l.split(";")[0].strip() for l in lines]
        assert not [l for l in code if l.startswith("scratch_")], name
        chunks = int(name.split("ELi")[1].split("E")[0]) if "rows" in name else 1
        if chunks <= 4:
            # per chunk and element one product for the output; the label's two; some for the sum's reciprocal and the loss
            products = sum(l.startswith(("v_mul_f32", "v_fma_mixlo", "v_fma_mixhi")) for l in code)
            assert products <= chunks * (8 + 8 + 2) + 24, (name, products)
        n += 1
    assert n == 20                                                       # eight row lengths, rows at any address or aligned; four for few rows
