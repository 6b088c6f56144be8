"""The closing launch of the batch-norm reductions waits for memory and for little else: its compiled form has eight partials of each sum
in flight before the first of them is waited for."""
import os
import shutil
import subprocess

import pytest

import asm_check

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_partials_are_fetched_together(tmp_path):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not (os.path.exists(hipcc) or shutil.which(hipcc)):
        pytest.skip("no hipcc")
    from paper_1710_03740_amd import build as mpt_build
    out = tmp_path / "norm.s"
    csrc = os.path.join(ROOT, "paper_1710_03740_amd", "csrc")
    cmd = [hipcc] + [f for f in mpt_build.HIP_FLAGS if f != "-fPIC"] + ["-x", "hip", "-S", "--cuda-device-only", "-o", str(out), os.path.join(csrc, "norm.hip")]
    subprocess.run(cmd, check=True, stdout=subprocess.PIPE, stderr=subprocess.STDOUT)
    together = []
    for name, lines in asm_check.kernels(out.read_text(), r"k_bn_finalize"):
        runs = [0]
        for l in lines:
            t = l.split(";")[0].strip()
            assert not t.startswith("scratch_"), name
            if t.startswith("global_load_dwordx2"):
                runs[-1] += 1
            elif t.startswith("s_waitcnt") and "vmcnt" in t:
                runs.append(0)
        together.append(max(runs))
    assert len(together) == 4 and min(together) >= 16, together     # in 16 and 64 groups of threads; two sums each
