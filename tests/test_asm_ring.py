"""The ring and any-alignment GEMM kernels, compiled for gfx950, never touch a register that an LDS read in flight will
still write (see asm_check.py).  Compiles csrc/gemm_ring.hip to device assembly and walks every instantiation."""
import os
import shutil
import subprocess

import pytest

import asm_check

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def assembly(tmp_path_factory):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not (os.path.exists(hipcc) or shutil.which(hipcc)):
        pytest.skip("no hipcc")
    from paper_1710_03740_amd import build as mpt_build
    out = tmp_path_factory.mktemp("asm") / "gemm_ring.s"
    csrc = os.path.join(ROOT, "paper_1710_03740_amd", "csrc")
    flags = [f for f in mpt_build.HIP_FLAGS if f != "-fPIC"]
    cmd = [hipcc] + flags + ["-I", os.path.join(ROOT, "include"), "-I", csrc, "-x", "hip", "-S", "--cuda-device-only", "-o", str(out), os.path.join(csrc, "gemm_ring.hip")]
    r = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert r.returncode == 0, r.stdout[-2000:]
    return out.read_text()


def test_ring_kernels_keep_in_flight_read_registers_untouched(assembly):
    n = 0
    for name, lines in asm_check.kernels(assembly, r"k_gemm_(ring|any|pieces)"):
        found = asm_check.check_kernel(lines)
        assert not found, "%s: %s" % (name, found[:5])
        assert sum("v_mfma" in l for l in lines) >= (4 if "ELi32ELi16E" in name else 8)      # (two blocks per half stage where a wavefront has 32 x 16)
        n += 1
    assert n >= 15


def test_no_wide_shift_takes_its_amount_from_the_last_register(assembly):
    registers = asm_check.vector_registers(assembly)
    n = 0
    for name, lines in asm_check.kernels(assembly, r"k_(gemm|conv)"):
        assert not asm_check.shifts_by_the_last_register(lines, registers[name]), name
        n += 1
    assert n >= 40
    assert asm_check.shifts_by_the_last_register(["\tv_lshlrev_b64 v[90:91], v127, v[86:87]"], 128) == [127]
    assert not asm_check.shifts_by_the_last_register(["\tv_lshlrev_b64 v[90:91], v127, v[86:87]"], 136)
