"""fp16_plan and fp16_launch (csrc/gemm_plan.h), compiled by themselves for the host: the pieces and tiles of FP16 results."""
import ctypes
import os
import random
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SOURCE = r"""
#include "gemm_plan.h"
using namespace mpt_gemm;
// out: fp16 pieces chosen (0: make_plan's stay), splits, stages per split, tile, make_plan's splits and stages
extern "C" void planned(long I, long J, long R, int ws, int a_rc, int b_rc, int relu, int aligned, int lines, int* out) {
  const Plan p = make_plan(I, J, R, ws != 0);
  const bool rows = (a_rc ? R : I) % 8 == 0 && (b_rc ? R : J) % 8 == 0;
  const bool own = !pieces_side_by_side(p, I, J, R, rows, a_rc, b_rc) && fp16_planned(p, J, R, a_rc && !b_rc, !a_rc, relu != 0);
  const Fp16Form f = fp16_launch(p, I, J, R, rows, rows && aligned, rows && aligned && lines);
  const int r[7] = {own, f.splits, f.ktiles_per_split, f.tile, p.splits, p.ktiles_per_split, rows};
  for (int k = 0; k < 7; ++k) out[k] = r[k];
}
extern "C" int edges(long I, long J, long R, int a_rc, int b_rc) {
  const Plan p = make_plan(I, J, R, true);
  if (p.splits > 1 && !fp16_planned(p, J, R, a_rc && !b_rc, !a_rc, false)) return 0;
  const Fp16Form f = fp16_launch(p, I, J, R, true, true, false);
  return f.splits == 1 && edges_in_256(I, J, R, f.cost);
}
"""
FORMS = {"f": (1, 0), "d": (1, 1), "w": (0, 0)}


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("no g++")
    d = tmp_path_factory.mktemp("plan16")
    (d / "plan.cpp").write_text(SOURCE)
    subprocess.run([cxx, "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC", "-I", os.path.join(ROOT, "paper_1710_03740_amd", "csrc"),
                    "-o", str(d / "plan.so"), str(d / "plan.cpp")], check=True)
    L = ctypes.CDLL(str(d / "plan.so"))
    L.planned.argtypes = [ctypes.c_long] * 3 + [ctypes.c_int] * 6 + [ctypes.c_void_p]

    def call(op, I, J, R, ws=1, relu=0, aligned=1, lines=0):
        out = (ctypes.c_int * 7)()
        L.planned(I, J, R, ws, *FORMS[op], relu, aligned, lines, ctypes.addressof(out))
        return tuple(out)
    L.edges.argtypes = [ctypes.c_long] * 3 + [ctypes.c_int] * 2
    call.edges = lambda op, I, J, R: L.edges(I, J, R, *FORMS[op])
    return call


def test_pieces_come_from_the_shape_alone_and_fit_the_workspace(plan):
    rng = random.Random(3)
    for _ in range(20000):
        I, J, R = (int(2 ** rng.uniform(0, 13)) for _ in range(3))
        if rng.random() < 0.6:
            I, J, R = (max(8, n // 8 * 8) for n in (I, J, R))
        op, kt = rng.choice("fdw"), -(-R // 64)
        first = plan(op, I, J, R)
        own, splits, per, _, most, _, rows = first
        for aligned, lines in ((1, 1), (0, 0)):
            assert plan(op, I, J, R, aligned=aligned, lines=lines)[:3] == first[:3]
        assert 1 <= splits <= most and (splits - 1) * per < kt <= splits * per
        assert plan(op, I, J, R, ws=0)[1:3] == (1, kt)


def test_pieces_that_stay(plan):
    """A ReLU's results, forward products that may be a convolution's gathered window, weight gradients that may be a convolution's, pieces that are summed side by side."""
    assert plan("f", 1000, 600, 4000)[0] == 1 and plan("f", 1000, 600, 4000, relu=1)[0] == 0
    assert plan("f", 784, 512, 3456)[0] == 0 == plan("f", 200, 1000, 72 * 60)[0] and plan("f", 784, 512, 3464)[0] == 1 == plan("d", 784, 512, 3456)[0]
    assert plan("w", 512, 576, 2000)[0] == 0 and plan("w", 512, 584, 2000)[0] == 1
    assert plan("f", 256, 1024, 1024)[0] == 0 and plan("f", 256, 1056, 1024)[0] == 1


def test_pieces_fill_the_chip_once(plan):
    tile64, tile12864, tile128 = 1, 3, 0
    for op, I, J, R, want in (("f", 256, 1024, 8192, (8, 16, tile12864)), ("d", 256, 1024, 32768, (16, 32, tile128)), ("d", 768, 1024, 8192, (5, 26, tile128)), ("f", 512, 1024, 8192, (4, 32, tile12864)), ("f", 128, 4096, 4096, (4, 16, tile12864)),
                              ("f", 1000, 600, 4000, (3, 21, tile12864)), ("f", 694, 613, 1711, (2, 14, tile64)), ("d", 1610, 2163, 3908, (1, 62, tile128)), ("f", 768, 824, 768, (1, 12, tile64))):
        assert plan(op, I, J, R)[1:4] == want, (op, I, J, R, plan(op, I, J, R))


def test_the_forms_run_on_the_gpu(plan):
    from test_gpu_gemm_fp16_pieces import LONG, REPLANNED, THROUGH_REGISTERS
    seen = set()
    for op, I, J, R in REPLANNED:
        own, splits, per, tile, most, planned, rows = plan(op, I, J, R)
        assert own and per != planned, (op, I, J, R)
        seen.add((op, rows, tile, splits > 1))
    every = {(op, rows, tile, split) for op in "fdw" for rows in (0, 1) for tile in (0, 1, 3) for split in (False, True)}
    assert every - seen == {(op, rows, 0, True) for op in "fdw" for rows in (0, 1)}          # (over more than 2047 only: LONG)
    for op, I, J, R in THROUGH_REGISTERS:
        _, _, _, tile, _, _, rows = plan(op, I, J, R)
        assert tile == 3 and not rows, (op, I, J, R)
    assert {plan(*p)[6] for p in LONG if plan(*p)[3] == 0 and plan(*p)[1] > 1} == {0, 1}


def test_large_outputs_that_are_no_whole_tiles(plan):
    """More than half the chip's tiles of 256 x 256, and the rule stands where both sides were measured."""
    for op, I, J, R, want in (("f", 3000, 3000, 3000, 1), ("f", 2480, 3528, 2448, 1), ("d", 904, 9240, 3504, 1), ("w", 3616, 3504, 776, 1), ("f", 2112, 2696, 1376, 0), ("w", 848, 7712, 1728, 0),
                              ("d", 1304, 5160, 1040, 0), ("f", 1616, 5200, 168, 0), ("d", 4752, 4736, 240, 0), ("w", 3568, 10688, 176, 0), ("f", 2000, 3000, 1000, 0)):
        assert plan.edges(op, I, J, R) == want, (op, I, J, R)
    from test_gpu_gemm_edges import SIZES
    assert all(plan.edges(*s) for s in SIZES)
