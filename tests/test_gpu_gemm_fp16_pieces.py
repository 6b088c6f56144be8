"""FP16 results in the pieces that fp16_plan (csrc/gemm_plan.h) chooses, and the 128 x 64 tiles of operands through registers: every tile that it takes, unsplit and
split, in each pass, on whole 16-byte pieces and on others.  Operands of -1, 0 and 1 over at most 2047 have exact sums in any order."""
import pytest
import torch

from paper_1710_03740_amd import binding as mpt
from test_gpu_gemm_ring import test_every_form_of_launch as check_form, ws_for

pytestmark = pytest.mark.gpu

# (pass, output rows, columns, reduction): the smallest of three million products in each tile, unsplit and split, aligned (the first of a line) and odd
REPLANNED = [("f", 2080, 1032, 1488), ("f", 1033, 2049, 1509), ("f", 2072, 232, 200), ("f", 324, 1516, 193), ("f", 8, 2064, 2000), ("f", 2077, 1, 1411),
             ("f", 712, 1368, 200), ("f", 898, 1940, 258), ("f", 1808, 136, 1568), ("f", 1997, 130, 1453),
             ("d", 2064, 1032, 1488), ("d", 1802, 1817, 977), ("d", 1263, 389, 200), ("d", 289, 1716, 196), ("d", 2064, 104, 1096), ("d", 5, 2059, 1836),
             ("d", 2072, 456, 200), ("d", 1612, 1089, 260), ("d", 1840, 136, 1560), ("d", 2029, 129, 1418),
             ("w", 1032, 2064, 1480), ("w", 2049, 1028, 1480), ("w", 1816, 272, 200), ("w", 1832, 259, 204), ("w", 2056, 8, 1848), ("w", 2063, 1, 1933),
             ("w", 1624, 592, 200), ("w", 963, 1793, 259), ("w", 136, 1816, 1672), ("w", 1937, 135, 1425)]
# 128 x 64 tiles through registers by four and by eight wavefronts, edges shifted and read over
THROUGH_REGISTERS = [("f", 1364, 2194, 65), ("f", 2436, 1537, 263), ("f", 1921, 928, 259), ("f", 2957, 577, 261), ("f", 2997, 72, 1445), ("f", 2958, 65, 1298),
                     ("d", 1366, 2223, 65), ("d", 2436, 709, 259), ("d", 2992, 65, 1286),
                     ("w", 1391, 2184, 65), ("w", 2696, 1411, 259), ("w", 1824, 1007, 261), ("w", 1795, 963, 259), ("w", 1847, 136, 1737), ("w", 2152, 65, 1966)]


def mnk(op, I, J, R):
    return {"f": (I, J, R), "d": (I, R, J), "w": (R, J, I)}[op]


@pytest.mark.parametrize("op,I,J,R", REPLANNED + THROUGH_REGISTERS)
def test_every_form(op, I, J, R):
    check_form(op, *mnk(op, I, J, R), True)


# (the last two in split 128 x 128 tiles)
LONG = [("f", 2080, 1032, 1488), ("f", 1808, 136, 1568), ("d", 2064, 104, 1096), ("d", 256, 1024, 8192), ("w", 2056, 8, 1848), ("w", 136, 1816, 1672),
        ("d", 256, 1024, 32768), ("w", 2673, 434, 3297)]


@pytest.mark.parametrize("op,I,J,R", LONG)
def test_the_pieces_do_not_depend_on_the_alignment(op, I, J, R):
    """The same bits from rows of whole cache lines, whole 16-byte pieces, odd strides and odd addresses; and within one FP16 step of the exact result where that is at
    least 2^-6 of its terms' sum (FP32 chains of up to 2^13 terms are off by less than 2^13 * 2^-24 = 2^-11 of it)."""
    M, N, K = mnk(op, I, J, R)
    gen = torch.Generator(device="cuda").manual_seed(I + J + R)
    a, b = (torch.empty(*s, device="cuda").normal_(generator=gen).half() for s in {"f": ((M, K), (K, N)), "d": ((M, N), (K, N)), "w": ((M, K), (M, N))}[op])
    call = {"f": mpt.mpt_gemm_fwd, "d": mpt.mpt_gemm_dgrad, "w": mpt.mpt_gemm_wgrad}[op]
    want = None
    for pad, offset in ((0, 0), (8, 8), (1, 0), (3, 5)):
        x, y = (torch.zeros(t.shape[0] * (t.shape[1] + pad) + offset, device="cuda", dtype=torch.float16)[offset:].view(t.shape[0], t.shape[1] + pad)[:, :t.shape[1]].copy_(t)
                for t in (a, b))
        out = torch.empty(I, J, device="cuda", dtype=torch.float16)
        print("alignment", op, (I, J, R), (pad, offset), flush=True)
        call(x, y, out, ws=ws_for("fdw".index(op), M, N, K))
        want = out if want is None else want
        assert torch.equal(out, want), (pad, offset)
    p, q = {"f": (a, b), "d": (a, b.t()), "w": (a.t(), b)}[op]
    p, q = p.double(), q.double()
    exact, terms = p @ q, p.abs() @ q.abs()
    well = exact.abs() >= terms / 64
    step = torch.exp2(torch.floor(torch.log2(exact.abs().clamp(min=2.0 ** -14))) - 10)
    assert ((want.double() - exact).abs() <= step)[well].all() and well.any()


@pytest.mark.parametrize("op,I,J,R", [("f", 1364, 2194, 65), ("w", 1391, 2184, 65)])
def test_strides_beyond_32_bit_offsets(op, I, J, R):
    """One operand of few rows, 4 MiB apart."""
    M, N, K = mnk(op, I, J, R)
    gen = torch.Generator(device="cuda").manual_seed(I)
    a, b = (torch.randint(-1, 2, s, device="cuda", generator=gen).half() for s in {"f": ((M, K), (K, N)), "w": ((M, K), (M, N))}[op])
    far = torch.empty(R, (1 << 21) + 8, device="cuda", dtype=torch.float16)[:, :b.shape[1]].copy_(b)
    out = torch.empty(I, J, device="cuda", dtype=torch.float16)
    (mpt.mpt_gemm_fwd if op == "f" else mpt.mpt_gemm_wgrad)(a, far, out, ws=ws_for("fdw".index(op), M, N, K))
    assert torch.equal(out.double(), (a.double() @ b.double() if op == "f" else a.double().t() @ b.double()))
