"""The ring and any-alignment GEMM kernels at the sizes where a tile, a stage or a 16-byte piece ends.

Operands are -1, 0 or 1, so every partial sum is a whole number below 2^11 and exact in FP32 and FP16: the results must equal
the matrix product exactly, whatever the order of the sums.  Operands are windows of buffers filled with NaN (a read outside a window that reaches
a result shows), outputs windows of buffers whose surroundings must stay as they were."""
import numpy as np
import pytest
import torch

from oracle import conv, fp16
from paper_1710_03740_amd import binding as mpt
from gpu_util import dev16, host, host16

pytestmark = pytest.mark.gpu

# (M, N, K): below, at and above tiles of 64 and 128, stages of 64 and pieces of 8
SIZES = [(1, 8, 8), (7, 3, 5), (63, 72, 200), (64, 64, 64), (65, 136, 72), (127, 129, 191), (128, 192, 256), (200, 56, 1000),
         (65, 63, 509), (520, 2000, 1992), (2056, 1544, 520), (3001, 3003, 517)]
# row padding in elements and offset of the window's first element: whole 16-byte pieces; odd strides; odd bases
LAYOUTS = [(0, 0), (8, 0), (8, 16), (1, 0), (3, 5)]


def window(rows, cols, pad, offset, values=None, dtype=torch.float16):
    ld = cols + pad
    buf = torch.full((rows * ld + offset + 64,), float("nan"), dtype=dtype, device="cuda")
    view = buf[offset:offset + rows * ld].view(rows, ld)[:, :cols]
    if values is not None:
        view.copy_(dev16(values) if values.dtype == np.float16 else torch.from_numpy(values).cuda())
    return buf, view


def outside_untouched(buf, view):
    inside = torch.zeros_like(buf, dtype=torch.bool)
    inside.as_strided(view.shape, view.stride(), view.storage_offset()).fill_(True)
    return bool(torch.isnan(buf[~inside]).all())


def ws_for(op, M, N, K):
    need = mpt.mpt_gemm_workspace_bytes(op, M, N, K)
    return torch.empty(need // 4, dtype=torch.float32, device="cuda") if need else None


@pytest.mark.parametrize("pad,offset", LAYOUTS)
@pytest.mark.parametrize("M,N,K", SIZES)
def test_edges_of_tiles_stages_and_pieces(M, N, K, pad, offset):
    if M > 1000 and (pad, offset) not in ((0, 0), (3, 5)):
        pytest.skip("the large sizes are there for their tiles: two layouts do")
    rng = np.random.default_rng(M + 3 * N + 7 * K + pad)
    X, W, G, H = (rng.integers(-1, 2, s).astype(np.float16) for s in ((M, K), (K, N), (M, N), (M, K)))
    x, w, g, h = (window(*a.shape, pad, offset, a)[1] for a in (X, W, G, H))
    X, W, G = (a.astype(np.float64) for a in (X, W, G))
    want = {"fwd": X @ W, "dgrad": G @ W.T, "wgrad": X.T @ G}
    for split in (False, True):
        def run(name, op, shape, call, expect):
            print(name, (M, N, K), (pad, offset), split, flush=True)
            buf, out = window(*shape, pad, offset)
            call(out, ws_for(op, M, N, K) if split else None)
            assert np.array_equal(host16(out.contiguous()).astype(np.float64), expect), name
            assert outside_untouched(buf, out), name
        run("fwd", 0, (M, N), lambda o, ws: mpt.mpt_gemm_fwd(x, w, o, ws), want["fwd"])
        run("fwd relu", 0, (M, N), lambda o, ws: mpt.mpt_gemm_fwd_relu(x, w, o, ws), np.maximum(want["fwd"], 0))
        run("dgrad", 1, (M, K), lambda o, ws: mpt.mpt_gemm_dgrad(g, w, o, ws), want["dgrad"])
        run("dgrad relu", 1, (M, K), lambda o, ws: mpt.mpt_gemm_dgrad_relu(g, w, h, o, ws), np.where(H > 0, want["dgrad"], 0))
        flag = torch.zeros(1, dtype=torch.int32, device="cuda")
        run("wgrad", 2, (K, N), lambda o, ws: mpt.mpt_gemm_wgrad(x, g, o, flag=flag, ws=ws), want["wgrad"])
        assert int(flag.item()) == 0
        buf, out = window(K, N, pad, offset, dtype=torch.float32)
        mpt.mpt_gemm_wgrad(x, g, out, flag=flag, ws=ws_for(2, M, N, K) if split else None)
        mpt.mpt_gemm_wgrad(x, g, out, accumulate=True, flag=flag, ws=ws_for(2, M, N, K) if split else None)
        assert np.array_equal(host(out.contiguous()).astype(np.float64), 2 * want["wgrad"]) and outside_untouched(buf, out)
        assert int(flag.item()) == 0


# Products (pass, M, N, K, with workspace) for the forms of launch that the planner chooses: operands in whole pieces (sizes are multiples of 8) and through
# registers, tiles, two or four slots, split, cut and whole; some now sum their pieces side by side, and RING_FORMS of test_gpu_gemm_pieces.py stands in for them
FORMS = [("d", 577, 1549, 839, 1), ("d", 1415, 265, 2123, 0), ("d", 9, 211, 9, 1), ("d", 9, 329, 9, 1), ("d", 9, 9, 9, 0), ("d", 8048, 200, 800, 1),
         ("d", 672, 5904, 784, 1), ("d", 2888, 136, 2120, 0), ("d", 2336, 1488, 1040, 1), ("d", 776, 3104, 592, 1), ("d", 1168, 720, 2232, 0),
         ("d", 2888, 976, 1520, 1), ("d", 368, 2048, 648, 1), ("d", 136, 8, 11040, 0), ("d", 776, 216, 1328, 1), ("d", 344, 1320, 392, 1),
         ("d", 136, 8, 7768, 0), ("d", 8, 200, 8, 1), ("d", 8, 720, 8, 1), ("d", 8, 8, 8, 0), ("f", 691, 647, 1563, 1), ("f", 2151, 1477, 261, 0),
         ("f", 9, 9, 193, 1), ("f", 9, 11, 323, 1), ("f", 9, 9, 9, 0), ("f", 1824, 4040, 272, 1), ("f", 1040, 552, 5344, 1), ("f", 664, 8200, 144, 0),
         ("f", 2160, 1168, 1504, 1), ("f", 400, 968, 3144, 1), ("f", 1168, 2336, 656, 0), ("f", 2024, 2088, 1032, 1), ("f", 680, 392, 2120, 1),
         ("f", 11072, 144, 8, 0), ("f", 928, 1120, 208, 1), ("f", 368, 440, 1288, 1), ("f", 136, 7800, 8, 0), ("f", 8, 8, 200, 1), ("f", 8, 8, 712, 1),
         ("f", 8, 8, 8, 0), ("w", 1549, 647, 655, 1), ("w", 199, 1749, 1891, 0), ("w", 193, 9, 9, 1), ("w", 351, 9, 9, 1), ("w", 9, 9, 9, 0),
         ("w", 224, 1888, 3920, 1), ("w", 5832, 592, 840, 1), ("w", 144, 5568, 1048, 0), ("w", 1520, 1088, 2096, 1), ("w", 3304, 680, 704, 1),
         ("w", 712, 1688, 1552, 0), ("w", 1032, 3264, 1184, 1), ("w", 2024, 736, 328, 1), ("w", 8, 11056, 136, 0), ("w", 208, 984, 1088, 1),
         ("w", 1304, 328, 424, 1), ("w", 8, 136, 7992, 0), ("w", 200, 8, 8, 1), ("w", 720, 8, 8, 1), ("w", 8, 8, 8, 0)]


# And one for each instance through registers, or form of its launch, that neither those nor the edge tests reach: tiles, wavefronts, split, cut and whole, edges read
# over, operands apart, rows of fewer than 8 elements, in four wavefronts beside other workgroups and in eight alone (test_gemm_plan.py counts them)
INSTANCES = [("d", 590, 621, 449, 1), ("d", 771, 4059, 827, 1), ("d", 1048, 9, 6819, 0), ("d", 6857, 3, 1027, 0), ("f", 33, 5, 1293, 1), ("f", 70, 203, 2100, 1),
             ("f", 300, 5, 1173, 1), ("f", 352, 321, 2302, 1), ("f", 424, 594, 613, 1), ("f", 538, 921, 1640, 1), ("f", 898, 4144, 1505, 0), ("f", 1001, 1999, 1503, 1),
             ("f", 1054, 3264, 1313, 1), ("f", 1080, 283, 6950, 1), ("f", 1419, 4975, 3, 1), ("f", 2305, 264, 3827, 1), ("f", 2511, 1538, 1417, 0), ("f", 3005, 722, 271, 0),
             ("f", 4968, 1415, 11, 1), ("w", 5, 2508, 2823, 1), ("w", 194, 781, 1280, 1), ("w", 258, 1485, 3449, 0), ("w", 265, 387, 7085, 1), ("w", 272, 645, 778, 1),
             ("w", 321, 65, 130, 0), ("w", 821, 5, 300, 1), ("w", 901, 37, 5, 1), ("w", 2064, 38, 49, 1), ("w", 2386, 322, 326, 1), ("w", 4356, 774, 790, 1)]


@pytest.mark.parametrize("op,M,N,K,split", FORMS + INSTANCES)
def test_every_form_of_launch(op, M, N, K, split):
    g = torch.Generator(device="cuda").manual_seed(M + 3 * N + 7 * K)
    shapes = {"f": ((M, K), (K, N)), "d": ((M, N), (K, N)), "w": ((M, K), (M, N))}[op]
    a, b = (torch.randint(-1, 2, s, device="cuda", generator=g).half() for s in shapes)
    x, y = a.double(), b.double()
    want = {"f": lambda: x @ y, "d": lambda: x @ y.t(), "w": lambda: x.t() @ y}[op]()
    run = {"f": mpt.mpt_gemm_fwd, "d": mpt.mpt_gemm_dgrad, "w": mpt.mpt_gemm_wgrad}[op]
    for dtype in (torch.float16, torch.float32) if op == "w" else (torch.float16,):
        buf, out = window(*want.shape, 8, 16, dtype=dtype)
        print("form", op, (M, N, K), split, dtype, flush=True)
        run(a, b, out, ws=ws_for("fdw".index(op), M, N, K) if split else None)
        assert torch.equal(out.double(), want) and outside_untouched(buf, out)


@pytest.mark.parametrize("pad", [0, 1])
def test_special_values_stay_in_their_rows_and_columns(pad):
    """Pieces read past a ragged edge must not carry an Inf or NaN of one row or column into others."""
    M, N, K = 130, 72 + pad, 136 + pad
    X, W = np.ones((M, K), np.float16), np.ones((K, N), np.float16)
    X[M - 1, K - 1] = np.inf
    W[K - 1, N - 1] = np.nan
    y = torch.empty((M, N), dtype=torch.float16, device="cuda")
    mpt.mpt_gemm_fwd(dev16(X), dev16(W), y)
    got = host16(y)
    assert np.isnan(got[:, N - 1]).all()
    assert np.isinf(got[M - 1, :N - 1]).all()
    assert (got[:M - 1, :N - 1] == K).all()
    flag = torch.zeros(1, dtype=torch.int32, device="cuda")
    dw = torch.empty((K, N), dtype=torch.float16, device="cuda")
    G = np.ones((M, N), np.float16)
    mpt.mpt_gemm_wgrad(dev16(X), dev16(G), dw, flag=flag)
    got = host16(dw)
    assert np.isinf(got[K - 1]).all() and (got[:K - 1] == M).all() and int(flag.item()) == 1


# channel counts below, at and between the stages of 64; output columns around the tiles; images smaller than a stage and wider
@pytest.mark.parametrize("Nb,H,W,C,Kf", [(1, 3, 3, 8, 64), (2, 5, 70, 8, 72), (1, 1, 65, 16, 24), (3, 9, 1, 40, 136), (2, 7, 7, 64, 64), (2, 8, 6, 72, 200),
                                         (1, 13, 13, 192, 56), (4, 14, 14, 128, 64)])
def test_convolution_edges(Nb, H, W, C, Kf):
    rng = np.random.default_rng(Nb + H + W + C + Kf)
    x, w, dy = (rng.integers(-1, 2, s).astype(np.float16) for s in ((Nb, H, W, C), (Kf, 3, 3, C), (Nb, H, W, Kf)))
    d_x, d_w, d_dy = dev16(x), dev16(w), dev16(dy)
    want = (conv.conv3x3_fwd(x, w)[0], conv.conv3x3_dgrad(dy, w)[0], conv.conv3x3_wgrad(x, dy)[0])
    for split in (False, True):
        for op, shape, call in ((0, (Nb, H, W, Kf), lambda o, ws: mpt.mpt_conv3x3_fwd(d_x, d_w, o, ws)), (1, (Nb, H, W, C), lambda o, ws: mpt.mpt_conv3x3_dgrad(d_dy, d_w, o, ws)),
                                (2, (Kf, 3, 3, C), lambda o, ws: mpt.mpt_conv3x3_wgrad(d_x, d_dy, o, ws=ws))):
            need = mpt.mpt_conv3x3_workspace_bytes(op, Nb, H, W, C, Kf) if split else 0
            out = torch.full(shape, float("nan"), dtype=torch.float16, device="cuda")
            print("conv", op, (Nb, H, W, C, Kf), split, flush=True)
            call(out, torch.empty(need // 4, dtype=torch.float32, device="cuda") if need else None)
            got = host16(out)
            assert np.array_equal(got.astype(np.float64), want[op].astype(np.float64)), (op, split)      # (a zero may carry either sign)


# The weight gradient's 128 x 128 tile (test_gemm_plan.py holds the planner to it): split with the workspace, cut, and whole; a ragged last tile
# of output channels, of window columns and of pixels, and images whose rows a stage crosses once or many times
@pytest.mark.parametrize("Nb,H,W,C,Kf", [(4, 56, 56, 136, 72), (16, 9, 9, 1000, 384), (1, 14, 14, 768, 1000)])
def test_convolution_weight_gradient_in_wide_tiles(Nb, H, W, C, Kf):
    rng = np.random.default_rng(Nb + H + W + C + Kf)
    x, dy = (rng.integers(-1, 2, s).astype(np.float16) for s in ((Nb, H, W, C), (Nb, H, W, Kf)))
    want = conv.conv3x3_wgrad(x, dy)[0].astype(np.float64)
    d_x, d_dy = dev16(x), dev16(dy)
    need = mpt.mpt_conv3x3_workspace_bytes(2, Nb, H, W, C, Kf)
    flag = torch.zeros(1, dtype=torch.int32, device="cuda")
    for ws in (None, torch.empty(need // 4, dtype=torch.float32, device="cuda") if need else None):
        out = torch.full((Kf, 3, 3, C), float("nan"), dtype=torch.float16, device="cuda")
        print("conv weight gradient", (Nb, H, W, C, Kf), ws is not None, flush=True)
        mpt.mpt_conv3x3_wgrad(d_x, d_dy, out, flag=flag, ws=ws)
        assert np.array_equal(host16(out).astype(np.float64), want) and int(flag.item()) == 0


@pytest.mark.parametrize("ld", [1 << 21, (1 << 21) + 1])
def test_rows_too_far_apart_for_32_bit_offsets(ld):
    """Row strides from which the kernels form whole 64-bit addresses, aligned and odd, with ragged last stages and tiles."""
    rng = np.random.default_rng(ld)
    M, N, K = 70, 72, 136
    X, W, G = (rng.integers(-1, 2, s).astype(np.float16) for s in ((M, K), (K, N), (M, N)))
    x, w, g = (window(*a.shape, ld - a.shape[1], 0, a)[1] for a in (X, W, G))
    X, W, G = (a.astype(np.float64) for a in (X, W, G))
    for shape, call, want in (((M, N), lambda o: mpt.mpt_gemm_fwd(x, w, o), X @ W), ((M, K), lambda o: mpt.mpt_gemm_dgrad(g, w, o), G @ W.T),
                              ((K, N), lambda o: mpt.mpt_gemm_wgrad(x, g, o), X.T @ G)):
        print("far apart", ld, shape, flush=True)
        _, out = window(*shape, ld - shape[1], 0)
        call(out)
        assert np.array_equal(host16(out.contiguous()).astype(np.float64), want)


# (forward or input gradient, M, N, K): three and four workgroups on the busiest CU over reductions that are long enough for the operands
# to be fetched one after the other, whose last stage holds one element, all but one or about half of them, with the sums whole and in pieces
# (test_gemm_plan.py checks that they are of this kind)
APART = [("f", 2047, 2003, 1281), ("f", 1999, 1921, 1279), ("d", 1921, 1345, 2001), ("d", 1473, 2049, 1409), ("d", 1475, 2111, 1409)]


@pytest.mark.parametrize("op,M,N,K", APART)
@pytest.mark.parametrize("split", [False, True])
def test_operands_fetched_one_after_the_other(op, M, N, K, split):
    gen = torch.Generator(device="cuda").manual_seed(M)
    ints = lambda *s: torch.randint(-1, 2, s, device="cuda", generator=gen).to(torch.float16)  # noqa: E731
    print(op, (M, N, K), split, flush=True)
    w = ints(K, N)
    if op == "f":
        x, out = ints(M, K), torch.empty(M, N, device="cuda", dtype=torch.float16)
        mpt.mpt_gemm_fwd(x, w, out, ws_for(0, M, N, K) if split else None)
        want = x.float() @ w.float()
    else:
        g, out = ints(M, N), torch.empty(M, K, device="cuda", dtype=torch.float16)
        mpt.mpt_gemm_dgrad(g, w, out, ws_for(1, M, N, K) if split else None)
        want = g.float() @ w.float().t()
    assert torch.equal(out.float(), want)
