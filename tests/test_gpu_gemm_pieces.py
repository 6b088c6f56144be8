"""Products of few tiles whose pieces are summed side by side (k_gemm_pieces), at the edges of its tiles, stages, pieces and stores, and the
ring kernels' forms at sizes that still reach them.  Operands of -1, 0 and 1 have exact sums in any order; windows as in test_gpu_gemm_ring.py.
That the bits are those of the pieces added in order is checked here for FP16 results, in test_gpu_gemm_cut.py for FP32 weight gradients."""
import numpy as np
import pytest
import torch

from paper_1710_03740_amd import binding as mpt
from gpu_util import host, host16
from test_gpu_gemm_ring import outside_untouched, window, ws_for

pytestmark = pytest.mark.gpu

# (M, N, K): forward, input and weight gradient of each reduce over K, N, M.  2 .. 8 pieces, so four and eight wavefronts; rows and columns below, at and
# above a tile of 32; last columns of 1, 2 and 3; a last piece shorter than the others; rows of fewer than 8 elements
SIZES = [(129, 33, 31), (256, 10, 1024), (31, 257, 192), (33, 323, 130), (64, 512, 512), (1000, 24, 264), (97, 1100, 1030), (200, 2048, 40), (300, 5, 387),
         (190, 3, 7), (1, 1536, 1), (1280, 34, 1023), (500, 100, 1408), (200, 40, 1024), (640, 33, 100)]
LAYOUTS = [(0, 0), (8, 16), (1, 0), (3, 5)]


@pytest.mark.parametrize("pad,offset", LAYOUTS)
@pytest.mark.parametrize("M,N,K", SIZES)
def test_edges(M, N, K, pad, offset):
    rng = np.random.default_rng(M + 3 * N + 7 * K + pad)
    X, W, G, H = (rng.integers(-1, 2, s).astype(np.float16) for s in ((M, K), (K, N), (M, N), (M, K)))
    x, w, g, h = (window(*a.shape, pad, offset, a)[1] for a in (X, W, G, H))
    X, W, G = (a.astype(np.float64) for a in (X, W, G))
    y, dx, dw = X @ W, G @ W.T, X.T @ G
    flag = torch.zeros(1, dtype=torch.int32, device="cuda")
    for name, op, want, call in (("fwd", 0, y, lambda o, ws: mpt.mpt_gemm_fwd(x, w, o, ws)), ("fwd relu", 0, np.maximum(y, 0), lambda o, ws: mpt.mpt_gemm_fwd_relu(x, w, o, ws)),
                                 ("dgrad", 1, dx, lambda o, ws: mpt.mpt_gemm_dgrad(g, w, o, ws)), ("dgrad relu", 1, np.where(H > 0, dx, 0), lambda o, ws: mpt.mpt_gemm_dgrad_relu(g, w, h, o, ws)),
                                 ("wgrad", 2, dw, lambda o, ws: mpt.mpt_gemm_wgrad(x, g, o, flag=flag, ws=ws))):
        print(name, (M, N, K), (pad, offset), flush=True)
        buf, out = window(*want.shape, pad, offset)
        call(out, ws_for(op, M, N, K))
        assert np.array_equal(host16(out.contiguous()).astype(np.float64), want), name
        assert outside_untouched(buf, out), name
    buf, out = window(K, N, pad, offset, dtype=torch.float32)
    mpt.mpt_gemm_wgrad(x, g, out, flag=flag, ws=ws_for(2, M, N, K))
    mpt.mpt_gemm_wgrad(x, g, out, accumulate=True, flag=flag, ws=ws_for(2, M, N, K))
    assert np.array_equal(host(out.contiguous()).astype(np.float64), 2 * dw) and outside_untouched(buf, out)
    assert int(flag.item()) == 0


# (output rows, columns, reduction), forward and input gradient: two, three, four, five, seven and eight pieces, with and without a ragged last stage; whole 16-byte
# pieces where the sizes have them (test_gemm_plan.py checks that all take this route, at both numbers of wavefronts)
ORDERED = [(256, 10, 1024), (256, 1000, 1024), (100, 72, 1280), (40, 1000, 264), (300, 200, 424), (65, 63, 509), (264, 40, 640), (33, 35, 899), (31, 130, 1215)]


@pytest.mark.parametrize("odd", [False, True])
@pytest.mark.parametrize("I,J,R", ORDERED)
def test_fp16_results_are_the_pieces_added_in_order(I, J, R, odd):
    """Bit for bit: each planned piece as an FP32 product of its own (a weight gradient of the transposed operands, in one chain), added in FP32 and rounded once."""
    gen = torch.Generator(device="cuda").manual_seed(I + 3 * J + 7 * R)
    a, b = torch.empty(I, R, device="cuda").normal_(generator=gen).half(), torch.empty(R, J, device="cuda").normal_(generator=gen).half()
    h = torch.empty(I, J, device="cuda").normal_(generator=gen).half()
    pieces, total = mpt.mpt_gemm_workspace_bytes(mpt.OP_FWD, I, J, R) // (4 * I * J), None
    rows = -(-(-(-R // 64)) // pieces) * 64
    for r in range(0, R, rows):
        part = torch.empty(I, J, device="cuda")
        mpt.mpt_gemm_wgrad(a[:, r:r + rows].t().contiguous(), b[r:r + rows].contiguous(), part)
        total = part if total is None else total + part
    assert pieces >= 2 and -(-R // rows) == pieces
    want = total.half()

    def view(t):
        return window(*t.shape, int(odd), 0, host16(t.contiguous()))[1]
    x, w, g, wt, mask = view(a), view(b), view(a), view(b.t()), view(h)
    for name, op, expect, call in (("fwd", 0, want, lambda o, ws: mpt.mpt_gemm_fwd(x, w, o, ws)), ("fwd relu", 0, want.clamp(min=0), lambda o, ws: mpt.mpt_gemm_fwd_relu(x, w, o, ws)),
                                   ("dgrad", 1, want, lambda o, ws: mpt.mpt_gemm_dgrad(g, wt, o, ws)),
                                   ("dgrad relu", 1, torch.where(h > 0, want, torch.zeros_like(want)), lambda o, ws: mpt.mpt_gemm_dgrad_relu(g, wt, mask, o, ws))):
        print("in order", name, (I, J, R), odd, flush=True)
        ws = ws_for(op, *((I, J, R) if op == 0 else (I, R, J)))
        assert ws.numel() == pieces * I * J
        ws.fill_(float("nan"))
        out = torch.empty(I, J, device="cuda", dtype=torch.float16)
        call(out, ws)
        assert torch.isnan(ws).all()                                     # one launch, no partials
        assert torch.equal(out, expect), name


def test_strides_beyond_32_bit_offsets():
    M, N, K = 40, 70, 260
    ld = (1 << 21) + 8
    g = torch.Generator(device="cuda").manual_seed(1)
    x = torch.zeros(M, ld, device="cuda", dtype=torch.float16)[:, :K]
    x.copy_(torch.randint(-1, 2, (M, K), device="cuda", generator=g))
    w = torch.randint(-1, 2, (K, N), device="cuda", generator=g).half()
    y = torch.empty(M, N, device="cuda", dtype=torch.float16)
    mpt.mpt_gemm_fwd(x, w, y, ws_for(0, M, N, K))
    assert torch.equal(y.double(), x.double() @ w.double())


@pytest.mark.parametrize("where", [0, 30, 31])
@pytest.mark.parametrize("dtype", [torch.float16, torch.float32])
def test_a_special_value_is_seen_where_it_is_stored(where, dtype):
    """31 columns: the last three go out one by one."""
    x, g = torch.ones(200, 31, device="cuda").half(), torch.ones(200, 31, device="cuda").half()
    flag = torch.zeros(1, dtype=torch.int32, device="cuda")
    out = torch.empty(31, 31, device="cuda", dtype=dtype)
    if where < 31:
        g[100, where] = float("inf")
    mpt.mpt_gemm_wgrad(x, g, out, flag=flag, ws=ws_for(2, 200, 31, 31))
    assert int(flag.item()) == (where < 31)
    assert torch.isinf(out).any(0).tolist() == [k == where for k in range(31)]


# the ring kernels' split and cut launches of 64 x 64 and 128 x 64 tiles, at sizes beyond those that k_gemm_pieces takes, and two with ragged edges over many
# stages (test_gemm_plan.py counts them)
RING_FORMS = [("d", 1288, 197, 400, 1), ("d", 8, 1734, 8, 1), ("d", 856, 200, 592, 1), ("d", 8, 2064, 8, 1), ("d", 344, 2280, 656, 1), ("d", 680, 2344, 136, 1),
              ("f", 459, 1090, 196, 1), ("f", 9, 10, 1546, 1), ("f", 752, 680, 208, 1), ("f", 8, 8, 2184, 1), ("f", 136, 672, 2296, 1), ("w", 206, 295, 1776, 1),
              ("w", 1350, 8, 10, 1), ("w", 216, 720, 720, 1), ("w", 1936, 8, 8, 1), ("w", 1856, 272, 408, 1), ("f", 885, 586, 267, 1), ("w", 2130, 387, 981, 1)]


@pytest.mark.parametrize("op,M,N,K,split", RING_FORMS)
def test_ring_forms_beside_them(op, M, N, K, split):
    from test_gpu_gemm_ring import test_every_form_of_launch
    test_every_form_of_launch(op, M, N, K, split)
