"""With a workspace a product is summed in the pieces of the split reduction planned for its shape, whether the launch is split so
or not: an FP32 weight gradient must equal, bit for bit, the pieces computed one by one and added in order in FP32, and the
FP16 results must have the same bits at every alignment."""
import pytest
import torch

from paper_1710_03740_amd import binding as mpt

pytestmark = pytest.mark.gpu


# reductions of one to many pieces, with and without a ragged last stage; aligned, odd; a whole-tile output and ragged ones; then
# two for which a split into fewer partials than pieces looks the cheapest (16 pieces; 6 pieces of 2 stages) one for which tiles
# that the kernel does not cut do, and two whose partials are added up by more than 512 workgroups
@pytest.mark.parametrize("M,N,K", [(512, 264, 136), (256, 1024, 8192), (1000, 264, 136), (513, 263, 135), (130, 136, 264), (2048, 1024, 2048),
                                   (8192, 1024, 256), (714, 1157, 172), (2269, 991, 3139),
                                   (8192, 4096, 256), (8192, 1032, 1000)])
@pytest.mark.parametrize("accumulate", [False, True])
def test_fp32_sums_are_those_of_the_pieces(M, N, K, accumulate):
    need = mpt.mpt_gemm_workspace_bytes(mpt.OP_WGRAD, M, N, K)
    ws = torch.empty(need // 4, device="cuda") if need else None
    pieces, tiles = max(1, need // (4 * K * N)), -(-M // 64)
    rows = -(-tiles // pieces) * 64                                       # (for these sizes every piece but the last has so many)
    g = torch.Generator(device="cuda").manual_seed(M + N)
    x = torch.empty(M, K, device="cuda").normal_(generator=g).half()
    d = torch.empty(M, N, device="cuda").normal_(generator=g).half()
    start = torch.empty(K, N, device="cuda").normal_(generator=g) if accumulate else torch.zeros(K, N, device="cuda")
    dw = start.clone()
    mpt.mpt_gemm_wgrad(x, d, dw, accumulate=accumulate, ws=ws)
    total = None
    for r in range(0, M, rows):
        part = torch.empty(K, N, device="cuda")
        mpt.mpt_gemm_wgrad(x[r:r + rows].contiguous(), d[r:r + rows].contiguous(), part)
        total = part if total is None else total + part
    want = start + total if accumulate else total
    assert torch.equal(dw, want)
    exact = x.double().t() @ d.double() + start.double()
    assert ((dw.double() - exact).norm() / exact.norm()).item() < 5e-7


# A recurrent layer's projection (the input gradient, 256 x 1024 over 8192) and middle-sized products, with enough outputs that other
# sums show in some.  (Whole tiles of 128 x 256 at aligned addresses have unsplit launches of their own: its weight gradient is left out.)
@pytest.mark.parametrize("M,N,K", [(256, 8192, 1024), (608, 2392, 3528), (172, 1160, 712), (1000, 520, 2000)])
def test_results_do_not_depend_on_the_alignment(M, N, K):
    g = torch.Generator(device="cuda").manual_seed(M + N + K)
    x, w, d = (torch.empty(*s, device="cuda").normal_(generator=g).half() for s in ((M, K), (K, N), (M, N)))

    def window(t, pad, offset):
        rows, cols = t.shape
        v = torch.zeros(rows * (cols + pad) + offset, device="cuda", dtype=torch.float16)[offset:].view(rows, cols + pad)[:, :cols]
        return v.copy_(t)
    want = {}
    # whole cache lines where the sizes have them, whole 16-byte pieces, odd strides, odd addresses
    for pad, offset in ((0, 0), (8, 8), (1, 0), (3, 5)):
        X, W, D = (window(t, pad, offset) for t in (x, w, d))
        for name, op, shape, call in (("fwd", mpt.OP_FWD, (M, N), lambda o, ws: mpt.mpt_gemm_fwd(X, W, o, ws)), ("dgrad", mpt.OP_DGRAD, (M, K), lambda o, ws: mpt.mpt_gemm_dgrad(D, W, o, ws)),
                                      ("wgrad", mpt.OP_WGRAD, (K, N), lambda o, ws: mpt.mpt_gemm_wgrad(X, D, o, ws=ws))):
            if shape[0] % 128 == 0 and shape[1] % 256 == 0 and shape[0] > 256:
                continue
            need = mpt.mpt_gemm_workspace_bytes(op, M, N, K)
            out = torch.empty(shape, device="cuda", dtype=torch.float16)
            call(out, torch.empty(need // 4, device="cuda") if need else None)
            assert torch.equal(out, want.setdefault(name, out)), (name, pad, offset)


def gathered(x, sgn):
    """[pixels][tap][channel]: what tap 3 * tr + ts of the window multiplies, (y + sgn * (tr - 1), x + sgn * (ts - 1)) or zeros."""
    Nb, H, W, C = x.shape
    z = torch.zeros(Nb, H + 2, W + 2, C, device="cuda", dtype=x.dtype)
    z[:, 1:-1, 1:-1] = x
    at = [(1 + sgn * (t // 3 - 1), 1 + sgn * (t % 3 - 1)) for t in range(9)]
    return torch.stack([z[:, a:a + H, b:b + W] for a, b in at], 3).reshape(Nb * H * W, 9 * C)


# Every form of launch: forward and input gradient in tiles of 64 x 64 and 128 x 128, cut, split and whole, and of 256 x 64, split and whole; the
# weight gradient in 64 x 64, at most and more than 512 workgroups, and 128 x 128, each cut, split and whole (test_gemm_plan.py counts them)
CONVOLUTIONS = [(1, 3, 3, 8, 8), (1, 3, 3, 24, 8), (1, 3, 3, 64, 8), (1, 3, 3, 8, 24), (1, 3, 3, 8, 64), (1, 14, 14, 8, 8), (18, 5, 5, 8, 8), (16, 7, 7, 384, 512),
                (32, 28, 28, 128, 128), (128, 13, 13, 128, 72), (128, 13, 13, 72, 128), (1, 56, 56, 200, 72), (1, 56, 56, 72, 200), (8, 56, 56, 8, 72), (8, 56, 56, 72, 8),
                (64, 13, 13, 192, 8), (64, 13, 13, 8, 192), (16, 56, 56, 8, 8), (4, 56, 56, 136, 72), (16, 9, 9, 1000, 384), (1, 14, 14, 768, 1000),
                (51, 7, 7, 712, 8), (12, 9, 9, 888, 264), (1, 3, 3, 912, 200)]


@pytest.mark.parametrize("Nb,H,W,C,Kf", CONVOLUTIONS)
@pytest.mark.parametrize("split", [False, True])
def test_convolutions_are_the_products_of_the_gathered_window(Nb, H, W, C, Kf, split):
    """The same sums in the same pieces, so the same bits."""
    g = torch.Generator(device="cuda").manual_seed(Nb + H + C + Kf)
    x, w, dy = (torch.empty(*s, device="cuda").normal_(generator=g).half() for s in ((Nb, H, W, C), (Kf, 3, 3, C), (Nb, H, W, Kf)))
    P = Nb * H * W

    def ws(need):
        return torch.empty(need // 4, device="cuda") if split and need else None
    for op, out, conv, plain, A, B, MNK in (
            (mpt.OP_FWD, torch.empty_like(dy), lambda o, s: mpt.mpt_conv3x3_fwd(x, w, o, s), mpt.mpt_gemm_fwd, gathered(x, 1), w.view(Kf, 9 * C).t().contiguous(), (P, Kf, 9 * C)),
            (mpt.OP_DGRAD, torch.empty_like(x), lambda o, s: mpt.mpt_conv3x3_dgrad(dy, w, o, s), mpt.mpt_gemm_fwd, gathered(dy, -1),
             w.view(Kf, 9, C).transpose(0, 1).reshape(9 * Kf, C), (P, C, 9 * Kf)),
            (mpt.OP_WGRAD, torch.empty_like(w), lambda o, s: mpt.mpt_conv3x3_wgrad(x, dy, o, ws=s), mpt.mpt_gemm_wgrad, dy.view(P, Kf), gathered(x, 1), (P, 9 * C, Kf))):
        print(op, (Nb, H, W, C, Kf), split, flush=True)
        conv(out, ws(mpt.mpt_conv3x3_workspace_bytes(op, Nb, H, W, C, Kf)))
        want = torch.empty(out.numel(), device="cuda", dtype=torch.float16).view(*((Kf, 9 * C) if op == mpt.OP_WGRAD else MNK[:2]))
        plain(A, B, want, ws=ws(mpt.mpt_gemm_workspace_bytes(mpt.OP_WGRAD if op == mpt.OP_WGRAD else mpt.OP_FWD, *MNK)))
        assert torch.equal(out.view_as(want), want), op
