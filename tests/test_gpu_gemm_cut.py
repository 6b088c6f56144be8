"""With a workspace a product is summed in the pieces of the split reduction planned for its shape, whether the launch is split so
or not: an FP32 weight gradient must equal, bit for bit, the pieces computed one by one and added in order in FP32, and the
FP16 results must have the same bits at every alignment."""
import pytest
import torch

from paper_1710_03740_amd import binding as mpt

pytestmark = pytest.mark.gpu


# reductions of one to many pieces, with and without a ragged last stage; aligned, odd; a whole-tile output and ragged ones; then
# two for which a split into fewer partials than pieces looks the cheapest (16 pieces; 6 pieces of 2 stages) and one for which tiles
# that the kernel does not cut do
@pytest.mark.parametrize("M,N,K", [(512, 264, 136), (256, 1024, 8192), (1000, 264, 136), (513, 263, 135), (130, 136, 264), (2048, 1024, 2048),
                                   (8192, 1024, 256), (714, 1157, 172), (2269, 991, 3139)])
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
