"""An FP32 weight gradient computed in one launch keeps the pieces that the split reduction of its workspace size sums it in: it
must equal, bit for bit, the pieces computed one by one and added in order in FP32."""
import pytest
import torch

from paper_1710_03740_amd import binding as mpt

pytestmark = pytest.mark.gpu


# reductions of one to many pieces, with and without a ragged last stage; aligned, odd; a whole-tile output and ragged ones
@pytest.mark.parametrize("M,N,K", [(512, 264, 136), (256, 1024, 8192), (1000, 264, 136), (513, 263, 135), (130, 136, 264), (2048, 1024, 2048)])
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
