"""Whole-tile products over short reductions, on both sides of where the small tiles take them from the streamed kernels, and sums
added to FP32 values whose rows and columns end inside a tile.

Operands are -1, 0 or 1: every sum is a whole number below 2^11 and exact, whatever its order."""
import pytest
import torch

from paper_1710_03740_amd import binding as mpt

pytestmark = pytest.mark.gpu


def ints(shape, seed, dtype=torch.float16):
    return torch.randint(-1, 2, shape, device="cuda", generator=torch.Generator(device="cuda").manual_seed(seed)).to(dtype)


# reductions of 1, 3 and 4 stages over 128 tiles of 256 x 256, 192 and 512 of them; then edges: one row and column more or less than tiles of 64 and 128
@pytest.mark.parametrize("R,I,J", [(64, 8192, 1024), (192, 8192, 1024), (256, 8192, 1024), (128, 2048, 6144), (64, 8192, 4096),
                                   (64, 65, 127), (72, 129, 65), (200, 191, 193), (33, 63, 3), (256, 1023, 641)])
@pytest.mark.parametrize("split", [False, True])
def test_fp32_outputs(R, I, J, split):
    x, g = ints((R, I), 1), ints((R, J), 2)
    want = (x.float().t() @ g.float())
    need = mpt.mpt_gemm_workspace_bytes(mpt.OP_WGRAD, R, J, I)
    ws = torch.empty(need // 4, device="cuda") if split and need else None
    buf = torch.full((I, J + 8), float("nan"), device="cuda")              # whole 16-byte pieces for rows of whole tiles, odd addresses for the others
    out = buf[:, :J]
    print("wgrad", R, I, J, split, flush=True)
    mpt.mpt_gemm_wgrad(x, g, out, ws=ws)
    assert torch.equal(out, want)
    start = ints((I, J), 3, torch.float32)
    out.copy_(start)
    mpt.mpt_gemm_wgrad(x, g, out, accumulate=True, ws=ws)
    assert torch.equal(out, want + start) and bool(torch.isnan(buf[:, J:]).all())


# 96, 128, 160 and 192 tiles of 128 x 256, below and above the line
@pytest.mark.parametrize("M,N,K", [(1536, 2048, 1024), (1536, 2048, 1088), (2048, 2048, 512), (2048, 2048, 832), (2560, 2048, 256), (3072, 2048, 256), (3072, 2048, 320)])
def test_fp16_outputs(M, N, K):
    x, w = ints((M, K), 1), ints((K, N), 2)
    want = x.float() @ w.float()
    y, h = torch.empty((M, N), device="cuda", dtype=torch.float16), torch.empty((M, N), device="cuda", dtype=torch.float16)
    need = mpt.mpt_gemm_workspace_bytes(mpt.OP_FWD, M, N, K)
    for ws in (None, torch.empty(need // 4, device="cuda") if need else None):
        print("fwd", M, N, K, ws is not None, flush=True)
        mpt.mpt_gemm_fwd(x, w, y, ws)
        mpt.mpt_gemm_fwd_relu(x, w, h, ws)
        assert torch.equal(y.float(), want) and torch.equal(h.float(), want.clamp(min=0))
