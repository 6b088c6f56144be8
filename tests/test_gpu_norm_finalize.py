"""The launch that adds up the row blocks' partial sums (k_bn_finalize in csrc/norm.hip) on both sides of its rules: up to and beyond 128 row blocks, up to and beyond
128 channels, channels that are no whole workgroup."""
import pytest
import torch

from paper_1710_03740_amd import binding as mpt

pytestmark = pytest.mark.gpu


# (rows, channels): 64 rows per block with 256 channels and more, 256 with 64, 4096 with one
@pytest.mark.parametrize("P,C", [(40000, 8), (600000, 3), (40000, 64), (20000, 120), (16384, 128), (16640, 128), (20011, 129), (9000, 136), (12544, 512), (70000, 1)])
def test_sums_of_many_row_blocks(P, C):
    """Chains of 16 rows in FP32 about the first row, the rest in FP64: a sum is off by at most (16 + 3) * 2^-24 of its terms' magnitudes, and rounded once."""
    g = torch.Generator(device="cuda").manual_seed(P + C)
    x, dy = (torch.empty(P, C, device="cuda").normal_(generator=g).half() for _ in range(2))
    mean, var, dgamma, dbeta = (torch.empty(C, device="cuda") for _ in range(4))
    ws = torch.empty((mpt.mpt_bn_workspace_bytes(P, C) + 3) // 4, device="cuda")
    ws.fill_(float("nan"))
    mpt.mpt_bn_stats(x, mean, var, ws)
    d = x.double()
    k = d[0]
    step = 19 * 2.0 ** -24
    off = (d - k).abs().mean(0) * step
    assert ((mean.double() - d.mean(0)).abs() <= off + 2.0 ** -24 * d.mean(0).abs()).all()
    assert ((var.double() - d.var(0, unbiased=False)).abs() <= 2 * step * ((d - k) ** 2).mean(0)).all()
    ws.fill_(float("nan"))
    mpt.mpt_bn_bwd_reduce(x, dy, mean, var, 1e-5, dgamma, dbeta, ws)
    xh, e = (d - mean.double()) / torch.sqrt(var.double() + 1e-5), dy.double()
    assert ((dbeta.double() - e.sum(0)).abs() <= step * e.abs().sum(0)).all()
    assert ((dgamma.double() - (e * xh).sum(0)).abs() <= (step + 4 * 2.0 ** -24) * (e * (xh.abs() + mean.double().abs() / torch.sqrt(var.double()))).abs().sum(0)).all()
