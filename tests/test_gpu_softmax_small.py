"""Few short rows with their mean are one workgroup's work: the same bits as the rows alone give, at the edges of its range and one row
beyond, and the mean of the row losses."""
import pytest
import torch

from paper_1710_03740_amd import binding as mpt

pytestmark = pytest.mark.gpu
F16, I32 = torch.float16, torch.int32


@pytest.mark.parametrize("B,C", [(1, 1), (100, 10), (512, 16), (513, 16), (128, 17), (128, 64), (129, 64), (32, 65), (32, 256), (33, 256), (16, 257), (16, 512),
                                 (17, 512), (3, 513), (1, 7), (1024, 8)])
@pytest.mark.parametrize("pad", [0, 3])
def test_rows_and_their_mean(B, C, pad):
    g = torch.Generator(device="cuda").manual_seed(B * 1000 + C)
    z = (torch.randn(B, C + pad, device="cuda", generator=g) * 3).to(F16)[:, :C]
    lab = torch.randint(0, C, (B,), device="cuda", dtype=I32, generator=g)
    out = [torch.full((B, C + pad), 7.0, device="cuda", dtype=F16) for _ in range(2)]
    rows = [torch.full((B + 8,), 7.0, device="cuda") for _ in range(2)]
    loss = torch.empty(1, device="cuda")
    mpt.mpt_softmax_xent_scaled(z, lab, 64.0, out[0][:, :C], loss, rows[0][:B])
    mpt.mpt_softmax_xent_scaled(z, lab, 64.0, out[1][:, :C], None, rows[1][:B])
    assert torch.equal(out[0], out[1]) and torch.equal(rows[0], rows[1])           # neighbours included: they keep their sevens
    r = rows[0][:B].double()
    # B - 1 additions and a division, each rounded once
    assert abs(loss.double().item() - r.mean().item()) <= (B + 1) * 2.0 ** -24 * r.abs().sum().item() / B
    zd = z.double()
    want = torch.logsumexp(zd, 1) - zd.gather(1, lab.long()[:, None])[:, 0]
    # exponentials to about 2 ulp each and C additions of positive terms; the maximum comes off exactly representable values
    assert ((r - want).abs() <= (C + 8) * 2.0 ** -23 * (1.0 + want.abs() + zd.abs().amax(1))).all()
