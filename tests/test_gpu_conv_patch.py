"""Convolutions of at most 64 channels over many pixels, which are taken a patch of pixels at a time: forward and input gradient at
the edges of its range against a 64-bit convolution.

An output is a sum of 9 * C products of FP16 values held exactly in FP32 and rounded once to FP16: |error| <= 2^-11 |sum| +
9 C 2^-24 sum |a b|, and half the smallest FP16 step."""
import pytest
import torch

from paper_1710_03740_amd import binding as mpt

F16, F64 = torch.float16, torch.float64

# (images, height, width, C, Kf): rows of images, single-pixel rows and columns, 256-pixel tiles that straddle images, a ragged last
# tile, the fewest pixels, the widest rows, one or two halves of 32 channels, one to four tiles per workgroup
SIZES = [(64, 23, 23, 64, 64), (700, 7, 7, 8, 64), (512, 8, 8, 40, 32), (3, 95, 120, 64, 56), (33000, 1, 1, 16, 8), (300, 1, 111, 32, 24),
         (301, 113, 1, 24, 32), (41, 57, 56, 64, 64), (90, 56, 56, 48, 64)]


def _reference(x, w):
    """y[n, i, j, k] = sum over taps and channels, in 64 bits, with the sums of magnitudes."""
    Nb, H, W, C = x.shape
    pad = torch.zeros(Nb, H + 2, W + 2, C, device=x.device, dtype=F64)
    pad[:, 1:-1, 1:-1] = x.to(F64)
    y = torch.zeros(Nb * H * W, w.shape[0], device=x.device, dtype=F64)
    mag = torch.zeros_like(y)
    for a in range(3):
        for b in range(3):
            p = pad[:, a:a + H, b:b + W].reshape(-1, C).contiguous()
            f = w[:, a, b].to(F64).t().contiguous()
            y += p @ f
            mag += p.abs() @ f.abs()
    return y.view(Nb, H, W, -1), mag.view(Nb, H, W, -1)


def _check(got, ref, mag, terms):
    bound = 2.0 ** -11 * ref.abs() + terms * 2.0 ** -24 * mag + 2.0 ** -25
    assert ((got.to(F64) - ref).abs() <= bound).all()


@pytest.mark.gpu
@pytest.mark.parametrize("Nb,H,W,C,Kf", SIZES)
def test_patch_convolutions(Nb, H, W, C, Kf):
    g = torch.Generator(device="cuda")
    g.manual_seed(Nb + H)
    x = torch.randn(Nb, H, W, C, device="cuda", generator=g).to(F16)
    dy = torch.randn(Nb, H, W, Kf, device="cuda", generator=g).to(F16)
    w = (torch.randn(Kf, 3, 3, C, device="cuda", generator=g) * 0.1).to(F16)
    # the outputs between guards: nothing beside them is written
    buf = torch.full((Nb * H * W * max(C, Kf) + 512,), 7.0, device="cuda", dtype=F16)
    n = Nb * H * W * Kf
    y = buf[256:256 + n].view(Nb, H, W, Kf)
    mpt.mpt_conv3x3_fwd(x, w, y)
    _check(y, *_reference(x, w), 9 * C)
    assert (buf[:256] == 7).all() and (buf[256 + n:] == 7).all()
    n = Nb * H * W * C
    buf.fill_(7.0)
    dx = buf[256:256 + n].view(Nb, H, W, C)
    mpt.mpt_conv3x3_dgrad(dy, w, dx)
    _check(dx, *_reference(dy, w.flip(1, 2).permute(3, 1, 2, 0).contiguous()), 9 * Kf)
    assert (buf[:256] == 7).all() and (buf[256 + n:] == 7).all()


@pytest.mark.gpu
def test_pixels_outside_an_image_stay_outside():
    """An infinite pixel reaches its neighbours only, not the next row's first or the next image's."""
    Nb, H, W, C = 600, 8, 8, 64
    x = torch.ones(Nb, H, W, C, device="cuda", dtype=F16)
    x[5, 3, 7, 2] = float("inf")
    x[9, 7, 7, 60] = float("inf")
    w = torch.full((64, 3, 3, C), 2.0 ** -6, device="cuda", dtype=F16)
    y, want = torch.empty(Nb, H, W, 64, device="cuda", dtype=F16), torch.zeros(Nb, H, W, device="cuda", dtype=torch.bool)
    want[5, 2:5, 6:8] = True
    want[9, 6:8, 6:8] = True
    mpt.mpt_conv3x3_fwd(x, w, y)
    assert torch.equal(torch.isinf(y).all(-1), want) and not torch.isinf(y[~want]).any()
    mpt.mpt_conv3x3_dgrad(x, w, y)
    assert torch.equal(torch.isinf(y).all(-1), want) and not torch.isinf(y[~want]).any()
