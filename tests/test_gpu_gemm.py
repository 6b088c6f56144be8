"""GPU parity of the three FP16 contractions against the oracle."""
import numpy as np
import pytest
import torch

import workloads
from oracle import fp16, gemm
from paper_1710_03740_amd import binding as mpt
from gpu_util import dev, dev16, host, host16, gemm_check

pytestmark = pytest.mark.gpu


def _ws(op, M, N, K):
    b = mpt.mpt_gemm_workspace_bytes(op, M, N, K)
    return torch.empty(max(b, 16) // 4, dtype=torch.float32, device="cuda") if b else None


def run_fwd(X, W, split=False):
    M, K = X.shape; N = W.shape[1]
    Y = torch.full((M, N), float("nan"), dtype=torch.float16, device="cuda")
    mpt.mpt_gemm_fwd(dev16(X), dev16(W), Y, _ws(0, M, N, K) if split else None)
    return host16(Y)


def run_dgrad(dY, W, split=False):
    M, N = dY.shape; K = W.shape[0]
    dX = torch.full((M, K), float("nan"), dtype=torch.float16, device="cuda")
    mpt.mpt_gemm_dgrad(dev16(dY), dev16(W), dX, _ws(1, M, N, K) if split else None)
    return host16(dX)


def run_wgrad(X, dY, split=False, flag=None):
    M, K = X.shape; N = dY.shape[1]
    dW = torch.full((K, N), float("nan"), dtype=torch.float16, device="cuda")
    mpt.mpt_gemm_wgrad(dev16(X), dev16(dY), dW, flag=flag, ws=_ws(2, M, N, K) if split else None)
    return host16(dW)


SHAPES = [(1, 1, 1), (3, 5, 7), (33, 10, 65), (8, 16, 64), (130, 70, 200), (257, 129, 65), (300, 264, 136)]


@pytest.mark.parametrize("M,N,K", SHAPES)
def test_integer_inputs_bit_exact(M, N, K):
    """Small-integer operands with short reductions: every partial sum is exact in
    FP32, so all three passes must equal integer arithmetic bit-for-bit."""
    rng = np.random.default_rng(M + N + K)
    lim = 4 if max(M, N, K) <= 65 else 2
    X = rng.integers(-lim, lim + 1, (M, K)).astype(np.float16)
    W = rng.integers(-lim, lim + 1, (K, N)).astype(np.float16)
    dY = rng.integers(-lim, lim + 1, (M, N)).astype(np.float16)
    Xi, Wi, dYi = X.astype(np.int64), W.astype(np.int64), dY.astype(np.int64)
    for split in (False, True):
        assert np.array_equal(run_fwd(X, W, split).astype(np.int64), Xi @ Wi)
        assert np.array_equal(run_dgrad(dY, W, split).astype(np.int64), dYi @ Wi.T)
        assert np.array_equal(run_wgrad(X, dY, split).astype(np.int64), Xi.T @ dYi)


@pytest.mark.parametrize("M,N,K", [(130, 72, 200), (257, 129, 65), (300, 264, 136), (256, 10, 1024), (512, 384, 1024),
                                   (1000, 520, 776)])
@pytest.mark.parametrize("split", [False, True])
def test_random_inputs_against_oracle(M, N, K, split):
    rng = np.random.default_rng(M * 7 + N * 3 + K)
    X = rng.standard_normal((M, K)).astype(np.float16)
    W = (rng.standard_normal((K, N)) * 0.05).astype(np.float16)
    dY = (np.exp2(rng.uniform(-20, -3, (M, N))) * rng.choice([-1, 1], (M, N))).astype(np.float16)
    y, sa, s = gemm.gemm_fwd(X, W, full=True)
    gemm_check(run_fwd(X, W, split), y, sa, s, "fwd %s" % ((M, N, K),))
    dx, sa, s = gemm.gemm_dgrad(dY, W, full=True)
    gemm_check(run_dgrad(dY, W, split), dx, sa, s, "dgrad")
    dw, sa, s = gemm.gemm_wgrad(X, dY, full=True)
    gemm_check(run_wgrad(X, dY, split), dw, sa, s, "wgrad")


def test_leading_dimensions_and_unaligned_bases():
    rng = np.random.default_rng(5)
    M, N, K = 70, 52, 90
    Xb = rng.standard_normal((M, K + 5)).astype(np.float16)
    Wb = rng.standard_normal((K, N + 3)).astype(np.float16)
    d_X, d_W = dev16(Xb), dev16(Wb)
    Yb = torch.zeros((M, N + 7), dtype=torch.float16, device="cuda")
    mpt.mpt_gemm_fwd(d_X[:, 1:K + 1], d_W[:, 2:N + 2], Yb[:, 3:N + 3])
    X, W = np.ascontiguousarray(Xb[:, 1:K + 1]), np.ascontiguousarray(Wb[:, 2:N + 2])
    y, sa, s = gemm.gemm_fwd(X, W, full=True)
    out = host16(Yb)
    gemm_check(np.ascontiguousarray(out[:, 3:N + 3]), y, sa, s, "fwd strided")
    assert not out[:, :3].any() and not out[:, N + 3:].any()       # nothing written outside the view


@pytest.mark.parametrize("pad", [0, 8, 4, 1])
def test_whole_tile_kernels_over_more_tiles_than_cus(pad):
    """272 whole 256 x 256 tiles (more than one per CU), reduction depth of 4, 6 and 10 stages, with output row strides
    that keep 16-byte, 8-byte and 2-byte alignment: every store path of the whole-tile kernels."""
    M, N = 4352, 4096
    rng = np.random.default_rng(77 + pad)
    for K in ((128, 192, 320) if pad == 0 else (128,)):      # 4, 6 and 10 stages: whole trips of the 4-stage loop, with and without its 2-stage tail
        X = rng.standard_normal((M, K)).astype(np.float16)
        W = (rng.standard_normal((K, N)) * 0.05).astype(np.float16)
        Yb = torch.full((M, N + pad), 7.0, dtype=torch.float16, device="cuda")
        mpt.mpt_gemm_fwd(dev16(X), dev16(W), Yb[:, :N])
        y, sa, s = gemm.gemm_fwd(X, W, full=True)
        out = host16(Yb)
        gemm_check(np.ascontiguousarray(out[:, :N]), y, sa, s, "fwd pad %d K %d" % (pad, K))
        assert (out[:, N:] == 7.0).all()                          # nothing written outside the view
        if pad == 0:
            dY = (np.exp2(rng.uniform(-20, -3, (M, N))) * rng.choice([-1, 1], (M, N))).astype(np.float16)
            Wd = (rng.standard_normal((4096, N)) * 0.05).astype(np.float16)     # dgrad output 4352 x 4096, reduce over N
            dx, sa, s = gemm.gemm_dgrad(dY[:, :K], Wd[:, :K], full=True)
            gemm_check(run_dgrad(np.ascontiguousarray(dY[:, :K]), np.ascontiguousarray(Wd[:, :K])), dx, sa, s, "dgrad K %d" % K)
            Xw = rng.standard_normal((K, M)).astype(np.float16)                  # wgrad output 4352 x 4096, reduce over K rows
            dYw = np.ascontiguousarray(dY[:K, :])
            dw, sa, s = gemm.gemm_wgrad(Xw, dYw, full=True)
            gemm_check(run_wgrad(Xw, dYw), dw, sa, s, "wgrad K %d" % K)


def test_whole_tile_wgrad_flag():
    M, K, N = 64, 4352, 4096
    X = np.full((M, K), 2.0 ** -3, dtype=np.float16)
    dY = np.full((M, N), 2.0 ** -3, dtype=np.float16)
    flag = torch.zeros(1, dtype=torch.int32, device="cuda")
    run_wgrad(X, dY, flag=flag)
    assert int(flag.item()) == 0
    X[:, K - 1] = 300.0
    dY[:, N - 1] = 300.0                                           # one element of the last tile sums to 64 * 9e4 -> Inf
    dW = run_wgrad(X, dY, flag=flag)
    assert fp16.bits(dW)[K - 1, N - 1] == 0x7C00 and int(flag.item()) == 1
    assert np.isfinite(dW.astype(np.float32)).sum() == K * N - 1


def test_overflow_stores_inf_and_raises_wgrad_flag():
    X = np.full((64, 8), 200.0, dtype=np.float16)
    dY = np.full((64, 8), 100.0, dtype=np.float16)
    dY[:, 1] = 2.0 ** -10
    flag = torch.zeros(1, dtype=torch.int32, device="cuda")
    dW = run_wgrad(X, dY, flag=flag)
    want, _ = gemm.gemm_wgrad(X, dY)
    assert np.array_equal(fp16.bits(dW), fp16.bits(want))
    assert fp16.bits(dW)[0, 0] == 0x7C00 and int(flag.item()) == 1
    flag.zero_()
    dY[:, :] = 2.0 ** -10
    run_wgrad(X, dY, flag=flag)
    assert int(flag.item()) == 0


def test_subnormal_operands_and_results_are_kept():
    """Without loss scaling the upstream gradient is largely subnormal in FP16;
    neither operands nor results may be flushed."""
    rng = np.random.default_rng(8)
    M, N, K = 128, 64, 96
    X = rng.standard_normal((M, K)).astype(np.float16)
    dY = (np.exp2(rng.uniform(-24, -15, (M, N))) * rng.choice([-1, 1], (M, N))).astype(np.float16)
    assert ((fp16.bits(dY) & 0x7C00) == 0).mean() > 0.8
    W = (np.exp2(rng.uniform(-8, -1, (K, N)))).astype(np.float16)
    dw, sa, s = gemm.gemm_wgrad(X, dY, full=True)
    gemm_check(run_wgrad(X, dY), dw, sa, s, "wgrad subnormal operand")
    dx, sa, s = gemm.gemm_dgrad(dY, W, full=True)
    got = run_dgrad(dY, W)
    gemm_check(got, dx, sa, s, "dgrad subnormal result")
    assert (((fp16.bits(got) & 0x7C00) == 0) & ((fp16.bits(got) & 0x3FF) != 0)).any()


def test_power_of_two_invariance_and_determinism():
    rng = np.random.default_rng(10)
    X = rng.standard_normal((200, 300)).astype(np.float16)
    dY = (rng.uniform(0.5, 1.0, (200, 100)) * 2.0 ** -9).astype(np.float16)
    a = run_wgrad(X, dY, split=True)
    b = run_wgrad(X, dY, split=True)
    assert np.array_equal(fp16.bits(a), fp16.bits(b))
    c = run_wgrad(X, (dY.astype(np.float32) * 64).astype(np.float16), split=True)
    av, cv = fp16.to_f64(a), fp16.to_f64(c)
    normal = np.abs(av) >= 2.0 ** -14
    assert np.array_equal(cv[normal], av[normal] * 64)


def test_wgrad_fp32_store_and_accumulate():
    rng = np.random.default_rng(12)
    T, B, K, N = 5, 64, 72, 40
    X = rng.standard_normal((T, B, K)).astype(np.float16)
    dY = (rng.standard_normal((T, B, N)) * 2.0 ** -12).astype(np.float16)
    d_acc = torch.zeros((K, N), dtype=torch.float32, device="cuda")
    acc, sabs = None, 0.0
    for t in range(T):
        mpt.mpt_gemm_wgrad(dev16(X[t]), dev16(dY[t]), d_acc, accumulate=(t > 0))
        acc, sa = gemm.gemm_wgrad(X[t], dY[t], out_fp32=True, acc32=acc)
        sabs = sabs + sa
    got = host(d_acc)
    # FP32 accumulation allowance against the sum of magnitudes (cancellation makes ulp counts meaningless)
    from gpu_util import C_ACC, U32
    assert (np.abs(got.astype(np.float64) - acc.astype(np.float64)) <= C_ACC * U32 * sabs).all()
    well = np.abs(acc) >= sabs * 2.0 ** -4
    assert fp16.ulpdist32(got[well], acc[well]).max() <= 64
    flag = torch.zeros(1, dtype=torch.int32, device="cuda")
    d_acc[3, 3] = float("inf")
    mpt.mpt_gemm_wgrad(dev16(X[0]), dev16(dY[0]), d_acc, accumulate=True, flag=flag)
    assert int(flag.item()) == 1


@pytest.mark.parametrize("K,N,B", [(512, 256, 128), (256, 768, 64), (1024, 512, 256), (4096, 2048, 64), (4096, 2048, 576)])
def test_wgrad_fp32_whole_tiles(K, N, B):
    """FP32 store and accumulate with 16 bytes per lane: the general kernel on the small shapes, the streamed kernel's
    FP32 epilogues on the last two (128 tiles of 256 x 256: one stage of the reduction on the two-wavefront-per-SIMD
    kernel, nine on the depth-64 one).  Integer data so that the sums are exact, then real data
    against the oracle's allowance; the output is a column window of a wider buffer (row stride 8 floats longer than
    the matrix), and a planted Inf raises the flag."""
    rng = np.random.default_rng(K + N + B)
    T = 3
    Xi = rng.integers(-3, 4, (T, B, K)).astype(np.float16)
    dYi = rng.integers(-3, 4, (T, B, N)).astype(np.float16)
    buf = torch.full((K, N + 8), 7.0, dtype=torch.float32, device="cuda")
    out = buf[:, 4:4 + N]                                                  # 16-byte aligned rows, ld = N + 8
    want = np.zeros((K, N), dtype=np.int64)
    for t in range(T):
        mpt.mpt_gemm_wgrad(dev16(Xi[t]), dev16(dYi[t]), out, accumulate=(t > 0))
        want += Xi[t].astype(np.int64).T @ dYi[t].astype(np.int64)
    got = host(buf)
    assert np.array_equal(got[:, 4:4 + N].astype(np.int64), want)
    assert (got[:, :4] == 7.0).all() and (got[:, 4 + N:] == 7.0).all()     # nothing outside the window is touched
    X = rng.standard_normal((T, B, K)).astype(np.float16)
    dY = (rng.standard_normal((T, B, N)) * 2.0 ** -10).astype(np.float16)
    d_acc = torch.zeros((K, N), dtype=torch.float32, device="cuda")
    acc, sabs = None, 0.0
    for t in range(T):
        mpt.mpt_gemm_wgrad(dev16(X[t]), dev16(dY[t]), d_acc, accumulate=(t > 0))
        acc, sa = gemm.gemm_wgrad(X[t], dY[t], out_fp32=True, acc32=acc)
        sabs = sabs + sa
    from gpu_util import C_ACC, U32
    assert (np.abs(host(d_acc).astype(np.float64) - acc.astype(np.float64)) <= C_ACC * U32 * sabs).all()
    flag = torch.zeros(1, dtype=torch.int32, device="cuda")
    mpt.mpt_gemm_wgrad(dev16(X[0]), dev16(dY[0]), d_acc, accumulate=True, flag=flag)
    assert int(flag.item()) == 0
    d_acc[K - 1, N - 1] = float("inf")
    mpt.mpt_gemm_wgrad(dev16(X[0]), dev16(dY[0]), d_acc, accumulate=True, flag=flag)
    assert int(flag.item()) == 1


@pytest.mark.parametrize("scale", [1.0, 8192.0])
def test_cfg2_square_4096(scale):
    """The benchmark shape, in the benchmarked launch configuration, whole output compared."""
    c = workloads.square_gemm(4096, scale=scale)
    A, B, G = c["A"], c["B"], c["G"]
    y, sa, s = gemm.gemm_fwd(A, B, full=True)
    gemm_check(run_fwd(A, B), y, sa, s, "cfg2 fwd")
    dx, sa, s = gemm.gemm_dgrad(G, B, full=True)
    gemm_check(run_dgrad(G, B), dx, sa, s, "cfg2 dgrad S=%g" % scale)
    dw, sa, s = gemm.gemm_wgrad(A, G, full=True)
    gemm_check(run_wgrad(A, G), dw, sa, s, "cfg2 wgrad S=%g" % scale)
    gb = fp16.bits(G)
    flushed = float((c["g_true"] != 0)[(gb & 0x7FFF) == 0].mean()) if ((gb & 0x7FFF) == 0).any() else 0.0
    print("[cfg2] S=%g: upstream gradient flushed to zero %.3f, subnormal %.3f" %
          (scale, float(((gb & 0x7FFF) == 0).mean()), float((((gb & 0x7C00) == 0) & ((gb & 0x3FF) != 0)).mean())), flush=True)


@pytest.mark.parametrize("M,N,K", [(130, 72, 200), (257, 129, 65), (256, 1024, 1024), (512, 384, 1024)])
@pytest.mark.parametrize("split", [False, True])
def test_relu_folded_into_the_stores(M, N, K, split):
    rng = np.random.default_rng(M + N + K)
    X = rng.standard_normal((M, K)).astype(np.float16)
    W = (rng.standard_normal((K, N)) * 0.05).astype(np.float16)
    H = torch.full((M, N), float("nan"), dtype=torch.float16, device="cuda")
    mpt.mpt_gemm_fwd_relu(dev16(X), dev16(W), H, _ws(0, M, N, K) if split else None)
    h, sa, s = gemm.gemm_fwd_relu(X, W, full=True)
    got = host16(H)
    gemm_check(got, h, sa, s, "fwd_relu")
    y, _, s_raw = gemm.gemm_fwd(X, W, full=True)
    clear = np.abs(s_raw) > 8 * 2.0 ** -24 * sa                     # away from the sign boundary the zero pattern is fixed
    assert np.array_equal((got == 0)[clear], (s_raw <= 0)[clear]) and not np.signbit(got).any()
    # backward: mask by the stored activation of the layer below
    dY = (np.exp2(rng.uniform(-20, -3, (M, N))) * rng.choice([-1, 1], (M, N))).astype(np.float16)
    Hb = np.maximum(rng.standard_normal((M, K)), 0).astype(np.float16)
    dX = torch.full((M, K), float("nan"), dtype=torch.float16, device="cuda")
    mpt.mpt_gemm_dgrad_relu(dev16(dY), dev16(W), dev16(Hb), dX, _ws(1, M, N, K) if split else None)
    dx, sa, s = gemm.gemm_dgrad_relu(dY, W, Hb, full=True)
    got = host16(dX)
    gemm_check(got, dx, sa, s, "dgrad_relu")
    assert not got[Hb <= 0].any() and not np.signbit(got[Hb <= 0]).any()


def test_relu_folded_whole_tile_kernels():
    """Shapes that take the whole-tile streamed kernels (aligned and odd-stride outputs and masks)."""
    M, N, K = 4352, 4096, 128
    rng = np.random.default_rng(3)
    X = rng.standard_normal((M, K)).astype(np.float16)
    W = (rng.standard_normal((K, N)) * 0.05).astype(np.float16)
    h, sa, s = gemm.gemm_fwd_relu(X, W, full=True)
    for pad in (0, 4):
        Hb = torch.full((M, N + pad), 7.0, dtype=torch.float16, device="cuda")
        mpt.mpt_gemm_fwd_relu(dev16(X), dev16(W), Hb[:, :N])
        gemm_check(np.ascontiguousarray(host16(Hb)[:, :N]), h, sa, s, "fwd_relu pad %d" % pad)
    dY = (np.exp2(rng.uniform(-20, -3, (M, K))) * rng.choice([-1, 1], (M, K))).astype(np.float16)   # reduce over K=128
    Wd = (rng.standard_normal((N, K)) * 0.05).astype(np.float16)                                      # output M x N
    mask = np.maximum(rng.standard_normal((M, N)), 0).astype(np.float16)
    dx, sa, s = gemm.gemm_dgrad_relu(dY, Wd, mask, full=True)
    for pad in (0, 4):
        mb = torch.zeros((M, N + pad), dtype=torch.float16, device="cuda"); mb[:, :N] = dev16(mask)
        dX = torch.full((M, N), float("nan"), dtype=torch.float16, device="cuda")
        mpt.mpt_gemm_dgrad_relu(dev16(dY), dev16(Wd), mb[:, :N], dX)
        got = host16(dX)
        gemm_check(got, dx, sa, s, "dgrad_relu mask pad %d" % pad)
        assert not got[mask <= 0].any()


def test_relu_forms_through_a_split_reduction_of_whole_tiles():
    """512 x 2048 outputs over a reduction of 8192: 16 tiles of 256 x 256, split 16 ways on the streamed kernel's FP32
    partials; the ReLU and the backward mask are applied by the reduction, four columns per thread (mask rows 8-byte
    aligned) or one (mask at an odd row stride)."""
    M, N, K = 512, 2048, 8192
    rng = np.random.default_rng(9)
    X = rng.standard_normal((M, K)).astype(np.float16)
    W = (rng.standard_normal((K, N)) * 0.02).astype(np.float16)
    h, sa, s_ = gemm.gemm_fwd_relu(X, W, full=True)
    H = torch.full((M, N), float("nan"), dtype=torch.float16, device="cuda")
    mpt.mpt_gemm_fwd_relu(dev16(X), dev16(W), H, _ws(0, M, N, K))
    gemm_check(host16(H), h, sa, s_, "fwd_relu, split")
    dY = (np.exp2(rng.uniform(-20, -3, (M, K))) * rng.choice([-1, 1], (M, K))).astype(np.float16)   # reduce over K, output M x N
    Wd = (rng.standard_normal((N, K)) * 0.05).astype(np.float16)
    mask = np.maximum(rng.standard_normal((M, N)), 0).astype(np.float16)
    dx, sa, s_ = gemm.gemm_dgrad_relu(dY, Wd, mask, full=True)
    for pad in (0, 1):
        mb = torch.zeros((M, N + pad), dtype=torch.float16, device="cuda"); mb[:, :N] = dev16(mask)
        dX = torch.full((M, N), float("nan"), dtype=torch.float16, device="cuda")
        mpt.mpt_gemm_dgrad_relu(dev16(dY), dev16(Wd), mb[:, :N], dX, _ws(1, M, K, N))
        got = host16(dX)
        gemm_check(got, dx, sa, s_, "dgrad_relu, split, mask pad %d" % pad)
        assert not got[mask <= 0].any()


def test_outputs_with_few_rows_and_many_columns():
    """384 x 16384 outputs (three 128-row tiles by 64 column tiles): the 128-row whole-tile kernel, in all three
    passes, with the folded ReLU forms and the overflow vote."""
    I, J = 384, 16384
    rng = np.random.default_rng(21)
    for K in (64, 192, 320):                                 # 2, 6 and 10 stages (tail only; loop + tail; two trips + tail)
        X = rng.standard_normal((I, K)).astype(np.float16)
        W = (rng.standard_normal((K, J)) * 0.05).astype(np.float16)
        y, sa, s = gemm.gemm_fwd(X, W, full=True)
        gemm_check(run_fwd(X, W), y, sa, s, "fwd K %d" % K)
        dY = (np.exp2(rng.uniform(-20, -3, (I, K))) * rng.choice([-1, 1], (I, K))).astype(np.float16)
        Wd = (rng.standard_normal((J, K)) * 0.05).astype(np.float16)
        dx, sa, s = gemm.gemm_dgrad(dY, Wd, full=True)
        gemm_check(run_dgrad(dY, Wd), dx, sa, s, "dgrad K %d" % K)
        Xw = rng.standard_normal((K, I)).astype(np.float16)
        dYw = (np.exp2(rng.uniform(-20, -3, (K, J))) * rng.choice([-1, 1], (K, J))).astype(np.float16)
        dw, sa, s = gemm.gemm_wgrad(Xw, dYw, full=True)
        gemm_check(run_wgrad(Xw, dYw), dw, sa, s, "wgrad K %d" % K)
    H = torch.full((I, J), float("nan"), dtype=torch.float16, device="cuda")
    mpt.mpt_gemm_fwd_relu(dev16(X), dev16(W), H)
    h, sa, s = gemm.gemm_fwd_relu(X, W, full=True)
    gemm_check(host16(H), h, sa, s, "fwd_relu")
    mask = np.maximum(rng.standard_normal((I, J)), 0).astype(np.float16)
    dX = torch.full((I, J), float("nan"), dtype=torch.float16, device="cuda")
    mpt.mpt_gemm_dgrad_relu(dev16(dY), dev16(Wd), dev16(mask), dX)
    dx, sa, s = gemm.gemm_dgrad_relu(dY, Wd, mask, full=True)
    got = host16(dX)
    gemm_check(got, dx, sa, s, "dgrad_relu")
    assert not got[mask <= 0].any()
    flag = torch.zeros(1, dtype=torch.int32, device="cuda")
    Xo = np.full((64, I), 2.0 ** -3, dtype=np.float16); dYo = np.full((64, J), 2.0 ** -3, dtype=np.float16)
    run_wgrad(Xo, dYo, flag=flag)
    assert int(flag.item()) == 0
    Xo[:, I - 1] = 300.0; dYo[:, J - 1] = 300.0
    dW = run_wgrad(Xo, dYo, flag=flag)
    assert fp16.bits(dW)[I - 1, J - 1] == 0x7C00 and int(flag.item()) == 1


def test_random_shapes_strides_and_offsets():
    """A seeded sweep over shapes, leading dimensions and base offsets (every loader and store path of the general
    kernel, with and without the split workspace), each pass against the oracle."""
    rng = np.random.default_rng(2024)
    for case in range(24):
        M, N, K = (int(v) for v in rng.integers(1, 400, 3))
        if case % 6 == 0:
            M, N, K = M * 2 + 256, N + 256, (K // 8 + 1) * 8
        px, pw, py = (int(v) for v in rng.integers(0, 12, 3))
        ox, ow, oy = (int(v) for v in rng.integers(0, 5, 3))
        if case % 3 == 0:
            px = pw = py = ox = ow = oy = 0                     # contiguous, aligned
        X = rng.standard_normal((M, K)).astype(np.float16)
        W = (rng.standard_normal((K, N)) * 0.1).astype(np.float16)
        dY = (np.exp2(rng.uniform(-18, -2, (M, N))) * rng.choice([-1, 1], (M, N))).astype(np.float16)
        split = bool(case % 2)

        def view(a, pad, off):
            buf = torch.zeros((a.shape[0], a.shape[1] + pad + off), dtype=torch.float16, device="cuda")
            buf[:, off:off + a.shape[1]] = dev16(a)
            return buf[:, off:off + a.shape[1]]

        def out(rows, cols, pad, off):
            buf = torch.full((rows, cols + pad + off), 3.0, dtype=torch.float16, device="cuda")
            return buf, buf[:, off:off + cols]

        label = "case %d M=%d N=%d K=%d pads %s offs %s split %s" % (case, M, N, K, (px, pw, py), (ox, ow, oy), split)
        yb, yv = out(M, N, py, oy)
        mpt.mpt_gemm_fwd(view(X, px, ox), view(W, pw, ow), yv, _ws(0, M, N, K) if split else None)
        y, sa, s = gemm.gemm_fwd(X, W, full=True)
        got = host16(yb)
        gemm_check(np.ascontiguousarray(got[:, oy:oy + N]), y, sa, s, "fwd " + label)
        assert (got[:, :oy] == 3.0).all() and (got[:, oy + N:] == 3.0).all(), label
        xb, xv = out(M, K, px, ox)
        mpt.mpt_gemm_dgrad(view(dY, py, oy), view(W, pw, ow), xv, _ws(1, M, N, K) if split else None)
        dx, sa, s = gemm.gemm_dgrad(dY, W, full=True)
        gemm_check(np.ascontiguousarray(host16(xb)[:, ox:ox + K]), dx, sa, s, "dgrad " + label)
        wb, wv = out(K, N, pw, ow)
        mpt.mpt_gemm_wgrad(view(X, px, ox), view(dY, py, oy), wv, ws=_ws(2, M, N, K) if split else None)
        dw, sa, s = gemm.gemm_wgrad(X, dY, full=True)
        gemm_check(np.ascontiguousarray(host16(wb)[:, ow:ow + N]), dw, sa, s, "wgrad " + label)


def test_mfma_probe_runs_to_completion():
    """The diagnostic entry point: both operand kinds run to completion and leave the sink untouched (rates are
    reported by bench.py, not asserted here: they depend on the clock state of the box)."""
    sink = torch.zeros(1, dtype=torch.float32, device="cuda")
    for rnd in (0, 1):
        for _ in range(3):
            mpt.mpt_probe_mfma(1000, rnd, sink)
        torch.cuda.synchronize()
    assert float(sink.item()) == 0.0


def test_accumulation_inside_the_matrix_instruction():
    """The evidence for the acceptance rule's allowance (C_ACC in gpu_util): how the FP16 matrix instruction adds.
    Through mpt_gemm_wgrad with an FP32 store (no FP16 rounding in the way), one product of 1 is summed with sixteen
    equal small products placed in the same instruction or in the next one.  Round-to-nearest FP32 additions of the
    exact products would return the exact sum in every case below (all sums are FP32 numbers).  The hardware aligns
    the addends of an instruction to the largest of them and keeps only a few bits below that value's FP32 step, so
    small addends are partly or wholly lost: the test prints the stored sums, asserts that each lies within the
    allowance C_ACC * 2^-24 * sum|a*b| of the exact one (the rule holds on these adversarial inputs), and that the
    worst case is off by more than 2^-24 * sum|a*b| (so an allowance of one FP32 rounding per result would reject
    correct hardware results).  The large output takes the streamed kernel (instructions of depth 32), the small one
    the general kernel (depth 16)."""
    from gpu_util import C_ACC
    worst = 0.0
    for K, N in ((4096, 2048), (256, 256)):
        M = 64
        for small in (-12, -13, -14, -15):                   # products 2^-25 .. 2^-28 next to a product of 1
            for where in (0, 32):                            # small products in the same instruction as the 1, or in the next one
                X = np.zeros((M, K), dtype=np.float16)
                dY = np.zeros((M, N), dtype=np.float16)
                X[0, :] = 1.0
                dY[0, :] = 1.0
                X[where + 1:where + 17, :] = 2.0 ** -13
                dY[where + 1:where + 17, :] = 2.0 ** small
                out = torch.empty((K, N), dtype=torch.float32, device="cuda")
                mpt.mpt_gemm_wgrad(dev16(X), dev16(dY), out)
                got = out.cpu().numpy().astype(np.float64)
                exact = 1.0 + 16 * 2.0 ** (small - 13)          # also sum|a*b|
                assert (got == got[0, 0]).all()                  # every output element sees the same sum
                err = abs(got[0, 0] - exact) / (2.0 ** -24 * exact)
                worst = max(worst, err)
                print("[mfma accumulation] %dx%d: 1 + 16 * 2^%d, small products in instruction %d: exact 1 + %g * 2^-24, stored 1 + %g * 2^-24, off by %.2f * 2^-24 * sum|a*b|"
                      % (K, N, small - 13, where // 32, 16 * 2.0 ** (small - 13 + 24), (got[0, 0] - 1.0) * 2.0 ** 24, err), flush=True)
                assert err <= C_ACC, (K, N, small, where, got[0, 0], exact)
    print("[mfma accumulation] worst case: %.2f * 2^-24 * sum|a*b| (allowance: %g)" % (worst, C_ACC), flush=True)
    assert worst > 1.0
    # a large accumulator swallows addends below a few bits under its FP32 step: 2^24 + 16 * 0.125 stays 2^24
    M, K, N = 64, 256, 256
    X = np.zeros((M, K), dtype=np.float16); dY = np.zeros((M, N), dtype=np.float16)
    X[0, :] = 4096.0; dY[0, :] = 4096.0                      # 2^24
    X[1:17, :] = 0.125; dY[1:17, :] = 1.0
    out = torch.empty((K, N), dtype=torch.float32, device="cuda")
    mpt.mpt_gemm_wgrad(dev16(X), dev16(dY), out)
    got = float(out.cpu().numpy()[0, 0])
    print("[mfma accumulation] 2^24 + 16 * 0.125: stored 2^24 + %g" % (got - 2.0 ** 24), flush=True)
    assert abs(got - (2.0 ** 24 + 2.0)) <= C_ACC * 2.0 ** -24 * (2.0 ** 24 + 2.0)


def test_odd_multiple_of_128_rows_with_a_split_reduction():
    """Outputs of 128 or 384 rows, few tiles, a long reduction and a workspace: 128 x 256 tiles of the streamed kernel
    with FP32 partials, then the ordered reduction - all three passes (the weight gradient's rows are K), the ReLU
    forms through the reduction's epilogue, and the overflow vote."""
    rng = np.random.default_rng(77)
    for (M, N, K) in ((384, 768, 8192), (128, 4096, 4160)):      # 9 tiles x 16 splits; 16 tiles x 8 splits, the last one short
        X = rng.standard_normal((M, K)).astype(np.float16)
        W = (rng.standard_normal((K, N)) * 0.05).astype(np.float16)
        assert mpt.mpt_gemm_workspace_bytes(0, M, N, K) > 0
        y, sa, s_ = gemm.gemm_fwd(X, W, full=True)
        gemm_check(run_fwd(X, W, split=True), y, sa, s_, "fwd %dx%dx%d" % (M, N, K))
        # dgrad: output M x K' with K' a multiple of 256, reduction over N'
        dY = (np.exp2(rng.uniform(-20, -3, (M, K))) * rng.choice([-1, 1], (M, K))).astype(np.float16)
        Wd = (rng.standard_normal((N, K)) * 0.05).astype(np.float16)
        dx, sa, s_ = gemm.gemm_dgrad(dY, Wd, full=True)
        gemm_check(run_dgrad(dY, Wd, split=True), dx, sa, s_, "dgrad %dx%dx%d" % (M, K, N))
        # wgrad: output rows = the weight's rows (M here), reduction over the batch (K here)
        Xw = rng.standard_normal((K, M)).astype(np.float16)
        dYw = (np.exp2(rng.uniform(-20, -3, (K, N))) * rng.choice([-1, 1], (K, N))).astype(np.float16)
        dw, sa, s_ = gemm.gemm_wgrad(Xw, dYw, full=True)
        flag = torch.zeros(1, dtype=torch.int32, device="cuda")
        gemm_check(run_wgrad(Xw, dYw, split=True, flag=flag), dw, sa, s_, "wgrad %dx%dx%d" % (K, M, N))
        assert int(flag.item()) == 0
        H = torch.full((M, N), float("nan"), dtype=torch.float16, device="cuda")
        mpt.mpt_gemm_fwd_relu(dev16(X), dev16(W), H, _ws(0, M, N, K))
        h, sa, s_ = gemm.gemm_fwd_relu(X, W, full=True)
        gemm_check(host16(H), h, sa, s_, "fwd_relu")
    Xo = np.full((8192, 384), 16.0, dtype=np.float16); dYo = np.full((8192, 768), 16.0, dtype=np.float16)
    flag = torch.zeros(1, dtype=torch.int32, device="cuda")
    got = run_wgrad(Xo, dYo, split=True, flag=flag)         # 8192 * 256 overflows FP16: Inf stored, vote raised
    assert np.isinf(got).all() and int(flag.item()) == 1


def test_smallest_outputs_over_the_longest_reductions():
    """256 x 1024 outputs over a reduction of 32768 (the recurrent input gradient of the projected-LSTM layer at its own
    size): 128 x 256 tiles, 32 splits.  Input-gradient and forward layouts."""
    rng = np.random.default_rng(5)
    M, N, K = 256, 32768, 1024
    dY = (np.exp2(rng.uniform(-20, -3, (M, N))) * rng.choice([-1, 1], (M, N))).astype(np.float16)
    W = (rng.standard_normal((K, N)) * 0.05).astype(np.float16)
    dx, sa, s_ = gemm.gemm_dgrad(dY, W, full=True)
    gemm_check(run_dgrad(dY, W, split=True), dx, sa, s_, "dgrad 256x1024 over 32768")
    X = rng.standard_normal((M, N)).astype(np.float16)
    Wf = (rng.standard_normal((N, K)) * 0.02).astype(np.float16)
    y, sa, s_ = gemm.gemm_fwd(X, Wf, full=True)
    gemm_check(run_fwd(X, Wf, split=True), y, sa, s_, "fwd 256x1024 over 32768")


# Products with room for partials that one launch sums in their pieces all the same, side by side (test_gpu_gemm_pieces.py compares those bit for bit) or
# by cutting its sums (test_gpu_gemm_cut.py)
UNSPLIT = {("fwd", 256, 1024, 1024), ("dgrad", 256, 1024, 1024), ("wgrad", 256, 1024, 1024), ("fwd", 256, 10, 1024), ("wgrad", 256, 10, 1024), ("wgrad", 256, 10, 2048),
           ("dgrad", 512, 384, 4096), ("wgrad", 512, 384, 4096), ("dgrad", 256, 1024, 8192), ("wgrad", 256, 1024, 8192)}


@pytest.mark.parametrize("M,N,K", [(256, 1024, 1024), (256, 10, 1024), (256, 10, 2048), (100, 72, 2048), (512, 384, 4096), (256, 1024, 8192), (384, 768, 8192)])
def test_split_reduction_adds_every_partial_in_split_order(M, N, K):
    """Few output tiles and a long reduction: the launcher splits the reduction and a second pass adds the FP32 partials
    up.  The partials stay in the caller's workspace as [split][I][J], so the stored FP16 result must be, bit for bit,
    the FP32 sum of those partials in split order, rounded once, and identical from launch to launch."""
    rng = np.random.default_rng(M + N + K)
    X = rng.standard_normal((M, K)).astype(np.float16)
    W = (rng.standard_normal((K, N)) * 0.05).astype(np.float16)
    dY = (rng.standard_normal((M, N)) * 0.01).astype(np.float16)
    dX_, dW_, dG_ = dev16(X), dev16(W), dev16(dY)
    cases = (("fwd", 0, (M, N), lambda out, ws: mpt.mpt_gemm_fwd(dX_, dW_, out, ws)),
             ("dgrad", 1, (M, K), lambda out, ws: mpt.mpt_gemm_dgrad(dG_, dW_, out, ws)),
             ("wgrad", 2, (K, N), lambda out, ws: mpt.mpt_gemm_wgrad(dX_, dG_, out, ws=ws)))
    for name, op, shape, call in cases:
        need = mpt.mpt_gemm_workspace_bytes(op, M, N, K)
        if need == 0:
            continue
        I, J = shape
        assert need % (I * J * 4) == 0 and need // (I * J * 4) >= 2          # room for a whole number of partial outputs
        ws = torch.full((need // 4,), float("nan"), dtype=torch.float32, device="cuda")
        first = None
        for rep in range(3):
            out = torch.full(shape, float("nan"), dtype=torch.float16, device="cuda")
            call(out, ws)
            got = host16(out)
            part = ws.cpu().numpy().reshape(-1, I, J)
            written = [k for k in range(part.shape[0]) if not np.isnan(part[k]).all()]
            assert written == list(range(len(written)))                       # the size asked for is an upper bound; the partials lead
            splits = len(written)
            part = part[:splits]
            assert splits == 0 or not np.isnan(part).any()
            assert (splits == 0) == ((name, M, N, K) in UNSPLIT), name
            if rep == 0 and splits == 0:
                # the workspace size is an upper bound over the kernels the launcher may pick; this shape went
                # through one launch without a split and left the workspace untouched
                print("[split order] %s %dx%dx%d: not split" % (name, M, N, K), flush=True)
                break
            acc = part[0].copy()
            for s_ in range(1, splits):
                acc = acc + part[s_]                      # float32 additions, split order
            assert acc.dtype == np.float32
            want = acc.astype(np.float16)
            assert np.array_equal(fp16.bits(got), fp16.bits(want)), (name, rep)
            if first is None:
                first = got
            assert np.array_equal(fp16.bits(got), fp16.bits(first)), (name, rep)
        else:
            print("[split order] %s %dx%dx%d: %d splits of %d x %d" % (name, M, N, K, splits, I, J), flush=True)
