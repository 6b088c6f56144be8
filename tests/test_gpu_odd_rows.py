"""Rows at any address and of any length in the softmax, the LSTM cell and the pointwise glue: the results must be, bit for bit,
those of the same values in aligned rows of a whole number of vectors."""
import pytest
import torch

from paper_1710_03740_amd import binding as mpt

pytestmark = pytest.mark.gpu
F16, F32, I32 = torch.float16, torch.float32, torch.int32


def window(rows, cols, pad, offset, fill):
    buf = torch.full((rows * (cols + pad) + offset + 16,), fill, dtype=F16, device="cuda")
    return buf, buf[offset:offset + rows * (cols + pad)].view(rows, cols + pad)[:, :cols]


# one wavefront a row, several, sixteen, chunks beyond the registers kept; lengths around the vector and the launch's brackets
@pytest.mark.parametrize("C", [1, 7, 8, 9, 15, 504, 505, 511, 513, 2047, 2049, 8185, 8191, 8193, 32761, 32767, 32769, 65535])
@pytest.mark.parametrize("pad,offset", [(0, 0), (1, 0), (3, 5)])
def test_softmax(C, pad, offset):
    B, whole = 5, -(-C // 8) * 8
    g = torch.Generator(device="cuda").manual_seed(C)
    z = torch.empty(B, C, device="cuda").normal_(0, 3, generator=g).half()
    labels = torch.tensor([0, C - 1, C // 2, C // 3, max(C - 2, 0)], device="cuda", dtype=I32)
    aligned = torch.full((B, whole), float("-inf"), device="cuda", dtype=F16)      # padded classes add exp(-inf) = 0 at the row's end
    aligned[:, :C] = z
    want, want_loss, want_rows = torch.empty_like(aligned), torch.empty(1, device="cuda"), torch.empty(B, device="cuda")
    mpt.mpt_softmax_xent_scaled(aligned, labels, 64.0, want, want_loss, want_rows)
    _, src = window(B, C, pad, offset, float("inf"))
    src.copy_(z)
    buf, out = window(B, C, pad, offset, 7.0)
    loss, rows = torch.empty(1, device="cuda"), torch.empty(B, device="cuda")
    mpt.mpt_softmax_xent_scaled(src, labels, 64.0, out, loss, rows)
    assert torch.equal(out, want[:, :C]) and torch.equal(rows, want_rows) and torch.equal(loss, want_loss)
    out.fill_(7.0)
    assert bool((buf == 7.0).all())                                                 # nothing beside the rows was written


@pytest.mark.parametrize("H", [1, 3, 4, 5, 31, 32, 1023, 1026])
@pytest.mark.parametrize("pad,offset", [(0, 0), (1, 1), (5, 2)])
def test_lstm_cell(H, pad, offset):
    B, wide = 6, -(-H // 8) * 8
    g = torch.Generator(device="cuda").manual_seed(H)
    v = lambda *s: torch.empty(*s, device="cuda").normal_(generator=g).half()  # noqa: E731
    gx, gr, cp, dh, dc, bias = v(B, 4, H), v(B, 4, H), v(B, H), v(B, H), v(B, H), torch.empty(4, H, device="cuda").normal_(generator=g)

    def run(h, put, new):
        def gates(t):
            q = torch.zeros(B, 4, h, device="cuda", dtype=F16)
            q[:, :, :H] = t
            return put(q.reshape(B, 4 * h))
        def one(t):
            q = torch.zeros(B, h, device="cuda", dtype=F16)
            q[:, :H] = t
            return put(q)
        b = torch.zeros(4, h, device="cuda")
        b[:, :H] = bias
        act, c, hh, da, dcp = new(4 * h), new(h), new(h), new(4 * h), new(h)
        mpt.mpt_lstm_cell_fwd(gates(gx), gates(gr), b.reshape(-1), one(cp), act, c, hh)
        mpt.mpt_lstm_cell_bwd(one(dh), one(dc), act, c, one(cp), da, dcp)
        return [t.reshape(B, -1, h)[:, :, :H].contiguous() for t in (act.contiguous(), c.contiguous(), hh.contiguous(), da.contiguous(), dcp.contiguous())]

    def put_odd(t):
        w = window(t.shape[0], t.shape[1], pad, offset, float("inf"))[1]
        w.copy_(t)
        return w

    want = run(wide, lambda t: t, lambda n: torch.empty(B, n, device="cuda", dtype=F16))
    got = run(H, put_odd, lambda n: window(B, n, pad, offset, 7.0)[1])
    for a, b in zip(got, want):
        assert torch.equal(a, b)


# more than 512 Ki cells take four per thread, with 0 to 3 left over in each row; the last moves more than the memory-side cache holds
@pytest.mark.parametrize("B,H", [(520, 1022), (520, 1023), (520, 1024), (520, 1025), (2300, 4099)])
@pytest.mark.parametrize("pad,offset", [(0, 0), (5, 2)])
def test_lstm_cell_has_the_same_bits_singly_and_in_fours(B, H, pad, offset):
    g = torch.Generator(device="cuda").manual_seed(H)

    def rows(n):
        w = window(B, n, pad, offset, 7.0)
        w[1].copy_(torch.empty(B, n, device="cuda").normal_(generator=g))
        return w[1]
    gx, gr, cp, dh, dc, bias = rows(4 * H), rows(4 * H), rows(H), rows(H), rows(H), torch.empty(4 * H, device="cuda").normal_(generator=g)
    out = [window(B, n, pad, offset, 7.0) for n in (4 * H, H, H, 4 * H, H)]
    act, c, h, da, dcp = (o[1] for o in out)
    mpt.mpt_lstm_cell_fwd(gx, gr, bias, cp, act, c, h)
    mpt.mpt_lstm_cell_bwd(dh, dc, act, c, cp, da, dcp)
    step = 64                                                               # (rows of at most 512 Ki cells: one per thread)
    for r in range(0, B, step):
        s = slice(r, min(r + step, B))
        want = [torch.empty(o[1][s].shape, device="cuda", dtype=F16) for o in out]
        mpt.mpt_lstm_cell_fwd(gx[s], gr[s], bias, cp[s], *want[:3])
        mpt.mpt_lstm_cell_bwd(dh[s], dc[s], want[0], want[1], cp[s], *want[3:])
        for o, w in zip(out, want):
            assert torch.equal(o[1][s], w), r
    for buf, view in out:                                                   # nothing beside the rows was written
        view.fill_(7.0)
        assert bool((buf == 7.0).all())


# More than the memory-side cache holds (205 MB, more than 192 MiB), in rows so short (276 threads where two workgroups have 512) that threads are
# dealt over the rows one after the other; a cell left over in each row
@pytest.mark.parametrize("pad,offset", [(0, 0), (5, 2)])
def test_lstm_cell_streamed_over_short_rows(pad, offset):
    test_lstm_cell_has_the_same_bits_singly_and_in_fours(6200, 1101, pad, offset)


@pytest.mark.parametrize("n", [1, 7, 8, 9, 2047, 4099])
@pytest.mark.parametrize("offset", [0, 1, 3])
def test_pointwise_glue(n, offset):
    g = torch.Generator(device="cuda").manual_seed(n)
    a, b = (torch.empty(n + offset, device="cuda").normal_(generator=g).half()[offset:] for _ in range(2))
    for call, want in ((lambda o: mpt.mpt_add_fp16(a, b, o), (a.float() + b.float()).half()), (lambda o: mpt.mpt_relu_fwd(a, o), a.clamp(min=0)),
                       (lambda o: mpt.mpt_relu_bwd(a, b, o), torch.where(b > 0, a, torch.zeros_like(a)))):
        buf = torch.full((n + offset + 16,), 7.0, device="cuda", dtype=F16)
        call(buf[offset:offset + n])
        assert torch.equal(buf[offset:offset + n], want)
        assert bool((buf[:offset] == 7.0).all()) and bool((buf[offset + n:] == 7.0).all())
