"""The binding's native calls: what they take ends as it does through the Python checks, bit for bit, and what is not plainly
as it should be is left to those (None)."""
import ctypes

import pytest
import torch

from paper_1710_03740_amd import binding as mpt

F16, F32, I32 = torch.float16, torch.float32, torch.int32


class Sub(torch.Tensor):
    pass


def test_host_tensors_subclasses_and_function_modes_are_left_to_the_python_checks():
    mpt.lib()
    X, W, Y = (torch.zeros(8, 8, dtype=F16) for _ in range(3))
    assert mpt._native.gemm_fwd(X, W, Y, None) is None                     # host tensors
    assert mpt._native.gemm_fwd(X, W, Y) is None                           # a call of another length
    assert mpt._native.gemm_fwd(X, None, 3, "ws") is None
    assert mpt._native.master_update_multi(iter([]), 1.0, 0.1, 0.9, None, None) is None
    assert mpt._native.master_update_multi([], 1.0, 0.1, 0.9, None, None) is None


@pytest.fixture
def unloaded(monkeypatch):
    """The binding as it is before its first call; as it was afterwards."""
    monkeypatch.setattr(mpt, "_lib", None)
    monkeypatch.setattr(mpt, "_native", mpt._NotLoaded())
    return monkeypatch


def _goes_on_through_the_checks():
    assert mpt.mpt_version() > 0 and mpt._native.gemm_fwd(*[torch.zeros(8, 8, dtype=F16)] * 3, None) is None
    with pytest.raises(ValueError, match="W: shape"):
        mpt.mpt_gemm_fwd(torch.zeros(8, 8, dtype=F16), torch.zeros(7, 8, dtype=F16), torch.zeros(8, 8, dtype=F16))


def test_a_library_without_the_native_calls_is_used_all_the_same(unloaded, tmp_path):
    unloaded.setattr(mpt, "CALLS_PATH", str(tmp_path / "_calls.so"))
    with pytest.warns(RuntimeWarning, match="_calls.so is not built"):
        mpt.lib()
    _goes_on_through_the_checks()
    unloaded.setattr(mpt, "LIB_PATH", str(tmp_path / "libmpt.so"))
    unloaded.setattr(mpt, "_lib", None)
    with pytest.raises(RuntimeError, match="libmpt.so is not built"):
        mpt.lib()


def test_native_calls_of_another_torch_are_left_alone(unloaded, tmp_path):
    """Compiled against other headers they could read a tensor's fields elsewhere."""
    unloaded.setattr(mpt.torch.version, "git_version", "0" * 40)
    with pytest.warns(RuntimeWarning, match="_calls.so is built for torch .*, this is .* 0{40}"):
        mpt.lib()
    _goes_on_through_the_checks()
    unloaded.setattr(mpt, "_lib", None)
    unloaded.setattr(mpt, "CALLS_PATH", str(tmp_path / "_calls.so"))
    (tmp_path / "_calls.so").write_bytes(b"no shared object")
    with pytest.warns(RuntimeWarning, match="_calls.so .*too short"):
        mpt.lib()
    _goes_on_through_the_checks()


def test_the_library_is_built_where_the_native_calls_cannot_be(monkeypatch, tmp_path):
    from paper_1710_03740_amd import build
    commands = []

    class Compiler:
        returncode = 0

        def __init__(self, cmd, **_):
            commands.append(cmd)

        def communicate(self):
            return "", None
    monkeypatch.setattr(build.subprocess, "Popen", Compiler)
    monkeypatch.setattr(build, "_run", commands.append)
    monkeypatch.setattr(build, "CALLS", str(tmp_path / "_calls.so"))
    for there in (True, False):
        (tmp_path / "_calls.so").write_bytes(b"of an earlier build")
        commands.clear()
        if not there:
            which = build.shutil.which
            monkeypatch.setattr(build.shutil, "which", lambda name: None if name == "g++" else which(name))
        assert build._calls_missing() == (None if there else "g++")
        assert build.build(verbose=False) == build.LIB and commands[-1][-1].endswith("host.cpp.o") and build.LIB in commands[-1]
        assert any(c[0] == "g++" for c in commands) == there == (tmp_path / "_calls.so").exists()


def _calls():
    g = torch.Generator(device="cuda")
    g.manual_seed(5)

    def n(*shape, dtype=F16):
        return torch.randn(shape, device="cuda", generator=g).to(dtype)

    def cut(*shape):                                                       # rows at an odd stride
        return n(shape[0], shape[1] + 3)[:, :shape[1]]

    fl = lambda: torch.zeros(1, device="cuda", dtype=I32)  # noqa: E731
    ws = torch.empty(1 << 20, device="cuda", dtype=F32)
    M, N, K, C = 40, 24, 72, 8
    x, w, vec = n(2, 5, 6, C), n(16, 3, 3, C), lambda: n(C, dtype=F32).abs_().add_(0.1)  # noqa: E731
    lab = torch.randint(0, N, (M,), device="cuda", dtype=I32, generator=g)
    p = [(n(s, dtype=F32), n(s, dtype=F32), n(s), n(s)) for s in (7, 300)]
    sc = mpt.scaler_to_device(mpt.mpt_scaler_init(8.0, 2))
    factor = n(1, dtype=F32).abs_()
    hp = mpt.mpt_opt_params(1e-2, 0.9, 0.99, 1e-8, 0.01, 0.1, 0.01, 0.5, 0.5, factor.data_ptr())
    hp.kept = factor
    sq, nws = torch.ones(1, device="cuda", dtype=torch.float64), torch.empty(mpt.mpt_grad_norm_workspace_bytes(), device="cuda", dtype=torch.uint8)
    second = n(300, dtype=F32).abs_()
    return [
        ("gemm_fwd", (n(M, K), n(K, N), n(M, N), ws), 2), ("gemm_fwd", (cut(M, K), cut(K, N), cut(M, N), None), 2),
        ("gemm_fwd_relu", (n(M, K), n(K, N), n(M, N), None), 2), ("gemm_dgrad", (n(M, N), n(K, N), n(M, K), ws), 2),
        ("gemm_dgrad_relu", (n(M, N), cut(K, N), cut(M, K), n(M, K), None), 3),
        ("gemm_wgrad", (n(M, K), n(M, N), n(K, N), False, fl(), ws), 2), ("gemm_wgrad", (n(M, K), n(M, N), n(K, N, dtype=F32), True, None, ws), 2),
        ("conv3x3_fwd", (x, w, n(2, 5, 6, 16), None), 2), ("conv3x3_dgrad", (n(2, 5, 6, 16), w, n(2, 5, 6, C), None), 2),
        ("conv3x3_wgrad", (x, n(2, 5, 6, 16), n(16, 3, 3, C), fl(), ws), 2), ("unscale_check", (n(99), 0.5, fl(), n(99, dtype=F32)), 3),
        ("master_update", (*p[0], 0.5, 1, 0.9, fl(), sc), 0), ("master_update", (p[1][0], None, n(300, dtype=F32), p[1][3], 0.5, 0.1, 0.0, None, None), 3),
        ("master_update_multi", (p, 0.5, 0.1, 0.9, fl(), None), None), ("loss_scale_update_dev", (sc.clone(), fl()), 0),
        ("master_update_fused", (*p[1][:3], n(300, dtype=F32), n(300, dtype=F32), n(300), 0.5, 0.1, 0.9, fl(), sc), 3),
        ("master_update_fused", (p[1][0], None, n(300, dtype=F32), n(300, dtype=F32), None, n(300), 0.5, 0.1, 0.9, fl(), None), 3),
        ("optimizer_update", ("adam", hp, p[1][0], second, second.clone(), p[1][2], p[1][3], 0.5, fl(), sc), 2),
        ("optimizer_update", ("adagrad", hp, p[1][0], second, None, n(300, dtype=F32), p[1][3], 0.5, None, None), 2),
        ("grad_sumsq", (p[1][2], 0.5, sq, nws, fl(), True, sc), 2), ("clip_factor", (sq, 0.5, n(1, dtype=F32), n(1, dtype=F32)), 3), ("clip_factor", (sq, 0.5, n(1, dtype=F32), None), 2),
        ("grad_stats", (n(999), torch.zeros(42, device="cuda", dtype=torch.int64), fl(), False), 1), ("relu_fwd", (n(77), n(77)), 1),
        ("softmax_xent_scaled", (n(M, N), lab, 64, n(M, N), fl().float(), n(M, dtype=F32)), 3), ("softmax_xent_scaled", (cut(M, N), lab, 64.0, cut(M, N), None, None), 3),
        ("add_fp16", (n(77), n(77), n(77)), 2), ("relu_bwd", (n(77), n(77), n(77)), 2), ("bn_stats", (n(60, C), vec(), vec(), ws), 2),
        ("bn_apply", (n(60, C), vec(), vec(), vec(), vec(), 1e-5, n(60, C), True), 6), ("bn_bwd_reduce", (n(60, C), n(60, C), vec(), vec(), 1e-5, vec(), vec(), ws), 6),
        ("bn_bwd_apply", (n(60, C), n(60, C), vec(), vec(), vec(), 1e-5, vec(), vec(), n(60, C)), 8),
        ("lstm_cell_fwd", (n(3, 32), None, None, n(3, 8), n(3, 32), n(3, 8), n(3, 8)), 6), ("lstm_cell_fwd", (n(3, 32), cut(3, 32), n(32, dtype=F32), n(3, 8), n(3, 32), cut(3, 8), n(3, 8)), 5),
        ("lstm_cell_bwd", (n(3, 8), None, n(3, 32), n(3, 8), n(3, 8), n(3, 32), n(3, 8)), 5), ("lstm_cell_bwd", (n(3, 8), n(3, 8), n(3, 32), n(3, 8), cut(3, 8), n(3, 32), n(3, 8)), 6),
    ]


def _copy(a):
    if isinstance(a, torch.Tensor):
        return torch.empty_strided(a.shape, a.stride(), dtype=a.dtype, device=a.device).copy_(a)
    return [tuple(_copy(t) for t in e) for e in a] if isinstance(a, list) else a


def _same(a, b):
    if isinstance(a, torch.Tensor):
        return torch.equal(a.contiguous().view(torch.uint8), b.contiguous().view(torch.uint8))
    return all(_same(x, y) for e, f in zip(a, b) for x, y in zip(e, f)) if isinstance(a, list) else a == b


@pytest.mark.gpu
def test_both_ways_lead_to_the_same_bits(monkeypatch):
    mpt.lib()
    native = mpt._native
    for name, args, out in _calls():
        mine, theirs = [_copy(a) for a in args], [_copy(a) for a in args]
        st = getattr(native, name)(*mine)
        assert st == 0, (name, st)
        with monkeypatch.context() as m:
            m.setattr(mpt, "_native", mpt._NotLoaded())
            getattr(mpt, "mpt_" + name)(*theirs)
        torch.cuda.synchronize()
        for k, (a, b) in enumerate(zip(mine, theirs)):
            if a is not b and not (isinstance(a, torch.Tensor) and (a.numel() == 1 << 20 or a.dtype is torch.uint8 and a.numel() > 32)):  # (not the workspaces)
                assert _same(a, b), (name, k)
        if out is not None:
            assert not _same(mine[out], args[out]), name                    # it did run


@pytest.mark.gpu
def test_errors_and_unusual_forms_end_as_they_did():
    mpt.lib()
    X, W, Y = (torch.zeros(64, 64, device="cuda", dtype=F16) for _ in range(3))
    nat = mpt._native
    assert nat.gemm_fwd(X, W, Y, None) == 0
    assert nat.gemm_fwd(X.as_subclass(Sub), W, Y, None) is None
    assert nat.gemm_fwd(X.t(), W, Y[:, ::2], None) is None and nat.gemm_fwd(X, W.float(), Y, None) is None
    assert nat.gemm_wgrad(X, W, Y, True, None, None) is None                # accumulating needs FP32
    w, s, h, hp = torch.zeros(8, device="cuda"), torch.zeros(8, device="cuda"), torch.zeros(8, device="cuda", dtype=F16), mpt.mpt_opt_params()
    assert nat.optimizer_update("adam", hp, w, s, None, h, h.clone(), 1.0, None, None) is None        # Adam without its second state
    assert nat.optimizer_update("lamb", hp, w, s, None, h, h.clone(), 1.0, None, None) is None
    assert nat.optimizer_update("nesterov", mpt.mpt_scaler(), w, s, None, h, h.clone(), 1.0, None, None) is None
    with torch.overrides.TorchFunctionMode():
        assert nat.gemm_fwd(X, W, Y, None) is None
    with pytest.raises(ValueError, match="W: shape"):
        mpt.mpt_gemm_fwd(X, W[:32], Y)
    with pytest.raises(mpt.MptError, match="mpt_gemm_fwd failed: -4"):      # workspace too small: the library's own answer
        mpt.mpt_gemm_fwd(torch.zeros(64, 8192, device="cuda", dtype=F16), torch.zeros(8192, 64, device="cuda", dtype=F16), Y, torch.zeros(4, device="cuda"))
    mpt.mpt_gemm_fwd(X.as_subclass(Sub), W, Y)


@pytest.mark.gpu
def test_numbers_and_switches_of_any_class_go_the_native_way(monkeypatch):
    """A learning rate or a scale out of numpy, a switch that is a number: what ctypes and Python's `if` take."""
    import numpy as np

    class Scale(float):
        def __float__(self):                                               # neither way asks for this
            return 3.0
    mpt.lib()
    native, g = mpt._native, torch.arange(64, device="cuda").to(F16)
    for x in (0.1, np.float64(0.1), Scale(0.1), np.float32(0.1), 1, True, np.int64(2), torch.tensor(0.1)):
        out, want, fl = torch.zeros(64, device="cuda"), torch.zeros(64, device="cuda"), torch.zeros(1, device="cuda", dtype=I32)
        assert native.unscale_check(g, x, fl, out) == 0, type(x)
        with monkeypatch.context() as m:
            m.setattr(mpt, "_native", mpt._NotLoaded())
            mpt.mpt_unscale_check(g, x, fl, want)
        assert torch.equal(out.view(I32), want.view(I32)) and float(out[10]) > 0
    assert native.unscale_check(g, np.float64(1e300), fl, out) == native.unscale_check(g, 1e300, fl, out) != 0     # infinite in 32 bits: refused
    for x in ("0.1", None, 10 ** 400, [0.1]):                              # left to the checks and ctypes, which say why
        assert native.unscale_check(g, x, fl, out) is None, type(x)
        with pytest.raises((TypeError, ctypes.ArgumentError)):
            mpt.mpt_unscale_check(g, x, fl, out)
    X, W = torch.ones(64, 64, device="cuda", dtype=F16), torch.zeros(64, 64, device="cuda")
    for switch, sum_ in ((0, 64), (1, 128), (np.bool_(True), 192), ("yes", 256), (None, 64)):
        assert native.gemm_wgrad(X, X, W, switch, None, None) == 0
        assert bool((W == sum_).all()), switch
    assert native.gemm_wgrad(X, X, W, np.zeros(2), None, None) is None    # neither true nor false
