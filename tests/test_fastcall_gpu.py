"""The native form of the Python calls (csrc/dwconv_fastcall.cpp) against the general one of binding.py: the same bits for what it takes,
and everything else left to binding.py - its errors, its conversions, wrappers of transforms, torch function and dispatch modes."""
import ctypes
import threading

import numpy as np
import pytest
import torch

from paper_2604_25422_amd import binding

pytestmark = pytest.mark.gpu


@pytest.fixture
def general(monkeypatch):
    """binding.py without the native calls, as a context to switch to."""
    binding.lib()

    def run(call):
        with monkeypatch.context() as m:
            m.setattr(binding, "_fast", binding._Declines)
            return call()
    return run


def _tensors(dtype=torch.float32, B=3, C=5, L=100, K=9):
    g = torch.Generator(device="cuda").manual_seed(1)
    x, dy = (torch.randn(B, C, L, device="cuda", generator=g).to(dtype) for _ in range(2))
    w = torch.randn(C, K, device="cuda", generator=g).to(dtype)
    return x, dy, w, binding.new_workspace(x, K, 4)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("given", [False, True])
def test_same_results(general, dtype, given):
    x, dy, w, ws = _tensors(dtype)
    from paper_2604_25422_amd import _fastcall
    assert _fastcall.fwd(x, w, 4, None) is not None and _fastcall.bwd(dy, x, w, 4, ws, None, None) is not None      # (it does take them)
    x.requires_grad_()
    w = torch.nn.Parameter(w)
    assert _fastcall.bwd_input(x, w, 4, None) is not None and _fastcall.bwd_weight(x, dy, 9, 4, ws, w.detach()) is not None
    w.data.copy_(_tensors(dtype)[2])
    out = lambda t: torch.full_like(t, float("nan")).detach() if given else None      # noqa: E731
    calls = (lambda: binding.dwconv_fwd(x, w, 4, out=out(x)), lambda: binding.dwconv_bwd_input(dy, w, 4, out=out(dy)),
             lambda: binding.dwconv_bwd_weight(x, dy, 9, 4, workspace=ws, out=out(w)),
             lambda: binding.dwconv_bwd(dy, x, w, 4, workspace=ws, out_dx=out(dy), out_dw=out(w)))
    for call in calls:
        a, b = call(), general(call)
        a, b = (a, b) if isinstance(a, tuple) else ((a,), (b,))
        for s, t in zip(a, b):
            assert type(s) is type(t) and s.dtype == t.dtype and s.shape == t.shape and s.device == t.device
            assert not s.requires_grad and torch.equal(s, t)
    y = torch.empty_like(x).detach()
    assert binding.dwconv_fwd(x, w, 4, out=y) is y


def test_takes_the_current_stream():
    x, dy, w, ws = _tensors(L=4096)
    want = binding.dwconv_fwd(x, w, 4)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    g = torch.cuda.CUDAGraph()
    y = torch.empty_like(x)
    with torch.cuda.graph(g, stream=side):                       # (a launch on another stream than the capture's would end it)
        binding.dwconv_fwd(x, w, 4, out=y)
        dw = binding.dwconv_bwd_weight(x, dy, 9, 4, workspace=ws)
    for _ in range(3):
        y.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(y, want) and torch.equal(dw, binding.dwconv_bwd_weight(x, dy, 9, 4, workspace=ws))


def test_leaves_errors_and_conversions_to_the_general_form(general):
    x, dy, w, ws = _tensors()
    wrong = (lambda: binding.dwconv_fwd(x.transpose(1, 2), w, 4), lambda: binding.dwconv_fwd(x, w.double(), 4),
             lambda: binding.dwconv_fwd(x, w[:3], 4), lambda: binding.dwconv_fwd(x.half(), w.half(), 4), lambda: binding.dwconv_fwd(x, w, 9),
             lambda: binding.dwconv_fwd(x, w, -1), lambda: binding.dwconv_fwd(x, w, 4, out=x[:2]), lambda: binding.dwconv_fwd(x, w.cpu(), 4),
             lambda: binding.dwconv_bwd_input(dy, w, "pad"), lambda: binding.dwconv_bwd_weight(x, dy[:2], 9, 4, workspace=ws),
             lambda: binding.dwconv_bwd_weight(x, dy, 9, 4, workspace=ws[:16]), lambda: binding.dwconv_bwd_weight(x, dy, 9, 4, workspace=ws[1:]),
             lambda: binding.dwconv_bwd_weight(x, dy, 0, 0, workspace=ws), lambda: binding.dwconv_bwd(dy, x, w, 4, workspace=ws.cpu()),
             lambda: binding.dwconv_fwd(x[:0], w, 4), lambda: binding.dwconv_fwd(x.cpu(), w, 4), lambda: binding.dwconv_fwd(None, w, 4))
    for i, call in enumerate(wrong):
        kinds = []
        for form in (lambda: call(), lambda: general(call)):
            with pytest.raises(Exception) as e:
                form()
            kinds.append((type(e.value), str(e.value)))
        assert kinds[0] == kinds[1], (i, kinds)
    for pad in (4.0, np.int64(4), True):
        assert torch.equal(binding.dwconv_fwd(x, w, pad), general(lambda: binding.dwconv_fwd(x, w, pad)))
    assert torch.equal(binding.dwconv_bwd_weight(x, dy, 9, 4), binding.dwconv_bwd_weight(x, dy, 9, 4, workspace=ws))


def test_leaves_modes_and_subclasses_to_the_general_form():
    from torch.overrides import TorchFunctionMode
    from torch.utils._python_dispatch import TorchDispatchMode
    x, dy, w, ws = _tensors()

    class Functions(TorchFunctionMode):
        seen = 0

        def __torch_function__(self, func, types, args=(), kwargs=None):
            Functions.seen += func is torch.empty_like
            return func(*args, **(kwargs or {}))

    class Dispatch(TorchDispatchMode):
        seen = 0

        def __torch_dispatch__(self, func, types, args=(), kwargs=None):
            Dispatch.seen += "empty_like" in str(func)
            return func(*args, **(kwargs or {}))

    class Sub(torch.Tensor):
        pass

    want = binding.dwconv_fwd(x, w, 4)
    for mode in (Functions, Dispatch):
        with mode():
            assert torch.equal(binding.dwconv_fwd(x, w, 4), want)
        assert mode.seen == 1
    assert type(binding.dwconv_fwd(x.as_subclass(Sub), w, 4)) is Sub


def test_leaves_wrappers_of_transforms_to_the_general_form(general):
    x, dy, w, ws = _tensors()
    mapped = lambda: torch.vmap(lambda t: binding.dwconv_fwd(t, w, 4))(torch.stack([x, x]))      # noqa: E731
    kinds = []
    for form in (lambda: mapped(), lambda: general(mapped)):
        with pytest.raises(Exception) as e:
            form()
        kinds.append((type(e.value), str(e.value)))
    assert kinds[0] == kinds[1]


def _all_calls(x, dy, w, ws, given):
    out = (lambda t: torch.empty_like(t)) if given else (lambda t: None)
    return (lambda: binding.dwconv_fwd(x, w, 4, out=out(x)), lambda: binding.dwconv_bwd_input(dy, w, 4, out=out(dy)),
            lambda: binding.dwconv_bwd_weight(x, dy, 9, 4, workspace=ws, out=out(w)),
            lambda: binding.dwconv_bwd(dy, x, w, 4, workspace=ws, out_dx=out(dy), out_dw=out(w)))


@pytest.mark.parametrize("given", [False, True])
def test_library_calls_run_without_the_interpreter_lock(given):
    """In the place of the library's functions one that says whether its thread holds the lock: 1, a status that is raised, or 0."""
    from paper_2604_25422_amd import _fastcall
    x, dy, w, ws = _tensors()
    held = ctypes.cast(ctypes.pythonapi.PyGILState_Check, ctypes.c_void_p).value
    assert ctypes.PYFUNCTYPE(ctypes.c_int)(held)() == 1
    _fastcall.setup(held, held, held, held, binding._current_device, binding._raw_stream, binding._check)
    try:
        for call in _all_calls(x, dy, w, ws, given):
            call()
        # ... and the lock is back when the status is raised
        status = ctypes.cast(ctypes.pythonapi.Py_IsInitialized, ctypes.c_void_p).value
        _fastcall.setup(status, status, status, status, binding._current_device, binding._raw_stream, binding._check)
        for call in _all_calls(x, dy, w, ws, given):
            with pytest.raises(binding.DwconvError):
                call()
    finally:
        binding._load_fastcall(binding.lib())


def test_calls_from_two_threads(general):
    """Each thread on a stream of its own, with tensors and a workspace of its own."""
    jobs, wrong = [], []
    for i, dtype in enumerate((torch.float32, torch.bfloat16)):
        x, dy, w, ws = _tensors(dtype, L=100 + 40 * i)
        jobs.append((_all_calls(x, dy, w, ws, False), [general(call) for call in _all_calls(x, dy, w, ws, False)]))
    torch.cuda.synchronize()

    def work(calls, want):
        try:
            with torch.cuda.stream(torch.cuda.Stream()):
                for _ in range(50):
                    got = [call() for call in calls]
                    torch.cuda.current_stream().synchronize()
                    for a, b in zip(got, want):
                        for s, t in zip(a, b) if isinstance(a, tuple) else ((a, b),):
                            if not torch.equal(s, t):
                                wrong.append("another result")
        except Exception as e:
            wrong.append(repr(e))

    threads = [threading.Thread(target=work, args=job) for job in jobs]
    for t in threads:
        t.start()
    for t in threads:
        t.join(60)
    assert not any(t.is_alive() for t in threads) and not wrong, wrong[:3]
