"""The autograd wrapper's native host path against the Python one: the same
library calls, so the same bits; and the cases it leaves to the Python path."""
import pytest
import torch

from paper_2608_10805_amd import autograd

pytestmark = pytest.mark.gpu


def params(C, k, L, bias, seed=0):
    g = torch.Generator(device="cuda").manual_seed(seed)
    r = lambda *s: (torch.rand(s, generator=g, device="cuda") - 0.5).requires_grad_(True)  # noqa: E731
    return r(C, k, k), r(C), r(C) if bias else None, [r(4 * C, k, k) for _ in range(L)], [r(4 * C) for _ in range(L)]


def grads_of(fn, x, p, dy, need_x=True):
    bw, bs, bb, lw, ls = p
    x = x.detach().requires_grad_(need_x)
    y = fn(x, bw, bs, lw, ls, bb)
    leaves = ([x] if need_x else []) + [t for t in (bw, bs, bb, *lw, *ls) if t is not None]
    return (y.detach(), *torch.autograd.grad(y, leaves, dy))


def python_path(x, bw, bs, lw, ls, bb):
    return autograd.WTConvFunction.apply(x, bw, bs, bb, *lw, *ls)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16, torch.float16])
@pytest.mark.parametrize("H,W,k,L,bias,need_x", [(13, 11, 5, 2, True, True), (28, 28, 3, 0, False, True),
                                                 (130, 128, 5, 2, True, False), (7, 7, 7, 1, False, False)])
def test_same_bits_as_the_python_path(dtype, H, W, k, L, bias, need_x):
    assert autograd._load_native(), "the native host path is not built"
    p = params(3, k, L, bias)
    x = torch.randn(4, 3, H, W, device="cuda").to(dtype)
    dy = torch.randn(4, 3, H, W, device="cuda").to(dtype)
    got = grads_of(autograd.wtconv, x, p, dy, need_x)
    want = grads_of(python_path, x, p, dy, need_x)
    assert len(got) == len(want) and all(torch.equal(a, b) for a, b in zip(got, want))
    # a gradient that is not contiguous, and on another stream
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        odd = grads_of(autograd.wtconv, x, p, dy.transpose(2, 3).contiguous().transpose(2, 3), need_x)
    torch.cuda.current_stream().wait_stream(s)
    assert all(torch.equal(a, b) for a, b in zip(odd, want))


def test_other_cases_take_the_python_path():
    bw, bs, bb, lw, ls = params(3, 5, 1, False)
    x = torch.randn(2, 3, 16, 16, device="cuda")
    ext = autograd._load_native()
    t = x.transpose(2, 3)  # not contiguous: converted
    assert ext.apply(t, bw, bs, None, [*lw, *ls]) is None
    assert torch.equal(autograd.wtconv(t, bw, bs, lw, ls), autograd.wtconv(t.contiguous(), bw, bs, lw, ls))
    with pytest.raises(ValueError):
        autograd.wtconv(x.double(), bw, bs, lw, ls)
    with pytest.raises(ValueError):
        autograd.wtconv(x, bw.detach().half(), bs, lw, ls)
    with pytest.raises(ValueError):
        autograd.wtconv(x[:, :2].contiguous(), bw, bs, lw, ls)
    with pytest.raises(Exception):  # forward-mode is refused, not ignored
        torch.func.jvp(lambda v: autograd.wtconv(v, bw, bs, lw, ls), (x,), (x,))
    with pytest.raises(Exception):  # so is vmap
        torch.vmap(lambda v: autograd.wtconv(v, bw, bs, lw, ls))(x[None])


def test_saved_tensor_hooks_see_the_saved_tensors():
    bw, bs, bb, lw, ls = params(3, 5, 1, True)
    x = torch.randn(2, 3, 16, 16, device="cuda", requires_grad=True)
    seen = []
    with torch.autograd.graph.saved_tensors_hooks(lambda v: (seen.append(v.shape), v)[1], lambda v: v.clone()):
        y = autograd.wtconv(x, bw, bs, lw, ls, bb)
    got = torch.autograd.grad(y, [x, bw], torch.ones_like(y))
    y = python_path(x, bw, bs, lw, ls, bb)
    want = torch.autograd.grad(y, [x, bw], torch.ones_like(y))
    assert len(seen) == 6 and all(torch.equal(a, b) for a, b in zip(got, want))


def test_dispatch_mode_around_the_backward_alone():
    """A mode that is entered after the forward sees the backward's
    allocations, as on the Python path; it does not make the call fail."""
    from torch.utils._python_dispatch import TorchDispatchMode

    class Count(TorchDispatchMode):
        n = 0

        def __torch_dispatch__(self, func, types, args=(), kwargs=None):
            self.n += 1
            return func(*args, **(kwargs or {}))

    bw, bs, bb, lw, ls = params(3, 5, 1, True)
    x = torch.randn(2, 3, 16, 16, device="cuda", requires_grad=True)
    got = []
    for fn in (autograd.wtconv, python_path):
        y = fn(x, bw, bs, lw, ls, bb)
        with Count() as mode:
            got.append(torch.autograd.grad(y, [x, bw, bb], torch.ones_like(y)))
        assert mode.n > 0
    assert all(torch.equal(a, b) for a, b in zip(*got))


class Tagged(torch.Tensor):
    """A subclass with torch functions of its own and no dispatch."""


class Counted(torch.Tensor):
    calls = 0

    @classmethod
    def __torch_function__(cls, func, types, args=(), kwargs=None):
        cls.calls += 1
        return super().__torch_function__(func, types, args, kwargs)


def test_tensor_subclasses_keep_their_type_and_functions():
    bw, bs, bb, lw, ls = params(3, 5, 1, True)
    x = torch.randn(2, 3, 16, 16, device="cuda")
    y = autograd.wtconv(x.as_subclass(Tagged), bw, bs, lw, ls, bb)
    assert type(y) is Tagged and torch.equal(y.as_subclass(torch.Tensor), autograd.wtconv(x, bw, bs, lw, ls, bb))
    for i in range(3):  # x, a kernel, a level's kernel
        t = [x, bw.detach(), lw[0].detach()]
        t[i] = t[i].as_subclass(Counted)
        before = Counted.calls
        autograd.wtconv(t[0], t[1], bs, [t[2]], ls, bb)
        assert Counted.calls > before


def test_torch_function_mode_sees_the_call():
    from torch.overrides import TorchFunctionMode

    class Names(TorchFunctionMode):
        def __torch_function__(self, func, types, args=(), kwargs=None):
            seen.append(func.__name__)
            return func(*args, **(kwargs or {}))

    bw, bs, bb, lw, ls = params(3, 5, 1, False)
    x, names = torch.randn(2, 3, 16, 16, device="cuda"), []
    for fn in (autograd.wtconv, python_path):
        seen = []
        with Names():
            fn(x, bw, bs, lw, ls, bb)
        names.append(seen)
    assert "empty_like" in names[1] and "empty_like" in names[0]


def test_a_type_error_of_a_pack_hook_is_raised_at_once():
    """The forward is not run a second time over it."""
    bw, bs, bb, lw, ls = params(3, 5, 1, False)
    x = torch.randn(2, 3, 16, 16, device="cuda", requires_grad=True)
    calls = []

    def pack(t):
        calls.append(t.shape)
        if len(calls) == 1:
            raise TypeError("pack")
        return t

    with torch.autograd.graph.saved_tensors_hooks(pack, lambda t: t), pytest.raises(TypeError, match="pack"):
        autograd.wtconv(x, bw, bs, lw, ls)
    assert len(calls) == 1


def test_errors_of_the_backward_are_the_python_path_s(monkeypatch):
    """Their types too: saved tensors that a hook hands back in another layout
    or dtype, and a call that the library refuses."""
    import ctypes

    from paper_2608_10805_amd import binding

    bw, bs, bb, lw, ls = params(3, 5, 1, True)
    x = torch.randn(2, 3, 16, 16, device="cuda", requires_grad=True)
    for unpack in (lambda t: t.mT.contiguous().mT if t.dim() == 4 else t, lambda t: t.half() if t.dim() == 3 else t):
        for fn in (autograd.wtconv, python_path):
            with torch.autograd.graph.saved_tensors_hooks(lambda t: t, unpack):
                y = fn(x, bw, bs, lw, ls, bb)
            with pytest.raises(ValueError, match="contiguous|float32"):
                y.sum().backward()

    ext, lib = autograd._load_native(), binding.load()
    refuse = ctypes.CFUNCTYPE(ctypes.c_int)(lambda: 8)  # WTCONV_ERR_UNSUPPORTED, whatever the arguments
    address = lambda f: ctypes.cast(f, ctypes.c_void_p).value  # noqa: E731
    try:
        ext.init(*(address(getattr(lib, n)) for n in ("wtconv_forward_workspace_bytes", "wtconv_forward",
                                                      "wtconv_backward_workspace_bytes")),
                 address(refuse), autograd._backward)
        monkeypatch.setattr(binding, "wtconv_backward", lambda *a: 8)
        y = autograd.wtconv(x, bw, bs, lw, ls, bb)
        with pytest.raises(binding.WTConvError) as e:
            y.sum().backward()
        assert e.value.status == 8
        monkeypatch.undo()  # the Python path is served: so is the call
        y = autograd.wtconv(x, bw, bs, lw, ls, bb)
        got = torch.autograd.grad(y, [x, bw, bb, *lw], torch.ones_like(y))
    finally:
        autograd._native = None
        autograd._load_native()
    y = python_path(x, bw, bs, lw, ls, bb)
    assert all(torch.equal(a, b) for a, b in zip(got, torch.autograd.grad(y, [x, bw, bb, *lw], torch.ones_like(y))))
