"""The binding's native calls: the ones they take give what the Python code
gives, and every other one reaches the Python code and its errors."""

import numpy as np
import pytest

from paper_2603_06492_amd import inputs as inp
from paper_2603_06492_amd import noble


def test_native_leaves_other_calls_to_python():
    """CPU tensors, wrong argument counts and non-tensors return None; the
    public call then raises its own error."""
    torch = pytest.importorskip("torch")
    n = noble._native()
    x, W = torch.zeros(4, 64), torch.zeros(64, 64)
    assert n.forward() is None and n.backward() is None
    assert n.module_forward() is None and n.module_backward() is None
    none = (None,) * 7
    assert n.forward(False, 0, 2, 1, x, W, None, *none, x, None, None) is None
    assert n.forward(False, 0, None, 1, x, W, None, *none, x, None, None) is None
    assert n.forward(False, 0, 2, 1, "x", W, None, *none, x, None, None) is None
    with pytest.raises(ValueError, match="must be on the GPU"):
        noble.noble_linear_fwd(x, W, None, *none, x, None, None)


@pytest.mark.parametrize("groups", [2 ** 63, 2 ** 70, -2 ** 70, -1, 0, 2 ** 40])
def test_native_leaves_groups_out_of_range_to_python(groups):
    """Past a C long too: no error of the native code's own."""
    torch = pytest.importorskip("torch")
    n = noble._native()
    x, W = torch.zeros(4, 64), torch.zeros(64, 64)
    none = (None,) * 7
    assert n.forward(False, 0, 2, groups, x, W, None, *none, x, None, None) is None
    assert n.backward(0, 2, groups, x, x, W, *none, None, x, W, None, *none, None) is None
    assert n.module_forward(True, 0, 2, groups, x, W, None, *none) is None
    assert n.module_backward(False, 0, 2, groups, x, x, W, *none, None) is None
    with pytest.raises(ZeroDivisionError if groups == 0 else ValueError):
        noble.noble_linear_fwd(x, W, None, *none, x, None, None, groups=groups)


class Recorder:
    """The native module, noting each call's name and whether it served the call (returned something)."""

    def __init__(self, native):
        self.native, self.calls = native, []

    def __getattr__(self, name):
        def call(*a):
            out = getattr(self.native, name)(*a)
            self.calls.append((name, out is not None))
            return out
        return call


# 1250 rows per batch entry: dW and the rank products split over K, so that the
# reduction stores their gradients; 37: the products themselves store dW and dW_up
CASES = [("cosnet", 1, 40, "bf16", 37), ("cosnet", 3, 16, "bf16", 37), ("gelu", 1, 40, "bf16", 37),
         ("cosnet3", 3, 24, "bf16", 37), ("cosnet", 1, 0, "bf16", 37), ("cosnet", 1, 24, "f32", 37),
         ("cosnet", 1, 64, "bf16", 1250), ("cosnet", 3, 32, "bf16", 1250), ("cosnet", 1, 0, "bf16", 1250)]


@pytest.mark.gpu
@pytest.mark.parametrize("act,G,r,dt,n", CASES, ids=[f"{a}_g{g}_r{r}_{d}_{n}" for a, g, r, d, n in CASES])
def test_native_equals_python(act, G, r, dt, n, monkeypatch):
    """Forward and gradients of the module, with the native calls and without,
    bit for bit (db and the frequency / phase gradients, summed atomically, to
    float32 rounding)."""
    import torch
    sd = torch.bfloat16 if dt == "bf16" else torch.float32
    print(f"[binding] {act} groups={G} r={r} {dt} {n}", flush=True)
    m = noble.NobleLinear(104, 264, r, dtype=sd, activation=act, groups=G, seed=3)
    g = torch.Generator(device="cuda").manual_seed(5)
    x = torch.randn(2, n, 104, device="cuda", generator=g).to(sd).requires_grad_(True)
    dy = torch.randn(2, n, 264, device="cuda", generator=g).to(sd)

    def step():
        m.zero_grad(set_to_none=True)
        x.grad = None
        y = m(x)
        y.backward(dy)
        with torch.no_grad():
            yi = m(x)
        return {"y": y.detach(), "yi": yi, "dx": x.grad, **{n: p.grad for n, p in m.named_parameters()}}

    native = noble._native()
    rec = Recorder(native)
    monkeypatch.setattr(noble, "_native_module", rec)
    fast = step()
    # the recorded forward, the backward and the inference forward, each served
    assert rec.calls == [("module_forward", True), ("module_backward", True), ("module_forward", True)]

    class Off:
        def __getattr__(self, name):
            return lambda *a: None

    monkeypatch.setattr(noble, "_native_module", Off())
    slow = step()
    monkeypatch.setattr(noble, "_native_module", native)
    assert fast.keys() == slow.keys()
    for k, a in fast.items():
        b = slow[k]
        assert a.shape == b.shape and a.dtype == b.dtype, k
        if k in ("b", "omega1", "phi1", "omega2", "phi2"):
            np.testing.assert_allclose(a.double().cpu(), b.double().cpu(), rtol=1e-4,
                                       atol=1e-5 * float(b.abs().max()), err_msg=k)
        else:
            assert torch.equal(a, b), k


@pytest.mark.gpu
@pytest.mark.parametrize("act,G,r,dt", [c[:4] for c in CASES[:6]], ids=[f"{a}_g{g}_r{r}_{d}" for a, g, r, d, _ in CASES[:6]])
def test_native_serves_the_public_functions(act, G, r, dt, monkeypatch):
    """noble_linear_fwd, _fwd_static and _bwd on ordinary tensors, the static forward's y as noble_linear_fwd's."""
    import torch
    sd = torch.bfloat16 if dt == "bf16" else torch.float32
    code = noble.NOBLE_BF16 if dt == "bf16" else noble.NOBLE_F32
    T, di, do = 37, 104, 264
    print(f"[binding] public {act} groups={G} r={r} {dt}", flush=True)
    m = noble.NobleLinear(di, do, r, dtype=sd, activation=act, groups=G, seed=3)
    reserve, scratch = noble.alloc_workspace(T, di, do, r, code, groups=G, activation=act)
    x, dy = torch.randn(T, di, device="cuda").to(sd), torch.randn(T, do, device="cuda").to(sd)
    y, ys, dx = dy.new_empty(T, do), dy.new_empty(T, do), torch.empty_like(x)
    with torch.no_grad():
        branch = m._branch()
        grads = [None if t is None else torch.empty(t.shape, device="cuda") for t in (m.W, m.b, *branch)]
    dW, db, dWd, do1, dp1, dM, do2, dp2, dWu = grads
    rec = Recorder(noble._native())
    monkeypatch.setattr(noble, "_native_module", rec)
    kw = dict(activation=act, groups=G)
    noble.noble_linear_fwd(x, m.W, m.b, *branch, y, reserve, scratch, **kw)
    noble.noble_linear_fwd_static(x, m.W, m.b, *branch, ys, None, **kw)
    noble.noble_linear_bwd(dy, x, m.W, *branch, reserve, dx, dW, db, dWd, dM, dWu, do1, dp1, do2, dp2, scratch, **kw)
    assert rec.calls == [("forward", True), ("forward", True), ("backward", True)]
    assert torch.equal(y, ys)


@pytest.mark.gpu
def test_errors_stay_the_binding_s(monkeypatch):
    import torch
    from paper_2603_06492_amd.runner import DeviceProblem
    p = inp.draw_projection("binding", 16, 64, 64, 8, "bf16", seed=4)
    dp = DeviceProblem(p)
    rec = Recorder(noble._native())
    monkeypatch.setattr(noble, "_native_module", rec)
    dp.fwd()
    assert rec.calls == [("forward", True)]
    y = dp.y
    for bad, err in ((y[:8], ValueError), (y.float(), TypeError), (y.cpu(), ValueError), (y.t(), ValueError)):
        dp.y = bad
        with pytest.raises(err):
            dp.fwd()
        assert rec.calls[-1] == ("forward", False)
    dp.y = y
    scratch, dp.scratch = dp.scratch, dp.scratch[:16]
    with pytest.raises(noble.NobleError):
        dp.fwd()
    assert rec.calls[-1] == ("forward", True)   # the library's own status
    dp.scratch = scratch
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):   # the current stream of the call
        dp.fwd()
    assert rec.calls[-1] == ("forward", True)
    s.synchronize()


@pytest.mark.gpu
def test_function_without_w_down_is_refused_by_the_forward():
    """The plain layer's W_down has no columns; None has no width, which the forward has to say and not the backward."""
    import torch
    x = torch.zeros(4, 64, device="cuda", requires_grad=True)
    W = torch.zeros(64, 64, device="cuda")
    with pytest.raises(AttributeError):
        noble.NobleLinearFunction.apply(x, W, None, *(None,) * 7)
    y = noble.NobleLinearFunction.apply(x, W, None, W.new_empty(64, 0), *(None,) * 5, W.new_empty(0, 64))
    y.sum().backward()
    assert x.grad.shape == x.shape
