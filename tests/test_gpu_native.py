"""The native path of the single call against the Python one it stands beside:
the same outputs and gradients, bitwise, under everything autograd does with a
node; and the routes that stay with the Python function."""
import pytest
import torch

from helpers import to_device
from paper_2601_10819_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ops():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2601_10819_amd import ops as o
    o._lib.load()
    return o


def operands(dtype=torch.float32, wdtype=torch.float32, needs=(True, True, True)):
    p = synth.small(seed=9, B=2, cams=3, levels=((9, 11), (4, 5)), C=32, G=4, A=6, P=3)
    feat, layout, loc, w = to_device(p, dtype)
    t = [x.detach().requires_grad_(n) for x, n in zip((feat, loc, w.to(wdtype)), needs)]
    return t, layout, synth.grad_out_like(p, seed=2).cuda()


def by_function(ops, t, layout, **kw):
    return ops.MSDAFunction.apply(*t, layout, kw.get("level_scale"), kw.get("deterministic", False),
                                  kw.get("tile"), kw.get("logits", False))


@pytest.mark.parametrize("dtype,wdtype,needs,kw", [
    (torch.float32, torch.float32, (True, True, True), {}),
    (torch.bfloat16, torch.bfloat16, (True, False, True), {"logits": True}),
    (torch.float16, torch.float32, (False, True, False), {"tile": {"order": "view"}}),
    (torch.float32, torch.float32, (True, True, True), {"deterministic": True}),
])
def test_same_as_the_function(ops, dtype, wdtype, needs, kw):
    t, layout, go = operands(dtype, wdtype, needs)
    ask = [x for x in t if x.requires_grad]
    a, b = ops.msda(t[0], layout, t[1], t[2], **kw), by_function(ops, t, layout, **kw)
    assert a.grad_fn.name() == "MSDABackward" and torch.equal(a, b)
    strided = go.transpose(1, 2).contiguous().transpose(1, 2)      # a gradient that is not contiguous
    for x, y in zip(torch.autograd.grad(a, ask, strided), torch.autograd.grad(b, ask, strided)):
        assert x.dtype == y.dtype and torch.equal(x, y)


def test_saved_tensors(ops):
    t, layout, go = operands()
    packed = []

    def pack(x):
        packed.append(x.shape)
        return x.cpu()

    with torch.autograd.graph.saved_tensors_hooks(pack, lambda x: x.cuda()):
        a = ops.msda(t[0], layout, t[1], t[2])
    assert sorted(packed) == sorted(x.shape for x in t)
    ref = torch.autograd.grad(by_function(ops, t, layout), t, go)
    for x, y in zip(torch.autograd.grad(a, t, go), ref):
        assert torch.equal(x, y)
    with pytest.raises(RuntimeError, match="second time"):
        torch.autograd.grad(a, t, go)
    b = ops.msda(t[0], layout, t[1], t[2])
    with torch.no_grad():
        t[1].add_(1.0)
    with pytest.raises(RuntimeError, match="modified by an inplace operation"):
        torch.autograd.grad(b, t, go)


def test_geometry_may_go_after_the_forward(ops):
    t, layout, go = operands()
    ref = torch.autograd.grad(by_function(ops, t, layout), t, go)
    a = ops.msda(t[0], layout, t[1], t[2])
    layout.host_shapes[:] = -1
    layout.host_starts[:] = -1
    del layout
    for x, y in zip(torch.autograd.grad(a, t, go), ref):
        assert torch.equal(x, y)


def test_no_gradient_asked(ops):
    t, layout, _ = operands(needs=(False, False, False))
    assert ops.msda(t[0], layout, t[1], t[2]).grad_fn is None
    t, layout, _ = operands()
    with torch.no_grad():
        assert ops.msda(t[0], layout, t[1], t[2]).grad_fn is None


def test_errors_are_the_bindings(ops):
    t, layout, go = operands()
    with pytest.raises(ValueError, match="sampling_loc must be torch.float32"):
        ops.msda(t[0], layout, t[1].double(), t[2])
    with pytest.raises(ValueError, match="contiguous"):
        ops.msda(t[0].transpose(1, 2), layout, t[1], t[2])
    with pytest.raises(ValueError, match="does not match"):
        ops.msda(t[0], layout, t[1][:, :5].contiguous(), t[2])
    with pytest.raises(ops._lib.MSDAError, match="UNSUPPORTED"):
        ops.msda(t[0], layout, t[1], t[2], tile={"waves_per_anchor": 3})
    # on the engine's thread: a gradient the library refuses
    a = ops.msda(t[0], layout, t[1], t[2], tile={"scatter": 9})
    with pytest.raises(ops._lib.MSDAError):
        torch.autograd.grad(a, t, go)


def test_followed_calls_stay_with_the_function(ops):
    t, layout, go = operands()
    class Through(torch.utils._python_dispatch.TorchDispatchMode):
        def __torch_dispatch__(self, func, types, args=(), kwargs=None):
            return func(*args, **(kwargs or {}))

    with Through():
        assert "MSDAFunction" in ops.msda(t[0], layout, t[1], t[2]).grad_fn.name()
    with pytest.raises(RuntimeError):                # no vmap rule
        torch.vmap(lambda f: ops.msda(f, layout, t[1], t[2]))(t[0].unsqueeze(0))
    with torch.autograd.forward_ad.dual_level():
        dual = torch.autograd.forward_ad.make_dual(t[0].detach(), torch.ones_like(t[0]))
        with pytest.raises(RuntimeError):            # no forward-mode rule
            ops.msda(dual, layout, t[1].detach(), t[2].detach())
