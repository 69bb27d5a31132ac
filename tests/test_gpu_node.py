"""The native autograd node where something other than the plain engine runs
it: compiled autograd gives the engine's own gradients. And no call of the
library is made with the interpreter lock held."""
import ctypes

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


def operands(dtype=torch.float32, needs=(True, True, True)):
    p = synth.small(seed=9, B=2, cams=3, levels=((9, 11), (4, 5)), C=32, G=4, A=6, P=3)
    feat, layout, loc, w = to_device(p, dtype)
    t = [x.detach().requires_grad_(n) for x, n in zip((feat, loc, w), needs)]
    return t, layout, synth.grad_out_like(p, seed=2).cuda()


@pytest.mark.parametrize("needs,kw", [
    ((True, True, True), {}),
    ((True, False, True), {"logits": True, "tile": {"order": "view"}}),
])
def test_compiled_autograd(ops, needs, kw):
    from torch._dynamo import compiled_autograd
    t, layout, go = operands(needs=needs)
    ask = [x for x in t if x.requires_grad]
    ref = torch.autograd.grad(ops.msda(t[0], layout, t[1], t[2], **kw), ask, go)
    for _ in range(2):                       # traced, then from its cache
        out = ops.msda(t[0], layout, t[1], t[2], **kw)
        assert out.grad_fn.name() == "MSDABackward"
        for x in ask:
            x.grad = None
        with compiled_autograd._enable(torch.compile(backend="eager")):
            out.backward(go)
        for x, y in zip(ask, ref):
            assert torch.equal(x.grad, y)


def test_interpreter_lock_is_free_in_the_library(ops):
    t, layout, go = operands()
    feat, loc, w = (x.detach() for x in t)
    lib = ops._lib.load()
    address = lambda f: ctypes.cast(f, ctypes.c_void_p).value
    sizes = address(lib.msda_forward_workspace_size), address(lib.msda_backward_workspace_size)
    holds = address(ctypes.pythonapi.PyGILState_Check)     # as a status: 0 is OK, 1 an error
    side = ops._lib.torch_side()
    side.bind(holds, sizes[0], holds, sizes[1])
    try:
        ops.forward(feat, layout, loc, w)
        ops.backward(feat, layout, loc, w, go)
        torch.autograd.grad(ops.msda(t[0], layout, t[1], t[2]), t, go)
    finally:
        side.bind(address(lib.msda_forward_ws), sizes[0], address(lib.msda_backward), sizes[1])
