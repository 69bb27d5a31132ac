"""Work order with 3 to 7 views of large maps: the library takes view order
when it has the workspace and anchor order when it has not. Both agree with
the order asked for by name, bitwise, and the orders with each other: the
forward to the rounding of an FP32 sum, the backward bitwise."""
import pytest
import torch

from helpers import host, normwise, to_device
from paper_2601_10819_amd import synth

pytestmark = pytest.mark.gpu

LEVELS = ((80, 176), (40, 88), (20, 44), (10, 22))      # 18,700 rows a camera
# FP32 sums of N*P*L terms added in two orders: eps * sqrt(terms), and a margin of 4
SUM_TOL = 1e-6


@pytest.fixture(scope="module")
def ops():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2601_10819_amd import ops as o
    o._lib.load()
    return o


@pytest.mark.parametrize("B,cams,dtype,logits", [
    (1, 3, torch.float32, False), (1, 7, torch.bfloat16, False), (2, 3, torch.float16, False),
    (1, 5, torch.float32, True)])
def test_few_views_of_large_maps(ops, B, cams, dtype, logits):
    A = 24576 // (B * cams * 13) + 1
    p = synth.small(seed=cams, B=B, cams=cams, levels=LEVELS, C=256, G=8, A=A, P=13)
    feat, layout, loc, w = to_device(p, dtype)
    kw = {"logits": True} if logits else {}
    assert ops.forward_workspace_bytes(feat, layout, loc, w, **kw) >= 8 * B * A * 256 * 4
    # fewer than 24,576 pairs: the anchor order's workspace
    less = (feat, layout, loc[:, :A - 2], w[:, :A - 2])
    assert (ops.forward_workspace_bytes(*less, **kw) ==
            ops.forward_workspace_bytes(*less, tile={"order": "anchor"}, **kw))
    auto, view, anchor = (ops.forward(feat, layout, loc, w, tile=t, **kw) for t in
                          (None, {"order": "view"}, {"order": "anchor"}))
    noalloc = ops.forward_noalloc(feat, layout, loc, w, torch.empty_like(auto), **kw)
    go = synth.grad_out_like(p, seed=1).cuda()
    grads = [ops.backward(feat, layout, loc, w, go, tile=t, **kw) for t in
             (None, {"order": "view"}, {"order": "anchor"})]
    torch.cuda.synchronize()
    assert torch.equal(auto, view) and torch.equal(auto, noalloc)
    assert normwise(host(auto), host(anchor)) <= SUM_TOL
    for other in grads[1:]:
        assert all(torch.equal(x, y) for x, y in zip(grads[0], other))
