"""Calls of more waves than one launch holds (2^32 work-items): the same results
as the calls on their halves, bitwise."""
import pytest
import torch

from paper_2601_10819_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ops():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2601_10819_amd import ops as o
    o._lib.load()
    return o


def operands(cams, L, A, P, C, fdtype, wdtype, scale=1.0):
    shapes, starts, rows = synth.layout([[(3 + l, 4 + l) for l in range(L)]] * cams)
    gen = torch.Generator("cuda").manual_seed(cams + A)
    feat = torch.randn(1, rows, C, device="cuda", generator=gen).to(fdtype)
    loc = torch.rand(1, A, P, cams, 2, device="cuda", generator=gen) * 1.1 - 0.05
    w = torch.rand(1, A, P, cams, L, 1, device="cuda", dtype=wdtype, generator=gen) * scale
    return feat, shapes, starts, loc, w


def test_view_order_forward_and_batch(ops):
    A = 1_060_000                                  # 64 rows: 67.8 M waves
    feat, shapes, starts, loc, w = operands(64, 8, A, 6, 4, torch.float32, torch.bfloat16)
    layout = ops.Layout(shapes, starts)
    out = ops.forward(feat, layout, loc, w)
    for lo, hi in ((0, A // 2), (A // 2, A)):
        assert torch.equal(out[:, lo:hi], ops.forward(feat, layout, loc[:, lo:hi], w[:, lo:hi]))
    batch = ops.SceneBatch([(feat[0], layout, loc[0], w[0])], need_feat=False, need_loc=False,
                           need_w=False)
    batch.forward()
    assert torch.equal(batch.out[0], out[0])


def test_view_order_backward_and_batch(ops):
    A = 1_060_000
    feat, shapes, starts, loc, w = operands(64, 1, A, 7, 4, torch.bfloat16, torch.float32)
    layout = ops.Layout(shapes, starts)
    go = torch.randn(1, A, 4, device="cuda")
    _, gl, gw = ops.backward(feat, layout, loc, w, go, need_feat=False)
    for lo, hi in ((0, A // 2), (A // 2, A)):
        _, hl, hw = ops.backward(feat, layout, loc[:, lo:hi], w[:, lo:hi],
                                 go[:, lo:hi].contiguous(), need_feat=False)
        assert torch.equal(gl[:, lo:hi], hl) and torch.equal(gw[:, lo:hi], hw)
    batch = ops.SceneBatch([(feat[0], layout, loc[0], w[0])], need_feat=False)
    batch.grad_out[0].copy_(go[0])
    batch.backward()
    assert torch.equal(batch.grad_loc[0], gl[0]) and torch.equal(batch.grad_w[0], gw[0])


def test_softmax_of_many_anchors(ops):
    A = 17_000_000                                 # a workgroup of 256 threads each
    feat, shapes, starts, loc, w = operands(1, 2, A, 1, 4, torch.float32, torch.float32, 4.0)
    layout = ops.Layout(shapes, starts)
    go = torch.randn(1, A, 4, device="cuda")
    out = ops.forward(feat, layout, loc, w, logits=True)
    gw = ops.backward(feat, layout, loc, w, go, False, False, True, logits=True)[2]
    for lo, hi in ((0, A // 2), (A // 2, A)):
        part = loc[:, lo:hi], w[:, lo:hi]
        assert torch.equal(out[:, lo:hi], ops.forward(feat, layout, *part, logits=True))
        assert torch.equal(gw[:, lo:hi], ops.backward(feat, layout, *part, go[:, lo:hi].contiguous(),
                                                      False, False, True, logits=True)[2])


def test_anchor_order(ops):
    A = 70_000_000                                 # a wave each
    feat, shapes, starts, loc, w = operands(1, 1, A, 1, 2, torch.bfloat16, torch.float32)
    layout = ops.Layout(shapes, starts)
    go = torch.randn(1, A, 2, device="cuda")
    out = ops.forward(feat, layout, loc, w)
    _, gl, gw = ops.backward(feat, layout, loc, w, go, need_feat=False)
    for lo, hi in ((0, A // 2), (A // 2, A)):
        part = loc[:, lo:hi], w[:, lo:hi]
        assert torch.equal(out[:, lo:hi], ops.forward(feat, layout, *part))
        _, hl, hw = ops.backward(feat, layout, *part, go[:, lo:hi].contiguous(), need_feat=False)
        assert torch.equal(gl[:, lo:hi], hl) and torch.equal(gw[:, lo:hi], hw)
