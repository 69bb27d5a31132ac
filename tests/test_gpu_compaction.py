"""The compaction of the visible (batch item, camera, anchor) items at the edges
of its blocks of 2048: the visible-view operator, whose items it lists, against
the dense one with the invisible views' weights set to zero."""
import pytest
import torch

from helpers import (FWD_F32_MAXREL, FWD_F32_TOL, GRAD_F32_MAXREL, GRAD_F32_TOL, assert_close,
                     host, to_device)
from paper_2601_10819_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,cams,A,share", [
    (1, 1, 2047, 0.5), (1, 1, 2048, 0.5), (1, 1, 2049, 0.5), (2, 3, 683, 0.3), (1, 2, 1024, 0.0),
    (1, 3, 1366, 1.0), (2, 5, 1231, 0.1)])
def test_compaction_edges(B, cams, A, share):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2601_10819_amd import ops
    p = synth.small(seed=A, B=B, cams=cams, levels=((5, 7), (3, 3)), C=32, G=4, A=A, P=2)
    feat, layout, loc, w = to_device(p)
    go = synth.grad_out_like(p, seed=1).cuda()
    g = torch.Generator().manual_seed(A)
    visible = (torch.rand(B, A, cams, generator=g) < share).to(torch.uint8).cuda()
    on = visible.view(B, A, 1, cams, 1, 1).float()
    out = ops.forward_visible(feat, layout, loc, w, visible)
    ref = ops.forward(feat, layout, loc, w * on)
    gf, gl, gw = ops.backward_visible(feat, layout, loc, w, visible, go)
    rf, rl, rw = ops.backward(feat, layout, loc, w * on, go)
    torch.cuda.synchronize()
    if share == 0.0:
        assert not any(x.any() for x in (out, gf, gl, gw))
        return
    assert_close(host(out), host(ref), FWD_F32_TOL, FWD_F32_MAXREL, "out")
    assert_close(host(gf), host(rf), GRAD_F32_TOL, GRAD_F32_MAXREL, "grad_feat")
    assert_close(host(gl), host(rl), GRAD_F32_TOL, GRAD_F32_MAXREL, "grad_loc")
    assert_close(host(gw), host(rw * on), GRAD_F32_TOL, GRAD_F32_MAXREL, "grad_w")
