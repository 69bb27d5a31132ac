"""The per-group softmax of the weight logits and its gradient at the edges of
its launch shapes: rounds of 16 entries per thread, 256, 512 or 1024 threads
per anchor (by entries and anchors), 1 to 64 groups. Against FP64 through the
plain operator: the forward on logits equals the forward on their softmax, and
the logits' gradient is w * (dw - sum of w * dw) of the plain grad_weights dw."""
import pytest
import torch

from helpers import (FWD_F32_MAXREL, FWD_F32_TOL, GRAD_F32_MAXREL, GRAD_F32_TOL, assert_close,
                     host, to_device)
from paper_2601_10819_amd import synth

pytestmark = pytest.mark.gpu

CASES = [
    # (cams, levels, C, G, A, P): entries per anchor = P * cams * len(levels) * G
    (1, 1, 4, 1, 3, 2),          # two entries
    (32, 4, 32, 8, 5, 4),        # 4096: one full round of 256 threads
    (57, 3, 32, 8, 5, 3),        # 4104: 1024 threads, mostly idle
    (57, 3, 32, 8, 520, 3),      # 4104 in more than 512 anchors: 512 threads
    (32, 4, 32, 8, 513, 8),      # 8192: one full round of 512 threads
    (32, 4, 32, 8, 3, 16),       # 16384: one full round of 1024 threads
    (683, 1, 32, 8, 3, 3),       # 16392: a second round of one entry per group
    (683, 1, 32, 8, 514, 3),     # the same in more than 512 anchors
    (5, 2, 256, 64, 4, 13),      # a group per lane
]


@pytest.fixture(scope="module")
def ops():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2601_10819_amd import ops as o
    o._lib.load()
    return o


@pytest.mark.parametrize("i", range(len(CASES)))
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16], ids=["f32", "bf16"])
def test_softmax_and_gradient(ops, i, dtype):
    cams, levels, C, G, A, P = CASES[i]
    p = synth.small(seed=i, B=1, cams=cams, levels=((3, 4), (2, 2), (2, 1), (1, 1))[:levels],
                    C=C, G=G, A=A, P=P)
    feat, layout, loc, w = to_device(p)
    x = (2 * torch.randn(w.shape, generator=torch.Generator().manual_seed(i))).to(dtype).cuda()
    if x[0, 0, ..., 0].numel() > 4:
        x[0, 0, ..., 0].view(-1)[1::2] = float("-inf")          # masked entries
    w64 = torch.softmax(x.double().view(1, A, -1, G), 2)
    w = w64.float().view(w.shape).contiguous()
    out = ops.forward(feat, layout, loc, x, logits=True)
    assert_close(host(out), host(ops.forward(feat, layout, loc, w)), FWD_F32_TOL, FWD_F32_MAXREL,
                 "out")
    go = synth.grad_out_like(p, seed=i).cuda()
    dw = ops.backward(feat, layout, loc, w, go, need_feat=False)[2].double().view(1, A, -1, G)
    dx = ops.backward(feat, layout, loc, x, go, need_feat=False, logits=True)[2]
    ref = w64 * (dw - (w64 * dw).sum(2, keepdim=True))
    assert_close(host(dx.double().view(1, A, -1, G)), host(ref), GRAD_F32_TOL, GRAD_F32_MAXREL,
                 "grad_logits")


def test_nan_stays_in_its_group(ops):
    p = synth.small(seed=1, B=1, cams=57, levels=((3, 4), (2, 2)), C=32, G=8, A=2, P=5)
    feat, layout, loc, w = to_device(p)
    x = torch.zeros_like(w)
    x[0, 1, 4, 50, 1, 3] = float("nan")
    out = ops.forward(feat, layout, loc, x, logits=True).view(2, 8, 4)
    assert out[1, 3].isnan().all() and not out[0].isnan().any()
    assert not out[1, [0, 1, 2, 4, 5, 6, 7]].isnan().any()
