"""The backward's softmax where few anchors have many logits, which are cut into
runs: against the softmax and its gradient in 64 bits, on both sides of the line,
runs that are not full, masked and infinite logits, BF16; and a batch bitwise its
scenes' calls."""
import pytest
import torch

from helpers import GRAD_F32_MAXREL, GRAD_F32_TOL, assert_close, host, to_device
from paper_2601_10819_amd import synth

pytestmark = pytest.mark.gpu

CASES = [
    # (B, cams, L, G, A, P, dtype): entries an anchor
    (1, 40, 2, 64, 3, 7, torch.float32),       # 35,840: 9 rounds of 4096
    (1, 33, 2, 64, 1, 8, torch.bfloat16),      # 33,792: 9, the last one short
    (2, 64, 4, 64, 5, 3, torch.float32),       # 49,152
    (1, 8, 4, 32, 127, 30, torch.float32),     # 30,720: 8 rounds, four runs
    (1, 8, 4, 32, 128, 30, torch.float32),     # too many anchors: a block each
    (1, 8, 4, 32, 20, 27, torch.float32),      # 27,648: 7 rounds, a block each
]


@pytest.fixture(scope="module")
def ops():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2601_10819_amd import ops as o
    o._lib.load()
    return o


def operands(i):
    B, cams, L, G, A, P, dtype = CASES[i]
    p = synth.small(seed=600 + i, B=B, cams=cams, levels=((4, 5), (3, 2), (2, 2), (1, 1))[:L], C=G,
                    G=G, A=A, P=P)
    feat, layout, loc, _ = to_device(p)
    gen = torch.Generator().manual_seed(i)
    x = 3 * torch.randn(p.weights.shape, generator=gen)
    x[..., ::7, :, :, 1] = float("-inf")                   # masked keypoints of one group
    x[..., 0, 0, 0, 2] = torch.finfo(torch.float32).min
    return p, feat, layout, loc, x.to(dtype), synth.grad_out_like(p, seed=i)


@pytest.mark.parametrize("i", range(len(CASES)))
def test_runs(ops, oracle_mod, i):
    B, cams, L, G, A, P, dtype = CASES[i]
    p, feat, layout, loc, x, go = operands(i)
    soft = torch.softmax(x.double().reshape(B, A, -1, G), 2)
    gw = oracle_mod.backward(p.feat, p.spatial_shapes, p.level_start_index, p.sampling_loc,
                             soft.reshape(x.shape), go, need_feat=False)[2]
    gw = torch.as_tensor(gw).reshape(soft.shape)
    ref = (soft * (gw - (soft * gw).sum(2, keepdim=True))).reshape(x.shape)
    grads = ops.backward(feat, layout, loc, x.cuda(), go.cuda(), logits=True)
    assert_close(host(grads[2]), ref, GRAD_F32_TOL, GRAD_F32_MAXREL, f"case {i} grad of logits")
    again = ops.backward(feat, layout, loc, x.cuda(), go.cuda(), logits=True)
    for a, b in zip(grads, again):
        assert torch.equal(a, b)


def test_infinite_and_missing_logits(ops):
    """A NaN, an infinity or nothing but masked entries make their group's
    gradient NaN and leave the others alone, in runs as in one block."""
    p, feat, layout, loc, x, go = operands(0)
    x[:, 0, 0, 0, 0, 5] = float("nan")
    x[:, 1, 3, 2, 1, 6] = float("inf")
    x[:, 2, :, :, :, 7] = float("-inf")
    gw = ops.backward(feat, layout, loc, x.cuda(), go.cuda(), logits=True)[2].cpu()
    bad = torch.isnan(gw).flatten(2, 4).any(2)
    want = torch.zeros_like(bad)
    want[:, 0, 5] = want[:, 1, 6] = want[:, 2, 7] = True
    assert torch.equal(bad, want)


def test_batch(ops):
    scenes, gos = [], []
    for i in (0, 0):
        p, feat, layout, loc, x, go = operands(i)
        scenes.append((feat[0], layout, loc[0], x[0].cuda()))
        gos.append(go[0].cuda() * (len(gos) + 1))
    batch = ops.SceneBatch(scenes, logits=True)
    for out, go in zip(batch.grad_out, gos):
        out.copy_(go)
    batch.backward()
    for i, (feat, layout, loc, x) in enumerate(scenes):
        gw = ops.backward(feat[None], layout, loc[None], x[None], gos[i][None], logits=True)[2]
        assert torch.equal(gw[0], batch.grad_w[i])
