"""The backward gather's units: one to eight levels, more pairs than a wave
stages at a time, few keypoints (several cameras per row), many groups, every
wave count, narrow rows. All gradients against the FP64 oracle, and both work
orders bit for bit."""
import pytest
import torch

from helpers import GRAD_F32_MAXREL, GRAD_F32_TOL, assert_close, host, to_device
from paper_2601_10819_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.fixture(scope="module")
def ops():
    from paper_2601_10819_amd import ops as o
    o._lib.load()
    return o


LEVELS = ((9, 13), (5, 7), (3, 4), (2, 3), (4, 4), (2, 5), (1, 3), (1, 1))
CASES = [
    # B, cams, levels, C, G, A, P, waves
    (1, 9, 1, 64, 4, 7, 70, 0),        # 64 pairs at a time
    (1, 9, 2, 128, 8, 5, 35, 2),       # 32
    (2, 9, 3, 256, 8, 4, 19, 0),       # 16, padded levels
    (1, 10, 8, 32, 4, 6, 11, 8),       # 8
    (1, 11, 4, 64, 4, 9, 1, 4),        # one keypoint: 7 cameras per row
    (1, 8, 4, 128, 64, 3, 3, 8),       # 64 groups
    (1, 13, 5, 4, 1, 5, 5, 1),         # one lane per sample
]


@pytest.mark.parametrize("i", range(len(CASES)))
def test_grads_match_oracle_in_both_orders(ops, oracle_mod, i):
    B, cams, L, C, G, A, P, waves = CASES[i]
    p = synth.small(seed=400 + i, B=B, cams=cams, levels=LEVELS[:L], C=C, G=G, A=A, P=P)
    print(f"case {i} {p.dims()} waves {waves}", flush=True)
    feat, layout, loc, w = to_device(p)
    go = synth.grad_out_like(p, seed=i)
    ref = oracle_mod.backward(p.feat, p.spatial_shapes, p.level_start_index, p.sampling_loc,
                              p.weights, go)
    got = {}
    for order in ("view", "anchor"):
        got[order] = ops.backward(feat, layout, loc, w, go.cuda(),
                                  tile={"order": order, "waves_per_anchor": waves})
        torch.cuda.synchronize()
    for k, name in enumerate(("grad_feat", "grad_loc", "grad_w")):
        assert_close(host(got["view"][k]), ref[k], GRAD_F32_TOL, GRAD_F32_MAXREL,
                     f"case {i} {name}")
        assert torch.equal(got["view"][k], got["anchor"][k]), f"case {i} {name}"
    # a part of the gradients alone is the same
    gl = ops.backward(feat, layout, loc, w, go.cuda(), need_feat=False, need_w=False,
                      tile={"order": "view", "waves_per_anchor": waves})[1]
    assert torch.equal(gl, got["view"][1])
