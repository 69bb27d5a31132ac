"""The line between 4 and 8 waves per coarse tile (96 samples per coarse tile),
both sides of it, and 8 waves with many groups, whose record tables take most of
a CU's LDS: grad_feat against the FP64 oracle, and a batch bitwise its scenes'
calls."""
import pytest
import torch

from helpers import GRAD_F32_MAXREL, GRAD_F32_TOL, assert_close, host, to_device
from paper_2601_10819_amd import synth

pytestmark = pytest.mark.gpu

LEVELS = ((32, 56), (16, 28), (8, 14), (4, 7))     # 2 coarse levels of 8 and 2 tiles
CASES = [
    # (cams, C, G, A, P)
    (2, 256, 8, 36, 13),               # 93.6 samples per coarse tile: 4 waves
    (2, 256, 8, 37, 13),               # 96.2: 8 waves
    (1, 64, 4, 40, 12),                # 96: 8 waves, sub-waves
    (2, 256, 32, 128, 13),             # 80 KB of record tables
    (2, 256, 64, 128, 13),             # 144 KB
    (1, 64, 64, 100, 13),              # one channel a lane
]


@pytest.mark.parametrize("i", range(len(CASES)))
def test_tile_waves(oracle_mod, i):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2601_10819_amd import ops
    cams, C, G, A, P = CASES[i]
    p = synth.small(seed=150 + i, cams=cams, levels=LEVELS, C=C, G=G, A=A, P=P)
    q = synth.small(seed=170 + i, cams=cams, levels=LEVELS, C=C, G=G, A=5, P=P)
    scenes, calls = [], []
    for x, seed in ((p, i), (q, 9), (p, i)):
        feat, layout, loc, w = to_device(x)
        go = synth.grad_out_like(x, seed=seed)
        calls.append(ops.backward(feat, layout, loc, w, go.cuda())[0])
        scenes.append(((feat[0], layout, loc[0], w[0]), go[0]))
    ref = oracle_mod.backward(p.feat, p.spatial_shapes, p.level_start_index, p.sampling_loc,
                              p.weights, synth.grad_out_like(p, seed=i))[0]
    assert_close(host(calls[0]), ref, GRAD_F32_TOL, GRAD_F32_MAXREL, f"case {i} grad_feat")
    batch = ops.SceneBatch([s for s, _ in scenes])
    for out, (_, go) in zip(batch.grad_out, scenes):
        out.copy_(go)
    batch.backward()
    for alone, gf in zip(calls, batch.grad_feat):
        assert torch.equal(alone[0], gf)
