"""The grad_feat tile reduction with 8 waves per block (few tiles, coarse tiles
of many records) and 4, whole-wave and narrow records, against the FP64 oracle:
the coarse tiles' records are split over the waves in chunks of 64 and the
partial sums added as a tree."""
import pytest
import torch

from helpers import GRAD_F32_MAXREL, GRAD_F32_TOL, assert_close, host, to_device
from paper_2601_10819_amd import synth

pytestmark = pytest.mark.gpu

CASES = [
    # (B, cams, levels, C, G, A, P)
    (1, 2, ((32, 56), (16, 28), (8, 14), (4, 7)), 256, 8, 128, 13),   # 8 waves, whole-wave
    (2, 1, ((32, 56), (16, 28), (8, 14), (4, 7)), 64, 4, 130, 13),    # 8 waves, sub-waves
    (1, 5, ((64, 112), (32, 56), (16, 28)), 256, 8, 80, 13),          # coarse: the last level only
    (1, 3, ((17, 19), (4, 3)), 256, 8, 2, 2),                         # 4: few records
    (1, 1, ((64, 64), (1, 1)), 256, 8, 40, 13),                       # one coarse tile of all
    (1, 2, ((5, 5), (5, 5)), 128, 8, 60, 13),                         # no coarse level
]


@pytest.mark.parametrize("i", range(len(CASES)))
def test_grad_feat_tiles(oracle_mod, i):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2601_10819_amd import ops
    B, cams, levels, C, G, A, P = CASES[i]
    p = synth.small(seed=50 + i, B=B, cams=cams, levels=levels, C=C, G=G, A=A, P=P)
    feat, layout, loc, w = to_device(p)
    go = synth.grad_out_like(p, seed=i)
    gf = ops.backward(feat, layout, loc, w, go.cuda())[0]
    again = ops.backward(feat, layout, loc, w, go.cuda())[0]
    torch.cuda.synchronize()
    ref = oracle_mod.backward(p.feat, p.spatial_shapes, p.level_start_index, p.sampling_loc,
                              p.weights, go)[0]
    assert_close(host(gf), ref, GRAD_F32_TOL, GRAD_F32_MAXREL, f"case {i} grad_feat")
    assert torch.equal(gf, again)


def test_batch_takes_each_scenes_waves():
    """A batch of a scene whose coarse tiles take 8 waves and one whose take 4:
    each grad_feat is bitwise that of the call on its scene alone."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2601_10819_amd import ops
    levels = ((32, 56), (16, 28), (8, 14), (4, 7))
    probs = [synth.small(seed=60 + i, cams=2, levels=levels, C=256, G=8, A=A, P=13)
             for i, A in enumerate((128, 3, 150))]
    scenes = []
    for p in probs:
        feat, layout, loc, w = to_device(p)
        scenes.append((feat[0], layout, loc[0], w[0]))
    batch = ops.SceneBatch(scenes)
    for i, go in enumerate(batch.grad_out):
        go.copy_(synth.grad_out_like(probs[i], seed=i)[0])
    batch.forward()
    batch.backward()
    for i, (feat, layout, loc, w) in enumerate(scenes):
        gf = ops.backward(feat[None], layout, loc[None], w[None], batch.grad_out[i][None])[0]
        torch.cuda.synchronize()
        assert torch.equal(gf[0], batch.grad_feat[i]), f"scene {i}"
