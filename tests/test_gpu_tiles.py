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
