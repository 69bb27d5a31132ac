"""The view-order forward where a camera has few samples, so that a partial row
holds several cameras: against the FP64 oracle, and the batched form bitwise
against the single calls."""
import pytest
import torch

from helpers import FWD_F32_MAXREL, FWD_F32_TOL, assert_close, host, to_device
from paper_2601_10819_amd import synth

pytestmark = pytest.mark.gpu

CASES = [
    # (B, cams, levels, C, G, A, P)
    (1, 17, ((5, 7),), 64, 4, 9, 1),                       # 48 cameras would fit a row: 8 rows
    (2, 29, ((9, 11), (5, 6), (3, 3)), 128, 4, 7, 7),      # 3 cameras: 16 rows
    (1, 70, ((6, 7), (3, 4)), 32, 4, 5, 2),                # 12 cameras: 8 rows
    (1, 24, ((6, 7), (3, 4), (2, 2), (1, 1)), 256, 8, 6, 11),   # 2 cameras: 16 rows
    (1, 24, ((6, 7), (3, 4), (2, 2), (1, 1)), 256, 8, 6, 12),   # exactly a row: 24 rows
]


@pytest.mark.parametrize("i", range(len(CASES)))
def test_short_rows(oracle_mod, i):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2601_10819_amd import ops
    B, cams, levels, C, G, A, P = CASES[i]
    p = synth.small(seed=90 + i, B=B, cams=cams, levels=levels, C=C, G=G, A=A, P=P)
    feat, layout, loc, w = to_device(p)
    out = ops.forward(feat, layout, loc, w, tile={"order": "view"})
    ref = oracle_mod.forward(p.feat, p.spatial_shapes, p.level_start_index, p.sampling_loc,
                             p.weights)
    assert_close(host(out), ref, FWD_F32_TOL, FWD_F32_MAXREL, f"case {i} out")
    small = torch.empty(8 * B * A * C * 4 + 256, dtype=torch.uint8, device="cuda")
    few = ops.forward(feat, layout, loc, w, tile={"order": "view"}, workspace=small)
    batch = ops.SceneBatch([(feat[b].contiguous(), layout, loc[b].contiguous(), w[b].contiguous())
                            for b in range(B)], tile={"order": "view"})
    batch.forward()
    torch.cuda.synchronize()
    assert torch.equal(few, out)
    for b in range(B):
        alone = ops.forward(feat[b:b + 1], layout, loc[b:b + 1].contiguous(),
                            w[b:b + 1].contiguous(), tile={"order": "view"})
        assert torch.equal(alone[0], batch.out[b])
