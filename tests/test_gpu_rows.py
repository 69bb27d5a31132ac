"""The view-order forward's partial rows: camera counts whose rows hold one or
two cameras, anchors of more than 64 samples, many groups (smaller staged
chunks), every wave count, and workspaces with room for fewer rows than the
call would take (the same sums in more launches)."""
import numpy as np
import pytest
import torch

from helpers import FWD_F32_MAXREL, FWD_F32_TOL, assert_close, host, to_device
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


CASES = [
    # B, cams, levels, C, G, A, P, tile
    (1, 17, ((9, 11), (5, 6)), 64, 4, 13, 3, {}),                       # rows of 1 and 2 cameras
    (2, 70, ((5, 7),), 32, 4, 3, 2, {}),                                # over 64 cameras
    (1, 8, ((9, 11), (5, 6), (3, 4), (2, 2)), 256, 8, 5, 17, {}),       # 68 samples: 64 + 4
    (1, 9, ((9, 11), (5, 6), (3, 4)), 128, 64, 4, 5, {"waves_per_anchor": 8}),
    (1, 8, ((9, 11), (5, 6)), 64, 32, 4, 7, {"waves_per_anchor": 4, "chans_per_lane": 2}),
    (1, 12, ((4, 5),), 4, 1, 7, 1, {"waves_per_anchor": 2}),            # one lane per sample
    (1, 64, ((2, 3),), 256, 8, 1, 1, {"waves_per_anchor": 1}),          # one sample per row
]


@pytest.mark.parametrize("i", range(len(CASES)))
def test_rows_match_oracle_with_any_workspace(ops, oracle_mod, i):
    B, cams, levels, C, G, A, P, tile = CASES[i]
    p = synth.small(seed=300 + i, B=B, cams=cams, levels=levels, C=C, G=G, A=A, P=P)
    print(f"case {i} {p.dims()} {tile}", flush=True)
    feat, layout, loc, w = to_device(p)
    tile = dict(tile, order="view")
    out = ops.forward(feat, layout, loc, w, tile=tile)
    torch.cuda.synchronize()
    ref = oracle_mod.forward(p.feat, p.spatial_shapes, p.level_start_index, p.sampling_loc,
                             p.weights)
    assert_close(host(out), ref, FWD_F32_TOL, FWD_F32_MAXREL, f"case {i} out")
    row = B * A * C * 4
    full = ops.forward_workspace_bytes(feat, layout, loc, w, tile=tile)
    assert full == -(-max(8, min(64, cams // 8 * 8)) * row // 256) * 256
    lib = ops._lib.load()
    for rows in (8, 9, 13):
        need = min(full, -(-rows * row // 256) * 256)
        ws = torch.empty(need + 256, dtype=torch.uint8, device="cuda")
        base = (ws.data_ptr() + 255) // 256 * 256
        got = torch.full_like(out, float("nan"))
        d = ops.make_desc(feat, layout, loc, w, tile=tile)
        ops._lib.check(lib.msda_forward_ws(
            ops._ptr(feat), ops._ptr(layout.shapes), ops._ptr(layout.starts), ops._ptr(loc),
            ops._ptr(w), ops._ptr(got), base, need, ops.ctypes.byref(d), ops._stream()))
        torch.cuda.synchronize()
        assert torch.equal(got, out), f"{rows} rows of workspace"


def test_infinite_features_stay_infinite(ops):
    """An infinity under a positive corner weight gives an infinity, not a NaN."""
    p = synth.small(seed=320, cams=9, levels=((6, 10), (3, 5)), C=64, G=4, A=6, P=3)
    p.sampling_loc[:] = 0.43
    p.feat.abs_().add_(0.1)
    p.feat[0, :, 5] = float("inf")
    p.weights.abs_().add_(0.1)
    for dtype in (torch.float32, torch.bfloat16, torch.float16):
        feat, layout, loc, w = to_device(p, dtype)
        out = ops.forward(feat, layout, loc, w, tile={"order": "view"}).cpu().numpy()
        assert np.all(np.isposinf(out[..., 5])), dtype
        assert np.all(np.isfinite(np.delete(out, 5, axis=-1))), dtype
