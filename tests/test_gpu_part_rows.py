"""The view-order forward with room for fewer partial rows than it takes: the same
sums, bitwise, in several launches, the statistics of logits after the rows, with
more than one batch item and with channels that are no multiple of four. Every
case takes more than the least workspace's eight rows, which is asserted."""
import pytest
import torch

from helpers import FWD_F32_MAXREL, FWD_F32_TOL, assert_close, host, to_device
from paper_2601_10819_amd import synth

pytestmark = pytest.mark.gpu

LEVELS = ((9, 11), (5, 6), (3, 3), (2, 2))
CASES = [
    # (B, cams, L, C, G, A, P, dtype, logits, rows)
    (2, 24, 4, 256, 8, 6, 12, torch.float32, False, 24),
    (1, 70, 4, 64, 4, 5, 13, torch.float32, False, 64),
    (2, 17, 4, 128, 4, 9, 13, torch.float32, True, 16),
    (3, 26, 3, 64, 4, 4, 16, torch.float16, True, 24),
    (2, 29, 3, 128, 4, 7, 7, torch.float32, False, 16),         # three cameras a row
    (2, 40, 4, 2, 1, 5, 13, torch.bfloat16, False, 40),
    (1, 32, 4, 128, 32, 5, 13, torch.float32, True, 32),
]


def rows_of(cams, P, L):
    """Partial rows: a multiple of 8, of cameras enough for 48 samples each."""
    per_row = -(-48 // (P * L))
    return min(min(cams // 8 * 8, 64), -(-(-(-cams // per_row)) // 8) * 8)


@pytest.mark.parametrize("i", range(len(CASES)))
def test_fewer_rows(oracle_mod, i):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2601_10819_amd import ops
    lib = ops._lib.load()
    B, cams, L, C, G, A, P, dtype, logits, rows = CASES[i]
    assert rows_of(cams, P, L) == rows > 8
    p = synth.small(seed=900 + i, B=B, cams=cams, levels=LEVELS[:L], C=C, G=G, A=A, P=P)
    feat, layout, loc, w = to_device(p, dtype)
    weights = p.weights
    if logits:
        gen = torch.Generator().manual_seed(i)
        raw = 2 * torch.randn(p.weights.shape, generator=gen)
        weights = torch.softmax(raw.double().reshape(B, A, -1, G), 2).reshape(raw.shape)
        w = raw.cuda()
    tile = {"order": "view"}
    out = ops.forward(feat, layout, loc, w, tile=tile, logits=logits)
    ref = oracle_mod.forward(p.feat.to(dtype).double(), p.spatial_shapes, p.level_start_index,
                             p.sampling_loc, weights)
    assert_close(host(out), ref, FWD_F32_TOL, FWD_F32_MAXREL, f"case {i} out")
    round_up = lambda n: -(-n // 256) * 256
    stats = round_up(B * A * G * 8) if logits else 0
    row = B * A * C * 4
    assert ops.forward_workspace_bytes(feat, layout, loc, w, tile=tile, logits=logits) >= \
        round_up(rows * row) + stats
    for n in (8, 9, 13, rows - 1):
        size = round_up(n * row) + stats
        ws = torch.full((size + 512,), 0xff, dtype=torch.uint8, device="cuda")    # NaNs
        base = (ws.data_ptr() + 255) // 256 * 256
        got = torch.full_like(out, float("nan"))
        d = ops.make_desc(feat, layout, loc, w, tile=tile, logits=logits)
        ops._lib.check(lib.msda_forward_ws(
            ops._ptr(feat), ops._ptr(layout.shapes), ops._ptr(layout.starts), ops._ptr(loc),
            ops._ptr(w), ops._ptr(got), base, size, ops.ctypes.byref(d), ops._stream()))
        torch.cuda.synchronize()
        assert torch.equal(got, out), f"{n} rows of workspace"
        assert bool((ws[base - ws.data_ptr() + size:] == 0xff).all()), "wrote past the workspace"
    d = ops.make_desc(feat, layout, loc, w, tile=tile, logits=logits)
    status = lib.msda_forward_ws(
        ops._ptr(feat), ops._ptr(layout.shapes), ops._ptr(layout.starts), ops._ptr(loc),
        ops._ptr(w), ops._ptr(got), base, round_up(8 * row) + stats - 256, ops.ctypes.byref(d),
        ops._stream())
    assert status == ops._lib.MSDA_ERR_WORKSPACE
