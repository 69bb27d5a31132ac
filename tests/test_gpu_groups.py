"""More than eight channel groups, whose weights the gathers stage lane after
lane: every storage form of the weights and features, samples that fill no round,
both work orders, against the FP64 oracle."""
import pytest
import torch

from helpers import (BF16_TOL, FWD_F32_MAXREL, FWD_F32_TOL, GRAD_F32_MAXREL, GRAD_F32_TOL,
                     assert_close, host, to_device)
from paper_2601_10819_amd import synth

pytestmark = pytest.mark.gpu

LEVELS = ((9, 13), (5, 7), (3, 4), (2, 3), (4, 4))
CASES = [
    # (B, cams, L, C, G, A, P, waves)
    (1, 9, 1, 64, 16, 7, 70, 0),       # 64 samples and 6; 4 lanes a group
    (2, 3, 3, 128, 16, 5, 5, 2),       # 15 samples a camera, padded levels
    (1, 10, 4, 256, 32, 6, 13, 4),
    (1, 9, 5, 64, 64, 3, 11, 8),       # a lane a group, FP32 of one channel
    (1, 8, 2, 256, 64, 4, 1, 1),       # fewer samples than a round
]


@pytest.mark.parametrize("order", ["view", "anchor"])
@pytest.mark.parametrize("i", range(len(CASES)))
def test_many_groups(oracle_mod, i, order):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2601_10819_amd import ops
    B, cams, L, C, G, A, P, waves = CASES[i]
    p = synth.small(seed=700 + i, B=B, cams=cams, levels=LEVELS[:L], C=C, G=G, A=A, P=P)
    feat, layout, loc, w = to_device(p)
    go = synth.grad_out_like(p, seed=i)
    geo = (p.spatial_shapes, p.level_start_index, p.sampling_loc)
    tile = {"order": order, "waves_per_anchor": waves}
    out = ops.forward(feat, layout, loc, w, tile=tile)
    ref = oracle_mod.forward(p.feat, *geo, p.weights)
    assert_close(host(out), ref, FWD_F32_TOL, FWD_F32_MAXREL, f"case {i} out")
    grads = ops.backward(feat, layout, loc, w, go.cuda(), tile=tile)
    refs = oracle_mod.backward(p.feat, *geo, p.weights, go)
    for x, r, name in zip(grads, refs, ("grad_feat", "grad_loc", "grad_w")):
        assert_close(host(x), r, GRAD_F32_TOL, GRAD_F32_MAXREL, f"case {i} {name}")
    # logits, in BF16: the softmax of what is stored
    logits = (3 * torch.randn(w.shape, generator=torch.Generator().manual_seed(i))).bfloat16()
    soft = torch.softmax(logits.double().reshape(B, A, -1, G), 2).reshape(w.shape)
    ref = oracle_mod.forward(p.feat, *geo, soft)
    got = ops.forward(feat, layout, loc, logits.cuda(), tile=tile, logits=True)
    assert_close(host(got), ref, FWD_F32_TOL, FWD_F32_MAXREL, f"case {i} logits")
    if C >= 4 * G:                     # FP8: four channels a lane at least
        codes, scale = ops.quantize_fp8(feat, layout)
        got = ops.forward(codes, layout, loc, w, level_scale=scale, tile=tile)
        stored = torch.zeros(p.feat.shape, dtype=torch.float64)
        value = codes.view(torch.float8_e4m3fn).float().double().cpu()
        for n in range(cams):
            for l in range(L):
                s0 = int(p.level_start_index[n, l])
                s1 = s0 + int(p.spatial_shapes[n, l, 0] * p.spatial_shapes[n, l, 1])
                stored[:, s0:s1] = value[:, s0:s1] * float(scale[l])
        ref = oracle_mod.forward(stored, *geo, p.weights)
        assert_close(host(got), ref, FWD_F32_TOL, FWD_F32_MAXREL, f"case {i} FP8")
    if C >= 2 * G:                     # two channels a lane at least
        half = p.feat.half()
        got = ops.forward(half.cuda(), layout, loc, w, tile=tile)
        ref = oracle_mod.forward(half.double(), *geo, p.weights)
        assert_close(host(got), ref, FWD_F32_TOL, FWD_F32_MAXREL, f"case {i} FP16")
        gh = ops.backward(half.cuda(), layout, loc, w, go.cuda(), tile=tile)
        refs = oracle_mod.backward(half.double(), *geo, p.weights, go)
        for x, r, tol in zip(gh, refs, (BF16_TOL, GRAD_F32_TOL, GRAD_F32_TOL)):
            assert_close(host(x.float()), r, tol, None, f"case {i} FP16 gradient")
