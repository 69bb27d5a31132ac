"""grad_feat of narrow records over light tiles of few samples, which take a
sub-wave each: one to eight tiles per wave, last waves that are not full, more
records in a tile than a sub-wave has lanes, against the FP64 oracle; and a batch
of sparse and other scenes, bitwise the calls on its scenes alone."""
import pytest
import torch

from helpers import BF16_TOL, GRAD_F32_MAXREL, GRAD_F32_TOL, assert_close, host, to_device
from paper_2601_10819_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ops():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2601_10819_amd import ops as o
    o._lib.load()
    return o


CASES = [
    # (B, cams, levels, C, G, A, P, dtype)
    (1, 3, ((125, 131), (63, 33)), 64, 4, 9, 3, torch.float32),         # 3600 tiles: one a wave
    (2, 3, ((125, 131), (63, 33)), 32, 4, 9, 3, torch.float32),         # 7392 tiles: one
    (1, 5, ((181, 203), (91, 50)), 64, 4, 30, 5, torch.float32),        # 14,960: 2
    (3, 4, ((211, 127), (50, 40)), 16, 2, 20, 3, torch.float32),        # 21,960: 4
    (1, 4, ((301, 402), (150, 201)), 4, 1, 40, 3, torch.float32),       # 38,456: 8
    (1, 6, ((180, 220), (9, 10)), 128, 8, 50, 4, torch.float16),        # 14,850: 2 sub-waves
    (1, 2, ((160, 200),), 8, 2, 300, 2, torch.float32),                 # several chunks a tile
]


@pytest.mark.parametrize("i", range(len(CASES)))
def test_sparse_tiles(ops, oracle_mod, i):
    B, cams, levels, C, G, A, P, dtype = CASES[i]
    p = synth.small(seed=80 + i, B=B, cams=cams, levels=levels, C=C, G=G, A=A, P=P)
    if i == 6:                                      # half of them in one place
        p.sampling_loc[:, ::2] = 0.5 + 0.01 * (p.sampling_loc[:, ::2] - 0.5)
    print(f"case {i} {p.dims()}", flush=True)
    feat, layout, loc, w = to_device(p, dtype)
    go = synth.grad_out_like(p, seed=i)
    gf = ops.backward(feat, layout, loc, w, go.cuda())[0]
    again = ops.backward(feat, layout, loc, w, go.cuda())[0]
    torch.cuda.synchronize()
    ref = oracle_mod.backward(p.feat, p.spatial_shapes, p.level_start_index, p.sampling_loc,
                              p.weights, go)[0]
    if dtype == torch.float32:
        assert_close(host(gf), ref, GRAD_F32_TOL, GRAD_F32_MAXREL, f"case {i} grad_feat")
    else:
        assert_close(host(gf.float()), ref, BF16_TOL, None, f"case {i} grad_feat")
    assert torch.equal(gf, again)


@pytest.mark.parametrize("kinds", ["sparse", "sparse dense", "wide sparse dense",
                                   "wide sparse", "both", "both dense"])
def test_batch_of_sparse_scenes(ops, kinds):
    shapes = {                                      # (cameras, levels, A)
        "sparse": (3, ((90, 110), (40, 50), (9, 10)), 12),
        "dense": (2, ((24, 32), (6, 8), (3, 3)), 60),
        "wide": (2, ((32, 56), (16, 28), (8, 14)), 128),
        "both": (1, ((120, 120), (8, 8), (3, 3)), 80),       # sparse, its coarse tiles 8 waves
    }
    probs = []
    for i, k in enumerate((kinds + " " + kinds).split()):
        cams, levels, A = shapes[k]
        probs.append(synth.small(seed=100 + i, cams=cams, levels=levels, C=64, G=4, A=A, P=13))
    scenes = []
    for p in probs:
        feat, layout, loc, w = to_device(p)
        scenes.append((feat[0], layout, loc[0], w[0]))
    batch = ops.SceneBatch(scenes)
    for i, go in enumerate(batch.grad_out):
        go.copy_(synth.grad_out_like(probs[i], seed=i)[0])
    batch.backward()
    for i, (feat, layout, loc, w) in enumerate(scenes):
        gf = ops.backward(feat[None], layout, loc[None], w[None], batch.grad_out[i][None])[0]
        torch.cuda.synchronize()
        assert torch.equal(gf[0], batch.grad_feat[i]), f"scene {i}"
