"""The FP8 quantiser's scales and codes, bitwise, against torch: more regions of a
level than a wave has lanes, several batch items and chunks per region, an
all-zero level, channels that do not divide by 4."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,cams,levels,C", [
    (3, 29, ((5, 7), (2, 3)), 32), (1, 2, ((150, 70), (9, 11), (1, 1)), 64), (2, 3, ((4, 5),), 6)])
def test_scales_and_codes(B, cams, levels, C):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2601_10819_amd import ops
    shapes = torch.tensor([levels] * cams)
    rows = (shapes[..., 0] * shapes[..., 1]).view(-1)
    starts = (rows.cumsum(0) - rows).view(cams, len(levels))
    x = torch.randn(B, int(rows.sum()), C, generator=torch.Generator().manual_seed(C)) * 3
    level = torch.arange(len(levels)).repeat(cams).repeat_interleave(rows)
    if len(levels) > 1:
        x[:, level == len(levels) - 1] = 0.0
    amax = torch.stack([x[:, level == l].abs().max() for l in range(len(levels))])
    scale = torch.where(amax > 0, amax / 448.0, torch.ones(()))
    want = (x / scale[level][None, :, None]).clamp(-448, 448).to(torch.float8_e4m3fn)
    codes, got = ops.quantize_fp8(x.cuda(), ops.Layout(shapes, starts, "cuda"))
    assert torch.equal(got.cpu(), scale)
    assert torch.equal(codes.cpu(), want.view(torch.uint8))
