"""The batched forward's workspace holds the partial rows its scenes take, not the
most that their cameras allow: few samples a camera make rows of several cameras."""
import ctypes

import pytest

from paper_2601_10819_amd import _lib
from test_abi import Geo, batch_desc


@pytest.mark.parametrize("points,rows", [(3, 8), (24, 64), (8, 24)])
def test_rows_of_64_cameras(points, rows):
    lib = _lib.load()
    b = batch_desc([Geo(ncam=64, levels=((6, 10), (3, 5)))], [1000])
    b.num_points = points                    # two levels: 6, 48 and 16 samples a camera
    size = lib.msda_batched_workspace_size(ctypes.byref(b), 0)
    row = 1000 * b.channels * 4
    assert rows * row <= size < rows * row + 65536
