"""Pyramid levels of long, thin and flat arrays: pieces of rows, windows of
rows that span planes, and the share of the chip they get, so that their time
follows their size."""
import numpy as np
import pytest

import gen
import oracle
from tests.helpers import median_us

pytestmark = pytest.mark.gpu


def level(src):
    import torch

    from paper_1804_08197_amd import sg
    t = torch.from_numpy(src).cuda()
    dst = torch.zeros([-(-n // 2) for n in src.shape], dtype=t.dtype, device="cuda")
    run = lambda: sg.sg_pyramid_level(t, dst)
    run()
    torch.cuda.synchronize()
    return dst.cpu().numpy(), run


# z, y, x: rows of several pieces (even and odd ones), one pair a row, one row
# a plane, and windows of 256 pairs that end inside a row or span planes
@pytest.mark.parametrize("dtype", [np.uint8, np.uint16])
@pytest.mark.parametrize("shape", [(2, 3, 8194), (1, 1, 5003), (3, 5, 2051), (300, 1, 3),
                                   (200, 301, 1), (130, 2, 5), (9, 300, 70), (40, 257, 258)])
def test_shapes(shape, dtype):
    src = gen.random_volume(shape, 3, dtype=dtype)
    assert np.array_equal(level(src)[0], oracle.downsample(src))


def test_long_rows_share_the_chip():
    us = {}
    for shape in ((64, 100, 1000), (8, 8, 100000)):  # 6.4 million voxels each
        us[shape] = median_us(level(np.zeros(shape, np.uint16))[1])
    print(us, flush=True)
    assert us[(8, 8, 100000)] <= 2 * us[(64, 100, 1000)], us
