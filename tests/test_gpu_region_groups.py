"""Brick regions where the route changes: thousands of small bricks (one
launch over groups of them, coordinates in device memory; under capture the
launches that carry them), and levels whose rows or planes need 64-bit
offsets, on both sides of each limit, against clamped indexing in numpy."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def level(dims, dtype, seed=6):
    r = np.random.default_rng(seed)
    return r.integers(0, np.iinfo(dtype).max, dims[::-1], dtype=dtype, endpoint=True)


def regions(lev, brick, coords, capture=False):
    import torch

    from paper_1804_08197_amd import sg
    S = brick + 2
    dev = torch.from_numpy(lev).cuda()
    out = torch.zeros((len(coords), S, S, S), dtype=dev.dtype, device="cuda")
    if not capture:
        sg.sg_brick_regions(dev, brick, coords, out)
        torch.cuda.synchronize()
        return out.cpu().numpy()
    g = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(g):
        sg.sg_brick_regions(dev, brick, coords, out)
    got = []
    for _ in range(3):
        out.zero_()
        g.replay()
        torch.cuda.synchronize()
        got.append(out.cpu().numpy())
    assert all(np.array_equal(got[0], x) for x in got[1:])
    return got[0]


def expected(lev, brick, coords):
    o = np.arange(-1, brick + 1)
    x, y, z = (np.clip(coords[:, i, None] * brick + o, 0, n - 1) for i, n in enumerate(lev.shape[::-1]))
    return lev[z[:, :, None, None], y[:, None, :, None], x[:, None, None, :]]


def some_bricks(dims, brick, n, seed=7):
    r = np.random.default_rng(seed)
    g = [-(-d // brick) for d in dims]
    c = np.stack([r.integers(0, k, n) for k in g], 1)
    c[:8] = [[(i >> a & 1) * (g[a] - 1) for a in range(3)] for i in range(8)]  # the corners
    return c.astype(np.int32)


@pytest.mark.parametrize("dtype", [np.uint8, np.uint16])
@pytest.mark.parametrize("brick", [2, 4, 8, 16])
@pytest.mark.parametrize("n", [3136, 3137, 3201, 9001])
def test_many_bricks(n, brick, dtype):
    # (16 keeps its launches; 3136 bricks are seven of them)
    dims = (61, 77, 43)
    lev, c = level(dims, dtype), some_bricks(dims, brick, n)
    assert np.array_equal(regions(lev, brick, c), expected(lev, brick, c))


@pytest.mark.parametrize("brick", [2, 8])
def test_many_bricks_under_capture(brick):
    dims = (61, 77, 43)
    lev, c = level(dims, np.uint16), some_bricks(dims, brick, 3500)
    assert np.array_equal(regions(lev, brick, c, capture=True), expected(lev, brick, c))


@pytest.mark.parametrize("dtype", [np.uint8, np.uint16])
@pytest.mark.parametrize("dims", [(2, 4095, 4096), (2, 4097, 4096), (3, 1, 20000)])
def test_many_bricks_of_large_planes(dims, dtype):
    # rows of all planes: 2^24 - 4096 and 2^24 + 4096, and few
    lev, c = level(dims, dtype), some_bricks(dims, 8, 4000)
    assert np.array_equal(regions(lev, 8, c), expected(lev, 8, c))


@pytest.mark.parametrize("dtype", [np.uint8, np.uint16])
@pytest.mark.parametrize("ny", [65027, 65029])
def test_rows_beyond_24_bits(ny, dtype):
    # a brick of 256 spans 258 planes: 258 ny rows, just below and above 2^24
    dims = (2, ny, 2)
    lev = level(dims, dtype)
    c = np.array([[0, 0, 0], [0, 127, 0], [0, ny // 256 - 1, 0], [0, ny // 256, 0]], np.int32)
    assert np.array_equal(regions(lev, 256, c), expected(lev, 256, c))


def test_cost_of_many_small_bricks():
    """A level of 256^3 in bricks of 4: one launch, not 586."""
    import torch

    from paper_1804_08197_amd import sg
    from tests.helpers import median_us
    dev = torch.zeros(256, 256, 256, dtype=torch.uint8, device="cuda")
    z, y, x = np.meshgrid(*[np.arange(64)] * 3, indexing="ij")
    c = np.stack([x.ravel(), y.ravel(), z.ravel()], 1).astype(np.int32)
    out = torch.empty((len(c), 6, 6, 6), dtype=torch.uint8, device="cuda")
    us = median_us(lambda: sg.sg_brick_regions(dev, 4, c, out), repeats=5, inner=1)
    print(us, flush=True)
    # host work and one launch 1.3 ms; 586 launches 2.9 ms
    assert us < 2300, us
