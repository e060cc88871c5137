"""The import kernels at the sizes and addresses where their words, rows and
launches end: levels and outputs that start one voxel past an aligned
address, rows of odd and even length, one-voxel axes, the smallest and the
largest brick, more bricks than one launch holds. Whole numbers: equal."""
import numpy as np
import pytest

import gen
import oracle

pytestmark = pytest.mark.gpu


def on_device(shape, dtype, shift):
    """An empty device tensor of the shape, `shift` voxels past an aligned address."""
    import torch
    n, item = int(np.prod(shape)), np.dtype(dtype).itemsize
    buf = torch.full(((n + 8) * item,), 0xA5, dtype=torch.uint8, device="cuda")
    dt = {1: torch.uint8, 2: torch.uint16}[item]
    return buf[shift * item:(shift + n) * item].view(dt).view(*shape)


def fill(t, a):
    import torch
    bits = torch.uint8 if a.itemsize == 1 else torch.int16
    t.view(bits).copy_(torch.from_numpy(a.view(np.uint8 if a.itemsize == 1 else np.int16)))
    return t


@pytest.mark.parametrize("dtype", [np.uint8, np.uint16], ids=["u8", "u16"])
@pytest.mark.parametrize("shift", [0, 1, 2, 3])
@pytest.mark.parametrize("shape", [(1, 1, 1), (2, 3, 4), (5, 6, 7), (9, 1, 33), (1, 20, 130),
                                   (16, 17, 256), (3, 2, 4101)])
def test_pyramid_level(shape, dtype, shift):
    from paper_1804_08197_amd import sg
    a = gen.random_volume(shape, sum(shape), dtype=dtype)
    src = fill(on_device(shape, dtype, shift), a)
    dst = on_device([-(-n // 2) for n in shape], dtype, shift)
    sg.sg_pyramid_level(src, dst)
    assert np.array_equal(dst.cpu().numpy(), oracle.downsample(a))


@pytest.mark.parametrize("dtype", [np.uint8, np.uint16], ids=["u8", "u16"])
@pytest.mark.parametrize("shift", [0, 1])
@pytest.mark.parametrize("shape,brick", [((3, 5, 7), 2), ((20, 19, 21), 2), ((17, 16, 31), 4),
                                         ((40, 33, 50), 8), ((70, 64, 66), 64), ((1, 1, 1), 32),
                                         ((5, 130, 129), 128), ((3, 9, 300), 256)])
def test_brick_regions(shape, brick, dtype, shift):
    from paper_1804_08197_amd import sg
    a = gen.random_volume(shape, brick + 1, dtype=dtype)
    level = fill(on_device(shape, dtype, shift), a)
    g = [-(-n // brick) for n in shape[::-1]]
    bz, by, bx = np.meshgrid(*[np.arange(k) for k in g[::-1]], indexing="ij")
    coords = np.stack([bx.ravel(), by.ravel(), bz.ravel()], 1)
    coords = coords[np.random.default_rng(1).permutation(len(coords))]
    S = brick + 2
    out = on_device((len(coords), S, S, S), dtype, shift)
    sg.sg_brick_regions(level, brick, coords, out)
    got = out.cpu().numpy()
    at = [np.clip(brick * coords[:, k:k + 1] - 1 + np.arange(S), 0, shape[2 - k] - 1)
          for k in range(3)]
    for i in range(len(coords)):
        assert np.array_equal(got[i], a[np.ix_(at[2][i], at[1][i], at[0][i])]), coords[i]
