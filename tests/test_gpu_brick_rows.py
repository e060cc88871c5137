"""The kernels that write and scan whole bricks by rows of four voxels
(upload, pyramid, apron, ranges, cache puts), at the sizes where their rows,
blocks and words end: stored edges that are and are not multiples of four,
bricks smaller and larger than a batch of rows, partial bricks at the far
faces, sources aligned to one voxel only.

A resident volume (uploaded level-0 cores, pyramid and aprons made on the
device) and a cache volume that received the oracle's bricks (pyramid and
clamped aprons in numpy) must render the same bits at every level, and their
skip flags must be those of the oracle's brick ranges."""
import numpy as np
import pytest

import gen
import oracle
from tests.helpers import LAYOUT_IDS, LAYOUTS

pytestmark = pytest.mark.gpu

CASES = [  # dims x, y, z; brick; levels
    ((9, 11, 10), 2, 4), ((37, 50, 41), 4, 4), ((37, 50, 41), 8, 3), ((64, 32, 48), 16, 3),
    ((65, 33, 47), 32, 3), ((70, 131, 66), 64, 2), ((150, 129, 128), 128, 2), ((1, 1, 5), 4, 2)]


def device_voxels(a, shift):
    """The array on the device, `shift` voxels past an aligned address."""
    import torch
    t = torch.from_numpy(np.ascontiguousarray(a).view(np.uint8).reshape(-1))
    buf = torch.empty(t.numel() + 64, dtype=torch.uint8, device="cuda")
    off = shift * a.itemsize
    buf[off:off + t.numel()] = t.cuda()
    dt = {1: torch.uint8, 2: torch.uint16}[a.itemsize]
    return buf[off:off + t.numel()].view(dt).view(a.shape) if off % 2 == 0 or a.itemsize == 1 \
        else None


def expected_empty(levels, brick, ids, n, start, domain):
    """Skip flags from the brick ranges: the table is zero below `start`."""
    out = []
    for L, bx, by, bz in oracle.node_decode(ids):
        _, hi = oracle.brick_minmax(levels[int(L)], brick, [int(bx), int(by), int(bz)])
        u = (hi - domain[0]) / (domain[1] - domain[0]) * (n - 1)
        out.append(min(int(np.floor(u)) + 2, n - 1) < start)
    return np.array(out)


@pytest.mark.parametrize("layout", LAYOUTS, ids=LAYOUT_IDS)
@pytest.mark.parametrize("dtype", [np.uint8, np.uint16], ids=["u8", "u16"])
@pytest.mark.parametrize("shift", [0, 1], ids=["aligned", "shifted"])
@pytest.mark.parametrize("dims,brick,levels", CASES, ids=["b%d" % c[1] for c in CASES[:-1]] + ["thin"])
def test_resident_and_cached_bricks_agree(dims, brick, levels, dtype, shift, layout):
    import torch

    from paper_1804_08197_amd import pack_bricks, sg
    vol = gen.random_volume(dims[::-1], 3 + brick, dtype=dtype)
    top = 255 if dtype == np.uint8 else 65535
    tf = gen.tf_hot(a_start=70)
    sgt = sg.SG_U8 if dtype == np.uint8 else sg.SG_U16
    kw = dict(dtype=sgt, brick=brick, levels=levels, layout=layout)
    res = sg.sg_volume_create(dims, **kw)
    pyr = oracle.pyramid(vol, levels)
    grids = [oracle.brick_grid(dims, brick, L) for L in range(levels)]
    cache = sg.sg_volume_create(dims, cache_slots=sum(int(np.prod(g)) for g in grids), **kw)
    try:
        coords, cores = pack_bricks(vol, brick)
        sg.sg_upload_bricks(res, 0, 0, 0, coords, device_voxels(cores, shift))
        sg.sg_build_lod(res, 0, 0)
        for L, g in enumerate(grids):
            bz, by, bx = np.meshgrid(*[np.arange(k) for k in g[::-1]], indexing="ij")
            bs = np.stack([bx.ravel(), by.ravel(), bz.ravel()], 1)
            reg = np.stack([oracle.brick_region(pyr[L], brick, b) for b in bs])
            sg.sg_cache_put(cache, 0, 0, L, bs, device_voxels(reg.astype(dtype), shift))
        c = np.array(dims) / 2.0
        v = gen.view(gen.look_at(c + 1.7 * max(dims) * gen.unit((1.0, 0.6, 0.5)), c), 61, 47, 0.6)
        images = {}
        for h in (res, cache):
            sg.sg_set_transfer_function(h, 0, tf, 0, top)
            for model in ("ea", "mip"):
                for bias in range(levels):
                    out = torch.full((47, 61, 4), float("nan"), device="cuda")
                    sg.sg_render_views(h, [v], {"lod": 0, "bias": bias, "model": model}, [out])
                    images.setdefault((model, bias), []).append(out.cpu().numpy())
        for k, (a, b) in images.items():
            assert np.isfinite(a).all() and np.array_equal(a, b), k
        for bias in range(levels):
            p = {"lod": 0, "bias": bias}
            ids, empty = sg.sg_get_lod_cut(res, v, p)
            cids, cempty = sg.sg_get_lod_cut(cache, v, p)
            assert np.array_equal(ids, cids)
            want = expected_empty(pyr, brick, ids, len(tf), 71, (0, top))
            assert np.array_equal(empty, want) and np.array_equal(cempty, want)
    finally:
        sg.sg_volume_destroy(res)
        sg.sg_volume_destroy(cache)
