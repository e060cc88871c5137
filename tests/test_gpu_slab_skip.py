"""Slabs that cannot contribute are passed over (staged kernel, images only):
the same image bit for bit as the gather kernel and as the staged kernel
without skipping (its instrumented instance samples everything), for every
optical model, slot layout, voxel type and channel count, on scenes where
most slabs are passed over, some are and none is.

Also where stepping over is not allowed: a step whose multiples are not exact
in FP32, a first sample that decides (ert <= 0, depth_alpha <= 0), tables
whose values are huge; and render graphs replayed after the table changed
what is transparent."""
import numpy as np
import pytest

import gen
from tests.helpers import LAYOUT_IDS, LAYOUTS, gpu_volume

pytestmark = pytest.mark.gpu

DIMS = (61, 70, 66)  # z, y, x


def sparse_volume(dtype, seed, background):
    """A few bright boxes and a diagonal line of voxels over a background."""
    top = 255 if dtype == np.uint8 else 65535
    r = np.random.default_rng(seed)
    v = r.integers(0, background + 1, DIMS).astype(dtype)
    for _ in range(4):
        z, y, x = (int(r.integers(2, n - 9)) for n in DIMS)
        v[z:z + 5, y:y + 3, x:x + 7] = top * 3 // 4
    n = np.arange(60)
    v[n, n, n] = top
    return v


def view(w=75, h=58, fov=0.5):
    c = np.array([33.0, 35.0, 30.5])
    return gen.view(gen.look_at(c + np.array([95.0, 60.0, 48.0]), c), w, h, fov)


def images(h, params, v=None, depth=True):
    """(staged, staged instrumented, gather) images and depths."""
    import torch

    from paper_1804_08197_amd import sg
    v = v or view()
    out = []
    for how in ("staged", "stats", "gather"):
        img = torch.full((v["height"], v["width"], 4), float("nan"), device="cuda")
        dep = [torch.full((v["height"], v["width"]), float("nan"), device="cuda")] if depth else None
        p = dict(params, gather=int(how == "gather"))
        if how == "stats":
            sg.sg_render_views_stats(h, [v], p, [img], dep)
        else:
            sg.sg_render_views(h, [v], p, [img], dep)
        torch.cuda.synchronize()
        out.append((img.cpu().numpy(), dep[0].cpu().numpy() if depth else None))
    return out


def same(h, params, **kw):
    a, b, c = images(h, params, **kw)
    for other in (b, c):
        assert np.array_equal(a[0], other[0]) and np.isfinite(a[0]).all()
        if a[1] is not None:
            assert np.array_equal(a[1], other[1])
    return a


@pytest.mark.parametrize("layout", LAYOUTS, ids=LAYOUT_IDS)
@pytest.mark.parametrize("dtype,channels", [(np.uint8, 1), (np.uint16, 1), (np.uint16, 2),
                                            (np.uint8, 3), (np.uint16, 4)])
@pytest.mark.parametrize("start", [0, 1, 40, 254])
def test_every_model_renders_the_same_bits(dtype, channels, start, layout):
    from paper_1804_08197_amd import sg
    top = 255 if dtype == np.uint8 else 65535
    vols = [sparse_volume(dtype, 5 + c, 20 * top // 255) for c in range(channels)]
    tf = gen.tf_hot(a_start=start)
    tf[:max(start, 1), :3] = 0.0  # dark where transparent, for emission-only
    h = gpu_volume(vols, 32, 3, [tf] * channels, [(0, top)] * channels, layout=layout)
    try:
        for model in ("ea", "eo", "mip"):
            for step in (0.5, 0.3, 1.0):
                for lod in (0, 1):
                    same(h, {"model": model, "step": step, "lod": lod, "tau": 2.0})
    finally:
        sg.sg_volume_destroy(h)


@pytest.mark.parametrize("params", [{"ert": 0.0}, {"ert": -1.0}, {"depth_alpha": 0.0},
                                    {"depth_alpha": -0.5}, {"step": 0.3}, {"ert": 2.0},
                                    {"bg": (0.1, 0.2, 0.3, 0.4)}, {"skip_empty": 0}])
def test_options_that_make_clear_samples_count(params):
    from paper_1804_08197_amd import sg
    tf = gen.tf_hot(a_start=60)
    h = gpu_volume([sparse_volume(np.uint16, 9, 3000)], 64, 1, [tf], [(0, 65535)], layout=1)
    try:
        same(h, dict({"lod": 0}, **params))
    finally:
        sg.sg_volume_destroy(h)


@pytest.mark.parametrize("domain", [(0.0, 65535.0), (-9000.0, 70000.0), (3000.0, 3000.5),
                                    (1e-30, 2e-30), (-1e300, 1e300), (0.0, 1e-42)])
def test_unusual_windows_and_tables(domain):
    from paper_1804_08197_amd import sg
    tf = gen.tf_hot(a_start=100)
    h = gpu_volume([sparse_volume(np.uint16, 3, 3000)], 32, 2, [tf], [domain], layout=0)
    try:
        for t in (tf, np.where(np.arange(256)[:, None] < 60, [3e38, -3e38, 1.0, 0.0], tf)):
            sg.sg_set_transfer_function(h, 0, t, *domain)
            a, b, c = images(h, {"lod": 0}, depth=False)
            for o in (b, c):
                assert np.array_equal(a[0], o[0], equal_nan=True)
    finally:
        sg.sg_volume_destroy(h)


def test_graph_replays_follow_the_table():
    """What is transparent is read when the graph runs, not when it is made."""
    import torch

    from paper_1804_08197_amd import sg
    tf = gen.tf_hot(a_start=200)
    h = gpu_volume([sparse_volume(np.uint16, 4, 20000)], 32, 2, [tf], [(0, 65535)], layout=1)
    try:
        v, p = view(), {"lod": 0}
        out = torch.empty(v["height"], v["width"], 4, device="cuda")
        g = sg.RenderGraph(h, [v], p, [out])
        for start in (200, 0, 90, 254, 10):
            sg.sg_set_transfer_function(h, 0, gen.tf_hot(a_start=start), 0, 65535)
            g.launch()
            torch.cuda.synchronize()
            got = out.cpu().numpy().copy()
            want = same(h, p, depth=False)[0]
            assert np.array_equal(got, want)
        g.destroy()
    finally:
        sg.sg_volume_destroy(h)
