"""Short frames of the gather kernel put four lanes to a ray, and pixels whose
rays cannot meet the volume are told by its projected corners: the same image,
depth and content flags bit for bit as the instrumented gather instance (one
lane to a ray, every ray set up) and, where steps add up exactly, as the
staged kernel; over image sizes that leave partial tiles, every option that
decides when a ray ends, and cameras for which the projection degenerates."""
import numpy as np
import pytest

import gen
from tests.helpers import LAYOUT_IDS, LAYOUTS, gpu_volume

pytestmark = pytest.mark.gpu

DIMS = (45, 52, 61)  # z, y, x
CENTRE = np.array([30.5, 26.0, 22.5])


def volume(dtype, brick, levels, layout, a_start=30):
    top = 255 if dtype == np.uint8 else 65535
    z, y, x = np.meshgrid(*(np.linspace(-1, 1, n) for n in DIMS), indexing="ij")
    v = np.clip(1.2 - np.sqrt(x * x + y * y + z * z), 0, 1) * (0.6 + 0.4 * np.sin(9 * x + 7 * y))
    v = np.maximum(v, np.random.default_rng(1).random(DIMS) * 0.3)
    return gpu_volume([(v * top).astype(dtype)], brick, levels, [gen.tf_hot(a_start=a_start)],
                      [(0, top)], layout=layout)


def view(w=75, h=58, fov=0.5, eye=(95.0, 60.0, 48.0), m=None, **kw):
    m = gen.look_at(CENTRE + np.array(eye), CENTRE) if m is None else m
    return dict(gen.view(m, w, h, fov), **kw)


def flags_of(v):
    import torch
    return torch.full(((v["height"] + 7) // 8, (v["width"] + 7) // 8), 9, dtype=torch.uint8,
                      device="cuda")


def render(h, views, params, how, depth=True):
    import torch

    from paper_1804_08197_amd import sg
    vs = [dict(v, tile_any=flags_of(v)) for v in views]
    nan = float("nan")
    img = [torch.full((v["height"], v["width"], 4), nan, device="cuda") for v in vs]
    dep = [torch.full((v["height"], v["width"]), nan, device="cuda") for v in vs] if depth else None
    p = dict(params, gather=int(how != "staged"))
    if how == "stats":
        sg.sg_render_views_stats(h, vs, p, img, dep)
    elif how == "noalloc":
        sg.sg_render_views_noalloc(h, vs, p, img, dep)
    elif how == "if":
        sg.sg_render_views_if(h, vs, p, img, torch.ones(1, dtype=torch.int32, device="cuda"), dep)
    else:
        sg.sg_render_views(h, vs, p, img, dep)
    torch.cuda.synchronize()
    return [t.cpu().numpy() for t in img + (dep or []) + [v["tile_any"] for v in vs]]


def same(h, views, params, depth=True, staged=True, ways=("gather",)):
    want = render(h, views, params, "stats", depth)
    assert np.isfinite(want[0]).all()
    for how in ways + (("staged",) if staged else ()):
        for a, b in zip(want, render(h, views, params, how, depth)):
            assert np.array_equal(a, b), how
    return want


@pytest.mark.parametrize("layout", LAYOUTS, ids=LAYOUT_IDS)
@pytest.mark.parametrize("dtype", [np.uint8, np.uint16])
@pytest.mark.parametrize("brick,levels", [(64, 1), (32, 2), (16, 3)])
def test_sizes_steps_and_levels(brick, levels, dtype, layout):
    from paper_1804_08197_amd import sg
    h = volume(dtype, brick, levels, layout)
    try:
        for w, y in ((1, 1), (7, 9), (8, 8), (17, 3), (75, 58), (130, 65)):
            for tile in (8, 16, 32):
                sg.sg_set_launch_config(h, {"kernel": 1, "tile": tile, "block": 32})
                same(h, [view(w, y), view(y, w, 0.3)], {"lod": 0}, depth=tile != 16)
        for step in (0.25, 1.0, 0.3, 1.7):
            for lod in (0, 1):
                same(h, [view()], {"step": step, "lod": lod, "tau": 1.5},
                     staged=step in (0.25, 1.0))
        if levels > 1:
            same(h, [view()], {"lod": 0, "bias": 1})
    finally:
        sg.sg_volume_destroy(h)


@pytest.mark.parametrize("a_start", [1, 60])
@pytest.mark.parametrize("params", [
    {"ert": 0.0}, {"ert": -1.0}, {"ert": 1e-30}, {"ert": 0.3}, {"ert": 1.0}, {"ert": 2.0},
    {"depth_alpha": 0.0}, {"depth_alpha": -0.5}, {"depth_alpha": 0.99}, {"depth_alpha": 1.5},
    {"bg": (0.1, 0.2, 0.3, 0.4)}, {"skip_empty": 0}, {"roi": (3.5, 2.0, 1.0, 40.0, 31.7, 44.0)},
    {"planes": ((0.6, 0.8, 0.0, -40.0), (0.0, 0.0, 1.0, -30.0))}])
def test_options(params, a_start):
    from paper_1804_08197_amd import sg
    h = volume(np.uint16, 32, 2, 0, a_start)
    try:
        for v in (view(), view(lens=(0.22, 0.24, 0.0, 0.0)), view(33, 41, 0.2)):
            same(h, [v], dict({"lod": 0}, **params))
    finally:
        sg.sg_volume_destroy(h)


def cameras():
    m = gen.look_at(CENTRE + np.array([95.0, 60.0, 48.0]), CENTRE)

    def with_(r=None, eye=None):
        n = m.copy()
        if r is not None:
            n[:3, :3] = m[:3, :3] @ np.asarray(r, float)
        if eye is not None:
            n[:3, 3] = eye
        return n
    yield "inside", view(m=with_(eye=CENTRE), fov=0.8)
    yield "corner", view(m=with_(eye=(0.0, 0.0, 0.0)))
    yield "near a face", view(m=with_(eye=(61.001, 26.0, 22.5)), fov=1.5)
    yield "face plane", view(m=with_(eye=(90.0, 52.0, 22.5)))
    yield "behind", view(m=with_(np.diag([-1.0, 1.0, -1.0])))
    yield "mirrored", view(m=with_(np.diag([-1.0, 1.0, 1.0])))
    yield "skewed", view(m=with_([[1.0, 0.4, 0.2], [0.0, 0.7, -0.3], [0.1, 0.0, 1.3]]))
    yield "flat", view(m=with_(np.diag([1.0, 1e-5, 1.0])))
    yield "large axes", view(m=with_(1e5 * np.eye(3)))
    yield "off screen", dict(view(), tan_left=2.0, tan_right=3.0)
    yield "partly off", dict(view(), tan_left=-0.02, tan_right=0.9, tan_bottom=-0.9, tan_top=0.01)
    yield "one pixel wide", view(w=1, h=300, fov=0.6)
    yield "narrow", view(fov=1e-9)
    yield "far", view(eye=(9.5e4, 6e4, 4.8e4), fov=5e-4)
    yield "very far", view(eye=(9.5e9, 6e9, 4.8e9), fov=5e-9)
    yield "grazing", view(eye=(95.0, 26.0 - 1e-9, 0.0), fov=0.7)


@pytest.mark.parametrize("name,v", list(cameras()), ids=[n for n, _ in cameras()])
def test_cameras(name, v):
    from paper_1804_08197_amd import sg
    h = volume(np.uint8, 32, 2, 1)
    try:
        for model in ("ea", "eo", "mip"):
            same(h, [v, view()], {"lod": 0, "model": model, "bg": (0.5, 0.0, 0.25, 1.0)})
    finally:
        sg.sg_volume_destroy(h)


def test_limits_routes_and_replays():
    """Ray limits, the render that allocates nothing, the gated one, and a
    graph whose views move the volume out of the image and back."""
    import torch

    from paper_1804_08197_amd import sg
    h = volume(np.uint16, 32, 2, 0)
    try:
        v, p = view(), {"lod": 0}
        lim = torch.from_numpy(np.random.default_rng(3).uniform(
            60, 160, (v["height"], v["width"])).astype(np.float32)).cuda()
        same(h, [dict(v, ray_limit=lim)], p, ways=("gather", "noalloc", "if"))
        away = dict(v, tan_left=2.0, tan_right=3.0)
        out = torch.empty(v["height"], v["width"], 4, device="cuda")
        g = sg.RenderGraph(h, [away], dict(p, gather=1), [out])
        for w in (away, v, away, view(eye=(60.0, -70.0, 40.0)), view(m=gen.look_at(
                CENTRE, CENTRE + 1.0))):
            g.set_views([w])
            g.launch()
            torch.cuda.synchronize()
            assert np.array_equal(out.cpu().numpy(), same(h, [w], p)[0])
        g.destroy()
    finally:
        sg.sg_volume_destroy(h)


def test_many_tiles_take_one_lane():
    """Both sides of the limits on the tiles (of the volume and of the image)."""
    from paper_1804_08197_amd import sg
    h = volume(np.uint8, 64, 1, 0)
    try:
        for w, n, fov in ((352, 1, 0.33), (368, 1, 0.33), (1024, 2, 1.5), (1032, 2, 1.5)):
            same(h, [view(w, w, fov)] * n, {"lod": 0})
    finally:
        sg.sg_volume_destroy(h)
