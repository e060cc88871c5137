"""Where four lanes to a ray cost more than they save, the frame runs with
one: an opaque table, small bricks, a small region of interest. The same frame
with a step that does not add up exactly always runs with one lane to a ray
and takes the same samples within a few, so it is the measure. And the screen
bounds of a region of interest leave the image as it is, bit for bit."""
import numpy as np
import pytest

import gen
from tests.helpers import gpu_volume, median_us
from tests.test_gpu_split_rays import CENTRE, same, view, volume

pytestmark = pytest.mark.gpu


def blobs(n):
    t = (np.arange(n) + 0.5) / n - 0.5
    r2 = (t ** 2)[:, None, None] + (t ** 2)[None, :, None] + (t ** 2)[None, None]
    return (160 * np.exp(-8 * r2) + np.random.default_rng(2).integers(0, 16, (n, n, n))).astype(np.uint8)


def ramp(floor=0.0):
    k = np.arange(256) / 255
    return np.stack([k, k, k, np.maximum(k, floor)], 1)


@pytest.mark.parametrize("what,n,brick,px,params", [
    ("opaque", 512, 64, 1100, {}), ("opaque", 256, 64, 800, {}),
    ("bricks of 4", 256, 4, 800, {}), ("bricks of 8", 512, 8, 1100, {}),
    ("region", 512, 64, 1100, {"roi": (217.0, 217.0, 217.0, 295.0, 295.0, 295.0)})])
def test_no_slower_than_one_lane(what, n, brick, px, params):
    import torch

    from paper_1804_08197_amd import sg
    # (the region holds nothing to see through either)
    floor = 0.0 if what.startswith("bricks") else 5.0 if what == "opaque" else 0.5
    h = gpu_volume([blobs(n)], brick, 1, [ramp(floor)], [(0, 255)])
    try:
        d = np.array((1.0, 0.7, 0.4))
        cam = gen.look_at(np.full(3, n / 2) + 1.6 * n * d / np.linalg.norm(d), np.full(3, n / 2))
        v = gen.view(cam, px, px, np.tan(np.radians(30)))
        img = [torch.empty(px, px, 4, device="cuda")]
        p = dict(params, lod=0, gather=1)
        us = [median_us(lambda: sg.sg_render_views(h, [v], dict(p, step=s), img))
              for s in (0.5, 0.4999, 0.5, 0.4999)]
        print(what, us, flush=True)
        assert min(us[0], us[2]) <= 1.2 * min(us[1], us[3]), us
    finally:
        sg.sg_volume_destroy(h)


def test_region_bounds_leave_the_image():
    from paper_1804_08197_amd import sg
    h = volume(np.uint8, 16, 2, 1)
    try:
        inside = gen.look_at(CENTRE, CENTRE + 1.0)
        for roi in ((20.0, 18.0, 15.0, 33.5, 29.0, 31.25), (-9.0, -9.0, -9.0, 20.0, 70.0, 9.0),
                    (61.0, 0.0, 0.0, 80.0, 52.0, 45.0), (70.0, 0.0, 0.0, 80.0, 52.0, 45.0),
                    (30.0, 30.0, 10.0, 30.0, 40.0, 20.0), (0.0, 0.0, 0.0, 0.125, 0.125, 0.125),
                    (-5.0, -5.0, -5.0, 100.0, 100.0, 100.0)):
            for v in (view(), view(33, 41, 0.2), view(lens=(0.22, 0.24, 0.0, 0.0)),
                      view(eye=(0.0, 95.0, 1e-9), fov=0.8), view(m=inside, fov=1.2)):
                for model in ("ea", "mip"):
                    same(h, [v], {"lod": 0, "roi": roi, "model": model,
                                  "bg": (0.5, 0.0, 0.25, 1.0)})
    finally:
        sg.sg_volume_destroy(h)
