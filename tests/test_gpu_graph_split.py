"""A render graph takes four lanes to a ray, or one, by the poses of each
launch, not by those it was made with: a graph whose views were moved runs as
fast as one made with the same views, in both directions across the limit,
and renders the same image."""
import numpy as np
import pytest

import gen
from tests.helpers import gpu_volume, median_us

pytestmark = pytest.mark.gpu


# 64^3 filling two images: 32768 tiles, far beyond the limit of its 128 samples
# a ray; 256^3 in some 150 of 16384 tiles, far below the limit of its 512
@pytest.mark.parametrize("n,views,fov", [(64, 2, 0.2), (256, 1, 3.0)])
def test_moved_graph_runs_as_one_made_there(n, views, fov):
    import torch

    from paper_1804_08197_amd import sg
    r = np.random.default_rng(5)
    vol = (np.linspace(0, 90, n)[None, None] + r.integers(0, 30, (n, n, n))).astype(np.uint8)
    h = gpu_volume([vol], 64, 1, [gen.tf_hot(a_start=20)], [(0, 255)])
    try:
        cam = gen.look_at((1.9 * n, 1.6 * n, 1.2 * n), (n / 2, n / 2, n / 2))
        there = [gen.view(cam, 1024, 1024, fov)] * views
        away = [dict(v, tan_left=4.0, tan_right=5.0) if fov < 1 else gen.view(cam, 1024, 1024, 0.2)
                for v in there]
        p = {"lod": 0, "gather": 1}
        img = [torch.empty(1024, 1024, 4, device="cuda") for _ in there]
        made, moved = (sg.RenderGraph(h, v, p, img) for v in (there, away))
        moved.set_views(there)
        us = [median_us(g.launch) for g in (made, moved, made, moved)]
        print(us, flush=True)
        assert min(us[1], us[3]) <= 1.2 * min(us[0], us[2]), us
        sg.sg_render_views(h, there, p, img)
        torch.cuda.synchronize()
        want = [t.clone() for t in img]
        for g, v in ((made, there), (moved, there), (moved, away), (moved, there)):
            g.set_views(v)
            for t in img:
                t.fill_(float("nan"))
            g.launch()
            torch.cuda.synchronize()
            if v is there:
                assert all(torch.equal(a, b) for a, b in zip(img, want))
        made.destroy()
        moved.destroy()
    finally:
        sg.sg_volume_destroy(h)
