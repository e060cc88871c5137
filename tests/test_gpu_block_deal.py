"""Screen blocks are dealt to the XCDs eight at a time, turned where a view is
a multiple of eight blocks wide or one more: every pixel is rendered once,
whatever the widths around those, with views of one size and of several."""
import numpy as np
import pytest

import gen
from tests.helpers import gpu_volume

pytestmark = pytest.mark.gpu


def images(h, views, params):
    import torch

    from paper_1804_08197_amd import sg
    out = [torch.full((v["height"], v["width"], 4), float("nan"), device="cuda") for v in views]
    sg.sg_render_views(h, views, params, out)
    torch.cuda.synchronize()
    return [o.cpu().numpy() for o in out]


@pytest.mark.parametrize("gather", [0, 1])
@pytest.mark.parametrize("sizes", [
    [(224, 70)], [(225, 33)], [(256, 70)], [(257, 100)], [(288, 64)], [(289, 97)], [(512, 40)],
    [(513, 65)], [(256, 32)], [(256, 97)] * 2, [(280, 97)] * 3, [(225, 33)] * 2,
    [(256, 33), (40, 90), (257, 65), (8, 8), (1, 1), (288, 97), (33, 500), (512, 31)],
    [(1, 1)] * 9 + [(256, 40)] + [(1, 1)] * 10 + [(280, 70)]])
def test_every_block_is_dealt_once(sizes, gather):
    from paper_1804_08197_amd import sg
    vol = gen.random_volume((30, 40, 50), 7, dtype=np.uint8)
    h = gpu_volume([vol], 32, 2, [gen.tf_hot(a_start=90)], [(0, 255)])
    c = np.array([25.0, 20.0, 15.0])
    views = [gen.view(gen.look_at(c + np.array([70.0, 40.0 + i, 35.0]), c), w, y, 0.5)
             for i, (w, y) in enumerate(sizes)]
    params = {"lod": 0, "gather": gather, "bg": (0.1, 0.2, 0.3, 1.0)}
    try:
        out = []
        for tile, block in ((8, 32), (16, 32), (16, 64), (16, 128), (32, 32)):
            sg.sg_set_launch_config(h, {"kernel": gather, "tile": tile, "block": block})
            out.append(images(h, views, params))
        one = [images(h, [v], params)[0] for v in views]
        for got in out:
            for a, b in zip(got, one):
                assert np.isfinite(a).all() and np.array_equal(a, b)
    finally:
        sg.sg_volume_destroy(h)
