"""Cache puts move host regions through a staging buffer kept by the volume:
more regions than it holds, sources of every kind, sources overwritten as soon
as a put returns, puts that alternate between streams, a put that does not
fit, and a stream under capture."""
import numpy as np
import pytest

import gen

pytestmark = pytest.mark.gpu


def regions(vol, B, coords):
    from paper_1804_08197_amd.container import brick_regions
    import torch
    return brick_regions(torch.from_numpy(vol).cuda(), B, coords)


def view(dims, w=90, h=70):
    c = np.array(dims) / 2.0
    return gen.view(gen.look_at(c + max(dims) * np.array([1.1, 0.7, 0.5]), c), w, h, 0.6)


def image(h, v):
    import torch

    from paper_1804_08197_amd import sg
    out = torch.full((v["height"], v["width"], 4), float("nan"), device="cuda")
    sg.sg_render_views(h, [v], {"lod": 0, "step": 1.0}, [out])
    torch.cuda.synchronize()
    return out.cpu().numpy()


@pytest.mark.parametrize("source", ["pageable", "scattered", "device"])
def test_more_regions_than_the_buffer_holds(source):
    """40 bricks of 128^3 uint16: 176 MB of regions through 128 MiB."""
    import torch

    from paper_1804_08197_amd import sg, upload_volume
    from paper_1804_08197_amd.container import grid_coords, level_grids
    dims, B = (640, 512, 256), 128
    vol = np.random.default_rng(3).integers(0, 65536, dims[::-1], dtype=np.uint16)
    coords = grid_coords(level_grids(dims, B, 1)[0])
    reg = regions(vol, B, coords)
    full = sg.sg_volume_create(dims, dtype=sg.SG_U16, brick=B, levels=1)
    cache = sg.sg_volume_create(dims, dtype=sg.SG_U16, brick=B, levels=1, cache_slots=len(coords))
    try:
        upload_volume(full, torch.from_numpy(vol).cuda(), B)
        for h in (full, cache):
            sg.sg_set_transfer_function(h, 0, gen.tf_hot(a_start=40), 0, 65535)
        if source == "device":
            sg.sg_cache_put(cache, 0, 0, 0, coords, reg)
        else:
            host = torch.empty(reg.shape, dtype=torch.uint16, pin_memory=source == "scattered")
            host.copy_(reg)
            if source == "scattered":
                sg.sg_cache_put_scattered(cache, 0, 0, 0, coords,
                                          [host[i].data_ptr() for i in range(len(coords))])
            else:
                sg.sg_cache_put(cache, 0, 0, 0, coords, host.numpy())
            host.view(torch.int16).zero_()  # consumed before the put returned
        v = view(dims)
        assert np.array_equal(image(cache, v), image(full, v))
    finally:
        sg.sg_volume_destroy(full)
        sg.sg_volume_destroy(cache)


def test_streams_evictions_overflow_and_capture():
    import torch

    from paper_1804_08197_amd import sg, upload_volume
    from paper_1804_08197_amd.container import build_levels, grid_coords, level_grids
    dims, B, T = (61, 50, 43), 8, 6
    vols = [gen.random_volume(dims[::-1], 20 + t, dtype=np.uint8) for t in range(T)]
    grids = level_grids(dims, B, 3)
    n0, n1 = (len(grid_coords(g)) for g in grids[:2])
    top = len(grid_coords(grids[2]))
    slots = T * top + n0 + n1 + 5  # the lower levels of one timepoint
    h = sg.sg_volume_create(dims, timepoints=T, dtype=sg.SG_U8, brick=B, levels=3,
                            cache_slots=slots)
    full = sg.sg_volume_create(dims, dtype=sg.SG_U8, brick=B, levels=3)
    streams = [torch.cuda.Stream(), torch.cuda.Stream(), torch.cuda.current_stream()]
    v = view(dims)
    out = torch.empty(v["height"], v["width"], 4, device="cuda")
    host = torch.empty(200 * (B + 2) ** 3, dtype=torch.uint8, pin_memory=True)
    turn = 0
    try:
        for k in (h, full):
            sg.sg_set_transfer_function(k, 0, gen.tf_hot(a_start=40), 0, 255)
        for t in range(T):
            torch.cuda.synchronize()
            for lev, arr in reversed(list(enumerate(build_levels(vols[t], 3)))):
                coords = grid_coords(grids[lev])
                reg = regions(arr if isinstance(arr, np.ndarray) else arr.cpu().numpy(), B,
                              coords).cpu().numpy()
                for i in range(0, len(coords), 37):
                    part = torch.from_numpy(reg[i:i + 37].reshape(-1))
                    host[:len(part)].copy_(part)
                    addr = host.data_ptr() + np.arange(len(coords[i:i + 37])) * (B + 2) ** 3
                    sg.sg_cache_put_scattered(h, 0, t, lev, coords[i:i + 37], addr,
                                              stream=streams[turn % 3])
                    turn += 1
                if lev == 2:  # a frame later: what is stored from here is the newest
                    torch.cuda.synchronize()
                    sg.sg_render_views(h, [v], {"timepoint": t}, [out])
            torch.cuda.synchronize()
            upload_volume(full, torch.from_numpy(vols[t]).cuda(), B)
            sg.sg_render_views(h, [v], {"lod": 0, "step": 1.0, "timepoint": t}, [out])
            torch.cuda.synchronize()
            assert np.array_equal(out.cpu().numpy(), image(full, v)), t
        # a put that cannot find room changes nothing
        small = sg.sg_volume_create(dims, dtype=sg.SG_U8, brick=B, levels=3, cache_slots=top + n1)
        src = regions(vols[0], B, grid_coords(grids[0]))
        try:
            with pytest.raises(sg.SgError) as ex:
                sg.sg_cache_put(small, 0, 0, 0, grid_coords(grids[0]), src.cpu().numpy())
            assert ex.value.status == sg.SG_ERR_OUT_OF_MEMORY
            assert sg.sg_cache_get_info(small)["resident"] == 0
        finally:
            sg.sg_volume_destroy(small)
        # a stream under capture is refused and the cache is as before
        before = sg.sg_cache_get_info(h)
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            with pytest.raises(sg.SgError) as ex:
                sg.sg_cache_put(h, 0, 0, 0, grid_coords(grids[0])[:1], src[:1])
        assert ex.value.status == sg.SG_ERR_DEVICE
        assert sg.sg_cache_get_info(h) == before
    finally:
        sg.sg_volume_destroy(h)
        sg.sg_volume_destroy(full)
