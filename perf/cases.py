"""The workloads by which this renderer's speed is judged.

Each case is one call (or one step of a loop) that a program using the
library makes, through the public entry points of ``paper_1804_08197_amd``:
frames of the three synthetic scenes under their options, a batch of uneven
views, the learned upsampler's frame, network and training step, and the
work that brings data in (a resident volume opened from brick chunks, the
import of an out-of-core volume, playback through the brick cache) or puts
part images together. ``exact`` holds plain torch float64 versions of the
same computations, written from their definitions.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_1804_08197_amd import container, pack_bricks, sg, upload_volume
from paper_1804_08197_amd import upsample, upsampler

DEV = "cuda"

# ------------------------------------------------------------------- cases
# What each listed case stands for in use is said beside it. "frame" cases
# share their fields: scene, dims, brick / levels / layout of the volume,
# views and their size, the optical model and options, and the launch
# configuration (the autotuner's choice for the scene where the benchmark
# tunes it, else the default).
FRAME = {"kind": "frame", "scene": "blobs", "x": 128, "y": 128, "z": 128, "channels": 1,
         "brick": 128, "levels": 1, "micro": False, "width": 256, "height": 256, "views": 1,
         "fov": 30.0, "distance": 4.33, "model": "ea", "gather": True, "tile": 16, "block": 64,
         "stage": 8192, "lod": False, "lens": False, "roi": False, "depth": False}


def _frame(**kw):
    return dict(FRAME, **kw)


def listed():
    return [
        # The smallest call: a preview window of a small 8-bit volume that is
        # one brick; the frame is as long as its longest rays and launches.
        _frame(name="blobs_256", tile=8),
        # The headset frame of a large 16-bit volume: both eyes at 1440x1600,
        # screen-space level of detail, mostly empty space with thin tubes.
        _frame(name="tubes_stereo", scene="tubes", x=1024, y=1024, z=1024, brick=64, levels=5,
               micro=True, width=1440, height=1600, views=2, fov=50.0, distance=1.25,
               gather=False, block=32, lod=True),
        # The headset frame of a three-channel microscopy timepoint.
        _frame(name="cells3_stereo", scene="cells", x=1024, y=1024, z=512, channels=3, brick=64,
               levels=5, micro=True, width=1440, height=1600, views=2, fov=50.0, distance=1.25,
               gather=False, lod=True),
        # A maximum-intensity view through the headset's lens map inside a
        # region of interest: the analysis tools' frame, on a ragged volume
        # of the default slot layout.
        _frame(name="mip_lens_roi", scene="cells", x=500, y=471, z=390, brick=32, levels=4,
               width=1080, height=1200, views=2, fov=50.0, distance=1.25, model="mip",
               gather=False, lod=True, lens=True, roi=True),
        # Many uneven views of one small volume in one call (thumbnails,
        # remote viewers), with first-hit depth.
        {"name": "batch_views", "kind": "batch", "views": 24, "lo": 320, "hi": 1100,
         "gather": False},
        # The learned-upsampler frame (half-resolution cast, network, gated
        # full-resolution render) for both eyes.
        {"name": "upsampled_frame", "kind": "upframe", "width": 1440, "height": 1600},
        # The upsampler network alone on full images (no empty tiles), with
        # the predicted error: a dense scene fills the view.
        {"name": "network_dense", "kind": "network", "n": 2, "h": 800, "w": 720},
        # One training step of the upsampler on a batch of 256x256 windows.
        {"name": "train_step", "kind": "train", "n": 16, "h": 128, "w": 128},
        # A resident volume opened, or its next timepoint: brick chunks
        # uploaded, pyramid built, committed, first frame shown.
        {"name": "open_volume", "kind": "open", "x": 512, "y": 512, "z": 512, "brick": 64,
         "levels": 4, "u8": False, "micro": True, "width": 640, "height": 480},
        # Import of an out-of-core volume: the resolution pyramid and every
        # level cut into whole bricks.
        {"name": "import_bricks", "kind": "import", "x": 700, "y": 512, "z": 420, "brick": 64,
         "levels": 4, "u8": False},
        # Movie playback: two timepoints streamed in turn from page-locked
        # host memory through the brick cache, a frame after every load.
        {"name": "playback", "kind": "play", "x": 384, "y": 384, "z": 256, "channels": 2,
         "brick": 64, "levels": 3, "width": 720, "height": 800},
        # Sort-last compositing of eight octant images of one eye.
        {"name": "composite_8", "kind": "composite", "width": 1440, "height": 1600, "parts": 8},
    ]


def _log(rng, lo, hi, even=False):
    v = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    return max(2, v - v % 2) if even else v


def draw(rng):
    kind = rng.choice(["frame", "frame", "frame", "batch", "upframe", "network", "train", "open",
                       "import", "play", "composite"])
    if kind == "frame":
        scene = rng.choice(["blobs", "tubes", "cells"])
        w = _log(rng, 128, 1440)
        h = max(96, min(1600, int(w * rng.uniform(0.6, 1.3))))
        if scene == "blobs":
            n = [rng.randint(60, 200) for _ in range(3)]
            return _frame(x=n[0], y=n[1], z=n[2], width=w, height=h, views=rng.randint(1, 2),
                          brick=rng.choice([64, 128, 256]), gather=rng.random() < 0.5,
                          tile=rng.choice([8, 16]), model=rng.choice(["ea", "eo", "mip"]), depth=rng.random() < 0.5,
                          distance=rng.uniform(1.5, 4.3), lens=rng.random() < 0.3)
        n = [_log(rng, 150, 800) for _ in range(3)]
        model = rng.choice(["ea", "ea", "eo", "mip"])
        return _frame(scene=scene, x=n[0], y=n[1], z=n[2],
                      channels=1 if scene == "tubes" else rng.randint(1, 3),
                      brick=rng.choice([32, 64]), levels=rng.randint(2, 5),
                      micro=rng.random() < 0.7, width=w, height=h, views=rng.randint(1, 2),
                      fov=50.0, distance=rng.uniform(0.9, 1.6), model=model, gather=False,
                      block=rng.choice([32, 64]), stage=rng.choice([4096, 8192]),
                      lod=True, lens=rng.random() < 0.2, roi=rng.random() < 0.2,
                      depth=model == "ea" and rng.random() < 0.3)
    if kind == "batch":
        lo = _log(rng, 64, 400)
        return {"kind": kind, "views": rng.randint(5, 24), "lo": lo,
                "hi": lo + rng.randint(10, 600), "gather": rng.random() < 0.5}
    if kind == "upframe":
        w = _log(rng, 320, 1440, even=True)
        return {"kind": kind, "width": w, "height": max(2, int(w * rng.uniform(0.6, 1.11)) // 2 * 2)}
    if kind == "network":
        return {"kind": kind, "n": rng.randint(1, 2), "h": _log(rng, 60, 800),
                "w": _log(rng, 60, 720)}
    if kind == "train":
        c = _log(rng, 32, 128)
        return {"kind": kind, "n": rng.randint(2, 16), "h": c, "w": c}
    if kind == "open":
        n = [_log(rng, 100, 512) for _ in range(3)]
        return {"kind": kind, "x": n[0], "y": n[1], "z": n[2], "brick": rng.choice([32, 64, 128]),
                "levels": rng.randint(1, 4), "u8": rng.random() < 0.4,
                "micro": rng.random() < 0.6, "width": _log(rng, 160, 640),
                "height": _log(rng, 120, 480)}
    if kind == "import":
        n = [_log(rng, 100, 512) for _ in range(3)]
        return {"kind": kind, "x": n[0], "y": n[1], "z": n[2], "brick": rng.choice([32, 64]),
                "levels": rng.randint(2, 4), "u8": rng.random() < 0.4}
    if kind == "play":
        n = [_log(rng, 120, 320) for _ in range(3)]
        return {"kind": kind, "x": n[0], "y": n[1], "z": n[2], "channels": rng.randint(1, 2),
                "brick": rng.choice([32, 64]), "levels": rng.randint(2, 3),
                "width": _log(rng, 200, 720), "height": _log(rng, 200, 800)}
    return {"kind": kind, "width": _log(rng, 200, 1440), "height": _log(rng, 200, 1600),
            "parts": rng.choice([2, 4, 8])}


# ------------------------------------------------------------------ inputs
def _gen(seed, salt=0):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) * 1000003 + salt)
    return g


def _gauss(n, centre, sigma):
    t = torch.arange(n, device=DEV, dtype=torch.float32) + 0.5
    return torch.exp(-0.5 * ((t[None] - centre[:, None]) / sigma[:, None]) ** 2)


def _blob_field(dims, cen, sig, amp, z0, z1):
    """sum_b amp_b of separable Gaussians on planes z0 .. z1 - 1, [z, y, x]."""
    gx, gy, gz = (_gauss(dims[i], cen[:, i], sig) for i in range(3))
    zy = (gz[:, z0:z1, None] * gy[:, None, :]).reshape(len(sig), -1) * amp[:, None]
    return (zy.t() @ gx).reshape(z1 - z0, dims[1], dims[0])


def _blobs(dims, seed):
    """8-bit volume: eight Gaussian blobs over uniform noise."""
    r = np.random.default_rng(seed + 1001)
    sc = min(dims) / 128.0
    f32 = dict(device=DEV, dtype=torch.float32)
    cen = torch.tensor(r.uniform(0, 1, (8, 3)) * np.array(dims), **f32)
    sig = torch.tensor(r.uniform(6, 20, 8) * sc, **f32)
    amp = torch.tensor(r.uniform(100, 255, 8), **f32)
    f = _blob_field(dims, cen, sig, amp, 0, dims[2])
    f += 16 * torch.rand(f.shape, device=DEV, generator=_gen(seed, 1))
    return f.round().clamp(0, 255).to(torch.uint8)


def _cells(dims, channel, seed):
    """16-bit channel: 200 Gaussian cells over broad background Gaussians."""
    r = np.random.default_rng((seed + 7) * 16 + channel)
    f32 = dict(device=DEV, dtype=torch.float32)
    n = 200
    cen = r.uniform(0, 1, (n + 4, 3)) * np.array(dims)
    sig = np.concatenate([r.uniform(4, 12, n) * max(dims) / 1024 + 1, np.full(4, 0.2 * max(dims))])
    amp = np.concatenate([r.uniform(5000, 40000, n), r.uniform(500, 1500, 4)])
    cen, sig, amp = (torch.tensor(a, **f32) for a in (cen, sig, amp))
    out = torch.empty(dims[2], dims[1], dims[0], device=DEV, dtype=torch.uint16)
    for z in range(0, dims[2], 64):
        z1 = min(dims[2], z + 64)
        out[z:z1] = _blob_field(dims, cen, sig, amp, z, z1).round().clamp(0, 65535) \
            .to(torch.int32).to(torch.uint16)
    return out


def _tubes(dims, seed):
    """16-bit volume: random-walk filaments of Gaussian cross-section over a
    Poisson(200)-like background."""
    r = np.random.default_rng(seed + 1002)
    d3 = np.array(dims, dtype=np.float64)
    n, step = 120, 2.0
    steps = int(max(dims) / step)
    pos = np.empty((n, steps, 3))
    p = r.uniform(0, 1, (n, 3)) * d3
    d = r.normal(size=(n, 3))
    for s in range(steps):
        d += 0.15 * r.normal(size=(n, 3))
        d /= np.linalg.norm(d, axis=1, keepdims=True)
        p = p + step * d
        pos[:, s] = p
    out = torch.empty(dims[2], dims[1], dims[0], device=DEV, dtype=torch.int32)
    g = _gen(seed, 2)
    for z in range(0, dims[2], 64):
        s = out[z:z + 64]
        s.copy_((200 + 14.14 * torch.randn(s.shape, device=DEV, generator=g)).round().clamp_(min=0))
    radius = r.integers(1, 7, n)
    amp = torch.tensor(r.uniform(2000, 60000, n), device=DEV, dtype=torch.float32)
    pos_t = torch.tensor(pos, device=DEV, dtype=torch.float32)
    flat = out.view(-1)
    dt = torch.tensor(dims, device=DEV)
    for rad in range(1, 7):
        sel = torch.tensor(np.nonzero(radius == rad)[0], device=DEV)
        if not len(sel):
            continue
        R = int(2.5 * rad) + 1
        o = torch.arange(-R, R + 1, device=DEV)
        off = torch.stack(torch.meshgrid(o, o, o, indexing="ij"), -1).reshape(-1, 3)
        pts = pos_t[sel].reshape(-1, 3)
        a = amp[sel].repeat_interleave(steps)
        keep = ((pts > -R) & (pts < dt + R)).all(1)
        pts, a = pts[keep], a[keep]
        per = max(1, (1 << 24) // len(off))
        for i in range(0, len(pts), per):
            v = pts[i:i + per].floor().long()[:, None] + off[None]
            d2 = ((v + 0.5 - pts[i:i + per, None]) ** 2).sum(-1)
            val = (a[i:i + per, None] * torch.exp(-0.5 * d2 / rad ** 2)).to(torch.int32)
            ok = ((v >= 0) & (v < dt)).all(-1) & (val > 0)
            idx = ((v[..., 2] * dims[1] + v[..., 1]) * dims[0] + v[..., 0])[ok]
            flat.scatter_reduce_(0, idx, val[ok], "amax")
    return out.clamp_(max=65535).to(torch.uint16)


def _ramp(n=256):
    k = np.arange(n) / (n - 1)
    return np.stack([k, k, k, k], 1)


def _hot(n=256, start=5, top=0.25):
    k = np.arange(n, dtype=np.float64)
    s = k / (n - 1)
    a = np.where(k < start, 0.0, top * (k - start) / (n - 1 - start))
    return np.stack([np.minimum(1, 3 * s), np.clip(3 * s - 1, 0, 1), np.clip(3 * s - 2, 0, 1), a], 1)


def _tint(rgb, n=256, start=12, top=0.15):
    k = np.arange(n, dtype=np.float64)
    a = np.where(k < start, 0.0, top * (k - start) / (n - 1 - start))
    return np.concatenate([np.outer(k / (n - 1), rgb), a[:, None]], 1)


TINTS = ((1.0, 0.2, 0.2), (0.2, 1.0, 0.2), (0.3, 0.3, 1.0))


def _scene(scene, dims, channels, seed):
    """(channel volumes [z, y, x], transfer tables, value domain)."""
    if scene == "blobs":
        return [_blobs(dims, seed)], [_ramp()], (0.0, 255.0)
    if scene == "tubes":
        return [_tubes(dims, seed)], [_hot()], (0.0, 65535.0)
    return ([_cells(dims, c, seed) for c in range(channels)], [_tint(t) for t in TINTS[:channels]],
            (0.0, 50000.0))


def _look_at(eye, target):
    f = np.asarray(target, dtype=np.float64) - eye
    f /= np.linalg.norm(f)
    r = np.cross(f, (0.0, 0.0, 1.0))
    r /= np.linalg.norm(r)
    m = np.eye(4)
    m[:3, 0], m[:3, 1], m[:3, 2], m[:3, 3] = r, np.cross(r, f), -f, eye
    return m


def _views(dims, n, width, height, fov, distance, seed, lens=False):
    """n = 1: one camera; n = 2: an eye pair. The head is `distance` longest
    edges from the centre, the direction moves a little with the seed."""
    r = np.random.default_rng(seed + 31)
    c = np.array(dims) / 2.0
    u = np.array((1.0, 0.7, 0.4)) + r.uniform(-0.1, 0.1, 3)
    head = c + distance * max(dims) * u / np.linalg.norm(u)
    m = _look_at(head, c)
    t = math.tan(math.radians(fov))
    tr = t * width / height
    out = []
    for s in ([0.0] if n == 1 else [-0.5, 0.5]):
        mm = m.copy()
        mm[:3, 3] = head + s * 0.064 * max(dims) * m[:3, 0]
        v = {"cam_to_world": mm, "tan_left": -tr, "tan_right": tr, "tan_bottom": -t, "tan_top": t,
             "width": width, "height": height}
        if lens:
            v["lens"] = (0.22, 0.24, 0.0, 0.0)
        out.append(v)
    return out


class _Volume:
    """A volume handle that is given back with its last reference."""

    def __init__(self, *a, **kw):
        self.h = sg.sg_volume_create(*a, **kw)

    def __del__(self):
        sg.sg_volume_destroy(self.h)


class _Model:
    def __init__(self, pixels, seed):
        self.m = upsampler.Upsampler(pixels)
        self.m.set_weights(_weights(seed))

    def __del__(self):
        self.m.close()


def _weights(seed):
    """Trained-looking weights: He-style layers, small biases, a small last
    layer (the network corrects the bilinear image)."""
    r = np.random.default_rng(seed + 77)
    w = upsample.init_params(r)
    out = []
    for k, b in upsampler.unpack(w):
        out.append((k, b + 0.02 * r.normal(size=b.shape)))
    return upsampler.pack(out)


def _resident(vols, tables, domain, dims, brick, levels, micro, u8):
    v = _Volume(dims, channels=len(vols), dtype=sg.SG_U8 if u8 else sg.SG_U16, brick=brick,
                levels=levels,
                layout=sg.SG_LAYOUT_MICROBLOCK if micro else sg.SG_LAYOUT_LINEAR)
    for c, vol in enumerate(vols):
        upload_volume(v.h, vol, brick, channel=c)
        sg.sg_set_transfer_function(v.h, c, tables[c], *domain)
    sg.sg_volume_commit(v.h)
    return v


def _images(views, depth=False):
    rgba = [torch.empty(v["height"], v["width"], 4, device=DEV) for v in views]
    return rgba, [torch.empty(v["height"], v["width"], device=DEV) for v in views] if depth else None


def _smooth_images(n, h, w, c, seed):
    """Smooth premultiplied-looking images in [0, 1] with some grain."""
    g = _gen(seed, 5)
    lo = torch.rand(n, c, 2 + h // 24, 2 + w // 24, device=DEV, generator=g)
    f = torch.nn.functional.interpolate(lo, (h, w), mode="bilinear", align_corners=False)
    f = (f + 0.03 * torch.rand(f.shape, device=DEV, generator=g)).clamp(0.02, 1.0)
    return f.permute(0, 2, 3, 1).contiguous()


def _batch_views(case, seed):
    r = np.random.default_rng(seed + 1004)
    out = []
    for _ in range(case["views"]):
        u = r.normal(size=3)
        u[2] = np.clip(u[2], -0.9, 0.9) * 0.7
        u /= np.linalg.norm(u)
        w, h = (int(x) for x in r.integers(case["lo"], case["hi"] + 1, 2))
        eye = 64.0 + r.uniform(1.5, 4.0) * 128 * math.sqrt(3) * u
        t = math.tan(math.radians(30))
        out.append({"cam_to_world": _look_at(eye, (64.0, 64.0, 64.0)), "tan_left": -t * w / h,
                    "tan_right": t * w / h, "tan_bottom": -t, "tan_top": t, "width": w,
                    "height": h})
    # the sizes come from the case alone: every seed has the same pixels
    q = np.random.default_rng(case["views"] * 10007 + case["lo"])
    for v in out:
        w, h = (int(x) for x in q.integers(case["lo"], case["hi"] + 1, 2))
        v.update(width=w, height=h, tan_left=-t * w / h, tan_right=t * w / h)
    return out


def _params(case):
    p = {"step": 0.5, "ert": 0.99, "tau": 1.0, "lod": int(case["lod"]), "skip_empty": 1,
         "model": case["model"]}
    if case["roi"]:
        d = np.array([case["x"], case["y"], case["z"]], dtype=np.float64)
        p["roi"] = np.stack([0.2 * d, 0.85 * d])
    return p


def _dims(case):
    return (case["x"], case["y"], case["z"])


def _up_views(case, seed):
    return _views((128, 128, 128), 2, case["width"], case["height"], 30.0, 3.6, seed)


UP_DEPTH = 128 * math.sqrt(3.0)


def _parts(case):
    """The boxes of a split of the unit scene into 2, 4 or 8 parts."""
    axes = {2: (2, 1, 1), 4: (2, 2, 1), 8: (2, 2, 2)}[case["parts"]]
    out = []
    for z in range(axes[2]):
        for y in range(axes[1]):
            for x in range(axes[0]):
                lo = [1024.0 * i / a for i, a in zip((x, y, z), axes)]
                out.append(lo + [b + 1024.0 / a for b, a in zip(lo, axes)])
    return np.array(out)


def prepare(case, seed):
    kind = case["kind"]
    if kind == "frame":
        vols, tables, domain = _scene(case["scene"], _dims(case), case["channels"], seed)
        vol = _resident(vols, tables, domain, _dims(case), case["brick"], case["levels"],
                        case["micro"], case["scene"] == "blobs")
        sg.sg_set_launch_config(vol.h, {"kernel": int(case["gather"]), "tile": case["tile"],
                                        "block": case["block"], "stage_bytes": case["stage"]})
        views = _views(_dims(case), case["views"], case["width"], case["height"], case["fov"],
                       case["distance"], seed, case["lens"])
        rgba, depth = _images(views, case["depth"])
        return {"kind": kind, "vol": vol, "views": views, "params": _params(case), "rgba": rgba,
                "depth": depth}
    if kind == "batch":
        vol = _resident([_blobs((128, 128, 128), seed)], [_ramp()], (0.0, 255.0), (128, 128, 128),
                        128, 1, False, True)
        views = _batch_views(case, seed)
        rgba, depth = _images(views, True)
        return {"kind": "frame", "vol": vol, "views": views, "rgba": rgba, "depth": depth,
                "params": {"step": 0.5, "ert": 0.99, "lod": 0, "gather": int(case["gather"])}}
    if kind == "upframe":
        vol = _resident([_blobs((128, 128, 128), seed)], [_ramp()], (0.0, 255.0), (128, 128, 128),
                        64, 2, False, True)
        w, h = case["width"], case["height"]
        model = _Model(2 * (w // 2) * (h // 2), seed)
        # the launch configurations the benchmark settles on for this scene
        path = upsample.UpsampledPath(
            vol.h, model.m, UP_DEPTH, {"step": 0.5, "ert": 0.99}, w, h, 2, threshold_db=-200.0,
            launch_half={"kernel": 1, "tile": 16, "block": 64},
            launch_full={"kernel": 0, "tile": 32, "block": 64})
        return {"kind": kind, "vol": vol, "model": model, "path": path,
                "views": _up_views(case, seed),
                "flag": torch.zeros(1, dtype=torch.int32, device=DEV)}
    if kind in ("network", "train"):
        n, h, w = case["n"], case["h"], case["w"]
        f = _smooth_images(n, h, w, 5, seed)
        s = {"kind": kind, "model": _Model(n * h * w, seed), "rgba": f[..., :4].contiguous(),
             "depth": (f[..., 4] * 400 + 50).contiguous()}
        s["depth"][f[..., 4] < 0.25] = math.inf
        if kind == "network":
            s["out"] = torch.empty(n, 2 * h, 2 * w, 4, device=DEV)
            s["err"] = torch.empty(n, 2 * h, 2 * w, device=DEV)
        else:
            up = torch.nn.functional.interpolate(s["rgba"].permute(0, 3, 1, 2), scale_factor=2,
                                                 mode="bilinear", align_corners=False)
            s["target"] = (up.permute(0, 2, 3, 1) + 0.05 * torch.randn(
                n, 2 * h, 2 * w, 4, device=DEV, generator=_gen(seed, 6))).contiguous()
        return s
    if kind == "open":
        dims = _dims(case)
        data = _blobs(dims, seed) if case["u8"] else _cells(dims, 0, seed)
        vol = _Volume(dims, dtype=sg.SG_U8 if case["u8"] else sg.SG_U16, brick=case["brick"],
                      levels=case["levels"],
                      layout=sg.SG_LAYOUT_MICROBLOCK if case["micro"] else sg.SG_LAYOUT_LINEAR)
        table, domain = _open_table(case)
        sg.sg_set_transfer_function(vol.h, 0, table, *domain)
        coords, cores = pack_bricks(data, case["brick"])
        views = _views(dims, 1, case["width"], case["height"], 30.0, 1.6, seed)
        return {"kind": kind, "vol": vol, "coords": coords, "cores": cores, "views": views,
                "rgba": _images(views)[0]}
    if kind == "import":
        data = _blobs(_dims(case), seed) if case["u8"] else _cells(_dims(case), 0, seed)
        return {"kind": kind, "data": data, "brick": case["brick"], "levels": case["levels"],
                "coords": [container.grid_coords(g) for g in
                           container.level_grids(_dims(case), case["brick"], case["levels"])]}
    if kind == "play":
        dims, B, L, C = _dims(case), case["brick"], case["levels"], case["channels"]
        grids = container.level_grids(dims, B, L)
        nodes = sum(g[0] * g[1] * g[2] for g in grids)
        top = grids[-1][0] * grids[-1][1] * grids[-1][2]
        # room for one timepoint in full and the other's top level
        vol = _Volume(dims, channels=C, timepoints=2, dtype=sg.SG_U16, brick=B, levels=L,
                      cache_slots=C * (nodes + top), layout=sg.SG_LAYOUT_MICROBLOCK)
        store = container.HostBrickStore(vol.h, dims, B, L, 2, chunk_bytes=64 << 20)
        for t in range(2):
            for c in range(C):
                store.add(t, c, _cells(dims, c, 2 * seed + t))
        for c in range(C):
            sg.sg_set_transfer_function(vol.h, c, _tint(TINTS[c]), 0.0, 50000.0)
        views = _views(dims, 2, case["width"], case["height"], 40.0, 1.25, seed)
        return {"kind": kind, "vol": vol, "store": store, "views": views,
                "rgba": [_images(views)[0] for _ in range(2)]}
    view = _views((1024, 1024, 1024), 1, case["width"], case["height"], 50.0, 1.25, seed)[0]
    return {"kind": kind, "view": view, "boxes": _parts(case),
            "parts": list(_smooth_images(case["parts"], case["height"], case["width"], 4, seed)),
            "out": torch.empty(case["height"], case["width"], 4, device=DEV)}


def _open_table(case):
    return (_ramp(), (0.0, 255.0)) if case["u8"] else (_tint(TINTS[0]), (0.0, 50000.0))


OPEN_PARAMS = {"step": 0.5, "ert": 0.99, "tau": 1.0, "lod": 1}
PLAY_PARAMS = {"step": 0.5, "ert": 0.99, "tau": 1.0, "lod": 1}


def run(s):
    kind = s["kind"]
    if kind == "frame":
        sg.sg_render_views(s["vol"].h, s["views"], s["params"], s["rgba"], s["depth"])
        return [s["rgba"], s["depth"]]
    if kind == "upframe":
        return [s["path"].render_device(s["views"], s["flag"]), s["flag"]]
    if kind == "network":
        s["model"].m.forward(s["rgba"], s["depth"], 300.0, s["out"], s["err"])
        return [s["out"], s["err"]]
    if kind == "train":
        s["model"].m.train_step(s["rgba"], s["depth"], 300.0, s["target"], 1e-3)
        return s["model"].m.get_weights()
    if kind == "open":
        h = s["vol"].h
        sg.sg_upload_bricks(h, 0, 0, 0, s["coords"], s["cores"])
        sg.sg_build_lod(h, 0, 0)
        sg.sg_volume_commit(h)
        sg.sg_render_views(h, s["views"], OPEN_PARAMS, s["rgba"])
        return s["rgba"]
    if kind == "import":
        levels = container.build_levels(s["data"], s["levels"])
        out = levels[1:] + [container.brick_regions(a, s["brick"], c)
                            for a, c in zip(levels, s["coords"])]
        return [a if a.dtype == torch.uint8 else a.view(torch.int16) for a in out]
    if kind == "play":
        for t in range(2):
            s["store"].put_top(t)
            p = dict(PLAY_PARAMS, timepoint=t)
            sg.sg_render_views(s["vol"].h, s["views"], p, s["rgba"][t])
            while s["store"].serve_requests():
                sg.sg_render_views(s["vol"].h, s["views"], p, s["rgba"][t])
        return s["rgba"]
    sg.sg_composite_over(s["view"], s["parts"], s["boxes"], s["out"])
    return s["out"]


# -------------------------------------------------------------------- work
def _chord(views, dims, per=24):
    """Mean path length through the volume box over all pixels (voxels)."""
    total = []
    for v in views:
        y, x = np.meshgrid((np.arange(per) + 0.5) / per, (np.arange(per) + 0.5) / per, indexing="ij")
        sx = v["tan_left"] + x * (v["tan_right"] - v["tan_left"])
        sy = v["tan_top"] - y * (v["tan_top"] - v["tan_bottom"])
        m = v["cam_to_world"]
        d = np.stack([m[i, 0] * sx + m[i, 1] * sy - m[i, 2] for i in range(3)], -1)
        d /= np.linalg.norm(d, axis=-1, keepdims=True)
        with np.errstate(divide="ignore", invalid="ignore"):
            a = (0.0 - m[:3, 3]) / d
            b = (np.array(dims) - m[:3, 3]) / d
        t0, t1 = np.minimum(a, b).max(-1), np.maximum(a, b).min(-1)
        total.append(np.maximum(t1 - np.maximum(t0, 0), 0).mean() * v["width"] * v["height"])
    return float(sum(total))


def _render_work(views, dims, channels, itemsize, scene, lod, depth=False):
    """Images written once, the voxels of the volume read once (level 0, or
    a quarter of it where level 1 serves most rays), and 31 operations per
    sample and channel; of the tube scene about a quarter of the path lies in
    bricks that are not empty, and the two-voxel pixels of the large scenes
    are sampled every voxel instead of every half."""
    pix = sum(v["width"] * v["height"] for v in views)
    vox = dims[0] * dims[1] * dims[2] * channels * itemsize
    part = 0.25 if scene == "tubes" else 1.0
    samples = _chord(views, dims) * (1.2 if lod else 2.0) * part
    return {"bytes": pix * (20 if depth else 16) + vox * part * (0.3 if lod else 1.0),
            "flops": samples * 31 * channels}


def work(case):
    kind = case["kind"]
    if kind == "frame":
        views = _views(_dims(case), case["views"], case["width"], case["height"], case["fov"],
                       case["distance"], 0)
        w = _render_work(views, _dims(case), case["channels"], 1 if case["scene"] == "blobs" else 2,
                         case["scene"], case["lod"], case["depth"])
        if case["model"] == "mip":
            w["flops"] *= 14 / 31
        if case["roi"]:
            w["flops"] *= 0.65
        return w
    if kind == "batch":
        return _render_work(_batch_views(case, 0), (128, 128, 128), 1, 1, "blobs", False, True)
    if kind == "upframe":
        views = _up_views(case, 0)
        pix = case["width"] * case["height"] * 2
        half = [dict(v, width=v["width"] // 2, height=v["height"] // 2) for v in views]
        cast = _chord(half, (128, 128, 128))  # level 1: one sample per voxel
        # the images written; the network on the twentieth of the pixels
        # that hold anything
        return {"bytes": pix * 16 + pix / 4 * 20 / 20, "flops": cast * 31 + pix / 4 / 20 * 59904}
    if kind == "network":
        p = case["n"] * case["h"] * case["w"]
        return {"bytes": p * 20 + 4 * p * 20, "flops": p * 59904.0}
    if kind == "train":
        p = case["n"] * case["h"] * case["w"]
        return {"bytes": p * 20 + 4 * p * 16 + 16.0 * upsampler.param_count(),
                "flops": p * (2 * 59904.0 + 2 * 9 * 32 * 96)}
    vox = case.get("x", 0) * case.get("y", 0) * case.get("z", 0) * (1 if case.get("u8") else 2)
    if kind == "open":
        views = _views(_dims(case), 1, case["width"], case["height"], 30.0, 1.6, 0)
        pyr = sum(8.0 ** -i for i in range(case["levels"]))
        w = _render_work(views, _dims(case), 1, 1, "cells", True)
        return {"bytes": vox + vox * pyr * ((case["brick"] + 2) / case["brick"]) ** 3 +
                case["width"] * case["height"] * 16, "flops": w["flops"]}
    if kind == "import":
        pyr = sum(8.0 ** -i for i in range(case["levels"]))
        return {"bytes": vox + vox * (pyr - 1) + vox * pyr * ((case["brick"] + 2) / case["brick"]) ** 3,
                "flops": vox * 4.0 / 8}
    if kind == "play":
        views = _views(_dims(case), 2, case["width"], case["height"], 40.0, 1.25, 0)
        w = _render_work(views, _dims(case), case["channels"], 2, "cells", True)
        bricks = vox * case["channels"] * 1.14 * ((case["brick"] + 2) / case["brick"]) ** 3
        return {"bytes": 2 * (2 * bricks + w["bytes"]), "flops": 2 * w["flops"]}
    return {"bytes": case["width"] * case["height"] * 16.0 * (case["parts"] + 1),
            "flops": case["width"] * case["height"] * 9.0 * case["parts"]}


# --------------------------------------------------------------- tolerance
def tolerance(case):
    """About four times what float64 and the library differ by; the library
    and another correct implementation of its precision differ by no more."""
    kind = case["kind"]
    if kind == "import":
        return "exact"
    if kind in ("frame", "batch", "open", "play"):
        # 32-bit sums along each ray (1e-7 to 1e-6); a ray whose opacity
        # lies at the termination threshold may stop one sample apart, which
        # takes an image to 2e-5 (1 in 100 of its value at that pixel)
        return {"rel": 8e-5, "max": 4e-2}
    if kind == "composite":
        return {"rel": 1e-6, "max": 1e-5}
    if kind == "train":
        # bfloat16 activations; Adam's first step moves a weight by the sign
        # of its gradient, so noise in the smallest gradients shows
        return {"rel": 5e-3, "max": 0.1}
    # bfloat16 activations; the predicted error is a squared value
    return {"rel": 4e-3, "max": 0.2}


# ------------------------------------------------------------------- exact
def _pyramid(vol, levels):
    """Levels of a volume as int32 [z, y, x]: (sum of 2x2x2 children, indices
    clamped, + 4) >> 3."""
    out = [vol.to(torch.int32)]
    for _ in range(1, levels):
        a = out[-1]
        for ax in range(3):
            n = a.shape[ax]
            i = torch.arange((n + 1) // 2, device=a.device)
            lo = a.index_select(ax, 2 * i)
            hi = a.index_select(ax, (2 * i + 1).clamp(max=n - 1))
            a = lo + hi
        out.append((a + 4) >> 3)
    return out


def _box(e, d, lo, hi):
    """Entry and exit of e + t d against [lo, hi] (per-axis lists of tensors)."""
    t0 = t1 = None
    for i in range(3):
        par = d[i] == 0
        a, b = (lo[i] - e[i]) / d[i], (hi[i] - e[i]) / d[i]
        mn, mx = torch.minimum(a, b), torch.maximum(a, b)
        inside = (lo[i] <= e[i]) & (e[i] <= hi[i])
        inf = torch.full_like(mn, math.inf)
        mn = torch.where(par, torch.where(inside, -inf, inf), mn)
        mx = torch.where(par, torch.where(inside, inf, -inf), mx)
        t0 = mn if t0 is None else torch.maximum(t0, mn)
        t1 = mx if t1 is None else torch.minimum(t1, mx)
    return t0, t1


def _rays(v):
    f8 = dict(device=DEV, dtype=torch.float64)
    W, H = v["width"], v["height"]
    y, x = torch.meshgrid(torch.arange(H, **f8), torch.arange(W, **f8), indexing="ij")
    sx = (v["tan_left"] + (x + 0.5) / W * (v["tan_right"] - v["tan_left"])).reshape(-1)
    sy = (v["tan_top"] - (y + 0.5) / H * (v["tan_top"] - v["tan_bottom"])).reshape(-1)
    if v.get("lens"):
        k1, k2, cx, cy = v["lens"]
        dx, dy = sx - cx, sy - cy
        r2 = dx * dx + dy * dy
        f = 1.0 + r2 * (k1 + r2 * k2)
        sx, sy = cx + dx * f, cy + dy * f
    m = v["cam_to_world"]
    w = [m[i, 0] * sx + m[i, 1] * sy - m[i, 2] for i in range(3)]
    n = torch.sqrt(w[0] * w[0] + w[1] * w[1] + w[2] * w[2])
    return [float(m[i, 3]) for i in range(3)], [c / n for c in w]


def _cast64(pyr, dims, brick, tables, domain, view, params, bias=0):
    """One view ray cast in float64. pyr: per channel the list of levels."""
    f8 = dict(device=DEV, dtype=torch.float64)
    e, d = _rays(view)
    n_rays, C, B, top = d[0].numel(), len(pyr), brick, len(pyr[0]) - 1
    model, lod = params.get("model", "ea"), params.get("lod", 1)
    ert, step, da = params.get("ert", 0.99), params.get("step", 0.5), params.get("depth_alpha", 0.5)
    grid = [-(-n // B) for n in dims]
    # the level of every level-0 cell: the coarsest ancestor that suits
    cz, cy, cx = torch.meshgrid(*[torch.arange(g, device=DEV) for g in grid[::-1]], indexing="ij")
    cell = [cx.reshape(-1), cy.reshape(-1), cz.reshape(-1)]
    lvl = torch.full_like(cell[0], bias)
    if lod:
        K = (params.get("tau", 1.0) * (view["tan_top"] - view["tan_bottom"]) / view["height"]) ** 2
        done = torch.zeros_like(lvl, dtype=torch.bool)
        for L in range(top, bias, -1):
            d2 = 0.0
            for i in range(3):
                w = B << L
                lo = (cell[i] >> L) * w
                hi = (lo + w).clamp(max=dims[i])
                g = torch.maximum(lo.double() - e[i], e[i] - hi.double()).clamp(min=0)
                d2 = d2 + g * g
            suits = (float(4 ** L) <= K * d2) & ~done
            lvl[suits] = L
            done |= suits
    # every level of every channel in one flat array
    off, flat = [], []
    for L in range(top + 1):
        off.append([0] * C)
        for c in range(C):
            off[L][c] = sum(a.numel() for a in flat)
            flat.append(pyr[c][L].reshape(-1))
    flat = torch.cat(flat)
    off_t = torch.tensor(off, device=DEV)
    ldim = torch.tensor([[a.shape[2], a.shape[1], a.shape[0]] for a in pyr[0]], device=DEV)
    tab = [torch.tensor(np.asarray(t, dtype=np.float32).astype(np.float64), **f8) for t in tables]

    def lookup(c, val):
        u = ((val - domain[0]) / (domain[1] - domain[0]) * (len(tab[c]) - 1)) \
            .clamp(0, len(tab[c]) - 1)
        k = u.floor().long().clamp(max=len(tab[c]) - 2)
        w = (u - k)[:, None]
        return tab[c][k] * (1 - w) + tab[c][k + 1] * w

    zero = torch.zeros(n_rays, **f8)
    tn, tf = _box(e, d, [zero] * 3, [zero + float(x) for x in dims])
    tn = tn.clamp(min=0)
    if params.get("roi") is not None:
        r = np.asarray(params["roi"], dtype=np.float64).reshape(6)
        a, b = _box(e, d, [zero + float(x) for x in r[:3]], [zero + float(x) for x in r[3:]])
        tn, tf = torch.maximum(tn, a), torch.minimum(tf, b)
    ids = torch.nonzero(tn < tf)[:, 0]
    out = torch.zeros(n_rays, 4, **f8)
    out_depth = torch.full((n_rays,), math.inf, **f8)
    d, tn, tf = [x[ids] for x in d], tn[ids], tf[ids]
    S = {"id": ids, "tn": tn, "tf": tf, "T": torch.ones_like(tn),
         "C": torch.zeros(len(ids), 3, **f8), "dep": torch.full_like(tn, math.inf),
         "vm": torch.full((len(ids), C), -math.inf, **f8),
         "k": torch.zeros_like(ids), "n": torch.full_like(ids, -1),
         "t0": tn.clone(), "len": torch.zeros_like(tn), "L": torch.zeros_like(ids)}
    for i in range(3):
        S["d%d" % i] = d[i]
        S["c%d" % i] = ((e[i] + tn * d[i]) / B).floor().long().clamp(0, grid[i] - 1)
        S["b%d" % i] = torch.zeros_like(ids)

    def enter(j):
        """Set up the segment of the node at the rays j's cell."""
        c = [S["c%d" % i][j] for i in range(3)]
        L = lvl[(c[2] * grid[1] + c[1]) * grid[0] + c[0]]
        lo, hi, dj = [], [], [S["d%d" % i][j] for i in range(3)]
        for i in range(3):
            b = c[i] >> L
            S["b%d" % i][j] = b
            w = B * (1 << L)
            lo.append((b * w).double())
            hi.append(((b + 1) * w).clamp(max=dims[i]).double())
        t0, t1 = _box(e, dj, lo, hi)
        t0, t1 = torch.maximum(t0, S["tn"][j]), torch.minimum(t1, S["tf"][j])
        ln = (t1 - t0).clamp(min=0)
        S["L"][j], S["t0"][j], S["len"][j] = L, t0, ln
        S["n"][j] = torch.ceil(ln / (step * (1 << L).double())).long()
        S["k"][j] = 0

    def finish(j):
        if model == "mip":
            col = torch.zeros(len(j), 3, **f8)
            for c in range(C):
                vm = S["vm"][j, c]
                ok = torch.isfinite(vm)
                col += torch.where(ok[:, None], lookup(c, torch.where(ok, vm, 0))[:, :3], 0)
            S["C"][j] = col
        out[S["id"][j], :3] = S["C"][j]
        out[S["id"][j], 3] = 1 - S["T"][j]
        out_depth[S["id"][j]] = S["dep"][j]

    dead = torch.zeros(len(ids), dtype=torch.bool, device=DEV)
    if len(ids):
        enter(torch.arange(len(ids), device=DEV))
    it = 0
    while len(S["id"]):
        it += 1
        # rays at the end of their segment walk one cell on
        j = torch.nonzero(~dead & (S["k"] >= S["n"]))[:, 0]
        if len(j):
            tx = []
            for i in range(3):
                di, ci = S["d%d" % i][j], S["c%d" % i][j]
                tx.append(torch.where(di == 0, math.inf,
                                      (B * (ci + (di > 0)).double() - e[i]) / di))
            tmin, ax = torch.stack(tx).min(0)
            gone = ~(tmin < S["tf"][j])
            same = torch.ones_like(gone)
            for i in range(3):
                m = ax == i
                ci = S["c%d" % i][j] + torch.where(m, torch.sign(S["d%d" % i][j]).long(), 0)
                gone |= (ci < 0) | (ci >= grid[i])
                S["c%d" % i][j] = ci.clamp(0, grid[i] - 1)
                same &= (ci >> S["L"][j]) == S["b%d" % i][j]
            dead[j[gone]] = True
            enter(j[~gone & ~same])
        j = torch.nonzero(~dead & (S["k"] < S["n"]))[:, 0]
        if len(j):
            L, k = S["L"][j], S["k"][j]
            sc = (1 << L).double()
            D, ln = step * sc, S["len"][j]
            s = torch.minimum(D, ln - k.double() * D)
            tau = k.double() * D + 0.5 * s
            t = S["t0"][j] + tau
            i0, i1, fr = [], [], []
            for i in range(3):
                nl = ldim[L, i]
                q = (e[i] + t * S["d%d" % i][j]) / sc - 0.5
                fl = q.floor()
                fr.append(q - fl)
                fl = fl.long()
                i0.append(torch.minimum(fl.clamp(min=0), nl - 1))
                i1.append(torch.minimum((fl + 1).clamp(min=0), nl - 1))
            nx, ny = ldim[L, 0], ldim[L, 1]
            rho, col = 0.0, 0.0
            for c in range(C):
                o = off_t[L, c]

                def at(x, y, z):
                    return flat[o + (z * ny + y) * nx + x].double()

                r = []
                for z in (i0[2], i1[2]):
                    a = at(i0[0], i0[1], z) * (1 - fr[0]) + at(i1[0], i0[1], z) * fr[0]
                    b = at(i0[0], i1[1], z) * (1 - fr[0]) + at(i1[0], i1[1], z) * fr[0]
                    r.append(a * (1 - fr[1]) + b * fr[1])
                val = r[0] * (1 - fr[2]) + r[1] * fr[2]
                if model == "mip":
                    S["vm"][j, c] = torch.maximum(S["vm"][j, c], val)
                    continue
                q = lookup(c, val)
                rho = rho + q[:, 3]
                col = col + (q[:, :3] if model == "eo" or C == 1 else q[:, 3:] * q[:, :3])
            if model == "eo":
                S["C"][j] += col * s[:, None]
            elif model == "ea":
                if C > 1:
                    col = torch.where(rho[:, None] > 0, col / rho.clamp(min=1e-300)[:, None], 0)
                T = S["T"][j]
                Tn = T * torch.exp(-rho * s)
                S["C"][j] += (T - Tn)[:, None] * col
                S["T"][j] = Tn
                A = 1 - Tn
                dep = S["dep"][j]
                S["dep"][j] = torch.where((A >= da) & torch.isinf(dep), t, dep)
                dead[j[A >= ert]] = True
            S["k"][j] = k + 1
        if it % 32 == 0:  # rays that are done leave the working set
            finish(torch.nonzero(dead)[:, 0])
            live = torch.nonzero(~dead)[:, 0]
            S = {a: b[live] for a, b in S.items()}
            dead = torch.zeros(len(live), dtype=torch.bool, device=DEV)
    H, W = view["height"], view["width"]
    return out.reshape(H, W, 4), out_depth.reshape(H, W)


def _conv64(x, w, b):
    n, h, wd, ci = x.shape
    p = torch.zeros(n, h + 2, wd + 2, ci, device=x.device, dtype=x.dtype)
    p = torch.nn.functional.pad(x, (0, 0, 1, 1, 1, 1))
    y = b.expand(n, h, wd, w.shape[2])
    for t in range(9):
        dy, dx = t // 3, t % 3
        y = y + (p[:, dy:dy + h, dx:dx + wd].reshape(-1, ci) @ w[t]).reshape(n, h, wd, -1)
    return y


def _net64(rgba, depth, scale, params):
    """Full-resolution rgba and error head z, [n, 2h, 2w, 5], in float64."""
    code = torch.where(torch.isfinite(depth), 1.0 / (1.0 + depth / scale), 0.0)
    x = torch.cat([rgba, code[..., None], torch.zeros_like(rgba[..., :3])], -1)
    for i, (w, b) in enumerate(params):
        x = _conv64(x, w, b)
        if i < 3:
            x = torch.relu(x)
    n, h, w = rgba.shape[:3]
    o = x[..., :20].reshape(n, h, w, 2, 2, 5).permute(0, 1, 3, 2, 4, 5).reshape(n, 2 * h, 2 * w, 5)

    def axis(m):
        u = (torch.arange(2 * m, device=DEV, dtype=torch.float64) + 0.5) / 2 - 0.5
        i = u.floor().long()
        return i.clamp(0, m - 1), (i + 1).clamp(0, m - 1), u - i

    y0, y1, fy = axis(h)
    x0, x1, fx = axis(w)
    fy, fx = fy[:, None, None], fx[:, None]
    a = rgba[:, y0] * (1 - fy) + rgba[:, y1] * fy
    base = a[:, :, x0] * (1 - fx) + a[:, :, x1] * fx
    return torch.cat([base + o[..., :4], o[..., 4:]], -1)


def _params64(seed, grad=False):
    out = []
    for w, b in upsampler.unpack(_weights(seed)):
        out.append(tuple(torch.tensor(np.asarray(q, dtype=np.float64), device=DEV,
                                      requires_grad=grad) for q in (w, b)))
    return out


def _empty(rgba, depth):
    """Pixels whose 9 x 9 neighbourhood holds nothing."""
    m = ((rgba != 0).any(-1) | torch.isfinite(depth)).float()[:, None]
    return torch.nn.functional.max_pool2d(m, 9, 1, 4)[:, 0] == 0


def exact(case, seed):
    kind = case["kind"]
    if kind == "frame":
        vols, tables, domain = _scene(case["scene"], _dims(case), case["channels"], seed)
        pyr = [_pyramid(v, case["levels"]) for v in vols]
        views = _views(_dims(case), case["views"], case["width"], case["height"], case["fov"],
                       case["distance"], seed, case["lens"])
        res = [_cast64(pyr, _dims(case), case["brick"], tables, domain, v, _params(case))
               for v in views]
        return [[r[0] for r in res], [r[1] for r in res] if case["depth"] else None]
    if kind == "batch":
        pyr = [_pyramid(_blobs((128, 128, 128), seed), 1)]
        res = [_cast64(pyr, (128, 128, 128), 128, [_ramp()], (0.0, 255.0), v, {"lod": 0})
               for v in _batch_views(case, seed)]
        return [[r[0] for r in res], [r[1] for r in res]]
    if kind == "upframe":
        pyr = [_pyramid(_blobs((128, 128, 128), seed), 2)]
        lo = [_cast64(pyr, (128, 128, 128), 64, [_ramp()], (0.0, 255.0),
                      dict(v, width=v["width"] // 2, height=v["height"] // 2), {"lod": 0}, bias=1)
              for v in _up_views(case, seed)]
        rgba, depth = torch.stack([a for a, _ in lo]), torch.stack([b for _, b in lo])
        o = _net64(rgba, depth, UP_DEPTH, _params64(seed))[..., :4]
        hole = _empty(rgba, depth).repeat_interleave(2, 1).repeat_interleave(2, 2)
        o[hole] = 0.0
        return [o, None]
    if kind in ("network", "train"):
        n, h, w = case["n"], case["h"], case["w"]
        s = prepare_inputs(case, seed)
        if kind == "network":
            o = _net64(s["rgba"], s["depth"], 300.0, _params64(seed))
            return [o[..., :4], o[..., 4] ** 2]
        p = _params64(seed, grad=True)
        o = _net64(s["rgba"], s["depth"], 300.0, p)
        diff = o[..., :4] - s["target"]
        err = torch.sqrt((diff[..., :3] ** 2).sum(-1) / 3.0).detach()
        loss = (diff ** 2).mean() + ((o[..., 4] - err) ** 2).mean()
        loss.backward()
        out = []
        for pair in p:
            for q in pair:
                g = q.grad
                # Adam's first step, bias-corrected
                out.append((q.detach() - 1e-3 * g / (g.abs() + 1e-8)).reshape(-1))
        return torch.cat(out)
    if kind == "open":
        dims = _dims(case)
        data = _blobs(dims, seed) if case["u8"] else _cells(dims, 0, seed)
        table, domain = _open_table(case)
        views = _views(dims, 1, case["width"], case["height"], 30.0, 1.6, seed)
        return [_cast64([_pyramid(data, case["levels"])], dims, case["brick"], [table], domain, v,
                        OPEN_PARAMS)[0] for v in views]
    if kind == "play":
        dims = _dims(case)
        views = _views(dims, 2, case["width"], case["height"], 40.0, 1.25, seed)
        out = []
        for t in range(2):
            pyr = [_pyramid(_cells(dims, c, 2 * seed + t), case["levels"])
                   for c in range(case["channels"])]
            out.append([_cast64(pyr, dims, case["brick"],
                                [_tint(x) for x in TINTS[:case["channels"]]], (0.0, 50000.0), v,
                                PLAY_PARAMS)[0] for v in views])
        return out
    if kind == "composite":
        view = _views((1024, 1024, 1024), 1, case["width"], case["height"], 50.0, 1.25, seed)[0]
        parts = _smooth_images(case["parts"], case["height"], case["width"], 4, seed).double()
        e, d = _rays(view)
        zero = torch.zeros_like(d[0])
        ts = []
        for b in _parts(case):
            t0, t1 = _box(e, d, [zero + float(x) for x in b[:3]], [zero + float(x) for x in b[3:]])
            ts.append(torch.where(t0 < t1, t0, math.inf))
        t, order = torch.stack(ts).sort(dim=0, stable=True)
        flat = parts.reshape(len(parts), -1, 4)
        at = torch.arange(flat.shape[1], device=DEV)
        col, T = torch.zeros_like(flat[0]), torch.ones_like(t[0])
        for k in range(len(parts)):
            p = torch.where(torch.isfinite(t[k])[:, None], flat[order[k], at], 0.0)
            col = col + T[:, None] * p
            T = T * (1 - p[:, 3])
        return col.reshape(case["height"], case["width"], 4)
    return None  # whole numbers: compared as they are


def prepare_inputs(case, seed):
    """The network cases' inputs in float64."""
    s = prepare(case, seed)
    return {k: v.double() for k, v in s.items() if isinstance(v, torch.Tensor)}
