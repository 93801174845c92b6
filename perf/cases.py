"""Performance cases of the hybrid depth-of-field library.

Each case is one call (or one short sequence of calls) that a program makes
through the public entry points of ``paper_2210_04981_amd.hdof``, on seeded
synthetic inputs: the procedural indoor scenes the library is tested on
(a close cushion partly covering a far one, spheres and boxes in a room) and,
for the stages that take images, images of the same make-up.

kinds: frame    one hdof_frame without history
       path     the next hdof_frame of a camera path, with every history
       batch    one replay of a captured batch of uneven views
       rebuild  hdof_build_bvh of new geometry and the G-buffer of it
       filter   hdof_postfilter of an image and its depth
       train    HybridDoFPost forward and backward (colour, focus, aperture)
       trace    hdof_trace_thin_lens of every pixel (the reference image)
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2210_04981_amd import hdof

TAN_HALF_FOV = 0.36
FOCAL = 0.05
VIEW_SIZES = ((640, 360), (1280, 720), (1920, 1080), (2560, 1440))


def listed():
    room = dict(objects=20, spp=8, fnum=1.4, focus=2.0, tile=8, blades=0, sa=0.0, glossy=False)
    return [
        # the smallest useful frame: a thumbnail or preview of a few hundred triangles, bound by latency
        dict(room, name="frame_64", kind="frame", w=64, h=64, objects=0, spp=4, fnum=2.0),
        # a real-time frame at the usual size: the library's headline workload
        dict(room, name="frame_1080p", kind="frame", w=1920, h=1080),
        # an odd-sized window with a shaped, aberrated lens and the mask resolution scaled by the blur
        dict(room, name="frame_hexagon_odd", kind="frame", w=1363, h=765, tile=0, blades=6, sa=0.6),
        # a glossy scene with the specular bokeh rule at the largest size of the batch's views
        dict(room, name="frame_glossy_1440p", kind="frame", w=2560, h=1440, glossy=True),
        # walking through a large scene: variance, temporal and spatial histories carried along
        dict(room, name="path_1m_tris", kind="path", w=1920, h=1080, objects=100, spp=16, focus=1.5),
        # offline serving: many views of one scene, uneven in size and lens, as one captured graph
        dict(room, name="batch_16", kind="batch", views=16),
        # geometry that changes from frame to frame: the acceleration structure anew, then what is seen
        dict(room, name="rebuild_200k", kind="rebuild", w=1280, h=720),
        # the post-filter alone on an application's own image, with fine CoC tiles
        dict(name="filter_tile8_720p", kind="filter", w=1280, h=720, taps=48, pp_tile=8, r_cap=64.0, fnum=1.4, focus=2.0),
        # the post-filter alone at its defaults, on an odd-sized window
        dict(name="filter_odd", kind="filter", w=853, h=479, taps=48, pp_tile=16, r_cap=64.0, fnum=1.4, focus=2.0),
        # one step of fitting focus and aperture (and the image) to a target, at full and at preview size
        dict(name="train_1080p", kind="train", w=1920, h=1080, taps=48, pp_tile=16, r_cap=64.0, fnum=1.4, focus=2.0),
        dict(name="train_preview", kind="train", w=333, h=187, taps=48, pp_tile=16, r_cap=64.0, fnum=2.0, focus=2.5),
        # the full ray-traced reference image that hybrid frames are judged by
        dict(room, name="trace_reference", kind="trace", w=960, h=540, spp=16),
    ]


def draw(rng):
    kind = rng.choice(("frame", "frame", "frame", "path", "batch", "rebuild", "filter", "filter", "train", "train", "trace"))

    def size(lo, hi):
        w = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
        return dict(w=w, h=max(16, int(w / rng.choice((16 / 9, 4 / 3, 1.85, 1.0)))))

    lens = dict(fnum=rng.choice((1.4, 2.0, 2.8)), focus=round(rng.uniform(0.9, 4.0), 3))
    post = dict(taps=rng.choice((24, 48, 48, 61, 96)), pp_tile=rng.choice((4, 8, 16, 16)), r_cap=rng.choice((24.0, 48.0, 64.0)))
    room = dict(lens, objects=rng.randint(6, 60), spp=rng.choice((4, 8, 8, 16)), tile=8, blades=0, sa=0.0, glossy=False)
    if kind == "frame":
        shape = rng.choice((dict(), dict(), dict(blades=rng.randint(5, 9), sa=round(rng.uniform(-0.5, 0.8), 2)), dict(glossy=True)))
        return dict(room, kind=kind, tile=rng.choice((0, 4, 8, 8, 16)), **size(64, 2560)) | shape
    if kind == "path":
        return dict(room, kind=kind, **size(320, 1920))
    if kind == "batch":
        return dict(room, kind=kind, views=rng.randint(2, 12))
    if kind == "rebuild":
        return dict(room, kind=kind, **size(160, 1280))
    if kind == "filter":
        return dict(lens, kind=kind, **post, **size(64, 2560))
    if kind == "train":
        return dict(lens, kind=kind, **dict(post, taps=min(post["taps"], 61)), **size(64, 1920))
    return dict(room, kind=kind, **size(64, 960))


# ----------------------------------------------------------------------------
# scenes
# ----------------------------------------------------------------------------

def _t(x):
    return torch.as_tensor(np.asarray(x, np.float32), device="cuda")


def _room(lo, hi):
    x0, y0, z0 = lo
    x1, y1, z1 = hi
    p = np.array([(x0, y0, z0), (x1, y0, z0), (x1, y1, z0), (x0, y1, z0),
                  (x0, y0, z1), (x1, y0, z1), (x1, y1, z1), (x0, y1, z1)])
    quads = [(0, 1, 2, 3), (5, 4, 7, 6), (4, 0, 3, 7), (1, 5, 6, 2), (4, 5, 1, 0), (3, 2, 6, 7)]
    return _t(np.stack([p[list(t)].reshape(9) for a, b, c, d in quads for t in ((a, b, c), (a, c, d))]))


def _grid_triangles(g):
    """(objects, patches, m, n, 3) grids of points as triangles (objects, t, 9)."""
    a, b, c, d = g[:, :, :-1, :-1], g[:, :, 1:, :-1], g[:, :, 1:, 1:], g[:, :, :-1, 1:]
    return torch.stack([torch.cat([a, b, c], -1), torch.cat([a, c, d], -1)], 4).reshape(g.shape[0], -1, 9)


def _boxes(cen, half, n=29):
    t = torch.linspace(-1, 1, n + 1, device="cuda")
    u, v = torch.meshgrid(t, t, indexing="ij")
    one = torch.ones_like(u)
    faces = [torch.stack([(s * one, u, v)[(k - a) % 3] for k in range(3)], -1) for a in range(3) for s in (-1.0, 1.0)]
    return _grid_triangles(cen[:, None, None, None] + half[:, None, None, None, None] * torch.stack(faces)[None])


def _spheres(cen, radius, stacks=70, slices=72):
    th = torch.linspace(0, math.pi, stacks + 1, device="cuda")[:, None]
    ph = torch.linspace(0, 2 * math.pi, slices + 1, device="cuda")[None]
    unit = torch.stack([th.sin() * ph.cos(), th.cos() + 0 * ph, th.sin() * ph.sin()], -1)
    tri = _grid_triangles(cen[:, None, None, None] + radius[:, None, None, None, None] * unit[None, None])
    keep = torch.ones(stacks, slices, 2, dtype=torch.bool, device="cuda")
    keep[-1, :, 0] = keep[0, :, 1] = False  # the triangles of no area at the poles
    return tri[:, keep.reshape(-1)]


def _scene(case, seed):
    """Triangles (n, 9), albedo (n, 3) and specular table (n, 2) of a room."""
    rng = np.random.default_rng(seed)
    if case["objects"] == 0:
        xy, z = rng.uniform(-1, 1, (256, 3, 2)), rng.uniform(1, 4, (256, 3, 1))
        parts = [_room((-2, -2, -1), (2, 2, 6)), _t(np.concatenate([xy, z], -1).reshape(256, 9))]
        albedo = [_t([0.8, 0.75, 0.7]).expand(12, 3), _t(rng.uniform(0, 1, (256, 3)))]
        spec = [_t([0.0, 1.0]).expand(12, 2), _t([0.5, 24.0]).expand(256, 2)]
    else:
        n = case["objects"]
        far = 8.0 if n > 60 else 6.0
        size = rng.uniform(0.15, 0.5, n)
        z = rng.uniform(np.maximum(1.2, size + 0.8), far)
        pos = np.stack([rng.uniform(-0.9, 0.9, n) * TAN_HALF_FOV * z, rng.uniform(-0.9, 0.9, n) * TAN_HALF_FOV * z * 9 / 16, z], -1)
        pos[0], size[0] = (0.072, -0.036, 0.6), 0.1  # the cushions
        pos[1], size[1] = (0.125, 0.05, 2.5), 0.3
        pos, size = _t(pos), _t(size)
        n_box = (n + 1) // 2
        box, ball = _boxes(pos[:n_box], size[:n_box]), _spheres(pos[n_box:], size[n_box:])
        parts = [_room((-3.0, -1.2, -0.5), (3.0, 1.8, far + 1.0)), box.reshape(-1, 9), ball.reshape(-1, 9)]
        alb = _t(rng.uniform(0, 1, (n, 3)))
        gloss = _t(np.stack([rng.uniform(0.3, 1, n), np.where(np.arange(n) < n_box, rng.uniform(4, 32, n), rng.uniform(16, 256, n))], -1))
        albedo, spec = [_t([0.8, 0.75, 0.7]).expand(12, 3)], [_t([0.0, 1.0]).expand(12, 2)]
        for a, b, tri in ((0, n_box, box), (n_box, n, ball)):
            albedo.append(alb[a:b, None].expand(-1, tri.shape[1], 3).reshape(-1, 3))
            spec.append(gloss[a:b, None].expand(-1, tri.shape[1], 2).reshape(-1, 2))
    return torch.cat(parts).contiguous(), torch.cat(albedo).contiguous(), torch.cat(spec).contiguous()


def _camera(eye, yaw_deg, w, h):
    a = math.radians(yaw_deg)
    return hdof.camera(eye, (math.cos(a), 0.0, -math.sin(a)), (0.0, 1.0, 0.0), (math.sin(a), 0.0, math.cos(a)), TAN_HALF_FOV, w, h)


def _light(case):
    if case["objects"] == 0:
        return hdof.light((0.0, 1.5, 1.0), (4.0,) * 3, (0.05,) * 3)
    return hdof.light((0.6, 1.5, 0.2), (6.0,) * 3, (0.05,) * 3)


def _lens(case):
    return hdof.lens(FOCAL, FOCAL / case["fnum"], case["focus"], case.get("blades", 0), 0.3 if case.get("blades", 0) else 0.0, case.get("sa", 0.0))


def _params(case, histories=False):
    mask = hdof.mask_params(spp_max=case["spp"], tile=case["tile"])
    comp = hdof.composite_params(spec_y=0.3 if case["glossy"] else 0.0)
    on = int(histories)
    return hdof.FrameParams(mask, hdof.pp_params(), comp, hdof.ReconParams(on, 0.2), hdof.SpatialParams(on, 24, 64.0, 0.01))


def _built(case, seed):
    verts, albedo, spec = _scene(case, seed)
    ctx = hdof.Context(0)
    scene = hdof.hdof_build_bvh(ctx, verts, albedo)
    if case["glossy"]:
        hdof.hdof_scene_set_specular(scene, spec)
    return ctx, scene


# ----------------------------------------------------------------------------
# images (the stages that take one): a slanted wall, fronto-parallel discs at
# many depths, smooth and sharp texture, ray counts along the depth edges
# ----------------------------------------------------------------------------

def _image(case, seed):
    H, W = case["h"], case["w"]
    g = torch.Generator(device="cuda").manual_seed(seed)
    rng = np.random.default_rng(seed)
    y, x = torch.meshgrid((torch.arange(H, device="cuda") + 0.5) / H, (torch.arange(W, device="cuda") + 0.5) / H, indexing="ij")
    depth = 4.0 + 2.0 * x * H / W + 0.5 * y
    color = torch.stack([0.4 + 0.3 * torch.sin(rng.uniform(5, 40) * x + rng.uniform(5, 40) * y + c) for c in range(3)])
    n = 14
    for z, r, cx, cy in sorted(zip(rng.uniform(0.6, 4.0, n), rng.uniform(0.08, 0.35, n), rng.uniform(0, W / H, n), rng.uniform(0, 1, n)), reverse=True):
        on = (x - cx) ** 2 + (y - cy) ** 2 < r * r
        depth = torch.where(on, z + 0.1 * (x - cx), depth)
        color = torch.where(on, _t(rng.uniform(0.1, 1.2, 3))[:, None, None] * (0.75 + 0.25 * torch.sin(60 * (x + y)))[None], color)
    color = color * (0.8 + 0.4 * torch.rand(3, H, W, device="cuda", generator=g))
    d = depth.float()
    edge = torch.zeros(H, W, device="cuda")
    edge[:, 1:] = (d[:, 1:] - d[:, :-1]).abs()
    edge[1:] = torch.maximum(edge[1:], (d[1:] - d[:-1]).abs())
    near = torch.nn.functional.max_pool2d((edge > 0.05)[None, None].float(), 25, 1, 12)[0, 0]
    spp = (near * (2 + torch.randint(0, 7, (H, W), device="cuda", generator=g))).to(torch.uint8)
    on = (spp > 0).float()
    rt = dict(c_near=torch.rand(3, H, W, device="cuda", generator=g) * on, c_far=torch.rand(3, H, W, device="cuda", generator=g) * on,
              hit_ratio=torch.rand(H, W, device="cuda", generator=g) * on, lum_m1=on * 0.5, lum_m2=on * 0.3)
    grad = (color.roll(3, 2) - color + 0.05 * torch.randn(3, H, W, device="cuda", generator=g)).float()
    return dict(color=color.float().contiguous(), depth=d.contiguous(), spp=spp, rt=rt, grad=grad.contiguous())


# ----------------------------------------------------------------------------
# what a program has in hand, and one pass
# ----------------------------------------------------------------------------

def prepare(case, seed):
    kind = case["kind"]
    if kind in ("filter", "train"):
        s = dict(kind=kind, ctx=hdof.Context(0), cam=_camera((0, 0, 0), 0.0, case["w"], case["h"]), lens=_lens(case),
                 pp=hdof.pp_params(case["taps"], case["pp_tile"], case["r_cap"]), **_image(case, seed))
        if kind == "filter":
            return dict(s, out=torch.empty_like(s["color"]))
        s["color"].requires_grad_()
        s["focus"] = torch.tensor(case["focus"], device="cuda", requires_grad=True)
        s["aperture"] = torch.tensor(FOCAL / case["fnum"], device="cuda", requires_grad=True)
        return dict(s, rt=hdof.RTResult(**s["rt"]), comp=hdof.composite_params())
    if kind == "rebuild":
        verts, albedo, _ = _scene(case, seed)
        return dict(kind=kind, ctx=hdof.Context(0), verts=verts, albedo=albedo, cam=_camera((0, 0, 0), 0.0, case["w"], case["h"]),
                    lens=_lens(case), light=_light(case), gb=hdof.GBuffer.empty(case["h"], case["w"]))
    ctx, scene = _built(case, seed)
    s = dict(kind=kind, ctx=ctx, scene=scene, light=_light(case), seed=seed & 0xffff)
    if kind == "batch":
        rng = np.random.default_rng(seed + 1)
        views, outs = [], []
        for v in range(case["views"]):
            w, h = VIEW_SIZES[v % 4]
            cam = _camera((*rng.uniform(-0.2, 0.2, 2), 0.0), rng.uniform(-10, 10), w, h)
            lens = hdof.lens(FOCAL, FOCAL / (1.4, 2.0, 2.8)[v % 3], rng.uniform(0.8, 5.0))
            views.append((cam, lens, s["seed"], 0, v))
            outs.append(torch.empty(3, h, w, device="cuda"))
        return dict(s, batch=hdof.Batch(ctx, scene, s["light"], _params(case), views, outs))
    H, W = case["h"], case["w"]
    s.update(lens=_lens(case), cam=_camera((0, 0, 0), 0.0, W, H))
    if kind == "trace":
        n = H * W
        return dict(s, spp_max=case["spp"], spp=torch.full((H, W), case["spp"], dtype=torch.uint8, device="cuda"),
                    offsets=(torch.arange(n, device="cuda", dtype=torch.int32) * case["spp"]).view(H, W),
                    total=torch.tensor([n * case["spp"]], dtype=torch.int32, device="cuda"), rt=hdof.RTResult.empty(H, W))
    s.update(params=_params(case, kind == "path"), out=torch.empty(3, H, W, device="cuda"), t=0)
    if kind == "path":
        # a dolly of 1 cm and a yaw of 0.2 degrees a frame, forth and back; the histories of its first frames are there
        s["cams"] = [_camera((0.0, 0.0, 0.01 * t), 0.2 * t, W, H) for t in range(16)]
        for _ in range(4):
            run(s)
    return s


def run(s):
    kind = s["kind"]
    if kind == "frame":
        return hdof.hdof_frame(s["ctx"], s["scene"], s["cam"], None, s["lens"], s["light"], s["params"], seed=s["seed"], out=s["out"])
    if kind == "path":
        t, s["t"] = s["t"], s["t"] + 1
        at = lambda i: s["cams"][15 - abs(i % 30 - 15)]  # noqa: E731
        return hdof.hdof_frame(s["ctx"], s["scene"], at(t), at(t - 1) if t else None, s["lens"], s["light"], s["params"], seed=s["seed"],
                               frame=t, out=s["out"])
    if kind == "batch":
        return list(s["batch"].launch())
    if kind == "rebuild":
        scene = hdof.hdof_build_bvh(s["ctx"], s["verts"], s["albedo"])
        gb = hdof.hdof_gbuffer(s["ctx"], scene, s["cam"], s["lens"], s["light"], out=s["gb"])
        scene.close()
        return dict(depth=gb.depth, normal=gb.normal, albedo=gb.albedo, color=gb.color, tri_id=gb.tri_id)
    if kind == "filter":
        return hdof.hdof_postfilter(s["ctx"], s["color"], s["depth"], s["cam"], s["lens"], s["pp"], out=s["out"])
    if kind == "train":
        out = hdof.HybridDoFPost.apply(s["color"], s["focus"], s["aperture"], s["depth"], s["spp"], s["rt"], s["cam"], FOCAL, s["pp"], s["comp"], s["ctx"])
        grads = torch.autograd.grad(out, (s["color"], s["focus"], s["aperture"]), s["grad"])
        return dict(out=out.detach(), color=grads[0], lens=torch.stack(grads[1:]))
    rt = hdof.hdof_trace_thin_lens(s["ctx"], s["scene"], s["cam"], s["lens"], s["light"], s["spp_max"], s["spp"], s["offsets"], s["total"],
                                   seed=s["seed"], out=s["rt"])
    return dict(c_near=rt.c_near, c_far=rt.c_far, hit_ratio=rt.hit_ratio, lum_m1=rt.lum_m1, lum_m2=rt.lum_m2)


# ----------------------------------------------------------------------------
# what a pass cannot do without
# ----------------------------------------------------------------------------

def _triangles(case):
    n = case["objects"]
    return 268 if n == 0 else 12 + (n + 1) // 2 * 12 * 29 * 29 + n // 2 * 2 * 72 * 69


def work(case):
    """Each input read once, each output written once; per gather tap a
    bilinear sample of four channels and its weight (60 operations), per ray
    one path down a binary tree (two boxes of 24 a level) and one triangle."""
    kind = case["kind"]
    if kind == "filter":
        px = case["w"] * case["h"]
        return dict(bytes=28 * px, flops=60 * case["taps"] * px)
    if kind == "train":  # colour, depth, counts, traced planes and gradient in; image and gradient out; the filter and its transpose
        px = case["w"] * case["h"]
        return dict(bytes=(12 + 4 + 1 + 28 + 12 + 12 + 12) * px, flops=3 * 60 * case["taps"] * px)
    tris = _triangles(case)
    ray = 48 * math.log2(tris) + 150
    if kind == "rebuild":  # triangles in, tree and triangles out; Morton codes, eight sorting passes and the clustering
        px = case["w"] * case["h"]
        return dict(bytes=48 * tris + 112 * tris + 8 * 24 * tris + 44 * px, flops=ray * px + 32 * 20 * 2 * tris)
    if kind == "trace":
        px = case["w"] * case["h"]
        return dict(bytes=48 * tris + 41 * px, flops=(ray + 100) * px * case["spp"])
    sizes = [VIEW_SIZES[v % 4] for v in range(case["views"])] if kind == "batch" else [(case["w"], case["h"])]
    px = sum(w * h for w, h in sizes)
    history = 2 * 49 if kind == "path" else 0
    return dict(bytes=48 * tris + (12 + history) * px, flops=(ray + 60 * 48) * px)


# ----------------------------------------------------------------------------
# the post-filter and composite in 64 bits
# ----------------------------------------------------------------------------

def _filter64(case, color, z, S1, A):
    """The gather filter of color (3, H, W) with depth z, focus S1, aperture A."""
    H, W, n, tile, cap = case["h"], case["w"], case["taps"], case["pp_tile"], case["r_cap"]
    c = A * (1 / S1 - 1 / z) * W / (2 * float(np.float32(TAN_HALF_FOV)))
    r = c.abs() / 2
    TH, TW, K = -(-H // tile), -(-W // tile), math.ceil(cap / tile)
    rp = torch.nn.functional.pad(r, (0, TW * tile - W, 0, TH * tile - H))
    rt = rp.view(TH, tile, TW, tile).permute(0, 2, 1, 3).reshape(TH, TW, -1).amax(-1)
    rt = torch.nn.functional.max_pool2d(rt[None, None], 2 * K + 1, 1, K)[0, 0].clamp(max=cap)
    R = rt.repeat_interleave(tile, 0).repeat_interleave(tile, 1)[:H, :W]
    y, x = torch.meshgrid(torch.arange(H, device="cuda"), torch.arange(W, device="cuda"), indexing="ij")
    tex = torch.cat([color, c[None]]).permute(1, 2, 0).reshape(-1, 4)
    w0 = 1 / r.clamp(min=0.5) ** 2
    num, den = w0 * color, w0
    for k in range(1, n + 1):
        u, a = math.sqrt((k - 0.5) / n), k * math.pi * (3 - math.sqrt(5))
        ox, oy = R * (u * math.cos(a)), R * (u * math.sin(a))
        fx, fy = ox.detach().floor(), oy.detach().floor()
        ax, ay, s = ox - fx, oy - fy, 0
        for dx, dy, b in ((0, 0, (1 - ax) * (1 - ay)), (1, 0, ax * (1 - ay)), (0, 1, (1 - ax) * ay), (1, 1, ax * ay)):
            q = (y + fy.long() + dy).clamp(0, H - 1) * W + (x + fx.long() + dx).clamp(0, W - 1)
            s = s + b[..., None] * tex.index_select(0, q.reshape(-1)).view(H, W, 4)
        cq = s[..., 3]
        rq = cq.abs() / 2
        reff = rq - (cq - c).clamp(0, 1) * (rq - r).clamp(min=0)
        w = R * R / n * (reff - R * u + 0.5).clamp(0, 1) / rq.clamp(min=0.5) ** 2
        num, den = num + w * s[..., :3].permute(2, 0, 1), den + w
    return torch.where(R > 0, num / den, color), c


def exact(case, seed):
    """The image stages in 64 bits; nothing for what rays return (their hits
    need the library's scale of scene and search)."""
    if case["kind"] not in ("filter", "train"):
        return None
    im = _image(case, seed)
    S1 = torch.tensor(float(np.float32(case["focus"])), dtype=torch.float64, device="cuda")
    A = torch.tensor(float(np.float32(FOCAL / case["fnum"])), dtype=torch.float64, device="cuda")
    color, z = im["color"].double(), im["depth"].double()
    if case["kind"] == "filter":
        return _filter64(case, color, z, S1, A)[0]
    color.requires_grad_(), S1.requires_grad_(), A.requires_grad_()
    pp, c = _filter64(case, color, z, S1, A)
    h = im["rt"]["hit_ratio"].double()
    crt = h * im["rt"]["c_near"].double() + (1 - h) * im["rt"]["c_far"].double()
    traced = (im["spp"] > 0).double()
    phi = (c.abs() - math.sqrt(2)).clamp(0, 1)
    nu = (0.5 - c / (2 * math.sqrt(2))).clamp(0, 1)
    beta = traced * (1 - h / 0.5).clamp(0, 1)
    off = nu * (traced * crt + (1 - traced) * pp) + (1 - nu) * (beta * crt + (1 - beta) * pp)
    out = (1 - phi) * color + phi * off
    grads = torch.autograd.grad(out, (color, S1, A), im["grad"].double())
    return dict(out=out.detach(), color=grads[0], lens=torch.stack(grads[1:]))
