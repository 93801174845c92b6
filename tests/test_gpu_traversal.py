"""GPU parity of the per-lane traversal's half-precision boxes and ray slots.

The boxes are halves about their node's centre in a power-of-two unit of the
scene, widened outwards, so they are tried where that could lose a hit:
scenes scaled by powers of ten, far from the origin, flat, and of one to a
few triangles; and the slots at queue lengths around a wave's 64 rays and
with rays of one pixel only.  Expected values: the FP64 oracle's closest hit
per ray, ids equal except on the rays it flags (within 1e-5 of an edge)."""
from __future__ import annotations

from dataclasses import replace

import numpy as np
import pytest
import torch

import scenegen as sg

pytestmark = pytest.mark.gpu

import oracle  # noqa: E402
from gpu_common import DEV, excl_cumsum, print_case, to_dev, upload_scene  # noqa: E402


@pytest.fixture(scope="module")
def hd():
    from paper_2210_04981_amd import hdof
    return hdof


@pytest.fixture(scope="module")
def ctx(hd):
    c = hd.hdof_create(0)
    yield c
    c.close()


def check_hits(hd, ctx, scene, cfg, spp, z_rel):
    H, W = spp.shape
    osc = oracle.Scene(scene.verts, scene.albedo)
    ref = oracle.trace(osc, cfg.camera, cfg.lens, cfg.light, spp, seed=5, frame=1, view=2, per_ray=True)
    sc = upload_scene(hd, ctx, scene)
    smax = max(1, int(spp.max()))
    cap = H * W * smax
    rid = torch.full((cap,), -7, dtype=torch.int32, device=DEV)
    rz = torch.zeros(cap, dtype=torch.float32, device=DEV)
    n = int(spp.sum())
    hd.hdof_trace_thin_lens(ctx, sc, hd.camera_of(cfg.camera), hd.lens_of(cfg.lens), hd.light_of(cfg.light), smax,
                            to_dev(spp.astype(np.uint8)), to_dev(excl_cumsum(spp).astype(np.int32)),
                            to_dev(np.array([n], np.int32)), seed=5, frame=1, view=2, ray_tri_id=rid, ray_depth=rz)
    torch.cuda.synchronize()
    ctx.sync()
    g_id, g_z = rid.cpu().numpy(), rz.cpu().numpy()[:n].astype(np.float64)
    assert (g_id[n:] == -7).all()
    bad = (g_id[:n] != ref["ray_id"]) & (ref["ray_amb"] == 0)
    assert not bad.any(), f"{bad.sum()} of {n} unambiguous rays hit other triangles"
    same = (g_id[:n] == ref["ray_id"]) & (g_id[:n] >= 0)
    rel = np.abs(g_z[same] - ref["ray_z"][same]) / np.abs(ref["ray_z"][same])
    assert rel.size == 0 or rel.max() < z_rel, rel.max()
    sc.close()


# fp32 hit distances: 1e-3 relative at worst (grazing hits), as for the
# library's other traversal tests; a scene at distance d from the origin adds
# the rounding of its coordinates, 2^-24 d over the hit's own scale
@pytest.mark.parametrize("scale,shift", [(1.0, 0.0), (1e-3, 0.0), (1e3, 0.0), (1.0, 64.0)])
def test_scaled_and_shifted_scene(hd, ctx, scale, shift):
    print_case(f"half boxes: scale {scale} shift {shift}")
    cfg = sg.config_tiny(aperture_override=0.2)
    scene = sg.tiny_scene(3)
    # the shift keeps every coordinate exact in float32, so both sides trace the same triangles
    verts = (np.round(scene.verts * 4096) / 4096 * scale + shift).astype(np.float32)
    cam = replace(cfg.camera, eye=(np.asarray(cfg.camera.eye) * scale + shift).astype(np.float32))
    lens = replace(cfg.lens, aperture=float(np.float32(cfg.lens.aperture * scale)),
                   focus_distance=float(np.float32(cfg.lens.focus_distance * scale)),
                   focal_length=float(np.float32(cfg.lens.focal_length * scale)))
    spp = np.full((cam.height, cam.width), 2, np.int32)
    check_hits(hd, ctx, sg.Scene(verts, scene.albedo), replace(cfg, camera=cam, lens=lens), spp, 1e-3)


@pytest.mark.parametrize("n", [1, 2, 4, 5, 9])
def test_flat_scene_of_few_triangles(hd, ctx, n):
    """Triangles in one plane facing the camera: node boxes of no extent in z."""
    print_case(f"half boxes: {n} coplanar triangles")
    rng = np.random.default_rng(n)
    v = np.concatenate([rng.uniform(-1, 1, (n, 3, 2)), np.full((n, 3, 1), 2.5)], -1).reshape(n, 9).astype(np.float32)
    cfg = sg.config_tiny(aperture_override=0.2)
    check_hits(hd, ctx, sg.Scene(v, rng.uniform(0, 1, (n, 3)).astype(np.float32)), cfg,
               np.full((64, 64), 1, np.int32), 1e-5)


@pytest.mark.parametrize("total", [1, 7, 63, 64, 65, 129, 511, 4097])
@pytest.mark.parametrize("refill", [1, 47, 64])
def test_queue_lengths(hd, ctx, total, refill):
    """Queues shorter than the segments, around a wave's slots, and of a
    single pixel's rays."""
    print_case(f"ray slots: {total} rays, refill {refill}")
    hd.hdof_set_tuning(ctx, refill=refill)
    cfg = sg.config_tiny(aperture_override=0.2)
    spp = np.zeros((64, 64), np.int32)
    left, p = total, 1000
    while left > 0:
        spp.reshape(-1)[p] = min(255, left)
        left -= min(255, left)
        p += 37
    check_hits(hd, ctx, sg.tiny_scene(1), cfg, spp, 1e-3)
    hd.hdof_set_tuning(ctx)


@pytest.mark.parametrize("n", [300, 20000])
def test_deep_stacks(hd, ctx, n):
    """Large overlapping triangles: nearly every ray reaches both children of
    every node on its way, so the stacks of all lanes grow to the tree's depth
    (about 9 and 17 levels and more), past the rows kept in LDS."""
    print_case(f"deep stacks: {n} overlapping triangles")
    rng = np.random.default_rng(n)
    z = rng.uniform(1, 4, (n, 1, 1))
    v = np.concatenate([rng.uniform(-2.5, 2.5, (n, 3, 2)), z + rng.uniform(-0.3, 0.3, (n, 3, 1))], -1)
    scene = sg.Scene(v.reshape(n, 9).astype(np.float32), rng.uniform(0, 1, (n, 3)).astype(np.float32))
    cfg = sg.config_tiny(aperture_override=0.2)
    cam = replace(cfg.camera, width=16, height=16)
    check_hits(hd, ctx, scene, replace(cfg, camera=cam), np.full((16, 16), 3, np.int32), 1e-3)


@pytest.mark.parametrize("smax,sa", [(1, 0.0), (3, 0.4), (16, 0.0), (255, 0.0)])
def test_reduction_any_entry_order(hd, ctx, smax, sa):
    """The reduction stages a wave's entries together where its pixels' lie
    together, else each lane reads its own: the same sums bit for bit for
    offsets in row-major order, in reverse (each wave's together, descending),
    column by column and in random order (spread over the queue, a lane per
    pixel), the last being the plain sum."""
    print_case(f"reduction smax {smax} sa {sa}")
    cfg = sg.config_tiny(aperture_override=0.2)
    W, H = (147, 131) if smax < 255 else (65, 7)
    cfg = replace(cfg, camera=replace(cfg.camera, width=W, height=H), lens=replace(cfg.lens, sa=sa))
    rng = np.random.default_rng(smax)
    spp = rng.integers(0, smax + 1, H * W)
    spp[rng.uniform(size=H * W) < 0.4] = 0
    sc = upload_scene(hd, ctx, sg.tiny_scene(3))
    orders = [np.arange(H * W), np.arange(H * W)[::-1], np.arange(H * W).reshape(H, W).T.ravel(),
              rng.permutation(H * W)]
    out = []
    for order in orders:
        off = np.zeros(H * W, np.int64)
        off[order] = np.cumsum(spp[order]) - spp[order]
        rt = hd.hdof_trace_thin_lens(ctx, sc, hd.camera_of(cfg.camera), hd.lens_of(cfg.lens), hd.light_of(cfg.light),
                                     smax, to_dev(spp.reshape(H, W).astype(np.uint8)),
                                     to_dev(off.reshape(H, W).astype(np.int32)),
                                     to_dev(np.array([spp.sum()], np.int32)), seed=5)
        torch.cuda.synchronize()
        out.append([t.cpu().numpy() for t in (rt.c_near, rt.c_far, rt.hit_ratio, rt.lum_m1, rt.lum_m2)])
    for o in out[1:]:
        for a, b in zip(out[0], o):
            assert np.array_equal(a, b)
    sc.close()


@pytest.mark.parametrize("eye,yaw,S1", [((0.17, 0.03, -0.1), -3.0, 4.0), ((0.05, 0.1, 0.0), 3.0, 0.7)])
def test_half_boxes_find_the_hits_of_full_boxes(hd, ctx, eye, yaw, S1):
    """33M rays by the per-lane walk (half-precision boxes) and by the
    wave-coherent one (the full boxes): the same triangles and depths.  At the
    very edge of a triangle its leaf's box decides, and the wider half boxes
    must not add hits there."""
    print_case(f"half boxes against full boxes {eye} {yaw} {S1}")
    W, H, smax = 1920, 1080, 16
    cfg = sg.config_1080p(W, H)
    cfg = replace(cfg, camera=sg.look_camera(eye, yaw, W, H), lens=replace(cfg.lens, focus_distance=S1))
    sc = upload_scene(hd, ctx, sg.living_room_scene(0))
    n = W * H * smax
    spp = torch.full((H, W), smax, dtype=torch.uint8, device=DEV)
    off = (torch.arange(H * W, dtype=torch.int32, device=DEV) * smax).view(H, W)
    total = torch.tensor([n], dtype=torch.int32, device=DEV)
    got = []
    for wave in (0, 1):
        hd.hdof_set_tuning(ctx, wave=wave)
        rid = torch.full((n,), -7, dtype=torch.int32, device=DEV)
        rz = torch.zeros(n, dtype=torch.float32, device=DEV)
        hd.hdof_trace_thin_lens(ctx, sc, hd.camera_of(cfg.camera), hd.lens_of(cfg.lens), hd.light_of(cfg.light), smax,
                                spp, off, total, seed=11, ray_tri_id=rid, ray_depth=rz)
        got.append((rid, rz))
    hd.hdof_set_tuning(ctx)
    torch.cuda.synchronize()
    diff = int((got[0][0] != got[1][0]).sum())
    assert diff == 0, f"{diff} of {n} rays"
    assert torch.equal(got[0][1], got[1][1])
    sc.close()


def far_room(hd, ctx, shift=0.0, ground=0.0, w=320, h=180, smax=8):
    """The living room moved along (1, 1, 1), or on a ground plane far wider
    than itself: its scene, and the arguments of a trace of every pixel."""
    cfg = sg.config_1080p(w, h)
    scene = sg.living_room_scene(0)
    verts, albedo = scene.verts, scene.albedo
    if ground:
        g, y = ground, float(verts.reshape(-1, 3)[:, 1].min()) - 0.05
        q = np.array([(-g, y, -g), (g, y, -g), (g, y, g), (-g, y, g)], np.float32)
        verts = np.concatenate([verts, q[[0, 1, 2]].reshape(1, 9), q[[0, 2, 3]].reshape(1, 9)])
        albedo = np.concatenate([albedo, np.full((2, 3), 0.5, albedo.dtype)])
    cam = replace(cfg.camera, eye=(np.asarray(cfg.camera.eye) + shift).astype(np.float32))
    sc = upload_scene(hd, ctx, sg.Scene((verts + np.float32(shift)).astype(np.float32), albedo))
    spp = torch.full((h, w), smax, dtype=torch.uint8, device=DEV)
    off = (torch.arange(h * w, dtype=torch.int32, device=DEV) * smax).view(h, w)
    total = torch.tensor([h * w * smax], dtype=torch.int32, device=DEV)
    return sc, (hd.camera_of(cam), hd.lens_of(cfg.lens), hd.light_of(cfg.light), smax, spp, off, total), h * w * smax


@pytest.mark.parametrize("wave", [0, 1])
def test_counted_rays_are_the_queue(hd, ctx, wave):
    """A ray that is walked a second time (its hit lies at the very edge of a
    triangle; far from the origin every hundredth does) is one ray."""
    print_case(f"counters, wave {wave}")
    sc, args, n = far_room(hd, ctx, 1000.0)
    hd.hdof_set_tuning(ctx, wave=wave)
    hd.hdof_counters_begin(ctx)
    hd.hdof_trace_thin_lens(ctx, sc, *args, seed=3)
    c = hd.hdof_counters_end(ctx)
    hd.hdof_set_tuning(ctx)
    assert c["trace_rays"] == n and c["trace_visits"] >= n, c
    sc.close()


def both_forms(hd, ctx, sc, args, n):
    """Hits of the per-lane walk and of the wave-coherent one, and the per-lane walk's work per ray."""
    out = []
    for wave in (0, 1):
        hd.hdof_set_tuning(ctx, wave=wave)
        rid = torch.full((n,), -7, dtype=torch.int32, device=DEV)
        rz = torch.zeros(n, dtype=torch.float32, device=DEV)
        hd.hdof_trace_thin_lens(ctx, sc, *args, seed=3, ray_tri_id=rid, ray_depth=rz)
        out.append((rid, rz))
    hd.hdof_set_tuning(ctx)
    hd.hdof_counters_begin(ctx)
    hd.hdof_trace_thin_lens(ctx, sc, *args, seed=3)
    c = hd.hdof_counters_end(ctx)
    ctx.sync()
    return out, (c["trace_visits"] + c["trace_tests"]) / n


@pytest.mark.parametrize("shift,ground,full,share", [
    (0.0, 0.0, 34.37, 0.0), (1e4, 0.0, 38.60, 1e-4), (1e5, 0.0, 40.58, 5e-4), (0.0, 1e4, 51.18, 0.0),
    (0.0, 1e5, 43.68, 0.0), (0.0, 1e8, 56.96, 0.0), (0.0, 1e10, 48.31, 0.0), (0.0, 1e14, 48.31, 0.0)])
def test_far_geometry_keeps_the_boxes_tight(hd, ctx, shift, ground, full, share):
    """A room far from the origin, or on a ground far wider than itself: the
    half boxes stay as tight as the room's size asks, and the hits are those
    of the full boxes.  full: node visits and triangle tests per ray of the
    per-lane walk by fp32 boxes on these inputs; share: the rays that may hit
    another triangle (at 1e4 and 1e5 the coordinates' own steps are 1e-3 and
    8e-3, and two walks by fp32 boxes in another order differ in 5 and 36 of
    these 460800 rays)."""
    print_case(f"half boxes: shift {shift} ground {ground}")
    sc, args, n = far_room(hd, ctx, shift, ground)
    (half, wave), work = both_forms(hd, ctx, sc, args, n)
    sc.close()
    differ = int(((half[0] != wave[0]) | (half[1] != wave[1])).sum())
    print(f"work per ray {work:.2f} against {full}, {differ} rays differ")
    assert work <= 1.25 * full
    assert differ <= share * n


def test_rays_along_an_axis_in_a_vast_scene(hd, ctx):
    """No aperture and an odd width: the middle column's rays have a direction
    component of exactly 0, whose inverse is clamped to 1e30.  Geometry of 1e7
    units' size inside 1e13: the scene's box unit times that inverse has to
    stay finite."""
    print_case("half boxes: axis rays, vast scene")
    rng = np.random.default_rng(1)
    c = rng.uniform(0, 1, (4000, 1, 3)) * [6e7, 6e7, 1e8] + [3e7, 3e7, 2e7]
    v = (c + rng.uniform(-3e6, 3e6, (4000, 3, 3))).reshape(-1, 9)
    g, y = 1e13, -1e6
    q = np.array([(-g, y, -g), (g, y, -g), (g, y, g), (-g, y, g)])
    v = np.concatenate([v, q[[0, 1, 2]].reshape(1, 9), q[[0, 2, 3]].reshape(1, 9)]).astype(np.float32)
    sc = upload_scene(hd, ctx, sg.Scene(v, np.full((len(v), 3), 0.5, np.float32)))
    W, H, smax = 65, 65, 1
    cfg = sg.config_1080p(W, H)
    cam = sg.look_camera((8.2e7, 7.1e7, 0.0), 0.0, W, H)
    lens = replace(cfg.lens, aperture=0.0, focus_distance=1e7)
    spp = torch.ones((H, W), dtype=torch.uint8, device=DEV)
    off = torch.arange(H * W, dtype=torch.int32, device=DEV).view(H, W)
    args = (hd.camera_of(cam), hd.lens_of(lens), hd.light_of(cfg.light), smax, spp, off,
            torch.tensor([H * W], dtype=torch.int32, device=DEV))
    (half, full), _ = both_forms(hd, ctx, sc, args, H * W)
    sc.close()
    assert int((full[0] >= 0).sum()) > H * W // 4
    assert torch.equal(half[0], full[0]) and torch.equal(half[1], full[1])


@pytest.mark.parametrize("W,H", [(256, 255), (256, 256)])
@pytest.mark.parametrize("count", [16, 17, 70])
def test_reduction_of_many_rays_a_pixel(hd, ctx, W, H, count):
    """Either side of the counts and image sizes from which a small image's
    pixels read their own entries: the same sums bit for bit as for entries
    in random order, which every lane reads for itself."""
    print_case(f"reduction {W}x{H}, {count} rays a pixel")
    cfg = sg.config_tiny(aperture_override=0.2)
    cfg = replace(cfg, camera=replace(cfg.camera, width=W, height=H))
    sc = upload_scene(hd, ctx, sg.tiny_scene(3))
    n, out = W * H, []
    for order in (np.arange(n), np.random.default_rng(count).permutation(n)):
        off = np.zeros(n, np.int64)
        off[order] = np.arange(n) * count
        rt = hd.hdof_trace_thin_lens(ctx, sc, hd.camera_of(cfg.camera), hd.lens_of(cfg.lens), hd.light_of(cfg.light),
                                     count, torch.full((H, W), count, dtype=torch.uint8, device=DEV),
                                     to_dev(off.reshape(H, W).astype(np.int32)),
                                     to_dev(np.array([n * count], np.int32)), seed=5)
        torch.cuda.synchronize()
        out.append([t.cpu().numpy() for t in (rt.c_near, rt.c_far, rt.hit_ratio, rt.lum_m1, rt.lum_m2)])
    for a, b in zip(*out):
        assert np.array_equal(a, b)
    sc.close()
