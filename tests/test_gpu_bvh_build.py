"""GPU BVH build at the triangle counts where its passes change form: the
sort's blocks of 1024 keys, the clustering rounds' blocks of 256, the one
block that does the last rounds (1024 clusters) with its split searches, and
degenerate inputs (equal triangles, all Morton codes alike).  Each build's
G-buffer against the FP64 oracle: ids equal except on the rays it flags."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import oracle
import scenegen as sg
from gpu_common import print_case, upload_scene

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def hd():
    from paper_2210_04981_amd import hdof
    return hdof


@pytest.fixture(scope="module")
def ctx(hd):
    c = hd.hdof_create(0)
    yield c
    c.close()


def soup(n, seed, size):
    rng = np.random.default_rng(seed)
    c = np.concatenate([rng.uniform(-1, 1, (n, 1, 2)), rng.uniform(1, 4, (n, 1, 1))], -1)
    v = (c + rng.uniform(-size, size, (n, 3, 3))).reshape(n, 9).astype(np.float32)
    return sg.Scene(v, rng.uniform(0, 1, (n, 3)).astype(np.float32))


def check(hd, ctx, scene):
    cfg = sg.config_tiny()
    sc = upload_scene(hd, ctx, scene)
    st = sc.stats()
    assert st["n_tris"] == scene.n_tris and 1 <= st["max_depth"] <= 64
    gb = hd.hdof_gbuffer(ctx, sc, hd.camera_of(cfg.camera), hd.lens_of(cfg.lens), hd.light_of(cfg.light))
    torch.cuda.synchronize()
    ctx.sync()
    ref = oracle.gbuffer(oracle.Scene(scene.verts, scene.albedo), cfg.camera, cfg.lens, cfg.light)
    bad = (gb.tri_id.cpu().numpy() != ref["tri_id"]) & (ref["amb"] == 0)
    assert not bad.any(), f"{bad.sum()} unambiguous hits differ"
    sc.close()


@pytest.mark.parametrize("n", [2, 3, 17, 128, 129, 255, 257, 512, 1023, 1024, 1025, 2049, 5000, 70001])
def test_counts(hd, ctx, n):
    print_case(f"build of {n} triangles")
    check(hd, ctx, soup(n, n, 0.9 / n ** (1 / 3)))


def test_builds_in_turn_share_scratch(hd, ctx):
    """A large build between two small ones: the context's kept scratch."""
    print_case("builds in turn")
    for n in (300, 40000, 301):
        check(hd, ctx, soup(n, n + 1, 0.05))


def test_equal_triangles(hd, ctx):
    """Every triangle the same: all codes and areas tie, each ray hits the lowest index."""
    print_case("equal triangles")
    one = soup(1, 5, 0.8)
    scene = sg.Scene(np.repeat(one.verts, 1500, 0), np.repeat(one.albedo, 1500, 0))
    cfg = sg.config_tiny()
    sc = upload_scene(hd, ctx, scene)
    gb = hd.hdof_gbuffer(ctx, sc, hd.camera_of(cfg.camera), hd.lens_of(cfg.lens), hd.light_of(cfg.light))
    torch.cuda.synchronize()
    ctx.sync()
    assert set(np.unique(gb.tri_id.cpu().numpy())) <= {-1, 0}
    sc.close()


@pytest.mark.parametrize("n,what", [(2, "inf"), (300, "inf"), (1500, "inf"), (300, "far"), (3000, "far")])
def test_geometry_that_does_not_cluster_is_refused(hd, ctx, n, what):
    """An infinite vertex, or two groups so far apart that the area of their
    union overflows: rounds make progress, then none merges.  The build is
    refused and the context builds on."""
    print_case(f"refused build: {n} triangles, {what}")
    scene = soup(n, n, 0.05)
    v = scene.verts.copy()
    if what == "inf":
        v[n // 3, 4] = np.inf
    else:
        v *= np.float32(1e13)
        v.reshape(n, 3, 3)[n // 2:, :, :2] += np.float32(1e20)
    with pytest.raises(hd.HdofError, match="no progress"):
        upload_scene(hd, ctx, sg.Scene(v, scene.albedo))
    check(hd, ctx, soup(400, 9, 0.1))


def gbuffer_of(hd, ctx, scene):
    cfg = sg.config_tiny()
    sc = upload_scene(hd, ctx, scene)
    gb = hd.hdof_gbuffer(ctx, sc, hd.camera_of(cfg.camera), hd.lens_of(cfg.lens), hd.light_of(cfg.light))
    torch.cuda.synchronize()
    ctx.sync()
    sc.close()
    return gb


def test_equal_triangles_cover_what_one_does(hd, ctx):
    """1500 equal triangles are hit where the one is, all as the lowest index, at its depth."""
    print_case("equal triangles against one")
    one = soup(1, 5, 0.8)
    a = gbuffer_of(hd, ctx, one)
    b = gbuffer_of(hd, ctx, sg.Scene(np.repeat(one.verts, 1500, 0), np.repeat(one.albedo, 1500, 0)))
    assert int((a.tri_id == 0).sum()) > 50
    assert torch.equal(a.tri_id, b.tri_id) and torch.equal(a.depth, b.depth)


def test_more_triangles_than_the_blocks_sum_by_themselves(hd, ctx):
    """A plane of 2.12M triangles: above 8192 blocks of clusters (2.10M) the
    rounds' counts are scanned by one block, and the scratch is larger than a
    context keeps.  Each pixel's triangle is known from where its ray meets
    the plane, but for rays within a thousandth of a cell of an edge; the
    scratch's memory is given back; the next build gets its own."""
    print_case("build of 2.12M triangles")
    nx, ny, z, ext = 1060, 1000, 3.0, 2.0
    free0 = torch.cuda.mem_get_info()[0]
    x = torch.linspace(-ext, ext, nx + 1, dtype=torch.float64, device="cuda").float()
    y = torch.linspace(-ext, ext, ny + 1, dtype=torch.float64, device="cuda").float()
    p = torch.stack([*torch.meshgrid(y, x, indexing="ij")[::-1], torch.full((ny + 1, nx + 1), z, device="cuda")], -1)
    q = [p[:-1, :-1], p[:-1, 1:], p[1:, 1:], p[1:, :-1]]
    v = torch.stack([torch.cat([q[0], q[1], q[2]], -1), torch.cat([q[0], q[2], q[3]], -1)], 2).reshape(-1, 9).contiguous()
    assert v.shape[0] > 8192 * 256
    W, H = 200, 150
    cfg = sg.config_1080p(W, H)
    cam = sg.look_camera((0, 0, 0), 0.0, W, H)
    sc = hd.hdof_build_bvh(ctx, v, torch.full((v.shape[0], 3), 0.5, device="cuda"))
    assert 1 <= sc.stats()["max_depth"] <= 64
    gb = hd.hdof_gbuffer(ctx, sc, hd.camera_of(cam), hd.lens_of(cfg.lens), hd.light_of(cfg.light))
    torch.cuda.synchronize()
    ctx.sync()
    sc.close()
    got = gb.tri_id.cpu().numpy()
    t = float(cam.tan_half_fov_x)
    px = ((2 * np.arange(W) + 1) / W - 1) * t * z
    py = (1 - (2 * np.arange(H) + 1) / H) * t * H / W * z
    cx, cy = np.meshgrid((px + ext) / (2 * ext) * nx, (py + ext) / (2 * ext) * ny)
    fx, fy = cx % 1, cy % 1
    clear = np.minimum.reduce([fx, 1 - fx, fy, 1 - fy, np.abs(fx - fy)]) > 1e-3
    want = 2 * (np.floor(cy).astype(int) * nx + np.floor(cx).astype(int)) + (fy > fx)
    assert clear.mean() > 0.9 and (got[clear] == want[clear]).all(), (got[clear] != want[clear]).sum()
    assert np.abs(gb.depth.cpu().numpy() - z).max() < 1e-5 * z
    del v, p, q, gb
    torch.cuda.empty_cache()
    assert free0 - torch.cuda.mem_get_info()[0] < 320 << 20
    check(hd, ctx, soup(300, 2, 0.1))
