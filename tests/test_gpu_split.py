"""How a frame's work is cut: binning workgroups and cluster quarters
(needs an MI355X).

Every cut must give the oracle's image: the sizes lie at the edges of the
primitive counts where the number of binning workgroups changes, at cluster
and quarter remainders, and at one and many renders per launch.
"""
import dataclasses

import numpy as np
import pytest

from oracle import compare, osplat
from paper_2501_12750_amd import scenes
from tests.gpu_util import assert_clean, run_render

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def vtx():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a visible GPU"
    from paper_2501_12750_amd import vtx as v
    return v


@pytest.fixture(scope="module")
def ctx(vtx):
    c = vtx.vtx_context_create(0, 0)
    yield c
    vtx.vtx_context_destroy(c)


def workload(n, bonded, width, height):
    wl = scenes.plain_small(n_atoms=n, width=width, height=height, seed=n)
    if bonded and n > 1:
        k = np.arange(n - 1, dtype=np.uint32)
        b = np.stack([k, k + 1], axis=1)[: max(1, n // 3)]
        wl.scene = dataclasses.replace(wl.scene, radii=np.full(n, 0.4, np.float32), bonds=np.ascontiguousarray(b))
    return wl


def assert_identical(a, b, what):
    for k in ("depth", "id", "rgba"):
        assert np.array_equal(a[k], b[k]), f"{what}: {k} differs at {np.count_nonzero(a[k] != b[k])} pixels"


@pytest.mark.parametrize("n", [1, 63, 64, 65, 255, 257, 511, 513, 1025, 4097, 65536, 65537, 131073, 262145])
@pytest.mark.parametrize("bonded", [False, True])
def test_binning_cuts_give_the_oracle_image(vtx, ctx, n, bonded):
    import torch
    wl = workload(n, bonded, 97, 83)
    ds = vtx.DeviceScene(wl.scene)
    rs = vtx.ResidentScene(ctx, ds)
    args = (wl.camera, wl.options, wl.width, wl.height)
    plain = run_render(vtx, ds, *args)
    one = rs.render(*args)
    frames = [vtx.Frame(wl.width, wl.height) for _ in range(3)]
    vtx.vtx_render_batch(ctx, [vtx.make_job(rs.handle, 0, *args, f.rgba, f.depth, f.id) for f in frames])
    torch.cuda.synchronize()
    ref = osplat.render(wl.scene, wl.camera, wl.options, wl.width, wl.height)
    print("atoms", n, "bonds", wl.scene.n_bonds, "hits", int(np.count_nonzero(plain["id"] != 0xFFFFFFFF)), flush=True)
    assert_clean(compare.check_gbuffer(plain["depth"], plain["id"], ref), f"{n} atoms")
    assert_identical(one.numpy(), plain, "scene")
    for f in frames:
        assert_identical(f.numpy(), plain, "batch")
    rs.close()


def two_ways(vtx, ctx, wl, flags_a, flags_b):
    """The scene's images and statistics with two sets of flags, once its lists are sized."""
    import torch
    rs = vtx.ResidentScene(ctx, vtx.DeviceScene(wl.scene))
    out = []
    for flags in (0, flags_a, flags_b):
        fr = rs.render(wl.camera, dataclasses.replace(wl.options, flags=flags), wl.width, wl.height)
        torch.cuda.synchronize()
        out.append((fr.numpy(), vtx.vtx_read_stats()))
    rs.close()
    return out[1:]


@pytest.mark.parametrize("n", [1, 256, 257, 2049, 4096, 65536 + 255, 300_001])
@pytest.mark.parametrize("bonded", [False, True])
def test_pre_pass_at_few_and_odd_cluster_counts(vtx, ctx, n, bonded):
    wl = workload(n, bonded, 211, 133)
    (two, st_two), (one, st_one) = two_ways(vtx, ctx, wl, vtx.VTX_FLAG_TWO_PASS, vtx.VTX_FLAG_ONE_PASS)
    assert_identical(two, one, f"{n} atoms")
    print("atoms", n, "binned in two passes", st_two["visible"], "in one", st_one["visible"], flush=True)
    assert st_two["visible"] <= st_one["visible"]


def test_a_large_opaque_scene_takes_the_pre_pass_unasked(vtx, ctx):
    """17M atoms in a ball, seen whole: over 16M in view, its faces covered
    hundreds of times.  The same scene seen from inside, with an eighth of it
    in view, keeps to one pass."""
    n = 17_000_000
    rng = np.random.default_rng(17)
    radius = (3.0 * n / (4.0 * np.pi * 0.1)) ** (1.0 / 3.0)
    d = rng.normal(size=(n, 3)).astype(np.float32)
    d *= (radius * np.cbrt(rng.uniform(size=n)) / np.linalg.norm(d, axis=1)).astype(np.float32)[:, None]
    scene = scenes.Scene(d, np.full(n, 1.6, np.float32), np.full(n, scenes.pack_rgba(200, 180, 160), np.uint32),
                         np.zeros((0, 2), np.uint32))
    wl = scenes.Workload("ball", scene, scenes.orbit_camera((0.0, 0.0, 0.0), 1.2 * radius, 0.4),
                         scenes.Options(ssao_samples=8), 640, 480)
    (auto, st_auto), (one, st_one) = two_ways(vtx, ctx, wl, 0, vtx.VTX_FLAG_ONE_PASS)
    assert_identical(auto, one, "whole")
    assert st_auto["visible"] < st_one["visible"] // 2, (st_auto["visible"], st_one["visible"])
    wl.camera = scenes.Camera(eye=(0.0, 0.0, 0.0), target=(1.0, 0.2, 0.1))
    (auto, st_auto), (one, st_one) = two_ways(vtx, ctx, wl, 0, vtx.VTX_FLAG_ONE_PASS)
    assert_identical(auto, one, "inside")
    assert st_auto["visible"] == st_one["visible"]


def test_a_clip_plane_on_the_near_side_keeps_to_one_pass(vtx, ctx):
    """The scene of the test above, cut: where the nearest part of it goes,
    the front pass would have nothing to draw, and the frame stays in one
    pass; a cut of the far half or of a rim leaves it the pre-pass."""
    n = 17_000_000
    rng = np.random.default_rng(18)
    radius = (3.0 * n / (4.0 * np.pi * 0.1)) ** (1.0 / 3.0)
    d = rng.normal(size=(n, 3)).astype(np.float32)
    d *= (radius * np.cbrt(rng.uniform(size=n)) / np.linalg.norm(d, axis=1)).astype(np.float32)[:, None]
    scene = scenes.Scene(d, np.full(n, 1.6, np.float32), np.full(n, scenes.pack_rgba(200, 180, 160), np.uint32),
                         np.zeros((0, 2), np.uint32))
    cam = scenes.orbit_camera((0.0, 0.0, 0.0), 1.2 * radius, 0.4)
    view = np.asarray(cam.target, float) - np.asarray(cam.eye, float)
    view /= np.linalg.norm(view)
    side = np.cross(view, cam.up)
    side /= np.linalg.norm(side)
    for name, normal, d0, one_pass in (("near half", view, 0.0, True), ("nearest fifth", view, 0.45 * radius, True),
                                       ("far half", -view, 0.0, False), ("rim", side, 0.6 * radius, False)):
        wl = scenes.Workload("ball", scene, cam, scenes.Options(clip_plane=tuple(float(v) for v in normal) + (float(d0),)),
                             640, 480)
        (auto, st_auto), (one, st_one) = two_ways(vtx, ctx, wl, 0, vtx.VTX_FLAG_ONE_PASS)
        print(name, "pairs", st_auto["pairs"], "in one pass", st_one["pairs"], flush=True)
        assert_identical(auto, one, name)
        # of two passes the counters hold the larger one's pairs
        assert (st_auto["pairs"] == st_one["pairs"]) == one_pass, name


@pytest.mark.parametrize("size", [(3845, 2049), (3840, 2064)])
def test_wide_shade_tiles_of_a_large_batch(vtx, ctx, size):
    """Over 128M pixels a launch shades in 64x16 tiles: the images are the
    single renders', at widths that end inside a tile and inside a block."""
    import torch
    W, H = size
    wl = scenes.plain_small(n_atoms=3000, width=W, height=H, seed=7)
    opts = dataclasses.replace(wl.options, ssao_samples=8, outline_depth=0.05, outline_color=scenes.pack_rgba(9, 9, 9))
    rs = vtx.ResidentScene(ctx, vtx.DeviceScene(wl.scene))
    n = (128 << 20) // (W * H) + 1
    cams = [scenes.orbit_camera((0.0, 0.0, 0.0), 36.0, 0.3 * k) for k in range(n)]
    frames = [vtx.Frame(W, H) for _ in range(n)]
    vtx.vtx_render_batch(ctx, [vtx.make_job(rs.handle, 0, cams[k], opts, W, H, f.rgba, f.depth, f.id)
                               for k, f in enumerate(frames)])
    one = vtx.Frame(W, H)
    for k, f in enumerate(frames):
        rs.render(cams[k], opts, W, H, one)
        torch.cuda.synchronize()
        for name in ("rgba", "depth", "id"):
            assert torch.equal(getattr(one, name), getattr(f, name)), (k, name)
    rs.close()


@pytest.mark.parametrize("n,size", [(200, (40, 30)), (5000, (97, 83)), (60_000, (701, 403)), (200_000, (1111, 1017))])
@pytest.mark.parametrize("representation", [0, 3])
def test_stored_order_binning_equals_clusters(vtx, ctx, n, size, representation):
    """Small resident scenes are binned in stored order, without clusters; a
    two-pass request keeps the clusters.  Bad bonds, trajectory frames and
    bond-free representations go the same way in both."""
    import torch
    wl = workload(n, True, *size)
    wl.scene.bonds[::7, 1] = n + 5          # out of range: dropped from the scene
    wl.options = dataclasses.replace(wl.options, representation=representation)
    rs = vtx.ResidentScene(ctx, vtx.DeviceScene(wl.scene))
    moved = torch.from_numpy(wl.scene.positions + np.float32(0.25)).cuda()
    rs.add_frames(moved, 1)
    out = {}
    for flags in (0, vtx.VTX_FLAG_TWO_PASS):
        opts = dataclasses.replace(wl.options, flags=flags)
        for again in range(2):              # the first sizes the lists
            frames = [vtx.Frame(*size) for _ in range(2)]
            vtx.vtx_render_batch(ctx, [vtx.make_job(rs.handle, k, wl.camera, opts, *size, f.rgba, f.depth, f.id)
                                       for k, f in enumerate(frames)])
            one = rs.render(wl.camera, opts, *size)
            torch.cuda.synchronize()
        out[flags] = [f.numpy() for f in frames + [one]]
    for a, b in zip(*out.values()):
        assert_identical(a, b, "stored and clusters")
    assert_identical(out[0][0], out[0][2], "batch and single")
    rs.close()


# The scatter scans the tile counts at every size: in one part up to 8192
# tiles, in two parts of 8192 above.
@pytest.mark.parametrize("size", [(8, 8), (1016, 64), (1024, 64), (1032, 64), (448, 256), (456, 256), (1024, 512),
                                  (1032, 512)])
@pytest.mark.parametrize("capacity", [0, 3000])
def test_list_offsets_at_the_edges_of_their_scan(vtx, size, capacity):
    """Up to 8192 tiles the scatter scans the tile counts itself, in rows of
    1024, and past 1792 tiles they are resolved by falling list length: the
    image is the one of 64-pixel tiles (at most 144 of them), also where part
    of the lists overflows."""
    import torch
    wl = workload(20_000, True, *size)
    ds = vtx.DeviceScene(wl.scene)
    s = torch.cuda.Stream()
    out = {}
    for tile in (64, 8):
        vtx.vtx_set_bin_capacity(capacity if tile == 8 else 0, s)
        opts = dataclasses.replace(wl.options, tile_size=tile)
        out[tile] = run_render(vtx, ds, wl.camera, opts, *size, stream=s)
        st = vtx.vtx_read_stats(s)
        if tile == 8:
            assert (st["overflow_tiles"] > 0) == (0 < capacity < st["pairs"]), st
    vtx.vtx_set_bin_capacity(0, s)
    assert_identical(out[8], out[64], "8-pixel tiles")


@pytest.mark.parametrize("n", [9, 63, 64, 65, 255, 256, 257, 700])
@pytest.mark.parametrize("tile,size", [(16, (45, 27)), (16, (8, 5)), (32, (45, 27)), (64, (149, 75))])
@pytest.mark.parametrize("view", ["perspective", "orthographic", "clipped"])
def test_blocks_front_to_back_equal_all_fragments(vtx, ctx, n, tile, size, view):
    """Deep tiles of large footprints go front to back by 8x8 blocks: the
    image is the one of a statistics frame, which tests every fragment, with
    coinciding atoms (equal depths), bonds, and images that end inside a
    tile and a block; counting frames see early-outs."""
    import torch
    rng = np.random.default_rng(n)
    wl = workload(n, True, *size)
    pos = rng.uniform(-3.0, 3.0, size=(n, 3)).astype(np.float32)
    pos[1::5] = pos[0::5][: len(pos[1::5])]
    wl.scene = dataclasses.replace(wl.scene, positions=pos, radii=rng.uniform(0.3, 1.8, n).astype(np.float32))
    wl.camera = scenes.Camera(eye=(0.5, 0.25, 14.0), target=(0.0, 0.0, 0.0), projection=1 if view == "orthographic" else 0,
                              ortho_half_height=5.0)
    wl.options = dataclasses.replace(wl.options, tile_size=tile, bond_radius=0.6,
                                     clip_plane=(0.2, 0.1, -1.0, 1.0) if view == "clipped" else (0.0,) * 4)
    ds = vtx.DeviceScene(wl.scene)
    out, tested = {}, {}
    for flags in (0, vtx.VTX_FLAG_STATS, vtx.VTX_FLAG_COUNT):
        out[flags] = run_render(vtx, ds, wl.camera, dataclasses.replace(wl.options, flags=flags), *size)
        tested[flags] = vtx.vtx_read_stats()["fragments_tested"]
    assert_identical(out[0], out[vtx.VTX_FLAG_STATS], "all fragments")
    assert_identical(out[0], out[vtx.VTX_FLAG_COUNT], "counted")
    assert 0 < tested[vtx.VTX_FLAG_COUNT] <= tested[vtx.VTX_FLAG_STATS]
    if n >= 256:
        assert tested[vtx.VTX_FLAG_COUNT] < tested[vtx.VTX_FLAG_STATS]
    ref = osplat.render(wl.scene, wl.camera, wl.options, *size)
    assert_clean(compare.check_gbuffer(out[0]["depth"], out[0]["id"], ref), f"{n} atoms")


@pytest.mark.parametrize("size", [(1024, 768), (701, 403), (257, 33)])
def test_noise_tiles_of_a_large_launch(vtx, ctx, size):
    """From 3M pixels on, a launch with the noise form of the ambient
    occlusion shades in 32x32 tiles: its images are the single renders', with
    and without the noise, at sizes that end inside a tile and a block."""
    import torch
    W, H = size
    wl = scenes.plain_small(n_atoms=3000, width=W, height=H, seed=7, eye_distance=60.0)
    rs = vtx.ResidentScene(ctx, vtx.DeviceScene(wl.scene))
    n = (3 << 20) // (W * H) + 1
    opts = [dataclasses.replace(wl.options, ssao_samples=8, ssao_noise=1 if k % 3 else 0) for k in range(n)]
    cams = [scenes.orbit_camera((0.0, 0.0, 0.0), 60.0, 0.3 * k) for k in range(n)]
    frames = [vtx.Frame(W, H) for _ in range(n)]
    vtx.vtx_render_batch(ctx, [vtx.make_job(rs.handle, 0, cams[k], opts[k], W, H, f.rgba, f.depth, f.id)
                               for k, f in enumerate(frames)])
    one = vtx.Frame(W, H)
    for k, f in enumerate(frames):
        rs.render(cams[k], opts[k], W, H, one)
        torch.cuda.synchronize()
        for name in ("rgba", "depth", "id"):
            assert torch.equal(getattr(one, name), getattr(f, name)), (k, name)
    rs.close()
