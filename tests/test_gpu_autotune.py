"""vtx_autotune: the tile-size tuner and its cache (needs an MI355X)."""
import json

import numpy as np
import pytest

from paper_2501_12750_amd import scenes
from tests.gpu_util import with_opts

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def vtx():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a visible GPU"
    from paper_2501_12750_amd import vtx as v
    return v


def _setup(vtx, ctx, n_atoms=4000):
    import torch
    scene0, frames, cams, opts, _ = scenes.trajectory(n_atoms=n_atoms, n_frames=3)
    rs = vtx.ResidentScene(ctx, vtx.DeviceScene(scene0))
    rs.add_frames(torch.from_numpy(np.ascontiguousarray(frames[1:])).to("cuda"), 2)
    return rs, cams, opts


def _batch(vtx, ctx, rs, cams, opts, tile, W=480, H=270):
    import torch
    imgs = [vtx.Frame(W, H) for _ in range(6)]
    jobs = [vtx.make_job(rs.handle, i % 3, cams[i % 4], with_opts(opts, tile_size=tile), W, H,
                         fr.rgba, fr.depth, fr.id) for i, fr in enumerate(imgs)]
    vtx.vtx_render_batch(ctx, jobs)
    torch.cuda.synchronize()
    return jobs, [fr.numpy() for fr in imgs]


def test_autotune_chooses_caches_and_applies(vtx, tmp_path):
    ctx = vtx.vtx_context_create(0, 0)
    rs, cams, opts = _setup(vtx, ctx)
    jobs, ref = _batch(vtx, ctx, rs, cams, opts, 16)
    cache = tmp_path / "tuning.json"
    t = vtx.vtx_autotune(ctx, jobs, cache)
    print(t)
    assert t["tile_size"] in (8, 16, 32, 64) and not t["from_cache"]
    assert set(t["ms_by_tile"]) == {8, 16, 32, 64} and min(t["ms_by_tile"].values()) > 0
    assert t["ms_by_tile"][t["tile_size"]] == min(t["ms_by_tile"].values())
    entries = json.loads(cache.read_text())["vtx_tuning"]
    assert [e["tile_size"] for e in entries if e["key"] == t["key"]] == [t["tile_size"]]
    # the images do not depend on the tile size, tuned or explicit
    for tile in (0, 8, 32, 64):
        _, got = _batch(vtx, ctx, rs, cams, opts, tile)
        for a, b in zip(got, ref):
            for k in ("depth", "id", "rgba"):
                assert np.array_equal(a[k], b[k]), f"tile {tile}: {k}"
    # a second context reads the choice back without timing anything
    ctx2 = vtx.vtx_context_create(0, 0)
    t2 = vtx.vtx_autotune(ctx2, jobs, cache)
    assert t2["from_cache"] and t2["tile_size"] == t["tile_size"] and t2["key"] == t["key"]
    # another shape is added to the same file, the first entry kept
    jobs3, _ = _batch(vtx, ctx, rs, cams, opts, 16, W=200, H=120)
    t3 = vtx.vtx_autotune(ctx, jobs3, cache)
    assert not t3["from_cache"] and t3["key"] != t["key"]
    keys = {e["key"]: e["tile_size"] for e in json.loads(cache.read_text())["vtx_tuning"]}
    assert keys == {t["key"]: t["tile_size"], t3["key"]: t3["tile_size"]}
    rs.close()
    vtx.vtx_context_destroy(ctx)
    vtx.vtx_context_destroy(ctx2)


def test_autotune_rejects_bad_arguments(vtx):
    ctx = vtx.vtx_context_create(0, 0)
    with pytest.raises(vtx.VtxError) as e:
        vtx.vtx_autotune(ctx, [])
    assert e.value.code == vtx.VTX_EINVAL
    vtx.vtx_context_destroy(ctx)


def test_autotune_sizes_the_bins(vtx, tmp_path):
    """The tuner reserves 5/4 of a sample job's pairs (+1024) at the chosen
    tile size; renders of that shape then fit their lists."""
    import torch
    ctx = vtx.vtx_context_create(0, 0)
    rs, cams, opts = _setup(vtx, ctx)
    jobs, ref = _batch(vtx, ctx, rs, cams, opts, 16)
    t = vtx.vtx_autotune(ctx, jobs, tmp_path / "t.json")
    assert t["bin_capacity"] > 1024
    # the same batch at the tuned size, with statistics, on a fresh stream
    stream = torch.cuda.Stream()
    for j in jobs:
        j.options.tile_size = 0
        j.options.flags = vtx.VTX_FLAG_STATS
    with torch.cuda.stream(stream):
        vtx.vtx_render_batch(ctx, jobs, stream)
    stream.synchronize()
    st = vtx.vtx_read_stats(stream)
    print(t, st)
    assert st["overflow_tiles"] == 0
    assert st["pairs"] <= len(jobs) * (t["bin_capacity"] - 1024) * 4 // 5 + len(jobs)
    assert st["bin_capacity"] >= st["pairs"]
    entries = json.loads((tmp_path / "t.json").read_text())["vtx_tuning"]
    assert [e["bin_capacity"] for e in entries if e["key"] == t["key"]] == [t["bin_capacity"]]
    rs.close()
    vtx.vtx_context_destroy(ctx)


def test_autotune_picks_ssao_samples_within_a_budget(vtx, tmp_path):
    """Jobs that ask for VTX_SSAO_AUTO get the largest tried count whose
    time per render fits the budget; renders asking for it afterwards equal
    renders with that count given explicitly."""
    import torch
    ctx = vtx.vtx_context_create(0, 0)
    rs, cams, opts = _setup(vtx, ctx)
    auto = with_opts(opts, ssao_samples=vtx.VTX_SSAO_AUTO)
    jobs, _ = _batch(vtx, ctx, rs, cams, auto, 0)
    # no budget: 16 samples, nothing timed for them
    t0 = vtx.vtx_autotune(ctx, jobs)
    assert t0["ssao_samples"] == 16 and t0["ms_by_samples"] == {}
    # a generous budget: the most samples
    t1 = vtx.vtx_autotune(ctx, jobs, frame_budget_ms=1e6)
    assert t1["ssao_samples"] == 64 and list(t1["ms_by_samples"]) == [64]
    # a budget between the times of two counts: the larger count that fits
    t2 = vtx.vtx_autotune(ctx, jobs, frame_budget_ms=1e-6)
    assert t2["ssao_samples"] == 0 and set(t2["ms_by_samples"]) == set(vtx.SSAO_COUNTS)
    times = t2["ms_by_samples"]
    assert times[64] > times[0]
    # the budget as the tuner holds it (FP32), so that both sides compare the same value
    mid = float(np.float32(0.5 * (times[64] + times[0])))
    t3 = vtx.vtx_autotune(ctx, jobs, tmp_path / "s.json", frame_budget_ms=mid)
    fits = [k for k in vtx.SSAO_COUNTS if times[k] <= mid]
    print(times, t3)
    assert t3["ssao_samples"] in vtx.SSAO_COUNTS and t3["ms_by_samples"][t3["ssao_samples"]] <= mid
    assert all(t3["ms_by_samples"].get(k, 1e9) > mid for k in vtx.SSAO_COUNTS if k > t3["ssao_samples"])
    assert fits  # the cheapest count fits a budget above its own time
    # renders asking for the context's count equal explicit ones
    _, got = _batch(vtx, ctx, rs, cams, auto, 0)
    _, ref = _batch(vtx, ctx, rs, cams, with_opts(opts, ssao_samples=t3["ssao_samples"]), 0)
    for a, b in zip(got, ref):
        for k in ("depth", "id", "rgba"):
            assert np.array_equal(a[k], b[k]), k
    # the cache keeps the count; a second context reads it back untimed
    ctx2 = vtx.vtx_context_create(0, 0)
    t4 = vtx.vtx_autotune(ctx2, jobs, tmp_path / "s.json", frame_budget_ms=mid)
    assert t4["from_cache"] and t4["ssao_samples"] == t3["ssao_samples"] and t4["bin_capacity"] == t3["bin_capacity"]
    rs.close()
    vtx.vtx_context_destroy(ctx)
    vtx.vtx_context_destroy(ctx2)


# ---------------------------------------------------------------------------
# Scenes large and opaque enough to take the occlusion pre-pass unasked
# ---------------------------------------------------------------------------
W_BALL, H_BALL = 1280, 960   # too many 8-pixel tiles, which keep to one pass


@pytest.fixture(scope="module")
def ball():
    """17M atoms in a ball seen whole: its frames take two passes once their lists are sized."""
    n = 17_000_000
    rng = np.random.default_rng(17)
    radius = (3.0 * n / (4.0 * np.pi * 0.1)) ** (1.0 / 3.0)
    d = rng.normal(size=(n, 3)).astype(np.float32)
    d *= (radius * np.cbrt(rng.uniform(size=n)) / np.linalg.norm(d, axis=1)).astype(np.float32)[:, None]
    scene = scenes.Scene(d, np.full(n, 1.6, np.float32), np.full(n, scenes.pack_rgba(200, 180, 160), np.uint32),
                         np.zeros((0, 2), np.uint32))
    return scenes.Workload("ball", scene, scenes.orbit_camera((0.0, 0.0, 0.0), 1.2 * radius, 0.4),
                           scenes.Options(ssao_samples=0), W_BALL, H_BALL)


def _fresh_stream(vtx):
    """A stream without scratch (torch hands the same streams out again)."""
    import torch
    stream = torch.cuda.Stream()
    vtx.vtx_release_scratch(stream)
    return stream


def _frame_stats(vtx, rs, wl, flags, stream):
    """Statistics of the scene's next frame on the stream."""
    import torch
    with torch.cuda.stream(stream):
        rs.render(wl.camera, with_opts(wl.options, flags=flags), wl.width, wl.height, stream=stream)
    stream.synchronize()
    return vtx.vtx_read_stats(stream)


def _ball_job(vtx, rs, wl):
    fr = vtx.Frame(wl.width, wl.height)
    return fr, vtx.make_job(rs.handle, 0, wl.camera, wl.options, wl.width, wl.height, fr.rgba, fr.depth, fr.id)


def test_tuned_lists_hold_the_one_pass_frames_of_a_pre_pass_scene(vtx, ball, tmp_path):
    ctx = vtx.vtx_context_create(0, 0)
    rs = vtx.ResidentScene(ctx, vtx.DeviceScene(ball.scene))
    fr, job = _ball_job(vtx, rs, ball)
    t = vtx.vtx_autotune(ctx, [job], tmp_path / "t.json")
    two = _frame_stats(vtx, rs, ball, 0, _fresh_stream(vtx))
    for flags in (vtx.VTX_FLAG_ONE_PASS, vtx.VTX_FLAG_STATS):
        st = _frame_stats(vtx, rs, ball, flags, _fresh_stream(vtx))
        print("capacity", t["bin_capacity"], "pairs in one pass", st["pairs"], "the larger of two", two["pairs"], flush=True)
        assert two["pairs"] < st["pairs"] and st["bin_capacity"] == t["bin_capacity"]
        assert st["overflow_tiles"] == 0
        assert t["bin_capacity"] == st["pairs"] + st["pairs"] // 4 + 1024
    # read back from the cache, the capacity is the same
    ctx2 = vtx.vtx_context_create(0, 0)
    t2 = vtx.vtx_autotune(ctx2, [job], tmp_path / "t.json")
    assert t2["from_cache"] and t2["bin_capacity"] == t["bin_capacity"]
    rs.close()
    vtx.vtx_context_destroy(ctx)
    vtx.vtx_context_destroy(ctx2)


def test_a_cache_entry_of_unknown_passes_is_counted_anew(vtx, ball, tmp_path):
    """A cache that does not say its pairs were one pass's: the tile size is
    taken, the capacity is not, so that the first frame counts its pairs.  A
    shape too small for the pre-pass keeps its capacity."""
    ctx = vtx.vtx_context_create(0, 0)
    rs = vtx.ResidentScene(ctx, vtx.DeviceScene(ball.scene))
    fr, job = _ball_job(vtx, rs, ball)
    small, cams, opts = _setup(vtx, ctx)
    jobs, _ = _batch(vtx, ctx, small, cams, opts, 16)
    cache = tmp_path / "old.json"
    cache.write_text('{"vtx_tuning": [\n'
                     '  {"key": "1280x960/p24/persp", "tile_size": 32, "ssao_samples": -1, "bin_capacity": 2000, "ms_per_batch": 0.5},\n'
                     '  {"key": "480x270/p11/persp", "tile_size": 32, "ssao_samples": -1, "bin_capacity": 70000, "ms_per_batch": 0.5}\n'
                     ']}\n')
    t = vtx.vtx_autotune(ctx, [job], cache)
    assert t["from_cache"] and t["tile_size"] == 32 and t["bin_capacity"] == 0
    st = _frame_stats(vtx, rs, ball, vtx.VTX_FLAG_ONE_PASS, _fresh_stream(vtx))
    assert st["overflow_tiles"] == 0 and st["bin_capacity"] > st["pairs"] > 2000
    t = vtx.vtx_autotune(ctx, jobs, cache)
    assert t["from_cache"] and t["tile_size"] == 32 and t["bin_capacity"] == 70000
    rs.close()
    small.close()
    vtx.vtx_context_destroy(ctx)


def test_two_pass_pairs_size_no_other_stream(vtx, ball):
    """Frames of a fixed capacity take two passes without a count: what they
    bin is not taken for the pairs of the scene on another stream."""
    ctx = vtx.vtx_context_create(0, 0)
    rs = vtx.ResidentScene(ctx, vtx.DeviceScene(ball.scene))
    fixed, other = _fresh_stream(vtx), _fresh_stream(vtx)
    vtx.vtx_set_bin_capacity(60_000_000, fixed)
    for _ in range(2):
        two = _frame_stats(vtx, rs, ball, 0, fixed)
    st = _frame_stats(vtx, rs, ball, vtx.VTX_FLAG_ONE_PASS, other)
    print("two passes", two, "one", st, flush=True)
    assert two["overflow_tiles"] == 0 and two["pairs"] < st["pairs"]
    assert st["overflow_tiles"] == 0 and st["bin_capacity"] >= st["pairs"]
    rs.close()
    vtx.vtx_release_scratch(fixed)
    vtx.vtx_context_destroy(ctx)
