"""The frame counters the host reads (needs an MI355X).

A frame's counters reach host memory while its shade still runs: whatever
frame came before on the stream, vtx_read_stats right after a call has to give
that call's own numbers.
"""
import dataclasses

import numpy as np
import pytest

from paper_2501_12750_amd import scenes

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def vtx():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a visible GPU"
    from paper_2501_12750_amd import vtx as v
    return v


def test_stats_are_the_last_calls_own(vtx):
    import torch
    ctx = vtx.vtx_context_create(0, 0)
    stream = torch.cuda.Stream()
    calls, names, keep = [], [], []
    for n, flags in ((500, 0), (3000, 16), (40_000, 0), (40_000, 8), (1, 0), (3000, 1)):
        wl = scenes.plain_small(n_atoms=n, width=400 + n % 97, height=300, seed=n)
        opts = dataclasses.replace(wl.options, flags=flags, ssao_samples=16)
        ds = vtx.DeviceScene(wl.scene)
        rs = vtx.ResidentScene(ctx, ds)
        frames = [vtx.Frame(wl.width, wl.height) for _ in range(3)]
        jobs = [vtx.make_job(rs.handle, 0, wl.camera, opts, wl.width, wl.height, f.rgba, f.depth, f.id) for f in frames]
        keep.append((ds, rs, frames, jobs))
        calls += [lambda ds=ds, wl=wl, o=opts, f=frames[0]: vtx.vtx_render(*ds.args(), wl.camera, o, wl.width, wl.height,
                                                                           f.rgba, f.depth, f.id, stream),
                  lambda rs=rs, wl=wl, o=opts, f=frames[0]: rs.render(wl.camera, o, wl.width, wl.height, f, stream),
                  lambda jobs=jobs: vtx.vtx_render_batch(ctx, jobs, stream)]
        names += [f"{n} atoms, flags {flags}, {form}" for form in ("arrays", "scene", "batch of 3")]
    def own(st, name):
        keys = ["visible", "pairs", "overflow_tiles"]
        if "flags 16" not in name:   # how many tests the early-outs leave depends on the order of evaluation
            keys += ["fragments_tested", "fragments_hit"]
        return {k: st[k] for k in keys}

    want = []
    for call, name in zip(calls, names):
        for _ in range(2):   # the first sizes the lists
            call()
        stream.synchronize()
        want.append(own(vtx.vtx_read_stats(stream), name))
    assert len({tuple(w.values()) for w in want}) > 10
    rng = np.random.default_rng(3)
    for i in rng.integers(0, len(calls), 400):
        calls[i]()
        assert own(vtx.vtx_read_stats(stream), names[i]) == want[i], names[i]
    # several frames queued before the numbers are read
    for i in rng.integers(0, len(calls), (100, 4)):
        for k in i:
            calls[k]()
        assert own(vtx.vtx_read_stats(stream), names[i[-1]]) == want[i[-1]], names[i[-1]]
    stream.synchronize()
    for _, rs, _, _ in keep:
        rs.close()
    vtx.vtx_context_destroy(ctx)
