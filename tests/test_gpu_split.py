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
