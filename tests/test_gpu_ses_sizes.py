"""The surface's distance windows, grid remainders and runs of cubes against
the SES oracle (needs an MI355X): windows on both sides of the one a brick's
LDS holds, dimensions around the bricks', words' and cells' sizes, grids
smaller than a window, cuts through atoms, and little or no capacity."""
import numpy as np
import pytest

from oracle import oses
from tests.test_gpu_ses import run_ses

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def vtx():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a visible GPU"
    from paper_2501_12750_amd import vtx as v
    return v


def atoms(seed, n, extent):
    rng = np.random.default_rng(seed)
    return (rng.uniform(0.0, 1.0, size=(n, 3)) * extent).astype(np.float32), rng.uniform(1.1, 1.9, size=n).astype(np.float32)


def check(vtx, pos, rad, probe, origin, h, dims, capacity=None):
    origin = np.asarray(origin, np.float32)
    h = np.float32(h)
    ref = oses.ses_field(pos, rad, probe, origin, h, dims)
    mc = oses.marching_cubes(ref["f"], origin, h)["vertices"]
    f, tri, n = run_ses(vtx, pos, rad, probe, origin, h, dims, capacity)
    print("grid", dims, "h", float(h), "probe", probe, "triangles", n, flush=True)
    assert np.array_equal(f, ref["f"])
    assert n == mc.shape[0]
    m = n if capacity is None else min(n, capacity)
    assert tri.shape[0] == m
    # the oracle's vertices in FP64 against FP32 arithmetic of a few roundings
    assert np.all(np.abs(tri.astype(np.float64) - mc[:m]) <= 1e-5 * (np.abs(mc[:m]) + float(h)))
    return n


@pytest.mark.parametrize("window", [2, 3, 4, 5, 8, 11, 12, 13, 32, 33])
def test_every_kind_of_window(vtx, window):
    h = 0.3
    probe = 0.0 if window == 2 else float(np.float32(h)) * (window - 2.5)
    pos, rad = atoms(window, 9, np.array([5.0, 6.0, 4.0]))
    check(vtx, pos, rad, probe, (-2.3, -2.1, -2.2), h, (35, 37, 31))


@pytest.mark.parametrize("dims", [(2, 2, 2), (3, 70, 5), (31, 15, 17), (32, 16, 16), (33, 17, 16), (34, 18, 33), (64, 5, 4),
                                  (65, 33, 2), (129, 3, 20), (97, 48, 50)])
def test_grid_remainders(vtx, dims):
    h = 0.45
    pos, rad = atoms(sum(dims), 40, np.array(dims) * h)   # atoms past the border too: it cuts through them
    assert check(vtx, pos, rad, 1.4, (0.1, -0.2, 0.05), h, dims) >= 0


def test_capacity_ends_inside_a_run(vtx):
    pos, rad = atoms(5, 30, np.array([9.0, 8.0, 7.0]))
    n = check(vtx, pos, rad, 1.4, (-3.0, -3.0, -3.0), 0.4, (37, 35, 33))
    assert n > 2000
    for capacity in (1, 511, 513, n - 1):
        check(vtx, pos, rad, 1.4, (-3.0, -3.0, -3.0), 0.4, (37, 35, 33), capacity)


def test_no_atoms(vtx):
    import torch
    dims = (40, 20, 18)
    f, tri, n = run_ses(vtx, np.zeros((0, 3), np.float32), np.zeros(0, np.float32), 1.4, (0.0, 0.0, 0.0), 0.5, dims, 16)
    assert n == 0 and np.all(f < 0.0)
    torch.cuda.synchronize()


def test_positions_far_beyond_the_spacing(vtx):
    """Coordinates of 2^27 at a spacing of 1e-6: their rounding is 0.03 steps,
    so a point that the rounded sphere holds can lie past the rounded end of
    the atom's box by more than any fixed margin."""
    rng = np.random.default_rng(0)
    o = 2.0 ** 27
    left_out = 0
    for _ in range(2000):
        h = float(np.float32(1e-6 * rng.uniform(0.5, 2.0)))
        r = float(np.float32(h * rng.uniform(2.0, 9.0)))
        x = (o + h * np.arange(14)) - o
        if np.flatnonzero(x * x < r * r).max() > np.floor((o + r - o) * (1.0 / h) + 1e-3):
            left_out += 1
            check(vtx, np.full((1, 3), o, np.float32), np.array([r], np.float32), 0.0, (o, o, o), h, (14, 14, 14))
    assert left_out > 5


@pytest.mark.parametrize("n", [1, 2, 7, 8, 9, 15, 63, 65, 520, 4099])
@pytest.mark.parametrize("dims,h,scale", [((6, 5, 4), 1.5, 1.0), ((5, 5, 8), 0.7, 1.0), ((17, 9, 33), 2.5, 1.0), ((34, 18, 6), 0.4, 6.0)])
def test_many_atoms_per_wave(vtx, n, dims, h, scale):
    """Grids on both sides of 100 points per atom, below which a wave takes
    several atoms: remainders of the wave's atoms, boxes of one cell and of
    many, atoms beside the grid, and ones that mark nothing (no radius, no
    finite position) between them."""
    pos, rad = atoms(n, n, np.array(dims) * h * 1.5)
    pos -= np.float32(0.25) * np.array(dims, np.float32) * np.float32(h)
    rad *= np.float32(scale)
    origin = (0.1, -0.2, 0.05)
    ref = oses.ses_field(pos, rad, 0.6, origin, h, dims)
    k = n // 3
    pos_all = np.insert(pos, [0, k, k, n], [[np.nan, 0, 0], [1, np.inf, 1], [2, 2, 2], [3, 3, -np.inf]], axis=0).astype(np.float32)
    rad_all = np.insert(rad, [0, k, k, n], [2.0, 2.0, -1.0, 2.0]).astype(np.float32)
    for p, r in ((pos, rad), (pos_all, rad_all)):
        f, tri, count = run_ses(vtx, p, r, 0.6, np.asarray(origin, np.float32), np.float32(h), dims)
        assert np.array_equal(f, ref["f"])
        assert count == oses.marching_cubes(ref["f"], origin, h)["vertices"].shape[0]
    print("atoms", n, "points per atom", np.prod(dims) / n, "inside", int(np.count_nonzero(~ref["exterior"])), flush=True)


@pytest.mark.parametrize("window", [13, 32, 33, 50])
@pytest.mark.parametrize("dims", [(2, 3, 2), (5, 4, 3), (63, 4, 3), (64, 3, 4), (65, 2, 2), (255, 4, 3), (256, 3, 3), (257, 3, 4), (515, 3, 2)])
def test_rows_through_memory(vtx, window, dims):
    """The x pass of windows too large for a brick in LDS: rows around the
    sizes of its cells, words and blocks, with exterior points at every
    distance up to the window and past it."""
    h = 0.25
    probe = float(np.float32(h)) * (window - 2.5)
    rng = np.random.default_rng(window + dims[0])
    centre, reach, x = [], [], rng.uniform(-5.0, 3.0)
    while x < dims[0]:   # spheres along the row with gaps of a point or two between them
        r = rng.uniform(2.0, 1.5 * window)
        centre.append([x + r, (dims[1] - 1) / 2, (dims[2] - 1) / 2])
        reach.append(r)
        x += 2.0 * r + rng.uniform(0.3, 2.5)
    pos, rad = np.array(centre, np.float32) * np.float32(h), np.array(reach, np.float32) * np.float32(h) - np.float32(probe)
    check(vtx, pos, rad, probe, (0.0, 0.0, 0.0), h, dims)
