"""What must not cost the partner search a multiple: the same gas in other
places, units of the time step or orders, one search phase against another on
the same card (the results are other tests' matter)."""
import math

import numpy as np
import pytest

from paper_1210_8084_amd import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

R, P = W.REFLECT, W.PERIODIC


@pytest.fixture(scope="module")
def T():
    from paper_1210_8084_amd import tpkmc
    assert torch.cuda.is_available(), "GPU test without a visible GPU"
    tpkmc.lib()
    return tpkmc


def search_us(T, state, grid, params, precision, reps=6, also=None):
    """Shortest search phase (with the phase `also`) of a step on this state,
    in microseconds."""
    n = len(state["x"])
    eng = T.Engine(max_particles=n, max_cells=T.ncells(grid) + 1, max_obins=T.nobins(grid), precision=precision)
    first = T.to_device(state, precision)
    out = T.make_outputs(1, T.nobins(grid))
    best = math.inf
    for k in range(reps):
        dst = {a: t.clone() for a, t in first.items()}
        eng.profile(k > 0)
        eng.step(dst, grid, params, out, flags=T.ALLOW_REORDER)
        torch.cuda.synchronize()
        if k:
            ms = eng.profile_read()
            best = min(best, 1e3 * (ms["search"][0] + (ms[also][0] if also else 0.0)))
    pairs = int(out.host()["counters"][0][T.CNT["pairs"]])
    eng.close()
    print(f"n={n} ncell={grid['ncell']} fp={precision}: search {best:.1f} us, {pairs} pairs", flush=True)
    return best


def test_a_gas_that_moves_half_a_cbin_is_filtered(T):
    """Four times the time step brings 1.5 times the search (more candidates);
    3.2 times where 1% of the records are taken unfiltered."""
    us = []
    for dt in (0.1, 0.4):
        w = W.random_box(n=500_000, seed=1, ncell=(32, 32, 32), bc=(R, P, P), hi=(1, 1, 1), dt_over=dt, nobin=(1, 1, 1))
        us.append(search_us(T, w.state, w.grid, w.params, T.FP32))
    assert us[1] < 2.3 * us[0]


@pytest.mark.parametrize("precision", ["FP64", "FP32"])
def test_a_plane_at_the_edge_of_its_box(T, precision):
    """The plane's place along z is the caller's choice."""
    us = []
    for z in (0.0, -0.5):
        w = W.random_plane(n=500_000, seed=1, ncell=(158, 158), bc=(R, P), hi=(1, 1), dt_over=0.1, nobin=(1, 1))
        w.state["z"][:] = z
        us.append(search_us(T, w.state, w.grid, w.params, getattr(T, precision)))
    assert us[1] < 1.25 * us[0]


def test_a_box_far_from_the_origin(T):
    us = []
    for lo in (0.0, 1000.0):
        w = W.random_box(n=500_000, seed=1, ncell=(32, 32, 32), bc=(R, R, R), lo=(lo,) * 3, hi=(lo + 1.0,) * 3,
                         dt_over=0.1, nobin=(1, 1, 1))
        us.append(search_us(T, w.state, w.grid, w.params, T.FP32))
    assert us[1] < 1.5 * us[0]


@pytest.mark.parametrize("precision", ["FP64", "FP32"])
@pytest.mark.parametrize("beyond", [0.0, 1e-4])
def test_a_particle_on_the_edge_of_a_periodic_box(T, precision, beyond):
    """One coordinate at (or a little beyond) the upper edge, as FP32 rounding
    brings it about; sort cells are skipped as without it."""
    w = W.sod(n=400_000, ncell=100, nobin=1)
    us = [search_us(T, w.state, w.grid, w.params, getattr(T, precision))]
    w.state["y"][7] = w.grid["hi"][1] + beyond
    us.append(search_us(T, w.state, w.grid, w.params, getattr(T, precision)))
    assert us[1] < 1.5 * us[0]


def test_fp64_thin_along_either_axis(T):
    """A tube of one c-bin across costs the same along x, where its c-bins
    follow one another in a row, and along y, where each is a row."""
    us = []
    for ncell, hi in (((100_000, 1, 1), (1.0, 0.02, 0.02)), ((1, 100_000, 1), (0.02, 1.0, 0.02))):
        w = W.random_box(n=300_000, seed=1, ncell=ncell, bc=(R, P, P), hi=hi, dt_over=0.1, nobin=(1, 1, 1))
        us.append(search_us(T, w.state, w.grid, w.params, T.FP64))
    assert us[1] < 3.0 * us[0]


@pytest.mark.parametrize("precision", ["FP64", "FP32"])
def test_tube_of_three_cbins_across(T, precision):
    """A tile of a tube of 3 by 3 c-bins has no more partners within reach than
    one of 4 by 4 of them, images or not."""
    us = []
    for m in (4, 3):
        nx = 3000 // (m * m)
        w = W.random_box(n=300_000, seed=1, ncell=(nx, m, m), bc=(R, P, P), hi=(1.0, m / nx, m / nx), dt_over=0.1,
                         nobin=(1, 1, 1))
        us.append(search_us(T, w.state, w.grid, w.params, getattr(T, precision)))
    assert us[1] < 1.1 * us[0]


def test_small_fp64_tube(T):
    """One row of 17 c-bins holds 2261 particles, which the waves of a walk by
    rows cannot share; the tiles, FP32's search of it, can.  Twice the cost for
    twice the bytes, and the settling of ties."""
    w = W.sod(n=2261, ncell=17, nobin=17)
    us = [search_us(T, w.state, w.grid, w.params, p) for p in (T.FP32, T.FP64)]
    assert us[1] < 2.0 * us[0] + 15.0


def test_fp64_cost_follows_the_particles(T):
    """1e5 particles on 256^3 c-bins, whose counts alone (the scatter's share
    of the pair tests) had cost more than the search."""
    us = []
    for nc in (46, 256):
        w = W.random_box(n=100_000, seed=1, ncell=(nc,) * 3, bc=(R, P, P), hi=(1, 1, 1), dt_over=0.1, nobin=(1, 1, 1))
        us.append(search_us(T, w.state, w.grid, w.params, T.FP64, also="scatter"))
    assert us[1] < 3.0 * us[0]


def test_fp64_ties_are_settled_by_the_whole_card(T):
    """Every record of the lattice meets several candidates at the same closest
    distance; the same lattice a little out of place has none to settle."""
    k = np.arange(100) + 0.5
    x, y, z = (c.ravel() * 0.01 for c in np.meshgrid(k, k, k, indexing="ij"))
    v = np.where((np.arange(100 ** 3) + np.repeat(np.arange(10_000), 100) + np.repeat(np.arange(100), 10_000)) % 2, 1.0, -1.0)
    g = W.grid((0, 0, 0), (1, 1, 1), (50, 50, 50), (R, R, R), (1, 1, 1))
    p = W.params(sigma=np.pi * 0.012 ** 2, dt=0.01)
    us = []
    for jitter in (1e-4, 0.0):
        d = np.random.default_rng(1).uniform(-jitter, jitter, (3, len(x)))
        us.append(search_us(T, W.make_state(x + d[0], y + d[1], z + d[2], v, 0.0 * v, 0.0 * v), g, p, T.FP64))
    assert us[1] < 7.0 * us[0]
