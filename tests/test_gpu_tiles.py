"""The tile search where it can go wrong: tiles that are not full, c-bins
that hold many tiles and are cut into sort cells, periodic axes of one to
five c-bins (whose images are visited one by one up to three), particles
outside the box or several c-bins per step fast, and exact ties of the
ranking value, which the FP64 keys cannot tell apart and the library settles
apart.  FP64 against the oracle, bit for bit."""
import numpy as np
import pytest

from paper_1210_8084_amd import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

R, P, A = W.REFLECT, W.PERIODIC, W.ABSORB


@pytest.fixture(scope="module")
def T():
    from paper_1210_8084_amd import tpkmc
    assert torch.cuda.is_available(), "GPU test without a visible GPU"
    tpkmc.lib()
    return tpkmc


def check(T, oracle, state, grid, params, steps=2, tune=False):
    print(f"n={len(state['x'])} grid={grid['ncell']} bc={grid['bc']}", flush=True)
    n = len(state["x"])
    eng = T.Engine(max_particles=max(n, 1), max_cells=T.ncells(grid) + 1, max_obins=T.nobins(grid), precision=T.FP64)
    dst, want = T.to_device(state, T.FP64), W.copy_state(state)
    if tune:
        eng.autotune(dst, [(0, n, grid, params)])
    out = T.make_outputs(1, T.nobins(grid), pair_cap=n // 2 + 1)
    found = 0
    for s in range(steps):
        p = dict(params, step=s)
        eng.step(dst, grid, p, out, flags=T.EMIT_PAIRS)
        torch.cuda.synchronize()
        ref = oracle.step(want, grid, p)
        got, o = T.to_host(dst), out.host()
        for k in ("x", "y", "z", "vx", "vy", "vz"):
            assert np.array_equal(got[k], want[k]), f"step {s}: {k} differs at {np.flatnonzero(got[k] != want[k])[:5]}"
        assert sorted(map(tuple, o["pairs"].tolist())) == sorted(map(tuple, ref["pairs"].tolist()))
        keep = [k for k in range(8) if not (tune and k in (T.CNT["tests"], T.CNT["cand"]))]
        assert o["counters"][0][keep].tolist() == ref["counters"][keep].tolist()
        found += len(ref["pairs"])
    eng.close()
    return found


@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 127, 129, 257, 1025])
@pytest.mark.parametrize("bc", [(R, P, P), (P, P, P)], ids=["rpp", "ppp"])
def test_tile_edges(T, oracle, n, bc):
    w = W.random_box(n=n, seed=n, ncell=(5, 4, 3), bc=bc, d_over_w=0.7, dt_over=0.6, nobin=(2, 2, 1))
    check(T, oracle, w.state, w.grid, w.params)


# Periodic axes of 1 to 5 c-bins, with c-bins of a few records (one sort cell
# each) and of hundreds (many), small and large D and steps.
@pytest.mark.parametrize("n", [300, 6001])
@pytest.mark.parametrize("ncell", [(1, 1, 1), (2, 3, 4), (4, 4, 4), (5, 1, 2), (3, 5, 1), (9, 2, 5)])
@pytest.mark.parametrize("d_over_w,dt_over", [(0.05, 0.05), (0.6, 0.4), (0.3, 3.0)])
def test_few_periodic_cbins(T, oracle, n, ncell, d_over_w, dt_over):
    w = W.random_box(n=n, seed=17, ncell=ncell, bc=(P, P, P), d_over_w=d_over_w, dt_over=dt_over, nobin=(2, 2, 1))
    check(T, oracle, w.state, w.grid, w.params)


@pytest.mark.parametrize("tune", [False, True], ids=["configured", "tuned"])
def test_thin_tube_in_sort_cells(T, oracle, tune):
    """The Sod tube: hundreds of records per c-bin, one c-bin across."""
    w = W.sod(n=30_001, ncell=40, nobin=8)
    assert check(T, oracle, w.state, w.grid, w.params, tune=tune) > 1000


def test_plane_in_sort_cells(T, oracle):
    w = W.sod2d(n=20_003, ncell=30, nobin=6)
    assert check(T, oracle, w.state, w.grid, w.params) > 1000


@pytest.mark.parametrize("by_time", [False, True], ids=["closest", "first contact"])
def test_particles_outside_and_fast(T, oracle, by_time):
    """Positions up to a fifth of the box outside it, and a tenth of the
    particles ten times faster: they take part unfiltered."""
    w = W.random_box(n=4001, seed=5, ncell=(3, 2, 6), bc=(P, P, R), d_over_w=0.4, dt_over=0.5, nobin=(2, 2, 1))
    st = w.state
    rng = np.random.default_rng(6)
    for k, L in zip(("x", "y", "z"), (1.0, 0.8, 0.6)):
        st[k] = st[k] * 1.4 - 0.2 * L
        st["v" + k][::10] *= 10.0
    st["vx"][rng.integers(0, 4001, 5)] *= 1e6
    check(T, oracle, st, w.grid, dict(w.params, rank_time=by_time))


@pytest.mark.parametrize("by_time", [False, True], ids=["closest", "first contact"])
@pytest.mark.parametrize("tune", [False, True], ids=["configured", "tuned"])
def test_exact_ties_go_to_the_lower_id(T, oracle, by_time, tune):
    """A lattice of particles at rest crossed by particles along +x that pass
    four rows at exactly the same distance: every mover has candidates whose
    d_min^2 (and contact time) are equal to the last bit."""
    k = np.arange(8) * 1.0
    x, y, z = (c.ravel() for c in np.meshgrid(k, k, k, indexing="ij"))
    mx, my, mz = (c.ravel() for c in np.meshgrid(k[:-1] + 0.25, k[:-1] + 0.5, k[:-1] + 0.5, indexing="ij"))
    zero = np.zeros(len(x))
    st = W.make_state(np.r_[x, mx], np.r_[y, my], np.r_[z, mz], np.r_[zero, np.ones(len(mx))], np.zeros(len(x) + len(mx)),
                      np.zeros(len(x) + len(mx)))
    st = W.shuffle_state(st, seed=3)
    st["id"] = np.random.default_rng(4).permutation(len(st["x"])).astype(np.uint32)
    g = W.grid((-1, -1, -1), (9, 9, 9), (4, 4, 4), (R, R, R), (2, 2, 2))
    p = dict(W.params(sigma=np.pi * 0.75 ** 2, dt=1.0, seed=2), rank_time=by_time)
    # The lattice of the first step is what ties; the second is generic.
    assert check(T, oracle, st, g, p, steps=2, tune=tune) > 10
