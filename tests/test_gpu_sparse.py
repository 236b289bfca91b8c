"""The lane walks of the partner search: FP64 states of few particles per c-bin
or per row of c-bins (a record a lane, its rows shared between work-groups in
small calls), and FP32 states that are sparse on average and dense in places
or thin (staged through LDS, several chunks of 128 records a row).  FP64
against the oracle bit for bit, FP32 pair by pair."""
import numpy as np
import pytest

from paper_1210_8084_amd import workloads as W
from test_gpu_fp32_parity import SHAPES, check_against_oracle
from test_gpu_tiles import T, check  # noqa: F401  (T: fixture)

pytestmark = pytest.mark.gpu

R, P, A = W.REFLECT, W.PERIODIC, W.ABSORB


@pytest.mark.parametrize("n", [1, 2, 64, 255, 257, 2000])
@pytest.mark.parametrize("ncell,bc", [((16, 12, 9), (R, P, P)), ((1, 40, 30), (P, P, P)), ((2, 25, 20), (P, R, P)),
                                      ((3, 3, 60), (P, P, P)), ((4, 4, 40), (P, P, R)), ((1, 1, 500), (R, P, P))],
                         ids=str)
def test_fp64_sparse_boxes(T, oracle, n, ncell, bc):  # noqa: F811
    w = W.random_box(n=n, seed=n + ncell[0], ncell=ncell, bc=bc, hi=(0.7, 1.0, 0.8), d_over_w=0.9, dt_over=0.7,
                     nobin=(2, 2, 1))
    check(T, oracle, w.state, w.grid, w.params)


@pytest.mark.parametrize("n", [29_000, 130_001, 290_000])  # nine, two and one work-group a record's rows
def test_fp64_sparse_box_of_many(T, oracle, n):  # noqa: F811
    w = W.random_box(n=n, seed=2, ncell=(66, 66, 66), bc=(R, P, A), hi=(1, 1, 1), d_over_w=0.6, dt_over=0.4,
                     nobin=(2, 2, 1))
    assert check(T, oracle, w.state, w.grid, w.params, steps=1) > 500


@pytest.mark.parametrize("by_time", [False, True], ids=["closest", "first contact"])
def test_fp64_sparse_outside_fast_and_planar(T, oracle, by_time):  # noqa: F811
    w = W.random_box(n=4001, seed=5, ncell=(20, 2, 40), bc=(P, P, R), d_over_w=0.8, dt_over=0.5, nobin=(2, 2, 1))
    for k, L in zip(("x", "y", "z"), (1.0, 0.8, 0.6)):
        w.state[k] = w.state[k] * 1.4 - 0.2 * L
        w.state["v" + k][::10] *= 10.0
    check(T, oracle, w.state, w.grid, dict(w.params, rank_time=by_time))
    w = W.random_plane(n=3001, seed=6, ncell=(40, 30), bc=(R, P), nobin=(2, 2))
    check(T, oracle, w.state, w.grid, dict(w.params, rank_time=by_time))


@pytest.mark.parametrize("by_time", [False, True], ids=["closest", "first contact"])
@pytest.mark.parametrize("tune", [False, True], ids=["configured", "tuned"])
def test_fp64_sparse_exact_ties(T, oracle, by_time, tune):  # noqa: F811
    """The lattice of test_gpu_tiles on c-bins of one particle or two."""
    k = np.arange(8) * 1.0
    x, y, z = (c.ravel() for c in np.meshgrid(k, k, k, indexing="ij"))
    mx, my, mz = (c.ravel() for c in np.meshgrid(k[:-1] + 0.25, k[:-1] + 0.5, k[:-1] + 0.5, indexing="ij"))
    zero = np.zeros(len(x) + len(mx))
    st = W.make_state(np.r_[x, mx], np.r_[y, my], np.r_[z, mz], np.r_[zero[:len(x)], np.ones(len(mx))], zero, zero)
    st = W.shuffle_state(st, seed=3)
    st["id"] = np.random.default_rng(4).permutation(len(st["x"])).astype(np.uint32)
    g = W.grid((-1, -1, -1), (9, 9, 9), (8, 8, 8), (R, R, R), (2, 2, 2))
    p = dict(W.params(sigma=np.pi * 0.75 ** 2, dt=1.0, seed=2), rank_time=by_time)
    assert check(T, oracle, st, g, p, steps=2, tune=tune) > 10


def test_fp64_search_mix_and_batch_of_both(T, oracle):  # noqa: F811
    """A sparse and a dense instance in one call: each takes its own search."""
    ws = [W.random_box(n=3000, seed=7, ncell=(16, 12, 9), bc=(R, P, P), d_over_w=0.7, dt_over=0.5, nobin=(2, 2, 1)),
          W.random_box(n=9000, seed=8, ncell=(3, 4, 2), bc=(R, P, P), d_over_w=0.2, dt_over=0.2, nobin=(2, 2, 1))]
    st = {k: np.concatenate([w.state[k] for w in ws]) for k in ws[0].state}
    specs, off = [], 0
    for k, w in enumerate(ws):
        specs.append((off, w.n, w.grid, dict(w.params, instance=k)))
        off += w.n
    eng = T.Engine(max_particles=off, max_cells=sum(T.ncells(w.grid) + 1 for w in ws), max_obins=8, precision=T.FP64,
                   max_instances=2)
    dst, out = T.to_device(st, T.FP64), T.make_outputs(2, 8)
    mix = eng.search_mix(dst, specs)
    eng.step_batched(dst, specs, out)
    got, o = T.to_host(dst), out.host()
    eng.close()
    tests = 0
    for k, (w, (o0, n, g, p)) in enumerate(zip(ws, specs)):
        want = W.copy_state(w.state)
        ref = oracle.step(want, g, p)
        for a in ("x", "y", "z", "vx", "vy", "vz"):
            assert np.array_equal(got[a][o0:o0 + n], want[a]), (k, a)
        assert o["counters"][k].tolist() == ref["counters"].tolist()
        tests += int(ref["counters"][T.CNT["tests"]])
    assert mix[0] == tests


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: f"{s[0]}x{s[1]}")
@pytest.mark.parametrize("bc", [(R, P, P), (P, P, P)], ids=["reflect", "periodic"])
def test_fp32_clumps_in_a_sparse_box(T, oracle, shape, bc):  # noqa: F811
    """Five particles per c-bin on average, half of them in 1% of the box: row
    unions of several hundred records, walked in chunks."""
    w = W.random_box(n=20000, seed=4, ncell=(20, 16, 12), bc=bc, d_over_w=0.35, dt_over=0.3)
    for k, L in zip(("x", "y", "z"), (1.0, 0.8, 0.6)):
        w.state[k][::2] = 0.95 * L + (w.state[k][::2] - 0.5 * L) * 0.22
        w.state[k] %= L
    check_against_oracle(T, oracle, w, shape=shape)


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: f"{s[0]}x{s[1]}")
@pytest.mark.parametrize("ncell", [(8000, 1, 1), (3000, 1, 1)], ids=str)
def test_fp32_long_tube(T, oracle, shape, ncell):  # noqa: F811
    """A tube as thin as a c-bin is long, periodic across, 15 and 40 a c-bin:
    staged, as the tiles would visit nine images of it."""
    w = W.random_box(n=120_000, seed=9, ncell=ncell, bc=(R, P, P), hi=(1.0, 1.0 / ncell[0], 1.0 / ncell[0]),
                     d_over_w=0.3, dt_over=0.2, nobin=(4, 1, 1))
    check_against_oracle(T, oracle, w, shape=shape)
