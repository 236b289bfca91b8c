"""The o-bin sums in each place their exponents can lie: a line each (up to
4096 o-bins), packed (more), or in the sums' own lines (a call without
allocations whose scratch is short).  The sums are exact, so a handle's and the
allocation-free call's moments are the same bits; the counts are the oracle's."""
import numpy as np
import pytest

from paper_1210_8084_amd import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

R, P = W.REFLECT, W.PERIODIC


@pytest.mark.parametrize("nobin", [(1, 1, 1), (16, 16, 16), (17, 241, 1), (80, 80, 62)], ids=str)
def test_exponents_apart_packed_and_shared(oracle, nobin):
    from paper_1210_8084_amd import tpkmc as T
    w = W.random_box(n=20_011, seed=9, ncell=(10, 9, 8), bc=(R, P, P), d_over_w=0.7, dt_over=0.6, nobin=nobin)
    print(f"o-bins {nobin}", flush=True)
    nob = T.nobins(w.grid)
    eng = T.Engine(max_particles=w.n, max_cells=T.ncells(w.grid) + 1, max_obins=nob + 5000, precision=T.FP64)
    moments = []
    for noalloc in (False, True):
        dst, out = T.to_device(w.state, T.FP64), T.make_outputs(1, nob)
        if noalloc:
            T.step_noalloc(dst, w.grid, w.params, out, precision=T.FP64)
        else:
            eng.step(dst, w.grid, w.params, out)
        torch.cuda.synchronize()
        moments.append(out.host()["moments"])
    eng.close()
    assert np.array_equal(moments[0], moments[1])
    ref = oracle.step(W.copy_state(w.state), w.grid, w.params)["moments"]
    assert np.array_equal(moments[0][:, 0], ref[:, 0]) and np.array_equal(moments[0][:, 10], ref[:, 10])
