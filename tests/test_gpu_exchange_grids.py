"""Sigma^ex on grids of the frequency-space route (short, long and mixed line
lengths) and of the grid route (an edge of 162), for even and odd N_v and more
products than one chunk of 64, against the oracle.

Tolerance 1e-11 relative, the bar of the other exchange tests (a sum of positive
terms, each a few roundings from an FFT of at most 20,736 points)."""
import numpy as np
import pytest

import gw_inputs as gi
from oracle import exchange as EX

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("grid", [(12, 16, 18), (8, 27, 96), (144, 12, 12), (162, 8, 6)],
                         ids=lambda g: "x".join(map(str, g)))
@pytest.mark.parametrize("nv", [1, 4, 23])
def test_exchange_grid(grid, nv):
    import paper_2310_20103_amd as G
    print("[case] exchange", grid, nv, flush=True)
    wl = gi.workload("grid24_v8c32", name="xgrid", seed=500 + nv, grid=grid, box=0.4 * grid[0],
                     n_occ=nv, n_emp=4, n_qp_occ=1, n_qp_emp=1)
    s = gi.make_system(wl)
    states = list(range(nv)) + [nv + 3, nv]
    states = states[-6:]
    with G.Context(s.phi, s.energies_ev, nv, grid, tuple(0.4 * n for n in grid), poly_lo=0.01,
                   poly_hi=1.0) as ctx:
        got = ctx.sigma_x(states)
    ref = np.array([EX.sigma_x(s.phi, nv, m, grid, wl.h) for m in states])
    assert np.max(np.abs(got - ref) / np.abs(ref)) <= 1e-11
