"""Grids with one edge longer than the plane passes' lines and 64 x 64 points
across it: their 64-point lines have a path of their own.  Against the oracle's
FFT, 1e-12 (FP64) and 2e-6 (FP32) of the largest potential."""
import numpy as np
import pytest

import gw_inputs as gi
from oracle import poisson as PO

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

H = 0.4


@pytest.mark.parametrize("grid", [(162, 64, 64), (64, 162, 64), (64, 64, 162), (64, 256, 64)],
                         ids=lambda g: "x".join(map(str, g)))
def test_long_edge(grid):
    import paper_2310_20103_amd as G
    nr = int(np.prod(grid))
    print("[case] long edge", grid, flush=True)
    f = gi.random_fields(3, nr, seed=43)
    ref = PO.poisson(f, grid, H)
    with G.Context(f, [-5.0, 1.0, 2.0], 1, grid, tuple(H * n for n in grid), poly_lo=0.01,
                   poly_hi=1.0) as ctx:
        for prec, dt, tol in (("fp64", torch.float64, 1e-12), ("mixed", torch.float32, 2e-6)):
            got = ctx.poisson(torch.tensor(f, dtype=dt, device="cuda"), prec)
            err = np.max(np.abs(got.double().cpu().numpy() - ref)) / np.max(np.abs(ref))
            assert err <= tol, (prec, err)
