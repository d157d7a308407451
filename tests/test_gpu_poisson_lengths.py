"""The Hartree solve on every line length of the plane passes (each edge in
turn a short or a long line, along every axis), planes at the LDS limit, grids
they do not cover, and odd numbers of fields, against the oracle's FFT.

Tolerances as for the other Poisson tests: 1e-12 (FP64) and 2e-6 (FP32) of the
largest potential; the transforms are a few roundings per point deep."""
import numpy as np
import pytest

import gw_inputs as gi
from oracle import poisson as PO

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

H = 0.4


@pytest.mark.parametrize("grid", [
    (2, 3, 4), (4, 2, 6), (6, 8, 9), (9, 12, 8), (16, 18, 12), (18, 27, 24), (24, 16, 32),
    (32, 24, 27), (36, 54, 48), (48, 36, 64), (54, 48, 36), (27, 64, 54), (64, 72, 81),
    (72, 81, 96), (81, 96, 72), (96, 108, 16), (108, 12, 128), (128, 16, 108), (144, 9, 144),
    (12, 144, 6), (8, 128, 128), (162, 8, 6), (8, 162, 12), (6, 16, 192), (256, 4, 8),
], ids=lambda g: "x".join(map(str, g)))
def test_poisson_grid(grid):
    import paper_2310_20103_amd as G
    nr = int(np.prod(grid))
    print("[case] poisson", grid, flush=True)
    phi = gi.random_fields(3, nr, seed=40)
    with G.Context(phi, [-5.0, 1.0, 2.0], 1, grid, tuple(H * n for n in grid), poly_lo=0.01,
                   poly_hi=1.0) as ctx:
        for n_fields in (1, 3):
            f = gi.random_fields(n_fields, nr, seed=41)
            ref = PO.poisson(f, grid, H)
            for prec, dt, tol in (("fp64", torch.float64, 1e-12), ("mixed", torch.float32, 2e-6)):
                got = ctx.poisson(torch.tensor(f, dtype=dt, device="cuda"), prec)
                err = np.max(np.abs(got.double().cpu().numpy() - ref)) / np.max(np.abs(ref))
                assert err <= tol, (n_fields, prec, err)
