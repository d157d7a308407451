"""Quadrature of many pairs, whose tridiagonals do not fit in LDS at once,
against calls of a few pairs of the same coefficients, which do.

1e-10 of the largest value: the eigensolver's rounding is a small multiple of
200 u, and a value sums 200 poles at 0.3 eV from the axis."""
import numpy as np
import pytest

import gw_inputs as gi

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("n_pairs,length", [(10000, 200), (50000, 30), (600, 2700)])
def test_many_pairs(n_pairs, length):
    import paper_2310_20103_amd as G
    grid = (8, 8, 12)
    wl = gi.workload("grid24_v8c32", name="routes", seed=620, grid=grid, box=6.0, n_occ=3, n_emp=5,
                     n_qp_occ=1, n_qp_emp=1)
    s = gi.make_system(wl)
    print("[case] quadrature routes", n_pairs, length, flush=True)
    few = 8
    rng = np.random.default_rng(17)
    used = min(length, 200)
    a, b = np.zeros((few, length)), np.zeros((few, length))
    a[:, :used] = 1.0 + 0.1 * rng.random((few, used))
    b[:, :used - 1] = 0.2 * rng.random((few, used - 1))
    n2, ln, om = rng.random(few) + 0.5, np.full(few, used), np.linspace(-10, 10, 5)
    idx = np.arange(n_pairs) % few
    with G.Context(s.phi, s.energies_ev, 3, grid, tuple(n * wl.h for n in grid)) as c:
        c.set_quadrature(True)
        ref = c.sigma_from_coeffs(np.arange(few), a, b, n2, ln, om, 0.3)
        got = c.sigma_from_coeffs(idx, a[idx], b[idx], n2[idx], ln[idx], om, 0.3)
    assert np.max(np.abs(got - ref[idx])) <= 1e-10 * np.max(np.abs(ref))
