"""Edges of the dispatch on sizes: FP64 row GEMMs with half-filled tiles and more
than 32 splits, coefficients staged in LDS or in global memory, results large
enough for pinned staging, buffers kept between calls of different shapes."""
import numpy as np
import pytest

import gw_inputs as gi
from oracle import casida as CA

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def make(name, grid, nv, nc, **kw):
    import paper_2310_20103_amd as G
    wl = gi.workload("grid24_v8c32", name=name, seed=600 + nv, grid=grid, box=6.0, n_occ=nv,
                     n_emp=nc, n_qp_occ=1, n_qp_emp=1)
    s = gi.make_system(wl)
    return wl, s, lambda: G.Context(s.phi, s.energies_ev, nv, grid,
                                    tuple(n * wl.h for n in grid), **kw)


@pytest.fixture(scope="module")
def rows():
    wl, s, ctx = make("row_gemm", (24, 16, 12), 64, 192)
    with ctx() as c:
        yield wl, s, CA.pair_densities(s.phi, 64), c


@pytest.mark.parametrize("split", [0, 1, 5])
@pytest.mark.parametrize("n_vec", [1, 5, 33])
def test_row_gemms(rows, n_vec, split):
    """64 + 192 orbitals: an odd batch half-fills the last row tile of 128 and
    N_cp the last column tile.  1e-11 of the largest element: sums of 4,608
    rounded products, n u = 5e-13."""
    import paper_2310_20103_amd as G
    wl, s, pairs, c = rows
    print("[case] row GEMM", n_vec, split, flush=True)
    v = gi.random_fields(n_vec, wl.n_r, seed=42)
    ref = wl.h ** 3 * (v @ pairs.T)
    c.set_option(G.KEY_GEMM_SPLITK, split)
    got = c.potential_product(torch.tensor(v, device="cuda")).cpu().numpy()
    c.set_option(G.KEY_GEMM_SPLITK, 0)
    assert np.max(np.abs(got - ref)) <= 1e-11 * np.max(np.abs(ref))


def coefficients(n_pairs, length, ld):
    rng = np.random.default_rng(9)
    a, b = np.zeros((n_pairs, ld)), np.zeros((n_pairs, ld))
    a[:, :length] = 1.0 + 0.1 * rng.random((n_pairs, length))
    b[:, :length - 1] = 0.2 * rng.random((n_pairs, length - 1))
    return a, b, rng.random(n_pairs) + 0.5, np.full(n_pairs, length)


@pytest.mark.parametrize("quadrature", [False, True])
@pytest.mark.parametrize("length", [1, 2, 65])
def test_leading_dimension(length, quadrature):
    """The same coefficients with rows as long as needed, of 2,731 (the first
    past 64 KB of three rows in LDS) and of 4,000 (the longest).  1e-10: the
    eigensolver's rounding is a small multiple of 65 u."""
    wl, s, ctx = make("leading", (8, 8, 12), 3, 5)
    print("[case] leading dimension", length, quadrature, flush=True)
    om = np.linspace(-10, 10, 33)
    with ctx() as c:
        if quadrature:
            c.set_quadrature(True)
        out = [c.sigma_from_coeffs([0, 4, 7], *coefficients(3, length, ld), om, 0.3)
               for ld in (length, 2731, 4000)]
    assert np.all(np.isfinite(out[0]))
    for o in out[1:]:
        assert np.max(np.abs(o - out[0])) <= 1e-10 * np.max(np.abs(out[0]))


@pytest.mark.parametrize("n_omega", [20000, 54321])
def test_large_result(n_omega):
    """Whole chunks or a partial last one, against calls too small to be staged."""
    wl, s, ctx = make("leading", (8, 8, 12), 3, 5)
    print("[case] large result", n_omega, flush=True)
    om = np.linspace(-10, 10, n_omega)
    n = np.arange(16) % 8
    a, b, n2, ln = coefficients(16, 12, 12)
    with ctx() as c:
        for _ in range(2):
            whole = c.sigma_from_coeffs(n, a, b, n2, ln, om, 0.3)
        for i in range(16):
            one = c.sigma_from_coeffs(n[i:i + 1], a[i:i + 1], b[i:i + 1], n2[i:i + 1],
                                      ln[i:i + 1], om, 0.3)
            assert np.array_equal(whole[i:i + 1], one)


def test_gradient_buffers_reused():
    """Calls of other lengths, ranges and frequency counts in between change
    nothing: bitwise the first result and a fresh context's."""
    wl, s, ctx = make("leading", (8, 8, 12), 3, 5, block=4)
    print("[case] gradient buffers", flush=True)
    qp = s.qp_states

    def grad(c, length, nw, n_range=None):
        g = np.cos(np.arange(len(qp) * nw)).reshape(len(qp), nw) * (1 + 0.5j)
        sig, ge, go = c.sigma_c_vjp(qp, np.linspace(-10, 10, nw), 0.3, length, g,
                                    n_range=n_range)
        return sig, ge, go.cpu().numpy()

    with ctx() as c:
        first = grad(c, 6, 9)
        small = grad(c, 3, 2, (1, 4))
        grad(c, 9, 40)
        again = grad(c, 6, 9)
        small2 = grad(c, 3, 2, (1, 4))
    with ctx() as c:
        fresh = grad(c, 6, 9)
    for x, y, z in zip(first, again, fresh):
        assert np.array_equal(x, y) and np.array_equal(x, z)
    for x, y in zip(small, small2):
        assert np.array_equal(x, y)
