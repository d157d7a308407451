"""FP64 K product on the pair-density GEMMs: batches and orbital counts at the
edges of their tiles (16 vectors, 128 vectors per M tile, 16 pairs per K step,
64 or 128 pairs per N tile), against the oracle's dense C and C^1/2 start
vectors.

Tolerance: 1e-11 relative to the largest element, the bar of every FP64 step
(sums of at most N_r = 1,152 and N_vc = 2,310 rounded products: n u ~ 3e-13)."""
import numpy as np
import pytest

import gw_inputs as gi
import oracle

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

GRID = (12, 12, 8)


@pytest.fixture(scope="module", params=[(3, 5), (7, 33), (33, 70)], ids=["15", "231", "2310"])
def case(request):
    import paper_2310_20103_amd as G
    nv, nc = request.param
    wl = gi.workload("grid24_v8c32", name="pair_gemm", seed=300 + nv, grid=GRID, box=6.0,
                     n_occ=nv, n_emp=nc, n_qp_occ=1, n_qp_emp=1)
    s = gi.make_system(wl)
    pr = oracle.Problem(s.phi, s.energies_ev, nv, GRID, wl.h)
    lo, hi = oracle.default_interval(pr)
    ctx = G.Context(s.phi, s.energies_ev, nv, GRID, tuple(n * wl.h for n in GRID), poly_lo=lo,
                    poly_hi=hi)
    yield wl, s, pr, ctx
    ctx.close()


def rel(a, b):
    return float(np.max(np.abs(a - b)) / np.max(np.abs(b)))


@pytest.mark.parametrize("split", [0, 1, 5])
@pytest.mark.parametrize("n_vec", [1, 16, 17, 64])
def test_product(case, n_vec, split):
    import paper_2310_20103_amd as G
    wl, s, pr, ctx = case
    print("[case] product", wl.n_vc, n_vec, split, flush=True)
    x = gi.random_pair_vectors(n_vec, wl.n_vc, seed=31)
    ref = x @ pr.C.T
    ctx.set_option(G.KEY_GEMM_SPLITK, split)
    got = ctx.apply_c(torch.tensor(x, device="cuda")).cpu().numpy()
    ctx.set_option(G.KEY_GEMM_SPLITK, 0)
    assert rel(got, ref) <= 1e-11
    d2 = pr.delta ** 2
    assert rel(got - d2 * x, ref - d2 * x) <= 1e-9  # the coupling part alone (a few 1e-3 of C x)


@pytest.mark.parametrize("n_vec", [113, 129, 130])
def test_density_and_projection(case, n_vec):
    """Both halves alone, in batches of 128 (8 full row blocks) and of 1 or 2."""
    from oracle import casida as CA
    wl, s, pr, ctx = case
    print("[case] halves", wl.n_vc, n_vec, flush=True)
    pairs = CA.pair_densities(s.phi, wl.n_occ)
    x = gi.random_pair_vectors(n_vec, wl.n_vc, seed=32)
    rho = ctx.pair_density(torch.tensor(x, device="cuda")).cpu().numpy()
    assert rel(rho, (np.sqrt(pr.delta) * x) @ pairs) <= 1e-11
    v = gi.random_fields(n_vec, wl.n_r, seed=33)
    y = ctx.potential_product(torch.tensor(v, device="cuda")).cpu().numpy()
    assert rel(y, wl.h ** 3 * (v @ pairs.T)) <= 1e-11
