"""FP64 pair-density GEMMs in every form that their launch rules can take: one to
eight row blocks of 16 vectors, one or two M tiles, one or two column blocks per
wave, K steps shared by 1, 2 or 4 waves, conduction orbitals in whole K steps and
remainders.  test_host_runtime.py checks that CASES reach them.

pair_density and potential_product run one GEMM each.  Tolerance 1e-11 of the
largest element, the bar of the other FP64 product tests: sums of N_r <= 73,728
or N_vc <= 2,310 rounded products, whose rounding grows like the root of their
number (n u alone is 8e-12)."""
import numpy as np
import pytest

import gw_inputs as gi
from oracle import casida as CA

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

# grid, occupied, empty, split of the second GEMM (0: automatic), vectors
CASES = [
    ((48, 48, 32), 3, 37, 0, (1, 17, 65, 113, 128)),
    ((32, 32, 32), 13, 61, 0, (1, 17, 40, 128)),
    ((24, 24, 24), 7, 60, 0, (1, 33, 100)),
    ((24, 24, 18), 33, 70, 32, (1, 20, 90, 128)),
    ((24, 24, 18), 33, 70, 0, (20, 50, 75)),
    ((48, 48, 32), 1, 9, 0, (5, 80)),
]


@pytest.mark.parametrize("grid,nv,nc,split,counts", CASES,
                         ids=lambda a: "x".join(map(str, a)) if isinstance(a, tuple) else str(a))
def test_halves(grid, nv, nc, split, counts):
    import paper_2310_20103_amd as G
    wl = gi.workload("grid24_v8c32", name="pair_variants", seed=700 + nv, grid=grid, box=9.0,
                     n_occ=nv, n_emp=nc, n_qp_occ=1, n_qp_emp=1)
    phi = gi.random_fields(nv + nc, wl.n_r, seed=51)
    e = np.concatenate([np.linspace(-9, -5, nv), np.linspace(1, 9, nc)])
    sd = np.sqrt(((e[nv:][None] - e[:nv, None]) / 27.211386245988).ravel())
    pairs = CA.pair_densities(phi, nv)
    dv = 1.0
    box = tuple(float(n) for n in grid)  # dV = 1
    with G.Context(phi, e, nv, grid, box, poly_lo=0.01, poly_hi=1.0) as ctx:
        ctx.set_option(G.KEY_GEMM_SPLITK, split)
        for n in counts:
            print("[case] halves", grid, nv, nc, split, n, flush=True)
            x = gi.random_pair_vectors(n, nv * nc, seed=52)
            rho = ctx.pair_density(torch.tensor(x, device="cuda")).cpu().numpy()
            ref = (sd * x) @ pairs
            assert np.max(np.abs(rho - ref)) <= 1e-11 * np.max(np.abs(ref)), n
            v = gi.random_fields(n, wl.n_r, seed=53)
            y = ctx.potential_product(torch.tensor(v, device="cuda")).cpu().numpy()
            ref = dv * (v @ pairs.T)
            assert np.max(np.abs(y - ref)) <= 1e-11 * np.max(np.abs(ref)), n


# Lanczos slots: 160 are two M tiles of 80 vectors, 256 two of 128
SLOTS = [((12, 12, 8), 7, 33, 160), ((24, 24, 24), 7, 60, 256)]


@pytest.mark.parametrize("grid,nv,nc,slots", SLOTS,
                         ids=lambda a: "x".join(map(str, a)) if isinstance(a, tuple) else str(a))
def test_two_row_tiles(grid, nv, nc, slots):
    """A Lanczos block of more than 128 slots against blocks of 64, four steps.
    1e-10 relative: the recurrence multiplies the rounding of a product (1e-14)
    by the inverse of its b_k, here above 1e-3 of the spectrum's width."""
    import paper_2310_20103_amd as G
    wl = gi.workload("grid24_v8c32", name="row_tiles", seed=720 + nv, grid=grid, box=6.0, n_occ=nv,
                     n_emp=nc, n_qp_occ=1, n_qp_emp=1)
    s = gi.make_system(wl)
    n = np.arange(slots) % (nv + nc)
    m = (np.arange(slots) // (nv + nc)) + nv - 2
    print("[case] row tiles", grid, slots, flush=True)
    out = []
    for block in (slots, 64):
        with G.Context(s.phi, s.energies_ev, nv, grid, tuple(k * wl.h for k in grid), poly_lo=0.01,
                       poly_hi=4.0, block=block) as ctx:
            out.append(ctx.lanczos_pairs(m, n, np.full(slots, 4)))
    for a, b in zip(*out):
        assert np.max(np.abs(np.asarray(a) - np.asarray(b))) <= 1e-10 * np.max(np.abs(np.asarray(b)))
