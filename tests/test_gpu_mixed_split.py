"""Mixed second GEMM: the tile and split that the time model chooses against the
forced tiles and splits, for batches on both sides of 32 (where up to 64 splits
are allowed) and ragged orbital counts.

All of them multiply the same FP16 operands and differ in the order of the FP32
sums alone, so the difference of two results is at most 2 N_r u sum_r |terms|
(u = 2^-24: the worst case of any order), and a lost split would be of the
order of the result."""
import numpy as np
import pytest

import gw_inputs as gi
from oracle import casida as CA

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

GRID = (24, 24, 18)


@pytest.fixture(scope="module", params=[(5, 130), (70, 9)], ids=["5x130", "70x9"])
def case(request):
    import paper_2310_20103_amd as G
    nv, nc = request.param
    wl = gi.workload("grid24_v8c32", name="mixed_split", seed=500 + nv, grid=GRID, box=7.0,
                     n_occ=nv, n_emp=nc, n_qp_occ=1, n_qp_emp=1)
    s = gi.make_system(wl)
    args = (s.phi, s.energies_ev, nv, GRID, tuple(n * wl.h for n in GRID))
    with G.Context(*args, precision="mixed") as ctx, \
            G.Context(*args, precision="mixed") as forced:
        yield wl, CA.pair_densities(s.phi, nv), ctx, forced


@pytest.mark.parametrize("n_vec", [1, 5, 31, 32, 40])
def test_model_against_forced(case, n_vec):
    import paper_2310_20103_amd as G
    wl, pairs, ctx, other = case
    print("[case] mixed split", wl.n_occ, n_vec, flush=True)
    v = gi.random_fields(n_vec, wl.n_r, seed=41)
    vd = torch.tensor(v, device="cuda")
    bound = 2 * wl.n_r * 2.0 ** -24 * wl.h ** 3 * (np.abs(v) @ np.abs(pairs).T)
    ref = wl.h ** 3 * (v @ pairs.T)
    got = ctx.potential_product(vd, precision="mixed").cpu().numpy()  # the model's choice
    # operands rounded to FP16 (three factors of 2^-11 each at most) and FP32 sums
    assert np.all(np.abs(got - ref) <= bound * (1 + 3 * 2.0 ** 13 / (2 * wl.n_r)))
    for tile in (128, 256):
        other.set_option(G.KEY_BF16_TILE, tile)
        for split in (0, 1, 7, 32):
            other.set_option(G.KEY_GEMM_SPLITK, split)
            y = other.potential_product(vd, precision="mixed").cpu().numpy()
            assert np.all(np.abs(y - got) <= bound), (tile, split)

