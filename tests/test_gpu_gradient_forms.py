"""The two forms of the gradient (one call; forward, then backward) on one
context in turn, over calls of other shapes whose buffers are kept in between:
bitwise a fresh context's results."""
import numpy as np
import pytest

import gw_inputs as gi

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

GRID = (8, 8, 12)


def test_forms_interleaved():
    import paper_2310_20103_amd as G
    wl = gi.workload("grid24_v8c32", name="forms", seed=611, grid=GRID, box=6.0, n_occ=3, n_emp=5,
                     n_qp_occ=1, n_qp_emp=1)
    s = gi.make_system(wl)
    print("[case] gradient forms", flush=True)

    def ctx():
        return G.Context(s.phi, s.energies_ev, 3, GRID, tuple(n * wl.h for n in GRID), block=4)

    def cot(nw):
        return np.cos(np.arange(len(s.qp_states) * nw)).reshape(-1, nw) * (1 + 0.5j)

    def one(c, length, nw, rng=None):
        return c.sigma_c_vjp(s.qp_states, np.linspace(-10, 10, nw), 0.3, length, cot(nw), n_range=rng)

    def two(c, length, nw, rng=None):
        sig = c.sigma_c_vjp_forward(s.qp_states, np.linspace(-10, 10, nw), 0.3, length, n_range=rng)
        return (sig, *c.sigma_c_vjp_backward(cot(nw)))

    calls = [(one, 6, 9), (two, 6, 9), (one, 9, 40), (two, 3, 2, (1, 4)), (one, 3, 2, (1, 4)),
             (two, 9, 40), (one, 6, 9), (two, 6, 9)]
    with ctx() as c:
        got = [f(c, *a) for f, *a in calls]
    for (f, *a), y in zip(calls, got):
        with ctx() as c:
            ref = f(c, *a)
        for p, q in zip(y, ref):
            assert np.array_equal(np.asarray(getattr(p, "cpu", lambda: p)()),
                                  np.asarray(getattr(q, "cpu", lambda: q)()))
