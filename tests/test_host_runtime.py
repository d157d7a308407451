"""Host side of the library on the CPU: libgwl.so is loaded over a stand-in for
the HIP runtime (fake_hip.cpp: device memory in host memory, kernel launches
logged and not run), in a process of its own for each test.  What is checked is
allocation, its failures and the launches; results mean nothing here."""
import os
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
LIB = os.path.join(ROOT, "paper_2310_20103_amd", "_lib", "libgwl.so")

pytestmark = pytest.mark.skipif(not os.path.exists(LIB), reason="libgwl.so not built")

PREAMBLE = '''
import ctypes as ct, importlib.util, re, sys
import numpy as np
fake = ct.CDLL(sys.argv[1], mode=ct.RTLD_GLOBAL)
fake.fake_log.restype = ct.c_char_p
fake.fake_watched.restype = ct.c_double
for f, t in (("fake_live", ct.c_size_t), ("fake_mallocs", ct.c_long)):
    getattr(fake, f).restype = t
for f in ("fake_fail_malloc", "fake_fail_event", "fake_limit"):
    getattr(fake, f).argtypes = [ct.c_size_t if f == "fake_limit" else ct.c_long]
fake.fake_watch.argtypes = [ct.c_char_p, ct.c_int, ct.c_long]
sys.modules["torch"] = None  # (its own HIP runtime stays out of this process)
spec = importlib.util.spec_from_file_location("binding", sys.argv[2])
G = importlib.util.module_from_spec(spec)
spec.loader.exec_module(G)
L = G.lib()

def context(nv, nc, grid, **kw):
    rng = np.random.default_rng(1)
    kw.setdefault("poly_lo", 0.01)
    kw.setdefault("poly_hi", 1.0)
    e = np.concatenate([np.linspace(-9, -5, nv), np.linspace(1, 9, nc)])
    c = G.Context(rng.standard_normal((nv + nc, int(np.prod(grid)))), e, nv, grid, 6.0, **kw)
    fake.fake_reset()
    return c

def log():
    return fake.fake_log().decode().splitlines()

def call(name, c, n_vec, *a):
    """A component call on host arrays (the stand-in's device memory)."""
    width = {"gwl_apply_c": (c.n_vc, c.n_vc), "gwl_poisson": (c.n_r, c.n_r),
             "gwl_pair_density": (c.n_vc, c.n_r), "gwl_potential_product": (c.n_r, c.n_vc)}[name]
    x, y = np.zeros((n_vec, width[0])), np.zeros((n_vec, width[1]))
    return getattr(L, name)(c._h, G._ptr(x), G._ptr(y), n_vec, *(a or (0,)))

def gemms():
    """The FP64 GEMM launches in the log: [("gemm1_pd", "1", "2", "1"), ("gemm2_f64m",), ...]"""
    return [tuple(x for x in m if x)
            for m in re.findall(r"(gemm[12]_(?:pd|f64m))_kernel(?:ILi(\\d+)ELi(\\d+)ELi(\\d+)E)?",
                                "\\n".join(log()))]
'''


@pytest.fixture(scope="module")
def fake(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("fake") / "libfakehip.so")
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-o", so,
                    os.path.join(HERE, "fake_hip.cpp")], check=True)
    return so


def run(fake, body):
    r = subprocess.run([sys.executable, "-c", PREAMBLE + body, fake,
                        os.path.join(ROOT, "paper_2310_20103_amd", "binding.py")],
                       capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout[-2000:] + r.stderr[-4000:]


@pytest.mark.parametrize("k", range(0, 30, 3))
def test_growth_that_fails(fake, k):
    """The k-th allocation of a growth fails: the call says so, and a smaller
    one afterwards works on whole, cleared buffers."""
    run(fake, f'''
c = context(3, 5, (4, 6, 4))
assert call("gwl_apply_c", c, 4) == 0
fake.fake_reset()
fake.fake_fail_malloc({k})
code = call("gwl_apply_c", c, 40)
assert code in (0, G.GWL_ENOMEM) and (code or {k} >= 24), code  # (the last ones are optional)
fake.fake_reset()
# the buffers given up are allocated again before a kernel runs on them
assert call("gwl_poisson", c, 8) == 0
assert call("gwl_apply_c", c, 4) == 0
if code:
    assert fake.fake_mallocs() >= 1
    lines = log()
    assert lines and not any(l.endswith("unsynced") for l in lines), lines
    fake.fake_reset()
    assert call("gwl_apply_c", c, 40) == 0
    assert call("gwl_apply_c", c, 40) == 0
''')


def test_scratch_growth_that_fails(fake):
    """The Poisson scratch alone fails to grow: products afterwards have theirs."""
    run(fake, '''
c = context(3, 5, (4, 6, 4))
assert call("gwl_apply_c", c, 4) == 0
fake.fake_reset()
fake.fake_fail_malloc(0)
assert call("gwl_poisson", c, 60) == G.GWL_ENOMEM
fake.fake_reset()
assert call("gwl_apply_c", c, 4) == 0
assert fake.fake_mallocs() == 1  # the scratch
''')


@pytest.mark.parametrize("k", [0, 1])
@pytest.mark.parametrize("what", ["malloc", "event"])
def test_staging_that_cannot_be_made(fake, what, k):
    """A large result without its pinned chunks or an event: copied plainly, now
    and in the calls that follow, and nothing is left allocated."""
    run(fake, f'''
c = context(3, 5, (4, 6, 4))
args = ([0, 4], np.ones((2, 3)), np.ones((2, 3)), np.ones(2), [3, 3], np.linspace(-1, 1, 200000), 0.1)
c.sigma_from_coeffs([0, 4], *args[1:5], args[5][:9], 0.1)
big = 2 * 200000 * 16
live = fake.fake_live()
fake.fake_reset()
if "{what}" == "event":
    fake.fake_fail_event({k})
else:
    fake.fake_limit(live + big + 200000 * 8 + 10000 + {k} * (2 << 20))
for _ in range(2):
    c.sigma_from_coeffs(*args)
    assert fake.fake_live() < live + big + 200000 * 8 + 100000
    if "{what}" == "event":
        fake.fake_fail_event(0)
fake.fake_reset()
c.sigma_from_coeffs(*args)
assert fake.fake_live() >= live + big + (4 << 20)
''')


VJP = '''
def vjp(c, length, n_omega, n_range):
    om, g = np.linspace(-5, 5, n_omega), np.ones((1, n_omega, 2))
    q, sig = np.zeros(1, np.int32), np.zeros((1, n_omega, 2))
    ge, go = np.zeros(c.n_orb), np.zeros((c.n_orb, c.n_r))
    return L.gwl_sigma_c_range_vjp(c._h, G._ptr(q), 1, *n_range, G._ptr(om), n_omega, 0.1, length,
                                   G._ptr(g), G._ptr(sig), G._ptr(ge), G._ptr(go))
'''


def test_kept_gradient_buffers_make_way(fake):
    """With the card full but for what a gradient call left behind, a call that
    needs that memory gets it; a second gradient as well, whatever its shape."""
    run(fake, VJP + '''
c = context(3, 5, (4, 6, 4))
assert call("gwl_apply_c", c, 1) == 0
bare = fake.fake_live()
assert vjp(c, 6, 50, (0, 8)) == 0
assert call("gwl_apply_c", c, 8) == 0   # (the products' buffers of that call)
kept = fake.fake_live()
fake.fake_limit(kept + 1000)
assert call("gwl_apply_c", c, 9) == 0
assert fake.fake_live() < kept + 1000

c = context(3, 5, (4, 6, 4))
assert vjp(c, 3, 400, (0, 8)) == 0
fake.fake_reset()
fake.fake_limit(fake.fake_live() + 1000)
assert vjp(c, 9, 50, (0, 8)) == 0
''')


def test_forward_alone_has_a_zero_cotangent(fake):
    """Also after a gradient call whose cotangent is still in the kept buffer."""
    run(fake, VJP + '''
c = context(3, 5, (4, 6, 4))
fake.fake_watch(b"cf_adjoint_kernel", 11, 2 * 40)
assert vjp(c, 4, 40, (0, 8)) == 0
assert fake.fake_watched() == 1.0
fake.fake_watch(b"cf_adjoint_kernel", 11, 2 * 40)
c.sigma_c_vjp_forward.__func__.__globals__["_sync_torch"] = lambda: None
c.sigma_c_vjp_forward([0], np.linspace(-5, 5, 40), 0.1, 4)
assert fake.fake_watched() == 0.0
''')


@pytest.mark.parametrize("grid,nv,nc,n,form", [
    # measured C products (us): rows, pairs
    ((12, 12, 12), 100, 300, 33, "f64m"),   # 281, 1,095
    ((18, 16, 18), 64, 200, 64, "f64m"),    # 431, 655
    ((36, 32, 32), 76, 171, 8, "f64m"),     # 525, 806
    ((32, 32, 32), 87, 139, 8, "f64m"),     # 523, 789
    ((24, 24, 24), 8, 32, 1, "pd"),         # 90, 52
    ((24, 24, 24), 8, 32, 64, "pd"),
    ((32, 32, 32), 32, 128, 64, "pd"),      # 1,120, 631
])
def test_form_of_the_product(fake, grid, nv, nc, n, form):
    """Pair densities as the GEMM operand where that is the faster product, and
    both halves of a K product in one form."""
    run(fake, f'''
c = context({nv}, {nc}, {grid})
assert call("gwl_apply_c", c, {n}) == 0
assert {{k[0] for k in gemms()}} == {{"gemm1_{form}", "gemm2_{form}"}}, gemms()
c.set_option(G.KEY_KERNELS, 0)
fake.fake_reset()
assert call("gwl_apply_c", c, {n}) == 0
assert not gemms()
''')


@pytest.mark.parametrize("nv,nc", [(8, 32), (33, 70), (100, 300)])
@pytest.mark.parametrize("grid", [(4, 6, 4), (12, 12, 8), (18, 18, 18), (24, 24, 24), (16, 27, 18)],
                         ids=lambda g: "x".join(map(str, g)))
def test_every_split_holds_points(fake, grid, nv, nc):
    """No part of the second GEMM's grid sum is empty."""
    run(fake, f'''
c = context({nv}, {nc}, {grid})
n = -(-c.n_r // 256) * 256
for precision in (G.FP64, G.MIXED_F16):
    for nb in (1, 5, 16, 31, 33, 64):
        fake.fake_reset()
        assert call("gwl_apply_c", c, nb, precision) == 0
        parts = [tuple(map(int, m)) for m in re.findall(r"split (\\d+) (\\d+)", "\\n".join(log()))]
        assert parts
        assert all((s - 1) * k < n <= s * k for s, k in parts), (nb, parts)
''')


@pytest.mark.parametrize("n_pairs,length,in_lds", [
    (1, 4, True), (80, 30, True), (640, 200, True), (6400, 200, True), (50000, 30, True),
    (200, 2730, True), (513, 2730, False), (3, 2731, False), (10000, 200, False), (20000, 200, False),
    (20000, 600, False)])
def test_eigenvalues_in_lds(fake, n_pairs, length, in_lds):
    """The QL iteration works in LDS where all its blocks are resident at once
    (160 KB and 32 waves a CU, 256 CUs)."""
    run(fake, f'''
c = context(3, 5, (4, 6, 4))
c.set_quadrature(True)
a = np.ones(({n_pairs}, {length}))
c.sigma_from_coeffs(np.zeros({n_pairs}), a, a, a[:, 0], np.full({n_pairs}, {length}), [0.0], 0.1)
lines = [l for l in log() if "quad_eig_kernel" in l]
assert len(lines) == 1
assert ("ILb1E" in lines[0]) == {in_lds}, lines
if {in_lds}:
    blocks, _, threads = map(int, lines[0].split()[1:4])
    assert blocks * threads >= {n_pairs} > (blocks - 1) * threads
    lds = threads * 3 * {length} * 8
    assert lds <= 65536 and blocks <= 256 * min(32, 160 * 1024 // lds)
''')


@pytest.mark.parametrize("grid,in_frequency_space", [((8, 12, 16), True), ((162, 4, 6), False)])
@pytest.mark.parametrize("nv,states", [(1, 1), (3, 4), (40, 20)])
def test_exchange_memory(fake, grid, in_frequency_space, nv, states):
    """Sigma^ex takes the transform's scratch of at most 64 fields, or where it goes
    by potentials on the grid the buffers of min(N_v, 64) vectors; besides them
    only lists and energy shares."""
    run(fake, f'''
c = context({nv}, 24, {grid})
before = fake.fake_live()
c.sigma_x(np.arange({states}))
used = fake.fake_live() - before
if {in_frequency_space}:
    fields = min({states} * ({nv} + {nv} % 2), 64)
    most = fields // 2 * c.n_r * 16
else:
    d = context({nv}, 24, {grid})
    before = fake.fake_live()
    assert call("gwl_apply_c", d, {nv}) == 0
    most = fake.fake_live() - before
shares = {states} * {nv + 1} * max(12 * 16, 64) * 8
assert used <= most + shares + 100000, (used, most)
''')


def test_pair_gemm_cases_reach_every_form(fake):
    """The sizes that test_gpu_pair_variants.py runs launch the pair-density GEMMs
    in every form of their rules: (column blocks, K shares) and 1 to 8 row
    blocks, and two M tiles."""
    pytest.importorskip("torch")
    from test_gpu_pair_variants import CASES, SLOTS
    run(fake, f'''
seen = set()
for grid, nv, nc, split, counts in {CASES!r}:
    c = context(nv, nc, grid)
    c.set_option(G.KEY_GEMM_SPLITK, split)
    for n in counts:
        for name in ("gwl_pair_density", "gwl_potential_product"):
            assert call(name, c, n) == 0
    seen |= {{(k[0], *map(int, k[1:])) for k in gemms() if "pd" in k[0]}}
    c.close()
for g, forms in (("gemm1_pd", [(2, 1), (1, 1), (1, 2), (1, 4)]),
                 ("gemm2_pd", [(1, 1), (1, 2), (1, 4)])):
    for f in forms:
        rows = sorted(k[1] for k in seen if k[0] == g and k[2:] == f)
        assert rows and rows[0] <= 2 and rows[-1] >= 5, (g, f, rows)
    assert {{k[1] for k in seen if k[0] == g}} == set(range(1, 9))
for grid, nv, nc, slots in {SLOTS!r}:
    c = context(nv, nc, grid, block=slots)
    c.lanczos_pairs(np.zeros(slots), np.zeros(slots), np.full(slots, 2))
    rows = -(-slots // 32)
    assert {{k[0] for k in gemms() if k[1:] and int(k[1]) == rows}} == {{"gemm1_pd", "gemm2_pd"}}, gemms()
    c.close()
''')


@pytest.mark.parametrize("n_vec", [1, 20, 31, 40])
def test_products_without_the_optional_memory(fake, n_vec):
    """The pair-density operand and room for more than 32 splits are not worth a
    refusal: without them a product runs on the row GEMMs, and with 32 splits."""
    run(fake, f'''
c = context(7, 33, (18, 18, 18))
assert call("gwl_apply_c", c, {n_vec}) == 0
full = fake.fake_live()
assert {{k[0] for k in gemms()}} == {{"gemm1_pd", "gemm2_pd"}}
c.close()
c = context(7, 33, (18, 18, 18))
start = fake.fake_live()
optional = ({n_vec} + 16) * 7 * 33 * 8 + (max(64 * min({n_vec}, 31), 32 * {n_vec}) - 32 * {n_vec}) * 64 * 64 * 8
fake.fake_limit(full - optional + 1000)
for precision in (0, 1):
    for _ in range(2):
        fake.fake_reset()
        fake.fake_limit(full - optional + 1000)
        assert call("gwl_apply_c", c, {n_vec}, precision) == 0
        if precision == 0:
            assert {{k[0] for k in gemms()}} == {{"gemm1_f64m", "gemm2_f64m"}}
        parts = [int(m) for m in re.findall(r"split (\\d+) ", "\\n".join(log()))]
        assert parts and max(parts) <= 32
fake.fake_reset()
assert call("gwl_apply_c", c, {n_vec} + 1) == 0   # the next growth asks again
assert {{k[0] for k in gemms()}} == {{"gemm1_pd", "gemm2_pd"}}
''')
