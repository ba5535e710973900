"""GPU: the friction quadrature from piecewise-polynomial omega sums (many
wall nodes) against the oracle's term-by-term long double sums on sampled nodes."""
import ctypes as C

import numpy as np
import pytest

import oracle
from paper_2403_15768_amd import inputs

pytestmark = pytest.mark.gpu

# positive terms, so the relative error of a sum is that of its terms and of
# its additions: at most 1500 sequential additions of 1.1e-16, some 1e-13 at
# the very worst (the interpolation error, below 1e-17, does not show)
TOL = 2e-13


@pytest.fixture(scope="module")
def lbm():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2403_15768_amd import lbm as mod

    mod.load()
    return mod


def spectra(nq, nw, coupling, v_l, disp, gamma_s=None):
    sp = inputs.draw_spectral(inputs.rng_for("tube", 77), nq=nq, nw=nw)
    sp.coupling, sp.v_l, sp.dispersion = coupling, v_l, disp
    if gamma_s is not None:
        sp.gamma_s = gamma_s
    return sp


def oracle_spectra(sp):
    return oracle.Spectral(T=sp.T, omega0=sp.omega0, gamma_s=sp.gamma_s, omega_l=sp.omega_l,
                           gamma_l=sp.gamma_l, a_l=sp.a_l, d=sp.d, nq=sp.nq, nw=sp.nw,
                           lambda_target=sp.lambda_target, dispersion=sp.dispersion,
                           coupling=sp.coupling, v_l=sp.v_l)


def static(lbm, sp, om):
    import torch

    s = lbm.make_spectral(sp)
    d = torch.tensor(om, dtype=torch.float64, device="cuda")
    rc = lbm.load().lbm_friction_quadrature_static(
        C.byref(s), C.c_void_p(d.data_ptr()), len(om), C.c_void_p(d.data_ptr()),
        C.c_void_p(torch.cuda.current_stream().cuda_stream))
    assert rc == 0
    return d.cpu().numpy()


# (nx of a 16 x 16 duct with 60 wall columns, spectra, range of Omega / omega0):
# the smallest node counts that take the tables (2560 shared, 18432 per q) and
# fewer, a part of a group of 8 q, one omega, one Omega for every node,
# and frequencies down to zero
@pytest.mark.parametrize("nx,nq,nw,coupling,v_l,disp,lo,hi", [
    (42, 64, 100, 0, 0.0, 1, 0.4, 1.6),
    (43, 64, 100, 0, 0.0, 1, 0.4, 1.6),
    (43, 19, 1500, 0, 0.0, 0, 0.4, 1.6),
    (43, 5, 1, 0, 0.0, 1, 1.2, 1.2),
    (43, 33, 64, 0, 0.0, 1, 0.0, 2.0),
    (307, 33, 100, 1, 0.4, 1, 0.4, 1.6),
    (308, 33, 100, 1, 0.4, 1, 0.4, 1.6),
    (308, 256, 512, 1, 0.0, 1, 0.6, 1.4),
    (308, 17, 700, 1, 0.3, 0, 1.3, 1.3),
    (308, 16, 64, 0, 0.7, 1, 0.0, 2.0),
])
def test_piecewise_sums(lbm, nx, nq, nw, coupling, v_l, disp, lo, hi):
    check(lbm, nx, spectra(nq, nw, coupling, v_l, disp), lo, hi, TOL)


# spectra whose poles are so close to the axis that a table would be too long:
# summed term by term inside the evaluation.  There a resonance magnifies the
# roundings of P - w^2 (three of P, three of w^2, each 1.1e-16 relative) by
# P / (gamma_s w) ~ s / gamma_s, s <= Omega_max sqrt(q_max d)
@pytest.mark.parametrize("nx,nq,nw,coupling,v_l", [(43, 40, 600, 0, 0.0), (308, 18, 600, 1, 0.2)])
def test_spectra_without_tables(lbm, nx, nq, nw, coupling, v_l):
    sp = spectra(nq, nw, coupling, v_l, 1, gamma_s=0.002)
    s_max = 1.5 * sp.omega0 * np.sqrt(10.0)
    check(lbm, nx, sp, 0.5, 1.5, TOL + 6 * 1.1e-16 * s_max / sp.gamma_s)


def check(lbm, nx, sp, lo, hi, tol):
    print("piecewise sums", nx, sp, lo, hi, flush=True)
    G = lbm.Channel(19, lbm.DUCT, nx, 16, 16, tau=0.7, precision="f16s")
    n = G.wall_count
    assert n == 60 * nx
    om = sp.omega0 * np.random.default_rng(3).uniform(lo, hi, n)
    om[0], om[-1] = sp.omega0 * lo, sp.omega0 * hi
    G.set_friction_spectral(sp, om)
    lam, raw = G.get_friction(raw=True)
    pick = np.unique(np.r_[0, n - 1, np.random.default_rng(4).integers(0, n, 20)])
    raw_o, lam_o = oracle.friction(oracle_spectra(sp), om[pick], kind="f80")
    ok = raw_o > 0
    assert np.array_equal(raw[pick][~ok], raw_o[~ok])
    err = np.max(np.abs(raw[pick][ok] / raw_o[ok] - 1))
    print(f"  {n} nodes, max relative error {err:.2e}", flush=True)
    assert err < tol
    assert np.max(np.abs(lam[pick][ok] / lam_o[ok] - 1)) < 2 * tol
    # the static entry point, whose scratch holds more tables at once: the same bits
    assert np.array_equal(static(lbm, sp, om), lam)


@pytest.mark.parametrize("coupling", [0, 1])
def test_a_bad_frequency_stays_its_own(lbm, coupling):
    print("bad frequency", coupling, flush=True)
    sp = spectra(32, 64, coupling, 0.0, 1)
    om = sp.omega0 * np.random.default_rng(5).uniform(0.5, 1.5, 20000)
    clean = static(lbm, sp, om)
    bad = om.copy()
    bad[[7, 4000]] = np.nan, np.inf
    got = static(lbm, sp, bad)
    assert np.all(np.isnan(got[[7, 4000]]))
    rest = np.ones(len(om), bool)
    rest[[7, 4000]] = False
    # (the two nodes' own frequencies may have set the ends of the range)
    assert np.max(np.abs(got[rest] / clean[rest] - 1)) < 2 * TOL


@pytest.mark.parametrize("coupling,n", [(0, 5000), (1, 20000)])
def test_static_call_in_a_graph(lbm, coupling, n):
    # captured once, replayed between eager calls on other frequencies: every
    # replay gives the eager call's bits
    import torch

    print("static quadrature in a graph", coupling, n, flush=True)
    sp = spectra(32, 64, coupling, 0.0, 1)
    s = lbm.make_spectral(sp)
    om = [sp.omega0 * np.random.default_rng(k).uniform(0.5, 1.5, n) for k in (6, 7, 8)]
    eager = [static(lbm, sp, o) for o in om]
    d_om = torch.zeros(n, dtype=torch.float64, device="cuda")
    d_lam = torch.zeros(n, dtype=torch.float64, device="cuda")
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        rc = lbm.load().lbm_friction_quadrature_static(
            C.byref(s), C.c_void_p(d_om.data_ptr()), n, C.c_void_p(d_lam.data_ptr()),
            C.c_void_p(torch.cuda.current_stream().cuda_stream))
    assert rc == 0
    for o, want in zip(om, eager):
        d_om.copy_(torch.tensor(o, dtype=torch.float64))
        d_lam.zero_()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert np.array_equal(d_lam.cpu().numpy(), want)
        static(lbm, sp, om[0][::-1].copy())


# nearly equal frequencies (or one), all beyond the poles: the panels must not
# reach past the frequencies towards a pole.  Against the node-by-node kernel
# that fewer nodes take, whose factors outside the omega sum are the same; the
# rest differs by the roundings of v (4 u), of the denominator and its
# reciprocal (4 u), of the polynomial (4 u) and of the products (2 u),
# u = 1.1e-16
@pytest.mark.parametrize("lo,hi,w_max", [(1.0, 1.001, 3.0), (1.5, 1.5, 4.0), (1.0, 1.4, 4.0),
                                         (2.5, 2.501, 3.0)])
@pytest.mark.parametrize("coupling", [0, 1])
def test_panels_stay_inside_the_frequencies(lbm, lo, hi, w_max, coupling):
    print("panels", lo, hi, w_max, coupling, flush=True)
    sp = spectra(16, 1, coupling, 0.0, 0, gamma_s=2.0 ** -10)
    sp.T, sp.omega0, sp.omega_l, sp.gamma_l, sp.a_l, sp.d = 0.5, lo, 1.0, 0.5, 0.5, 1.0
    raw = {}
    few, many = ((42, 43), (307, 308))[coupling]
    om = np.linspace(lo, hi, 60 * few)
    for nx in (few, many):  # node by node; piecewise
        G = lbm.Channel(19, lbm.DUCT, nx, 16, 16, tau=0.7, precision="f16s")
        n = G.wall_count
        G.set_friction_spectral(make_w(sp, w_max), np.resize(om, n))
        raw[nx] = G.get_friction(raw=True)[1][: len(om)]
    assert np.all(raw[few] > 0)
    err = np.max(np.abs(raw[many] / raw[few] - 1))
    print(f"  {err:.2e}", flush=True)
    assert err < 14 * 1.1e-16


def make_w(sp, w_max):
    class WithRange:
        pass

    out = WithRange()
    out.__dict__.update({k: getattr(sp, k) for k in (
        "T", "omega0", "gamma_s", "omega_l", "gamma_l", "a_l", "d", "nq", "nw", "lambda_target",
        "dispersion", "coupling", "v_l")}, q_max=1.0, w_max=w_max)
    return out


# where a spectrum has no tables, the nodes from which tables may be taken cost
# what they cost below (the ratio: 1 to 1.1; 1.9 to 70 when the points without a
# table were summed in the evaluation)
@pytest.mark.parametrize("few,many,kw", [
    ((42, 16, 16), (43, 16, 16), dict()),
    ((1270, 3, 1), (1300, 3, 1), dict()), ((307, 16, 16), (308, 16, 16), dict(v_l=0.3)),
    ((307, 16, 16), (308, 16, 16), dict(coupling=1)),
    ((9200, 3, 1), (9300, 3, 1), dict(v_l=0.3)),
])
def test_without_tables_as_fast_as_node_by_node(lbm, few, many, kw):
    import time

    import torch

    print("time without tables", few, many, kw, flush=True)
    sp = spectra(256, 1024, kw.get("coupling", 0), kw.get("v_l", 0.0), 1, gamma_s=0.01)
    per_node = []
    for nx, ny, nz in (few, many):
        kind = (9, lbm.SLAB) if nz == 1 else (19, lbm.DUCT)
        G = lbm.Channel(*kind, nx, ny, nz, tau=0.7, precision="f16s")
        om = sp.omega0 * torch.linspace(0.5, 1.5, G.wall_count, dtype=torch.float64, device="cuda")
        best = 1e9
        for _ in range(6):
            torch.cuda.synchronize()
            t = time.perf_counter()
            G.set_friction_spectral(sp, om)
            best = min(best, time.perf_counter() - t)
        per_node.append(best / G.wall_count)
    print(f"  {per_node[0] * 1e9:.1f} -> {per_node[1] * 1e9:.1f} ns per node", flush=True)
    assert per_node[1] < 1.4 * per_node[0]


# the same without tables: a bad frequency spoils its own node only, and the
# static call replays in a graph
@pytest.mark.parametrize("coupling,n", [(0, 5000), (1, 20000)])
def test_without_tables_bad_frequency_and_graph(lbm, coupling, n):
    import torch

    print("without tables", coupling, n, flush=True)
    sp = spectra(70, 64, coupling, 0.0, 1, gamma_s=0.002)
    om = sp.omega0 * np.random.default_rng(5).uniform(0.5, 1.5, n)
    om[:2] = sp.omega0 * 0.5, sp.omega0 * 1.5  # the range stays
    clean = static(lbm, sp, om)
    assert np.all(np.isfinite(clean)) and np.all(clean > 0)
    bad = om.copy()
    bad[[7, 4000]] = np.nan, np.inf
    got = static(lbm, sp, bad)
    rest = np.ones(n, bool)
    rest[[7, 4000]] = False
    assert np.all(np.isnan(got[~rest])) and np.array_equal(got[rest], clean[rest])
    s = lbm.make_spectral(sp)
    d_om = torch.tensor(om, dtype=torch.float64, device="cuda")
    d_lam = torch.zeros(n, dtype=torch.float64, device="cuda")
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        rc = lbm.load().lbm_friction_quadrature_static(
            C.byref(s), C.c_void_p(d_om.data_ptr()), n, C.c_void_p(d_lam.data_ptr()),
            C.c_void_p(torch.cuda.current_stream().cuda_stream))
    assert rc == 0
    for _ in range(3):
        d_lam.zero_()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert np.array_equal(d_lam.cpu().numpy(), clean)
        static(lbm, spectra(32, 64, 1 - coupling, 0.0, 1), om[::-1].copy())


# no less precise than the sums node by node: the root mean square error of
# lambda over nodes and spectra, both against long double sums (1.6 times theirs
# when the groups of q were added in ascending order)
@pytest.mark.parametrize("coupling,v_l", [(0, 0.0), (1, 0.3)])
def test_as_precise_as_node_by_node(lbm, coupling, v_l):
    print("precision", coupling, v_l, flush=True)
    err = {40: [], 310: []}  # 2400 nodes: node by node; 18600: tables
    for seed in range(6):
        sp = inputs.draw_spectral(np.random.default_rng([seed, 1]))
        sp.coupling, sp.v_l, sp.dispersion = coupling, v_l, 1
        om = sp.omega0 * np.random.default_rng([seed, 2]).uniform(0.55, 1.45, 60 * 310)
        _, want = oracle.friction(oracle_spectra(sp), om[:12], kind="f80")
        for nx, e in err.items():
            G = lbm.Channel(19, lbm.DUCT, nx, 16, 16, tau=0.7)
            G.set_friction_spectral(sp, om[: G.wall_count])
            e += list(G.get_friction()[:12] / want - 1)
    rms = {nx: float(np.sqrt(np.mean(np.square(e)))) for nx, e in err.items()}
    print(f"  node by node {rms[40]:.2e}, tables {rms[310]:.2e}", flush=True)
    assert rms[310] < 1.2 * rms[40]
