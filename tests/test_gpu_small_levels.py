"""Small levels in one launch per leg of the V-cycle, and cycles queued ahead of
the stopping test, against the per-launch path (GRMG_SMALL_N=0, GRMG_AHEAD=0).

The legs update the points in the same order as the per-colour sweeps; only the
restriction and the norms add their terms in another order, so whole solves agree
to rounding: 1e-12 of the field's largest value for FP64, 1e-10 for the refined
mixed-precision solve (the bars of the single-workgroup cycle's tests).
"""
import numpy as np
import pytest

import oracle as O
from paper_1905_08890_amd import grmg, synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

PRM = dict(a=1.0, omega_m=synth.OMEGA_M, c_tilde=synth.C_TILDE)
KINDS = {"poisson": O.POISSON, "hamiltonian": O.HAMILTONIAN, "cmc": O.CMC}


def _problem(kind, n):
    rng = np.random.default_rng(100 + n)
    if kind == O.POISSON:
        return rng.standard_normal((n, n, n)), np.zeros((n, n, n))
    s0 = 1.0 + 0.3 * rng.standard_normal((n, n, n))
    if kind == O.HAMILTONIAN:
        return 1.5 * PRM["omega_m"] * (s0 - 1.0), 0.2 * np.abs(rng.standard_normal((n, n, n)))
    psi = 0.1 * rng.standard_normal((n, n, n)) / (2 * PRM["c_tilde"] ** 2)
    m2, f = O.build_cmc(psi, s0, np.zeros_like(s0), np.zeros_like(s0), prm=O.params(**PRM))
    return f, m2


def _grid(n, f, coef):
    g = grmg.Grid(n, **PRM)
    g.set_field("rhs", f)
    g.set_field("coef", coef)
    return g


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("kind", list(KINDS))
@pytest.mark.parametrize("n", [12, 16, 20, 24, 28, 40, 48, 56, 64, 128])
def test_small_legs_match_per_launch(n, kind, precision, monkeypatch):
    """Sides that tiles of 4 and 8 divide and sides they do not, both sweep counts."""
    print(f"[gpu] small legs n={n} {kind} {precision}", flush=True)
    f, coef = _problem(KINDS[kind], n)
    monkeypatch.setenv("GRMG_SMALL_N", "0")
    a = _grid(n, f, coef)
    monkeypatch.delenv("GRMG_SMALL_N")
    b = _grid(n, f, coef)
    for nu1, nu2 in ((2, 2), (1, 1), (2, 1)):
        out = []
        for g in (a, b):
            g.set_field("Vx", np.zeros((n, n, n)))
            g.solve_equation(KINDS[kind], "Vx", rtol=0, max_cycles=3, nu1=nu1, nu2=nu2, precision=precision)
            out.append(g.get_field("Vx"))
        tol = 1e-12 if precision == "fp64" else 1e-10
        assert float((out[0] - out[1]).abs().max()) <= tol * float(out[0].abs().max()), (nu1, nu2)


@pytest.mark.parametrize("kind", list(KINDS))
@pytest.mark.parametrize("n", [16, 32, 48, 64])
def test_cycles_queued_ahead_stop_alike(n, kind, monkeypatch):
    """Same cycles, status and residual for every way a solve can end, twice in a row."""
    print(f"[gpu] queued ahead n={n} {kind}", flush=True)
    k = KINDS[kind]
    f, coef = _problem(k, n)
    monkeypatch.setenv("GRMG_AHEAD", "0")
    a = _grid(n, f, coef)
    monkeypatch.delenv("GRMG_AHEAD")
    b = _grid(n, f, coef)
    allow = (grmg.OK, grmg.ENOTCONV, grmg.ENAN)
    for kw in (dict(rtol=1e-8), dict(rtol=0, max_cycles=3), dict(rtol=1e-12, max_cycles=2), dict(rtol=1e-8, max_cycles=0),
               dict(rtol=0, max_cycles=0), dict(rtol=1e-8)):
        rep, out = [], []
        for g in (a, b):
            g.set_field("Vx", np.zeros((n, n, n)))
            rep.append(g.solve_equation(k, "Vx", allow=allow, **kw))
            out.append(g.get_field("Vx"))
        assert rep[0]["status"] == rep[1]["status"], kw
        assert rep[0]["cycles"][0] == rep[1]["cycles"][0], kw
        assert abs(rep[0]["rel_res"][0] - rep[1]["rel_res"][0]) <= 1e-6 * rep[0]["rel_res"][0] + 1e-14, kw
        assert float((out[0] - out[1]).abs().max()) <= 1e-12 * float(out[0].abs().max()), kw
    f = f.copy()
    f[1, 2, 3] = np.nan
    for g in (a, b):
        g.set_field("rhs", f)
        assert g.solve_equation(k, "Vx", allow=allow, rtol=1e-8)["status"] == grmg.ENAN


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("n", [32, 36, 40, 48])
def test_concurrent_components_of_small_grids(n, precision, monkeypatch):
    """The vector components on three streams equal the ones solved in turn, bit for bit."""
    print(f"[gpu] concurrent components n={n} {precision}", flush=True)
    monkeypatch.setenv("GRMG_CONCURRENT", "0")
    a = grmg.Grid(n, **PRM)
    monkeypatch.delenv("GRMG_CONCURRENT")
    b = grmg.Grid(n, **PRM)
    pos, u, mass = synth.zeldovich(n, 5, 0.5)
    a.deposit_sources(pos, u, mass)
    for name in ("s0", "sx", "sy", "sz", "sm"):
        b.set_field(name, a.get_field(name))
    for _ in range(2):
        ra = a.solve_constraints(rtol=1e-9, precision=precision)
        rb = b.solve_constraints(rtol=1e-9, precision=precision)
        assert ra["cycles"] == rb["cycles"]
        for f in range(10):
            assert torch.equal(a.get_field(f), b.get_field(f)), f


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
@pytest.mark.parametrize("kind", list(KINDS))
@pytest.mark.parametrize("n", [12, 20, 28, 32, 48, 64, 128])
def test_small_legs_give_the_bits_of_the_per_launch_path(n, kind, precision, monkeypatch):
    """With the cycles measured alike (GRMG_AHEAD=0: queued ahead, the frozen means and
    norms are summed in another order) a leg in one launch changes no bit: its updates, its
    residuals and the sums of its restriction are in the per-launch order."""
    print(f"[gpu] small legs bit for bit n={n} {kind} {precision}", flush=True)
    f, coef = _problem(KINDS[kind], n)
    monkeypatch.setenv("GRMG_AHEAD", "0")
    a = _grid(n, f, coef)
    monkeypatch.setenv("GRMG_SMALL_N", "0")
    b = _grid(n, f, coef)
    for nu1, nu2 in ((2, 2), (1, 2)):
        out = []
        for g in (a, b):
            g.set_field("Vx", np.zeros((n, n, n)))
            g.solve_equation(KINDS[kind], "Vx", rtol=0, max_cycles=3, nu1=nu1, nu2=nu2, precision=precision)
            out.append(g.get_field("Vx"))
        assert torch.equal(out[0], out[1]), (nu1, nu2)
