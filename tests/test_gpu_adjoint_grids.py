"""The reverse kernels over the range of grids: the field adjoint's copies in
LDS (four, two and one, by the columns), the deposit's paired gathers with
their cyclic last column, and whole reverse steps on the narrowest and widest
grids.  Dot products against the oracle's tangents at 1e-12 of the terms'
magnitudes (1e-5 with FP32 grids); the step's gradient against a central
difference at 1e-6 (h^2 and the rounding of J over h are both below it)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import tangent
import oracle
from paper_1804_03901_amd import adjoint, avl, inputs

pytestmark = pytest.mark.gpu


def _state(nx, nv, ppc, precision=avl.AVL_FP64):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    w = inputs.bump_on_tail(nx=nx, nv=nv, ppc=ppc, seed=61).replace(L=0.25 * nx)
    rng = np.random.default_rng(nx)
    hv = (w.vmax[0] - w.vmin[0]) / nv
    n = nx * nv * ppc
    x = rng.uniform(0.0, w.L, n)
    v = rng.uniform(w.vmin[0] + hv, w.vmax[0] - hv, n)
    f = rng.uniform(0.2, 2.0, n)
    print(f"[case] nx={nx} n={n} prec={precision}", flush=True)
    return w, avl.Simulation(w, x, v, f, precision=precision), rng, x, v, f


def _t(a):
    return torch.tensor(np.ascontiguousarray(a, dtype=np.float64), device="cuda:0")


def _close(lhs_terms, rhs_terms, tol):
    lhs, rhs = (sum(float(np.sum(t)) for t in ts) for ts in (lhs_terms, rhs_terms))
    assert abs(lhs - rhs) <= tol * sum(float(np.sum(np.abs(t))) for t in lhs_terms + rhs_terms)


@pytest.mark.parametrize("nx", [8, 64, 1024, 2048, 4096])
def test_push_and_field_adjoint(nx):
    w, sim, rng, x, v, f = _state(nx, 6, 8)
    n = sim.n
    E, lx1, lv1 = rng.normal(size=nx), rng.normal(size=n), rng.normal(size=n)
    lx, lv, Eb = (torch.empty(k, dtype=torch.float64, device="cuda:0") for k in (n, n, nx))
    avl.avl_adjoint_push(sim.h, _t(x), _t(E), 1.0, _t(lx1), _t(lv1), lx, lv, Eb)
    lx, lv, Eb = (t.cpu().numpy() for t in (lx, lv, Eb))
    dx, dv, dE = rng.normal(size=n), rng.normal(size=n), rng.normal(size=nx)
    tx, tv = tangent.push_tangent(oracle.Grid.from_workload(w), x, v, E, 1.0, dx, dv, dE)
    _close([tx * lx1, tv * lv1], [dx * lx, dv * lv, dE * Eb], 1e-12)
    sim.close()


@pytest.mark.parametrize("nx,nv,ppc", [(8, 12, 8), (64, 9, 8), (1024, 6, 8), (4096, 5, 8)])
def test_reverse_step_against_a_difference(nx, nv, ppc):
    w, sim, rng, x, v, f = _state(nx, nv, ppc)
    xt, vt, ft = _t(x), _t(v), _t(f)
    _, g = adjoint.energy_and_gradient(sim, xt, vt, ft, 3, every=2)
    d = _t(rng.normal(size=f.size))
    h = 1e-6      # of weights of order one: the field of the widest grid grows with its length squared
    Jp, _ = adjoint.energy_and_gradient(sim, xt, vt, ft + h * d, 3, want_grad=False)
    Jm, _ = adjoint.energy_and_gradient(sim, xt, vt, ft - h * d, 3, want_grad=False)
    fd, ad = (float(Jp) - float(Jm)) / (2 * h), float((g * d).sum())
    scale = float((g * d).abs().sum())
    print(f"[result] adjoint {ad:.12e} fd {fd:.12e}", flush=True)
    assert abs(fd - ad) <= 1e-6 * scale
    sim.close()
