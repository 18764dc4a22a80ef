"""AVL_OPT_KAHAN32: what the compensated FP32 sums and their rho keep.

A corner sum keeps both of its words, so left are FP32 roundings of single terms: of
the product w f, and in N and in D of the term less the carried error, and of the
recovered error where the term exceeds the sum so far (the first few of a run).  One
is 2^-24 / sqrt(12) times the mean of 1/m over a binade, 1.24e-8 rms; a cell averages
4 ppc terms, and a Maxwellian of 16 thermal speeds effectively spans 0.22 nv rows of a
column.  rho sums the quotients in FP64.  The order of the terms, and with it the
roundings, changes from run to run: compared is the rms over the columns, which hardly
does, and the bound is three times the estimate, whose weights are all taken as equal.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

import oracle
from paper_1804_03901_amd import avl, inputs

pytestmark = pytest.mark.gpu

TERM = 1.24e-8


def _bound(terms, nv, ppc):
    return 3.0 * TERM * np.sqrt(terms / (4.0 * ppc * 0.22 * nv))


def _rms(a, b):
    return np.sqrt(np.mean((a - b) ** 2)) / np.max(np.abs(b))


def _rho(w, x, v, f):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"[case] {w.name} n={x.size}", flush=True)
    return avl.Simulation(w, x, v, f, precision=avl.AVL_FP32, options=avl.AVL_OPT_KAHAN32)


@pytest.mark.parametrize("nx,nv,ppc", [(64, 100, 8), (256, 96, 40), (512, 777, 5)])
def test_order_of_markers(nx, nv, ppc):
    # two orders of the same markers: both roundings of terms in N and D, twice
    w = inputs.bump_on_tail(nx=nx, nv=nv, ppc=ppc, seed=31)
    x, v, f = inputs.markers(w)
    v = v.reshape(-1)
    rho = []
    for order in (np.arange(x.size), np.random.default_rng(7).permutation(x.size)):
        sim = _rho(w, x[order], v[order], f[order])
        rho.append(sim.field()[1].cpu().numpy())
        sim.check()
        sim.close()
    assert _rms(*rho) <= _bound(8, nv, ppc)


def test_rho_against_the_oracle():
    # from the exported (FP32) markers: the products, and both roundings in N and D
    w = inputs.bump_on_tail(nx=512, nv=777, ppc=5, seed=32)
    x, v, f = inputs.markers(w)
    sim = _rho(w, x, v.reshape(-1), f)
    xs, vs, fs = (t.cpu().numpy() for t in sim.markers())
    g = oracle.Grid.from_workload(w)
    _, _, fo = oracle.reconstruct(g, xs, vs.reshape(1, -1), fs)
    rho_o, _, _ = oracle.moments(g, fo)
    assert _rms(sim.field()[1].cpu().numpy(), rho_o) <= _bound(5, 777, 5)
    sim.close()
