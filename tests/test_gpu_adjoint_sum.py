"""dL/dsigma where its sum leaves FP64's range: what the plain FP64 sum of the
sites' terms gives (an infinity of the overflowing sign, NaN from infinities of
both signs or from a NaN), not a NaN made by the summation.

With a fixed curvature of 1e12 a site's term, K (dL/dG . grad rho^N) / 2, is
some 1e10 times its other adjoints: adjoint inputs that push one site's
momenta make that site's term overflow while everything else stays finite (by
the oracle, the other sites' terms are below 1e-15 of it)."""
import numpy as np
import pytest
import torch

from oracle.lattice import C
from paper_2005_04642_amd import lbm, workloads as Wk

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
MAX = np.finfo(np.float64).max


# one tile per lattice, and several; one step, and a second one that adds the
# first one's parts
@pytest.mark.parametrize("kind", ["periodic", "walls", "mask"])
@pytest.mark.parametrize("nx,ny", [(24, 10), (131, 97)])
def test_overflow_of_dL_dsigma(nx, ny, kind):
    params = Wk.base_params(Lambda=10.0, sigma=1e-15)
    params.update(fixed_K=1e12, walls=kind == "walls")
    rng = np.random.default_rng(5)
    solid = None
    if kind == "mask":
        solid = np.zeros((ny, nx), dtype=bool)
        solid[:, nx // 2] = True
    sim = lbm.Simulation(nx, ny, params, 0.5 * rng.uniform(-1, 1, (ny, nx)), storage="f64", solid=solid)
    even = lbm.Simulation(nx, ny, params, np.full((ny, nx), 0.25), storage="f64", solid=solid)
    state, flat = sim.live_pops(), even.live_pops()
    c = torch.tensor(np.asarray(C, dtype=np.float64), device=DEV)
    push = c[:, 0] + 0.6 * c[:, 1]

    def dsigma(weights, steps=1):
        lam, out = sim.pops_like(), sim.pops_like()
        lam.zero_()
        for (y, x), w in weights.items():
            lam[:, :, y, x] = w * push
        total = torch.zeros(1, dtype=torch.float64, device=DEV)
        ws = sim.adjoint_workspace()
        states = [flat, state][2 - steps:]   # the uniform state's gradient and terms are zero
        lbm.lbm_adjoint_steps(sim.h, [s.data_ptr() for s in states], lam.data_ptr(), out.data_ptr(), ws.data_ptr(),
                              ws.numel(), total.data_ptr(), None, sim.stream())
        return float(total)

    a, b = (2, 3), (ny - 4, nx - 4)
    va, vb = dsigma({a: 1.0}), dsigma({b: 1.0})
    assert 1e8 < abs(va) < 1e14 and 1e8 < abs(vb) < 1e14
    one, other = MAX / va, MAX / vb          # the weight that takes a site's term to +MAX
    for steps in (1, 2):
        assert dsigma({a: 1.5 * one}, steps) == np.inf
        assert dsigma({b: -1.5 * other}, steps) == -np.inf
        assert dsigma({a: 0.7 * one, b: 0.7 * other}, steps) == np.inf
        assert np.isfinite(dsigma({a: 0.7 * one, b: -0.7 * other}, steps))
        assert abs(dsigma({a: 0.9 * one}, steps) / (0.9 * MAX) - 1.0) < 1e-9
        assert np.isnan(dsigma({a: 1.5 * one, b: -1.5 * other}, steps))
        assert np.isnan(dsigma({a: np.nan}, steps))
    sim.close()
    even.close()
