"""Which kernels an adjoint step runs does not change what it returns.

Passes 2-5 run in one kernel over tiles on most lattices and as separate
kernels on the others: FP64 lattices with a mask past one round of tiles, walls
around fewer than 4 fluid rows, and workspace rows of 2 GiB or more.  A large
lattice whose state and adjoint input repeat a small one's has, site by site,
the small lattice's adjoint, so the separate kernels are compared with the
tiles bit for bit; dL/dsigma is compared relative to the sum of its terms'
magnitudes."""
import numpy as np
import pytest
import torch

from gpu_helpers import *  # noqa: F401,F403
from oracle import chromo as O
from paper_2005_04642_amd import lbm, workloads as Wk
from test_gpu_adjoint import gpu_vjp, oracle_vjp, rel, state_and_params, torch_pull, torch_pull_masked

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


# 1, 2 and 3 fluid rows (separate passes: the walls' mirror images overlap) and
# 4 (the first the tiles take)
@pytest.mark.parametrize("stencil", [(3, 3, 3, 3), (3, 1, 1, 3), (1, 1, 1, 1)])
@pytest.mark.parametrize("ny", [3, 4, 5, 6])
def test_few_fluid_rows_match_oracle_autograd(ny, stencil):
    params, rn, S, lam, force = state_and_params(50, ny, seed=ny, stencil=stencil, walls=True)
    gS, gsig, gF = oracle_vjp(params, S, lam, force)
    aS, asig, aF = gpu_vjp(params, rn, S, lam, force)
    e = (rel(aS, gS), abs(asig - gsig) / abs(gsig), rel(aF, gF))
    print("adjoint walls f64 50x%d %s: pops %.2e sigma %.2e force %.2e" % (ny, stencil, *e))
    assert e[0] < 1e-11 and e[1] < 1e-10 and e[2] < 1e-11


def sum_of_magnitudes(params, S, dforce, solid):
    """Sum over the sites of |K (dL/dG . grad rho^N) / 2|, the terms of dL/dsigma."""
    ny, nx = S.shape[-2:]
    p = O.Params(nx=nx, ny=ny, solid=solid, **params)
    S = torch.as_tensor(S)
    P = torch_pull(S) if solid is None else torch_pull_masked(S, solid, torch.full_like(S, 0.05))
    d = O.interface_fields(P[0], P[1], p)
    t = 0.5 * d["K"] * (dforce[0] * d["gnx"] + dforce[1] * d["gny"])
    if solid is not None:
        t[torch.as_tensor(solid)] = 0.0
    return float(t.abs().sum())


def repeated(nx, ny, rx, ry, storage, stencil, masked):
    """An adjoint step of an nx x ny lattice, and of rx x ry copies of it side by side."""
    params = Wk.base_params(Lambda=10.0, sigma=0.01, stencil=stencil)
    rng = np.random.default_rng(nx + ny)
    rn = np.clip(np.tanh(2.0 * rng.standard_normal((ny, nx))), -1, 1)
    solid = Wk.random_solid_sites(nx, ny, nx * ny // 15, 3) if masked else None
    small = lbm.Simulation(nx, ny, params, rn, storage=storage, solid=solid)
    T = small.dtype
    S, lam = small.pops_like(), small.pops_like()
    S.copy_(small.live_pops())
    S.mul_(torch.as_tensor(Wk.random_state_perturbation(tuple(S.shape), 0.05, 7), device=DEV))
    lam.copy_(torch.as_tensor(rng.standard_normal(tuple(S.shape))))
    if masked:
        lam[:, :, torch.as_tensor(solid)] = 0.0

    def step(sim, S, lam):
        out = sim.pops_like()
        dsigma = torch.zeros(1, dtype=torch.float64, device=DEV)
        dforce = torch.zeros((2, sim.ny, sim.nx), dtype=T, device=DEV)
        sim.adjoint_step(S, lam, out, dsigma, dforce)
        torch.cuda.synchronize()
        return out, dforce, float(dsigma)

    print("adjoint %s %s %dx%d" % (storage, stencil, nx, ny), flush=True)
    a = step(small, S, lam)
    size = sum_of_magnitudes(params, S.double().cpu(), a[1].double().cpu(), solid)
    small.close()
    print("the same repeated: %dx%d" % (nx * rx, ny * ry), flush=True)
    big = lbm.Simulation(nx * rx, ny * ry, params, torch.as_tensor(rn).repeat(ry, rx), storage=storage,
                         solid=None if solid is None else torch.as_tensor(solid).repeat(ry, rx))
    Sb, lb = big.pops_like(), big.pops_like()
    Sb.copy_(S.repeat(1, 1, ry, rx))
    lb.copy_(lam.repeat(1, 1, ry, rx))
    b = step(big, Sb, lb)
    big.close()
    assert torch.equal(b[0], a[0].repeat(1, 1, ry, rx))
    assert torch.equal(b[1], a[1].repeat(1, ry, rx))
    # FP64 sums in blocks of 256, then strided: under 100 additions deep each
    n = rx * ry
    print("dL/dsigma %.15e, %d x %.15e, terms' magnitudes %.3e" % (b[2], n, a[2], n * size))
    assert abs(b[2] - n * a[2]) <= 100 * 2.0 ** -53 * 2 * n * size


# 100^2 in 27 tiles; 400^2 would take 340, more than one per CU
@pytest.mark.parametrize("stencil", [(3, 3, 3, 3), (3, 1, 3, 1), (1, 1, 1, 1)])
def test_masked_f64_past_one_round_equals_tiles(stencil):
    r = 4 if stencil == (3, 3, 3, 3) else 7
    repeated(100, 100, r, r, "f64", stencil, True)


# rows of 39 planes just past 2^31 bytes
@pytest.mark.parametrize("storage,ny,masked", [("f32", 1, False), ("f32", 4, True), ("f64", 1, False)])
def test_rows_past_31_bit_offsets_equal_tiles(storage, ny, masked):
    nx = 21001
    reps = -(-2 ** 31 // (39 * nx * (8 if storage == "f64" else 4)))
    repeated(nx, ny, reps, 1, storage, (3, 3, 3, 3), masked)
