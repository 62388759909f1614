"""The tile kernel against the march: the two forms of the step share a site's
arithmetic, so states and fields are equal bit for bit.

A plan for one CU sends a lattice of a few tiles through the march, the plan
for the whole device through the tiles."""
import itertools

import numpy as np
import pytest
import torch

from gpu_helpers import *  # noqa: F401,F403
from paper_2005_04642_amd import lbm, workloads as Wk

pytestmark = pytest.mark.gpu

PROFILES = [tuple(p) for p in itertools.product((1, 3), repeat=4)]


def run(nx, ny, storage, ncu, steps=3, stencil=(3, 3, 3, 3), walls=False, solid=False, force=False, **kw):
    p = Wk.base_params(Lambda=10.0, sigma=0.01, stencil=stencil)
    p.update(walls=walls, gx=1e-6 if walls else 0.0, gy=-2e-6 if walls else 0.0, **kw)
    y, x = np.mgrid[0:ny, 0:nx]
    rn = np.tanh((0.3 * min(nx, ny) - np.hypot(x - 0.4 * nx, y - 0.6 * ny)) / 2.0)
    mask = Wk.random_solid_sites(nx, ny, nx * ny // 15, 3) if solid else None
    f = 1e-5 * np.random.default_rng(5).standard_normal((2, ny, nx)) if force else None
    s = lbm.Simulation(nx, ny, p, rn, storage=storage, force=f, solid=mask)
    s.set_cu_budget(step=ncu)
    s.step(steps)
    rows = slice(1, -1) if walls else slice(None)
    state = s.live_words()[:, rows].contiguous().view(torch.uint8).cpu()
    fields = {k: v.cpu() for k, v in s.fields().items()}
    s.close()
    return state, fields


def check(nx, ny, storage, **kw):
    a, fa = run(nx, ny, storage, 0, **kw)
    b, fb = run(nx, ny, storage, 1, **kw)
    assert torch.equal(a, b)
    for k in fa:
        assert torch.equal(fa[k].nan_to_num(nan=7.0), fb[k].nan_to_num(nan=7.0)), k


# one strip and two of 46 columns; chunks of one tile height (14 or 30 rows),
# one row more, and a last chunk of one row; the widest lattice of two and
# three rounds on 256 CUs
@pytest.mark.parametrize("storage", ["f32", "f64", "f16", "bf16"])
@pytest.mark.parametrize("nx,ny", [(46, 75), (47, 85), (93, 61), (64, 64), (13, 200), (700, 333)])
def test_tile_equals_march(nx, ny, storage):
    check(nx, ny, storage)


@pytest.mark.parametrize("storage", ["f32", "f64", "f16"])
@pytest.mark.parametrize("kind", [dict(walls=True), dict(solid=True), dict(force=True), dict(walls=True, force=True),
                                  dict(fixed_K=0.02), dict(ghost_eq=1, recolor=False)],
                         ids=lambda d: "-".join(d))
@pytest.mark.parametrize("nx,ny", [(47, 85), (301, 147)])
def test_tile_equals_march_options(nx, ny, storage, kind):
    check(nx, ny, storage, **kind)


@pytest.mark.parametrize("stencil", PROFILES, ids=lambda p: "".join(map(str, p)))
def test_tile_equals_march_profiles(stencil):
    check(131, 97, "f32", stencil=stencil)
    check(131, 97, "f64", stencil=stencil, walls=True)


# 3 CUs and 2 strips of columns: one chunk each, or four rounds' shorter chunks
@pytest.mark.parametrize("storage,nx", [("f32", 300), ("f64", 90), ("f16", 300)])
@pytest.mark.parametrize("ny", [400, 403])
def test_march_in_rounds(storage, nx, ny):
    a, b = (run(nx, ny, storage, ncu) for ncu in (1, 3))
    assert torch.equal(a[0], b[0])


def adjoint(nx, ny, storage, ncu, stencil=(3, 3, 3, 3), walls=False, solid=False, force=False, **kw):
    p = Wk.base_params(Lambda=10.0, sigma=0.01, stencil=stencil)
    p.update(walls=walls, gx=1e-6 if walls else 0.0, **kw)
    rng = np.random.default_rng(11)
    y, x = np.mgrid[0:ny, 0:nx]
    rn = np.tanh((0.3 * min(nx, ny) - np.hypot(x - 0.4 * nx, y - 0.6 * ny)) / 2.0)
    mask = Wk.random_solid_sites(nx, ny, nx * ny // 15, 3) if solid else None
    f = 1e-5 * rng.standard_normal((2, ny, nx)) if force else None
    s = lbm.Simulation(nx, ny, p, rn, storage=storage, force=f, solid=mask)
    s.step(4)
    lam = s.pops_like()
    lam.copy_(torch.as_tensor(1e-3 * rng.standard_normal((2, 9, ny, nx))))
    out, state = s.pops_like(), s.pops_like()
    state.copy_(s.live_pops())
    dsigma = torch.zeros(1, dtype=torch.float64, device="cuda:0")
    dforce = torch.zeros((2, ny, nx), dtype=s.dtype, device="cuda:0")
    s.set_cu_budget(adjoint=ncu)
    for _ in range(2):
        s.adjoint_step(state, lam, out, dsigma, dforce)
    res = [t.cpu() for t in (out, dforce, dsigma)]
    s.close()
    return res


def check_adjoint(nx, ny, storage, **kw):
    a, b = (adjoint(nx, ny, storage, ncu, **kw) for ncu in (0, 1))
    assert torch.equal(a[0], b[0])
    assert torch.equal(a[1], b[1])
    # FP64 sums of the sites' FP64 terms in another order: nx ny roundings
    assert torch.allclose(a[2], b[2], rtol=nx * ny * 2.0 ** -53, atol=0.0)


@pytest.mark.parametrize("storage", ["f32", "f64"])
@pytest.mark.parametrize("nx,ny", [(46, 75), (47, 85), (93, 61), (64, 64), (13, 200), (500, 333)])
def test_adjoint_tile_equals_march(nx, ny, storage):
    check_adjoint(nx, ny, storage)


@pytest.mark.parametrize("storage", ["f32", "f64"])
@pytest.mark.parametrize("kind", [dict(walls=True), dict(solid=True), dict(force=True), dict(fixed_K=0.02),
                                  dict(ghost_eq=1, recolor=False)], ids=lambda d: "-".join(d))
def test_adjoint_tile_equals_march_options(storage, kind):
    check_adjoint(131, 97, storage, **kind)


@pytest.mark.parametrize("stencil", PROFILES, ids=lambda p: "".join(map(str, p)))
def test_adjoint_tile_equals_march_profiles(stencil):
    check_adjoint(131, 97, "f32", stencil=stencil)


# few lattices run as tiles, many as marches (a lattice in 24 of them as in 3)
@pytest.mark.parametrize("storage", ["f32", "f16", "f64"])
@pytest.mark.parametrize("count", [3, 24])
@pytest.mark.parametrize("walls", [False, True])
def test_batch_forms_equal_single_lattices(storage, count, walls):
    rng = np.random.default_rng(count)
    lats = []
    for k in range(count):
        nx, ny = int(rng.choice([47, 64, 131, 300])), int(rng.choice([33, 64, 97, 300]))
        p = Wk.base_params(Lambda=10.0, sigma=0.01)
        p.update(walls=walls, gx=1e-6 if walls else 0.0)
        y, x = np.mgrid[0:ny, 0:nx]
        lats.append((nx, ny, p, np.tanh((0.3 * min(nx, ny) - np.hypot(x - 0.4 * nx, y - 0.6 * ny)) / 2.0)))
    b = lbm.Batch(lats, storage=storage)
    b.step(4)
    live = b.pops[b.lib.lbm_batch_current_pops(b.h)]
    for k, (nx, ny, p, rn) in enumerate(lats):
        s = lbm.Simulation(nx, ny, p, rn, storage=storage)
        s.step(4)
        want = s.pops[lbm.lbm_current_pops(s.h)].view(torch.uint8)
        assert torch.equal(live[b.offsets[k]:b.offsets[k] + want.numel()], want), k
        s.close()
    b.close()
