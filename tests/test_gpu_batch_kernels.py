"""Both forms of the batch kernel, with and without tiles, for every kind of
lattice: each lattice evolves as it would alone.

On 256 CUs 256 lattices of 64^2 run as one march each, 30 of them (FP32
arithmetic) as several tiles each; masks lie on every other lattice."""
import numpy as np
import pytest
import torch

from gpu_helpers import *  # noqa: F401,F403
from paper_2005_04642_amd import lbm, workloads as Wk

pytestmark = pytest.mark.gpu

N = 64


@pytest.mark.parametrize("storage", ["f32", "f64", "f16", "bf16"])
@pytest.mark.parametrize("kind", ["periodic", "walls", "masks"])
@pytest.mark.parametrize("count", [30, 256])
@pytest.mark.parametrize("stencil", [(3, 3, 3, 3), (1, 1, 1, 1)])
def test_batch_kernel_equals_single_lattices(storage, kind, count, stencil):
    p = Wk.base_params(Lambda=10.0, sigma=0.01, stencil=stencil)
    p.update(walls=kind == "walls", gx=1e-6 if kind == "walls" else 0.0)
    y, x = np.mgrid[0:N, 0:N]
    profiles = [np.tanh((r - np.hypot(x - 25.0, y - 36.0)) / 2.0) for r in (12.0, 18.0)]
    masks = [Wk.random_solid_sites(N, N, N * N // 15, 3), None] if kind == "masks" else [None, None]
    singles = []
    for rn, mask in zip(profiles, masks):
        s = lbm.Simulation(N, N, p, rn, storage=storage, solid=mask)
        s.step(4)
        singles.append(s)
    b = lbm.Batch([(N, N, p, profiles[k % 2]) for k in range(count)], storage=storage)
    for k in range(count):
        if masks[k % 2] is not None:
            b.set_solid(k, masks[k % 2])
    items = b.plan_info()["items"]
    if storage != "f64":      # (FP64 marches in narrower strips, and never runs tiles in a batch)
        assert items == count if count == 256 else items > count
    b.step(4)
    live = b.pops[b.lib.lbm_batch_current_pops(b.h)]
    rows = slice(1, -1) if kind == "walls" else slice(None)
    for k in range(count):
        want = singles[k % 2].live_words()[:, rows]
        n = want.element_size() * singles[0].pops[0].numel()
        got = live[b.offsets[k]:b.offsets[k] + n].view(want.dtype).view(N, -1, N).permute(1, 0, 2)[:, rows]
        assert torch.equal(got, want), k
    b.close()
    for s in singles:
        s.close()
