"""Tiles against the march where the tiles take several rounds of workgroups,
and lattices beside the lines where the plan turns from tiles to the march
(counts for 256 CUs); states and fields bit for bit."""
import pytest

from gpu_helpers import *  # noqa: F401,F403
from test_gpu_tile import check

pytestmark = pytest.mark.gpu


# FP32 and 16-bit: two rounds, three (16-bit: 126 region rows against 12 march
# iterations stay tiles, 132 against 11 march); FP64: two, three, four within
# the cache and beyond; one strip of more rows than three rounds on one CU hold
@pytest.mark.parametrize("nx,ny,storage,stencil", [
    (724, 724, "f32", (3, 3, 3, 3)), (1061, 1063, "f32", (1, 1, 1, 1)),
    (881, 880, "f16", (3, 3, 3, 3)), (881, 880, "bf16", (3, 3, 3, 3)), (518, 1620, "f16", (3, 3, 3, 3)),
    (512, 512, "f64", (3, 3, 3, 3)), (762, 762, "f64", (3, 3, 3, 3)), (1019, 1021, "f64", (1, 1, 1, 1)),
    (1019, 1020, "f64", (3, 1, 3, 1)), (1146, 1147, "f64", (1, 1, 1, 1)),
    (46, 200, "f16", (3, 3, 3, 3)), (46, 200, "bf16", (3, 3, 3, 3)),
])
def test_rounds_of_tiles_equal_march(nx, ny, storage, stencil):
    check(nx, ny, storage, stencil=stencil, steps=2)


@pytest.mark.parametrize("storage,n,stencil", [("f32", 724, (3, 3, 3, 3)), ("f64", 762, (3, 3, 3, 3)),
                                               ("f64", 1146, (1, 1, 1, 1)), ("f16", 881, (3, 3, 3, 3))])
@pytest.mark.parametrize("kind", [dict(walls=True), dict(solid=True)], ids=lambda d: "-".join(d))
def test_rounds_of_tiles_equal_march_options(storage, n, stencil, kind):
    check(n, n, storage, stencil=stencil, steps=2, **kind)
