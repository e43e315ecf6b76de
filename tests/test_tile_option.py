"""DFT3D_OPT_TILE: the pencils per workgroup asked for are the ones that run,
for every kind of pass that has such a kernel."""
import numpy as np
import pytest

import oracle
from paper_1904_10119_amd import dft3d, inputs

# Bluestein lengths and the tiles they have, the default first
BLUESTEIN = {17: (16, 64), 31: (16, 64), 37: (16, 32, 8), 61: (16, 32, 8), 67: (16, 32, 8),
             127: (16, 32, 8), 131: (8, 4, 16), 251: (8, 4, 16), 263: (8, 16, 4),
             509: (8, 16, 4), 521: (4, 8, 2), 1021: (4, 8, 2), 1031: (4, 2, 1), 2053: (2, 1)}


def passes(shape, schedule="pencil", **kw):
    return dft3d.describe(shape, schedule, **kw)["passes"]


@pytest.mark.parametrize("n", sorted(BLUESTEIN))
def test_bluestein_tiles(n):
    default, *others = BLUESTEIN[n]
    for shape, schedule, at in (((3, 5, n), "pencil", 0), ((n, 3, 5), "slab", -1),
                                ((3, 5, n), "slab", 0)):
        def tile(**kw):
            p = passes(shape, schedule, rader=0, **kw)[at]
            assert p["bluestein"]
            return p["tile"]
        assert tile() == default
        for t in (default, *others):
            assert tile(tile=t) == t, (n, schedule, t)
        assert tile(tile=128) == default   # no such kernel


@pytest.mark.gpu
@pytest.mark.parametrize("n", [n for n in sorted(BLUESTEIN) if n < 1025])
def test_bluestein_tiles_on_the_gpu(n):
    """Every tile, rotating and in layout, ragged, both directions.  Tolerance:
    2 log2(m) + 3 rounding levels for the axis (m the power of two >= 2n - 1),
    log2 + 1 for the others, at 1e-6 / 18 a level."""
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    m = 1 << int(np.ceil(np.log2(2 * n - 1)))
    bar = 1e-6 * (2 * np.log2(m) + 3 + np.log2(3) + 1 + np.log2(7) + 1) / 18.0
    for shape, schedule in (((3, 7, n), "pencil"), ((n, 3, 7), "slab")):
        x = inputs.uniform_c64(shape, 91)
        for sign in (-1, 1):
            ref = oracle.dft3d(x.astype(np.complex128), sign, "direct")
            for t in BLUESTEIN[n]:
                print("case bluestein tile", shape, schedule, sign, t, flush=True)
                y = dft3d.fftn(torch.from_numpy(x).cuda(), schedule=schedule, inverse=sign == 1,
                               rader=0, tile=t)
                torch.cuda.synchronize()
                assert oracle.rel_l2(y.cpu().numpy(), ref) <= bar, (shape, schedule, sign, t)
