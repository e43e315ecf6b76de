"""GPU parity of kernels that the default plans of small shapes do not reach:
the staged mixed-radix kernels (asked for by a tile or a radix sequence) and
every tile and order of the power-of-two two-step passes.

Tolerances: log2(n) rounding levels for a power-of-two axis, log2(n) + 1 for
a mixed-radix one, at the tol(N) rate of 1e-6 / 18 a level; one level more for
a stage order of its own."""
import numpy as np
import pytest

import oracle
from paper_1904_10119_amd import dft3d, inputs


def bar(shape):
    return 1e-6 * sum(np.log2(n) + (n & (n - 1) != 0) for n in shape if n > 1) / 18.0


def gpu():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


def check(shape, schedule, seed, extra=0.0, **kw):
    torch = gpu()
    x = inputs.uniform_c64(shape, seed)
    for sign in (-1, 1):
        y = dft3d.fftn(torch.from_numpy(x).cuda(), schedule=schedule, inverse=sign == 1, **kw)
        torch.cuda.synchronize()
        err = oracle.rel_l2(y.cpu().numpy(), oracle.dft3d(x.astype(np.complex128), sign, "direct"))
        assert err <= bar(shape) + extra, (shape, schedule, kw, sign, err)


def staged_passes(shape, schedule, n, **kw):
    ps = [p for p in dft3d.describe(shape, schedule, **kw)["passes"]
          if p["mixed"] and n * p["pencils"] == np.prod(shape) and p["args"]["res_mask"] == n]
    assert ps and all(p["split"] == [] for p in ps), (shape, schedule, kw)
    return ps


# lengths of every bound of the staged kernel (32, 128, 512, 1024, 2048)
STAGED = [18, 30, 45, 96, 117, 125, 143, 250, 375, 486, 500, 539, 715, 1000, 1100, 1344, 1980]


def test_asked_tiles_reach_every_staged_kernel():
    """Over the lengths and tiles of the next test every bound of the staged
    kernel runs in its own tile."""
    seen = set()
    for n in STAGED:
        for tile in (2, 4, 8, 16, 64, 256):
            for p in staged_passes((5, 3, n), "pencil", n, tile=tile):
                seen.add((p["n"], p["tile"]))
    assert {b for b, _ in seen} >= {32, 128, 512, 1024, 2048}, seen
    assert {(512, 16), (1024, 8), (128, 64), (2048, 4), (32, 256)} <= seen, seen


@pytest.mark.gpu
@pytest.mark.parametrize("tile", [2, 4, 8, 16, 64, 256])
@pytest.mark.parametrize("n", STAGED)
def test_staged_kernels_by_tile(n, tile):
    """Rotating, row and column passes, ragged, both directions."""
    gpu()
    for shape, schedule in (((5, 3, n), "pencil"), ((5, 3, n), "slab"), ((n, 3, 7), "slab")):
        print("case staged", shape, schedule, "tile", tile, flush=True)
        staged_passes(shape, schedule, n, tile=tile)
        check(shape, schedule, 71, tile=tile)


@pytest.mark.gpu
@pytest.mark.parametrize("n,radices", [(143, [11, 13]), (1000, [10, 10, 2, 5]), (1000, [5, 10, 10, 2]),
                                       (96, [8, 4, 3]), (375, [3, 5, 5, 5]), (1001, [7, 11, 13]),
                                       (64, [4, 16]), (720, [8, 10, 3, 3])])
def test_staged_kernels_by_radix_sequence(n, radices):
    """Stage orders that are not the length's own, against the oracle."""
    gpu()
    assert int(np.prod(radices)) == n
    for shape, schedule in (((5, 3, n), "pencil"), ((5, 3, n), "slab"), ((n, 3, 7), "slab")):
        print("case radices", shape, schedule, radices, flush=True)
        for p in staged_passes(shape, schedule, n, radices=radices):
            assert p["radices"] == radices, (p["radices"], radices)
        check(shape, schedule, 72, 1e-6 / 18, radices=radices)


# (length, tile, load, store) of every registered two-step kernel of a power
# of two, and a plan whose pass it is
POWER = [((16, 16), [((8, 4, 16), "pencil"), ((8, 4, 16), "slab"), ((16, 8, 4), "slab")]),
         ((32, 16), [((8, 4, 32), "pencil"), ((8, 4, 32), "slab"), ((32, 8, 4), "slab")]),
         ((64, 16), [((8, 4, 64), "pencil"), ((8, 4, 64), "slab"), ((64, 8, 4), "slab")]),
         ((64, 32), [((256, 256, 64), "pencil"), ((256, 256, 64), "slab")]),
         ((128, 16), [((8, 4, 128), "pencil"), ((8, 4, 128), "slab"), ((128, 8, 4), "slab")]),
         ((256, 8), [((8, 4, 256), "pencil"), ((8, 4, 256), "slab"), ((256, 8, 4), "slab")]),
         ((256, 16), [((128, 128, 256), "pencil"), ((128, 128, 256), "slab"),
                      ((256, 128, 128), "slab")]),
         ((256, 32), [((512, 512, 256), "pencil"), ((512, 512, 256), "slab"),
                      ((256, 512, 512), "slab")]),
         ((512, 8), [((8, 4, 512), "pencil"), ((8, 4, 512), "slab"), ((512, 8, 4), "slab")]),
         ((512, 16), [((256, 128, 512), "pencil"), ((128, 128, 512), "slab")]),
         ((1024, 8), [((8, 4, 1024), "pencil"), ((8, 4, 1024), "slab"), ((1024, 16, 8), "slab")]),
         ((1024, 16), [((128, 128, 1024), "pencil"), ((128, 128, 1024), "slab")])]


def power_pass(shape, schedule, n, tile):
    kw = {"persistent": 0, "nontemporal": 0} if n == 256 and tile == 32 else {}
    if (n, shape[0]) == (1024, 1024):
        kw["halves"] = 0
    ps = [p for p in dft3d.describe(shape, schedule, fused_plane=0, **kw)["passes"]
          if p["n"] == n and p["tile"] == tile and p["split"] and not p["mixed"]]
    return ps, kw


def test_power_cases_reach_every_tile_and_order():
    for (n, tile), plans in POWER:
        orders = set()
        for shape, schedule in plans:
            ps, _ = power_pass(shape, schedule, n, tile)
            assert ps, (n, tile, shape, schedule)
            orders |= {(p["load"], p["store"]) for p in ps}
        want = {("row", "col"), ("row", "row"), ("col", "col")}
        if (n, tile) in ((64, 32), (512, 16), (1024, 16)):
            want.discard(("col", "col"))  # these grids leave for other kernels
        assert orders == want, (n, tile, orders)


@pytest.mark.gpu
@pytest.mark.parametrize("case", POWER, ids=lambda c: "%dx%d" % c[0])
def test_power_of_two_tiles_on_the_gpu(case):
    torch = gpu()
    (n, tile), plans = case
    for shape, schedule in plans:
        print("case power", n, tile, shape, schedule, flush=True)
        _, kw = power_pass(shape, schedule, n, tile)
        x = inputs.uniform_c64(shape, 73)
        xt = torch.from_numpy(x).cuda()
        y = dft3d.fftn(xt, schedule=schedule, fused_plane=0, **kw)
        torch.cuda.synchronize()
        if x.size <= 1 << 20:
            ref = oracle.dft3d(x.astype(np.complex128), -1, "fft")
            assert oracle.rel_l2(y.cpu().numpy(), ref) <= bar(shape), (shape, schedule)
        else:
            g = np.random.default_rng(n)
            k0 = np.concatenate([[0, shape[0] - 1], g.integers(0, shape[0], 4)])
            k1 = np.concatenate([[0, shape[1] - 1], g.integers(0, shape[1], 4)])
            got = y[torch.from_numpy(k0).cuda(), torch.from_numpy(k1).cuda(), :].cpu().numpy()
            ref = oracle.sample_pencils(x, k0, k1, -1)
            assert oracle.rel_l2(got, ref) <= bar(shape), (shape, schedule)
        back = dft3d.ifftn(y, schedule=schedule, fused_plane=0, **kw) / x.size
        rt = (torch.linalg.vector_norm(back - xt) / torch.linalg.vector_norm(xt)).item()
        assert rt <= 2 * bar(shape), (shape, schedule, rt)
