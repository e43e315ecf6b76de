"""Every compiled two-step mixed-radix kernel: each length 6..2000 that splits,
in each of its tiles and orders, launched on the GPU and compared element by
element with the DFT matrices in FP64.

Tolerance: log2(n) + 1 rounding levels an axis at the tol(N) rate of 1e-6 / 18
a level, the bar of every mixed-radix axis."""
import numpy as np
import pytest

from paper_1904_10119_amd import dft3d


def smooth13(n):
    for f in (2, 3, 5, 7, 11, 13):
        while n % f == 0:
            n //= f
    return n == 1


def split(n):
    """[A, B] of a length's two-step pass, [] if it has none."""
    if n & (n - 1) == 0 or not smooth13(n):
        return []
    return dft3d.describe((3, 5, n), "pencil")["passes"][0]["split"]


LENGTHS = [n for n in range(6, 2001) if split(n)]


def cases(n):
    """(shape, schedule, the pass of length n, its tile): small ragged grids,
    grids past the idle-CU rule, the wide tiles below 128 points and the tiles
    of 32 and 48 for rows off the 128-byte lines."""
    b = split(n)[1]
    base = 16 if b <= 40 and 16 * (n // b * (b | 1) | 1) * 8 <= 160 * 1024 else 8
    small = base if n < 360 else 8
    out = [((12, 10, n), "pencil", 0, small), ((12, 10, n), "slab", 0, small),
           ((n, 12, 10), "slab", -1, small)]
    if base == 16:
        out += [((84, 104, n), "pencil", 0, 16), ((84, 104, n), "slab", 0, 16),
                ((n, 84, 104), "slab", -1, 16)]
    if 48 <= n < 128:
        wide = [((364, 363), 64 if b <= 12 else 32)]
        if 12 < b <= 16:
            wide.append(((728, 726), 64))
        for k, t in wide:
            out += [(k + (n,), "pencil", 0, t), (k + (n,), "slab", 0, t),
                    ((n,) + k, "slab", -1, t)]
    if n >= 128 and base == 16:
        fits = [t for t in (32, 48) if t * b <= 1024 and
                t * (n // b * (b | 1) | 1) * 8 <= 160 * 1024]
        if fits:
            out.append(((255, 273, n), "pencil", 0, 32))
        if fits[1:]:
            out.append(((525, 507, n), "pencil", 0, 48))
    return out


def this_pass(n, shape, schedule, at):
    p = dft3d.describe(shape, schedule, fused_plane=0)["passes"][at]
    assert p["split"] == split(n) and p["fixed_n"] == n, (n, shape, schedule)
    return p


def test_cases_reach_every_tile():
    """The planner takes the tile each case is for."""
    assert len(LENGTHS) > 250
    for n in LENGTHS:
        for shape, schedule, at, tile in cases(n):
            assert this_pass(n, shape, schedule, at)["tile"] == tile, (n, shape, schedule)


def bar(shape):
    return 1e-6 * sum(np.log2(n) + 1 for n in shape if n > 1) / 18.0


def dft_matrix(torch, n):
    j = torch.arange(n, device="cuda", dtype=torch.int64)
    angle = (j[:, None] * j[None, :] % n).to(torch.float64) * (-2.0 * np.pi / n)
    return torch.complex(torch.cos(angle), torch.sin(angle))


def reference(torch, x):
    """The 3D DFT of x from the matrices of its axes, in FP64."""
    a, b, c = x.shape
    y = x.to(torch.complex128)
    y = (y.reshape(a * b, c) @ dft_matrix(torch, c)).reshape(a, b, c)
    y = y.transpose(1, 2).reshape(a * c, b) @ dft_matrix(torch, b)
    y = y.reshape(a, c, b).transpose(1, 2).reshape(a, b * c)
    return (dft_matrix(torch, a) @ y).reshape(a, b, c)


@pytest.mark.gpu
@pytest.mark.parametrize("part", range(32))
def test_every_kernel_on_the_gpu(part):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    g = torch.Generator(device="cuda")
    g.manual_seed(100 + part)
    for n in LENGTHS[part::32]:
        ref_of = None
        for shape, schedule, at, tile in cases(n):
            print("case length", n, shape, schedule, "tile", tile, flush=True)
            if ref_of != shape:
                x = torch.view_as_complex(
                    torch.empty(*shape, 2, device="cuda").uniform_(-1, 1, generator=g))
                ref, ref_of = reference(torch, x), shape
                norm = torch.linalg.vector_norm(ref)
            y = dft3d.fftn(x, schedule=schedule, fused_plane=0)
            err = (torch.linalg.vector_norm(y - ref) / norm).item()
            assert err <= bar(shape), (shape, schedule, tile, err)
        dft3d._plans.clear()
