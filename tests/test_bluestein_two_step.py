"""Bluestein axes with two-step FFTs of a convolution length m = A B (lengths
up to 1024): the chosen m and the steps' formulas on the CPU, GPU parity at
both ends of every m's range.

Tolerance on the GPU: 2 log2(m) + 3 rounding levels for the axis (two FFTs
and three complex products), log2(n) + 1 for the others, at the tol(N) rate
of 1e-6 / 18 per level."""
import numpy as np
import pytest

import oracle
from paper_1904_10119_amd import dft3d, inputs


def smooth13(n):
    for f in (2, 3, 5, 7, 11, 13):
        while n % f == 0:
            n //= f
    return n == 1


def axis_pass(n):
    return dft3d.describe((1, 1, n), "pencil", rader=0)["passes"][0]


LENGTHS = [n for n in range(17, 1024) if not smooth13(n)]


def edge_lengths():
    """The shortest and the longest length of every convolution length."""
    by_m = {}
    for n in LENGTHS:
        by_m.setdefault(axis_pass(n)["n"], []).append(n)
    return sorted({n for ns in by_m.values() for n in (ns[0], ns[-1])})


def test_convolution_lengths():
    """m = A B >= 2 n with A even, so that only the lower half of every
    column of the A x B table is loaded and stored; never above the power of
    two the longer lengths take; a tile option keeps the pass."""
    last = 0
    for n in LENGTHS:
        p = axis_pass(n)
        A, B = p["split"]
        assert p["bluestein"] and p["n"] == A * B and A % 2 == 0
        assert 2 * n <= p["n"] <= max(64, 1 << int(np.ceil(np.log2(2 * n)))) and p["n"] >= last
        last = p["n"]
        assert p["threads"] >= p["tile"] * max(A, B) and p["lds_bytes"] <= 160 * 1024
    assert axis_pass(1031)["split"] == []
    assert dft3d.describe((1, 1, 251), "pencil", tile=4)["passes"][0]["bluestein"]


@pytest.mark.parametrize("n", [17, 31, 37, 61, 101, 127, 131, 251, 263, 331, 509, 521, 557, 599, 613, 661, 701, 751, 821, 877,
                               941, 1021])
def test_steps_give_the_dft(n):
    """The three steps as the kernel documents them, in numpy."""
    A, B = axis_pass(n)["split"]
    m = A * B
    g = np.random.default_rng(n)
    x = g.standard_normal(n) + 1j * g.standard_normal(n)
    j = np.arange(n)
    w = np.exp(-1j * np.pi * (j * j % (2 * n)) / n)
    h = np.zeros(m, complex)
    h[:n] = np.conj(w)
    h[m - j[1:]] = np.conj(w[1:])
    filt = (np.fft.fft(h) / m).reshape(B, A).T                       # [tm][k]
    pad = np.zeros(m, complex)
    pad[:n] = x * w
    table = pad.reshape(A, B)                                        # [r][t]
    assert not table[A // 2:].any()
    tm, t = np.arange(A)[:, None], np.arange(B)[None, :]
    tw = np.exp(-2j * np.pi * (tm * t % m) / m)
    rows = np.fft.fft(np.fft.fft(table, axis=0) * tw, axis=1) * filt
    swap = rows.imag + 1j * rows.real
    cols = np.fft.fft(np.fft.fft(swap, axis=1) * tw, axis=0)
    y = (cols.imag + 1j * cols.real).reshape(m)[:n] * w
    ref = oracle.dft3d(x.reshape(n, 1, 1), -1, "direct").reshape(-1)
    assert oracle.rel_l2(y, ref) < 1e-12


@pytest.mark.gpu
@pytest.mark.parametrize("n", edge_lengths())
def test_edges_of_every_convolution_length(n):
    """Rotating, row and column passes over ragged tiles, both directions."""
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print("case bluestein two-step", n, flush=True)
    p = axis_pass(n)
    bar = 1e-6 * (2 * np.log2(p["n"]) + 3 + np.log2(3) + 1 + np.log2(7) + 1) / 18.0
    for shape, schedule in (((3, 7, n), "pencil"), ((n, 3, 7), "slab"), ((7, 3, n), "slab")):
        x = inputs.uniform_c64(shape, 70)
        for sign in (-1, 1):
            y = dft3d.fftn(torch.from_numpy(x).cuda(), schedule=schedule, inverse=sign == 1,
                           rader=0)
            torch.cuda.synchronize()
            ref = oracle.dft3d(x.astype(np.complex128), sign, "direct")
            assert oracle.rel_l2(y.cpu().numpy(), ref) <= bar, (shape, schedule, sign)
