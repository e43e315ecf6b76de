"""Rader axes with two-step FFTs of n - 1 = A B (compiled primes up to 1009):
the steps' formulas on the CPU, GPU parity over ragged tiles in the rotating,
row and column passes.

Tolerance on the GPU: 2 log2(n) + 3 rounding levels for the axis (two FFTs,
the filter product and the added x[0]), log2 + 1 for the others, at the
tol(N) rate of 1e-6 / 18 per level."""
import numpy as np
import pytest

import oracle
from paper_1904_10119_amd import dft3d, inputs

PRIMES = [197, 257, 281, 401, 577, 641, 769, 1009]


def axis_pass(n, **kw):
    return dft3d.describe((1, 1, n), "pencil", **kw)["passes"][0]


@pytest.mark.parametrize("n", PRIMES)
def test_steps_give_the_dft(n):
    """The three steps as the kernel documents them, in numpy."""
    p = axis_pass(n)
    assert p["rader"] and p["threads"] >= p["tile"] * max(p["split"])
    assert p["threads"] <= 1024 and p["lds_bytes"] <= 160 * 1024
    assert axis_pass(n, tile=4)["rader"] and axis_pass(n, tile=4)["split"] == []
    A, B = p["split"]
    L = A * B
    assert L == n - 1
    for g in range(2, n):
        pw = np.array([pow(g, j, n) for j in range(L)])
        if len(set(pw)) == L:
            break
    r = np.random.default_rng(n)
    x = r.standard_normal(n) + 1j * r.standard_normal(n)
    b = np.exp(-2j * np.pi * pw[-np.arange(L) % L] / n)              # w_n^(g^-m)
    filt = (np.fft.fft(b) / L).reshape(B, A).T                       # [tm][k]
    tm, t = np.arange(A)[:, None], np.arange(B)[None, :]
    tw = np.exp(-2j * np.pi * (tm * t % L) / L)
    table = x[pw].reshape(A, B)                                      # [r][t]
    rows = np.fft.fft(np.fft.fft(table, axis=0) * tw, axis=1)
    dc = rows[0, 0]
    # the second transform is a forward one: outputs at the inverse powers
    conv = np.fft.fft(np.fft.fft(rows * filt, axis=1) * tw, axis=0).reshape(L)
    y = np.empty(n, complex)
    y[0] = x[0] + dc
    y[pw] = x[0] + conv
    ref = oracle.dft3d(x.reshape(n, 1, 1), -1, "direct").reshape(-1)
    assert oracle.rel_l2(y, ref) < 1e-12


def test_order_of_large_arrays():
    """From 2.5 GiB up the cycle of axes 2, 0, 1, but the rotation where two
    or more axes take Rader passes."""
    order = lambda s: [p["label"][6] for p in dft3d.describe(s, "pencil")["passes"]]
    assert order((1009, 1000, 1000)) == ["2", "0", "1"]
    assert order((769, 769, 769)) == order((401, 1009, 1000)) == ["2", "1", "0"]


@pytest.mark.gpu
@pytest.mark.parametrize("n", PRIMES)
def test_ragged_tiles(n):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print("case rader two-step", n, flush=True)
    bar = 1e-6 * (2 * np.log2(n) + 3 + np.log2(3) + 1 + np.log2(11) + 1) / 18.0
    for shape, schedule in (((3, 11, n), "pencil"), ((n, 3, 11), "slab"), ((11, 3, n), "slab"),
                            ((1, 1, n), "pencil")):
        x = inputs.uniform_c64(shape, 71)
        for sign in (-1, 1):
            y = dft3d.fftn(torch.from_numpy(x).cuda(), schedule=schedule, inverse=sign == 1)
            torch.cuda.synchronize()
            ref = oracle.dft3d(x.astype(np.complex128), sign, "direct")
            assert oracle.rel_l2(y.cpu().numpy(), ref) <= bar, (shape, schedule, sign)
