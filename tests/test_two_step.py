"""Two-step mixed-radix passes (a length n = A B in two register DFTs and one
exchange): the split and its formulas on the CPU, the pass lists that use
them, and GPU parity against the oracle at the edges of the kernels' range.

Tolerance on the GPU: log2(n) + 1 rounding levels per axis at the tol(N) rate
of 1e-6 / 18 per level, the bar of every mixed-radix axis."""
import numpy as np
import pytest

import oracle
from paper_1904_10119_amd import dft3d, inputs

TWO_STEP = {6: [2, 3], 30: [5, 6], 96: [8, 12], 125: [5, 25], 143: [11, 13], 375: [15, 25],
            486: [18, 27], 720: [24, 30], 1000: [25, 40], 1008: [28, 36], 1024: [32, 32],
            343: [7, 49], 1089: [33, 33], 1100: [25, 44], 1600: [40, 40], 1980: [44, 45]}


def smooth13(n):
    for f in (2, 3, 5, 7, 11, 13):
        while n % f == 0:
            n //= f
    return n == 1


def first_pass(n, **kw):
    return dft3d.describe((3, 5, n), "pencil", **kw)["passes"][0]


def test_which_lengths_split():
    """Smooth lengths 6..2000 with a factor pair A <= B <= 50 (48 from 1700 up)
    take a two-step pass with the most even pair, in tiles of 16 pencils where
    B <= 40 and the LDS holds them, else 8; a tile option keeps the staged
    kernels."""
    for n in range(2, 2101):
        if n & (n - 1) == 0 or not smooth13(n):
            continue
        p = first_pass(n)
        most = 50 if n < 1700 else 48
        pairs = [a for a in range(2, 46) if n % a == 0 and a * a <= n and n // a <= most]
        assert p["split"] == ([max(pairs), n // max(pairs)] if pairs and 6 <= n <= 2000 else []), n
        if p["split"]:
            a, b = p["split"]
            fits = b <= 40 and 16 * (a * (b | 1) | 1) * 8 <= 160 * 1024
            assert p["fixed_n"] == n and p["tile"] == (16 if fits and n < 360 else 8)
            assert p["threads"] >= p["tile"] * b and p["lds_bytes"] <= 160 * 1024
        assert first_pass(n, tile=16)["split"] == []
    # tiles of 8 where 16 leave CUs idle: up to 256 tiles, from 512 up to 544
    for n, m in ((375, 64), (500, 64), (585, 136), (1000, 136), (1100, 136)):
        tiles = [dft3d.describe((k, 64, n), "pencil")["passes"][0]["tile"] for k in (m, m + 1)]
        assert tiles == ([8, 16] if n != 1100 else [8, 8]), n


@pytest.mark.parametrize("n", sorted(TWO_STEP))
def test_two_step_formulas(n):
    """Step 1: DFT_A of x[t + r B] over r; step 2: DFT_B over t of row tm
    times w_n^{tm t}, output j at tm + A j -- equals the direct sum."""
    p = first_pass(n)
    if n & (n - 1):
        assert p["split"] == TWO_STEP[n]
    A, B = TWO_STEP[n]
    g = np.random.default_rng(n)
    x = g.standard_normal(n) + 1j * g.standard_normal(n)
    rows = np.fft.fft(x.reshape(A, B), axis=0)                      # [tm][t]
    tm, t = np.arange(A)[:, None], np.arange(B)[None, :]
    y = np.fft.fft(rows * np.exp(-2j * np.pi * (tm * t % n) / n), axis=1)
    got = y.T.reshape(-1)                                           # [j][tm]
    ref = oracle.dft3d(x.reshape(n, 1, 1), -1, "direct").reshape(-1)
    assert oracle.rel_l2(got, ref) < 1e-12


def test_auto_schedule_of_other_lengths():
    """AUTO keeps the pencil rotation where its rows start on 128-byte lines,
    for small grids and for axes without a two-step pass, takes the slab
    schedule where they do not, and either gives way to options that name a
    pencil form; from 2.5 GiB up the pencil passes run in the cycle."""
    def sched(shape, **kw):
        return dft3d.describe(shape, "auto", **kw)["schedule"]
    assert sched((375, 486, 400)) == "slab" and sched((105, 105, 105)) == "slab"
    assert sched((324, 324, 324)) == "pencil" and sched((400, 400, 400)) == "pencil"
    assert sched((343, 343, 64)) == "slab" and sched((882, 882, 64)) == "pencil"
    assert sched((61, 75, 90)) == "pencil" and sched((101, 375, 375)) == "pencil"
    assert sched((675, 675, 675)) == "pencil" and sched((375, 375, 2048)) == "pencil"
    for kw in ({"tile": 16}, {"radices": [3, 5, 5, 5]}, {"pencil_order": 0}):
        assert sched((375, 375, 375), **kw) == "pencil", kw

    def cycled(shape, **kw):
        return [" cyc" in p["label"] for p in dft3d.describe(shape, "pencil", **kw)["passes"]]
    assert cycled((1000, 1000, 1000)) == [True] * 3
    assert cycled((1001, 1001, 1001)) == [True] * 3
    assert cycled((1024, 1000, 900)) == [True] * 3
    assert cycled((600, 600, 600)) == [False] * 3
    assert cycled((1000, 1000, 1000), pencil_order=0) == [False] * 3


@pytest.mark.parametrize("shape", [(1000, 700, 500), (1024, 1000, 900), (1001, 1009, 1013)])
def test_cycled_order_of_other_lengths(shape):
    """Each pass of the cycle reads and writes the documented orders: random
    pencils of every pass land on (A, B, C) -> (B, C, A) -> (C, A, B) -> (A,
    B, C), whatever the axis lengths."""
    A, B, C = shape
    d = dft3d.describe(shape, "pencil")
    g = np.random.default_rng(A)
    orders = [((0, 1, 2), (1, 2, 0), 2), ((1, 2, 0), (2, 0, 1), 0), ((2, 0, 1), (0, 1, 2), 1)]
    for p, (order_in, order_out, axis) in zip(d["passes"], orders):
        a = p["args"]
        assert a["B"] * shape[axis] == A * B * C
        # the pencil index runs over the slowest axis of the input fastest
        fast, slow = order_in[0], order_in[1]
        b = g.integers(0, a["B"], 200)
        if a["s0"] < 0:
            f0, f1, f2 = b % a["m0"], (b // a["m0"]) % a["m1"], b // (a["m0"] * a["m1"])
        else:
            f0, f1, f2 = b & a["m0"], (b >> a["s0"]) & a["m1"], b >> a["s1"]
        j = g.integers(0, shape[axis], 200)
        idx = {fast: b % shape[fast], slow: b // shape[fast], axis: j}

        def place(order):
            return (idx[order[0]] * shape[order[1]] + idx[order[1]]) * shape[order[2]] + idx[order[2]]
        got_in = f2 * a["is"][2] + f1 * a["is"][1] + f0 * a["is"][0] + j * a["ijs"]
        got_out = f2 * a["os"][2] + f1 * a["os"][1] + f0 * a["os"][0] + j * a["oks"]
        assert (got_in == place(order_in)).all() and (got_out == place(order_out)).all()


def test_power_of_two_passes_in_two_steps():
    """FP32 passes of 16..1024 points without a four-step twiddle: tiles by
    length and pencils, the pass kernels where an option asks for their forms,
    the halves kernels only where their tiles fill the CUs."""
    def pick(shape, schedule="pencil", **kw):
        return [(p["n"], p["tile"], bool(p["split"])) for p in
                dft3d.describe(shape, schedule, **kw)["passes"]]
    assert pick((64, 32, 16)) == [(16, 16, True), (32, 16, True), (64, 16, True)]
    assert pick((256, 256, 256)) == [(256, 16, True)] * 3
    assert pick((16, 256, 256)) == [(256, 8, True), (256, 8, True), (16, 16, True)]
    assert pick((1024, 1024, 1024)) == [(1024, 16, True)] * 3
    assert pick((256, 512, 512))[1] == (256, 32, True)             # cycled: axes 2, 0, 1
    assert pick((64, 1024, 64), "slab")[0] == (64, 32, True)
    assert pick((128, 512, 512))[1] == (128, 32, False)
    assert pick((16, 512, 512), "slab")[2] == (16, 256, False)
    assert pick((64, 32, 16), tile=64)[2] == (64, 64, False)
    assert not any(s for _, _, s in pick((1024, 1024, 1024), nontemporal=1))
    assert pick((1024, 16, 64), "slab")[-1] == (1024, 8, True)       # 32 halves tiles
    assert pick((1024, 128, 64), "slab")[-1] == (1024, 32, False)    # 256 of them
    assert pick((2048, 32, 32), "slab")[-1] == (2048, 4, False)
    assert pick((2048, 64, 64), "slab")[-1] == (2048, 16, False)


def bar(shape):
    return 1e-6 * sum(np.log2(n) + 1 for n in shape if n > 1) / 18.0


@pytest.mark.gpu
@pytest.mark.parametrize("schedule", ["pencil", "slab"])
@pytest.mark.parametrize("shape", [(6, 7, 30), (5, 17, 96), (125, 6, 16), (9, 143, 15),
                                   (3, 375, 33), (32, 486, 5), (720, 3, 7), (1, 1000, 17),
                                   (1008, 5, 1), (1024, 3, 5), (3, 1024, 6), (105, 49, 27),
                                   (343, 3, 17), (5, 1089, 9), (1100, 3, 3), (3, 7, 1250),
                                   (1600, 3, 3), (3, 1617, 3), (3, 3, 1980)])
def test_two_step_passes_on_the_gpu(shape, schedule):
    """Smallest, largest and ragged cases of every order (rotating, rows,
    columns), whole and ragged tiles, forward and inverse."""
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print("case two-step", shape, schedule, flush=True)
    x = inputs.uniform_c64(shape, 61)
    for sign in (-1, 1):
        y = dft3d.fftn(torch.from_numpy(x).cuda(), schedule=schedule, inverse=sign == 1)
        torch.cuda.synchronize()
        err = oracle.rel_l2(y.cpu().numpy(), oracle.dft3d(x.astype(np.complex128), sign, "direct"))
        assert err <= bar(shape), (shape, schedule, sign, err)


@pytest.mark.gpu
@pytest.mark.parametrize("shape", [(750, 720, 650), (225, 105, 75)])
def test_auto_choices_of_other_lengths_on_the_gpu(shape):
    """The cycle (above 2.5 GiB) and the slab choice of AUTO: sampled pencils
    against the oracle's direct sums, and the round trip."""
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print("case auto other lengths", shape, flush=True)
    x = inputs.uniform_c64(shape, 62)
    xt = torch.from_numpy(x).cuda()
    y = dft3d.fftn(xt)
    torch.cuda.synchronize()
    g = np.random.default_rng(62)
    k0 = np.concatenate([[0, shape[0] - 1], g.integers(0, shape[0], 4)])
    k1 = np.concatenate([[0, shape[1] - 1], g.integers(0, shape[1], 4)])
    got = y[torch.from_numpy(k0).cuda(), torch.from_numpy(k1).cuda(), :].cpu().numpy()
    assert oracle.rel_l2(got, oracle.sample_pencils(x, k0, k1, -1)) <= bar(shape)
    back = dft3d.ifftn(y) / x.size
    rt = (torch.linalg.vector_norm(back - xt) / torch.linalg.vector_norm(xt)).item()
    assert rt <= 2 * bar(shape)


@pytest.mark.gpu
@pytest.mark.parametrize("shape,schedule", [((16, 32, 64), "slab"), ((64, 1024, 64), "slab"),
                                            ((1024, 8, 256), "slab"), ((8, 512, 1024), "pencil"),
                                            ((2048, 64, 4), "slab"), ((4, 32, 16), "pencil")])
def test_power_of_two_passes_on_the_gpu(shape, schedule):
    """Every tile of the power-of-two two-step passes and the forms that
    replace the halves kernels on small grids, against the FP64 oracle."""
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print("case two-step powers", shape, schedule, flush=True)
    x = inputs.uniform_c64(shape, 63)
    tol = 1e-6 * np.log2(x.size) / 18
    for sign in (-1, 1):
        y = dft3d.fftn(torch.from_numpy(x).cuda(), schedule=schedule, inverse=sign == 1)
        torch.cuda.synchronize()
        err = oracle.rel_l2(y.cpu().numpy(), oracle.dft3d(x.astype(np.complex128), sign, "fft"))
        assert err <= tol, (shape, schedule, sign, err)
