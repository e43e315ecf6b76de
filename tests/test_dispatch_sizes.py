"""Which form of a pass large, misaligned and long shapes take, where the form
measured fastest depends on more than the pass length."""
import numpy as np
import pytest

import oracle
from paper_1904_10119_amd import dft3d, inputs


def passes(shape, schedule="pencil", **kw):
    return dft3d.describe(shape, schedule, **kw)["passes"]


@pytest.mark.parametrize("shape", [(2048, 1000, 300), (1000, 2048, 200), (300, 1000, 2048),
                                   (2048, 500, 700), (2048, 1009, 200), (2048, 2048, 100)])
def test_axes_of_2048_beside_other_lengths_keep_the_halves_kernel(shape):
    """From 2.5 GiB up the cycled order would run the 2048 pass as a staged
    mixed-radix one; such shapes keep the rotation."""
    for p, n in zip(passes(shape), reversed(shape)):
        assert " cyc" not in p["label"], p["label"]
        if n == 2048:
            assert p["halves"] and not p["mixed"], p["label"]
    assert all(" cyc" in p["label"] for p in passes((1024, 1000, 900)))


@pytest.mark.parametrize("schedule", ["pencil", "slab"])
def test_64_points_on_large_grids_take_the_pass_kernel(schedule):
    """Above 2^22 points the 64-point rows take the pass kernel's tiles of 64
    pencils."""
    for k, split in (((1024, 64), [8, 8]), ((1024, 128), []), ((1201, 1201), [])):
        p = passes(k + (64,), schedule, fused_plane=0)[0]
        assert p["n"] == 64 and p["split"] == split and (split or p["tile"] == 64), (k, p)


def test_512_points_on_middle_grids_take_the_pass_kernel():
    """From 2^23 points up strided axes of 512 whose points lie less than 2 KB or
    128 KB and more apart, and from 2^23 to 2^24 the rotation, take the pass
    kernel; the columns between, rows and the larger rotations two steps."""
    def split(shape, schedule, at):
        p = passes(shape, schedule, fused_plane=0)[at]
        assert p["n"] == 512
        return p["split"]
    assert split((512, 128, 64), "slab", -1) == [16, 32]      # 2^22
    assert split((512, 256, 64), "slab", -1) == []            # 2^23
    assert split((512, 512, 64), "slab", 1) == []             # 512 B apart
    assert split((64, 512, 256), "slab", 1) == [16, 32]       # 2 KB
    assert split((16, 512, 1024), "slab", 1) == [16, 32]
    assert split((8, 512, 4096), "slab", 1) == [16, 32]       # 32 KB
    assert split((512, 4, 4096), "slab", -1) == []            # 128 KB
    assert split((64, 512, 512), "slab", 0) == [16, 32]
    assert split((64, 256, 512), "pencil", 0) == []           # 2^23, rotated
    assert split((128, 256, 512), "pencil", 0) == [16, 32]    # 2^24
    assert split((64, 256, 512), "slab", 0) == [16, 32]


@pytest.mark.parametrize("precision", ["bf16x6", "bf16x9", "fp16x3", "bf16x1", "fp16x1"])
def test_split_passes_that_keep_the_layout_take_small_tiles_up_to_2_20(precision):
    """Above 2^20 points the in-layout split-precision passes keep 8192-point
    tiles; the rotating ones of 256 points take less up to 2^22."""
    def points(shape, schedule):
        return {p["n"]: p["tile"] * p["n"] for p in
                passes(shape, schedule, precision=precision, fused_plane=0)}
    assert points((16, 512, 256), "slab") == {256: 8192, 512: 8192, 16: 8192}
    assert points((16, 256, 256), "slab") == {256: 4096, 16: 4096}
    assert points((32, 256, 256), "pencil")[256] == 4096


def test_half_tiles_of_the_longest_lengths():
    """2048 and 4096 points take half the pencils where workgroups are few:
    fewer than 256, or 128 for columns of 4096."""
    def tile(shape, schedule, **kw):
        return next(p["tile"] for p in passes(shape, schedule, fused_plane=0, split_max=4096, **kw)
                    if p["n"] == max(shape))
    assert tile((4096, 16, 16), "slab") == 2
    assert tile((4096, 16, 32), "slab") == 4
    assert tile((16, 32, 4096), "slab") == 2
    assert tile((4096, 16, 32), "pencil") == 2
    assert tile((32, 32, 4096), "slab") == 4
    assert tile((2048, 32, 32), "slab", halves=0) == 4
    assert tile((2048, 64, 32), "slab", halves=0) == 8


def test_misaligned_rotation_of_powers_of_two():
    """Rotating passes of 64 and 256 points whose rows do not start on 128-byte
    lines take the pass kernel's longer tiles on large grids."""
    def split(shape):
        return next(bool(p["split"]) for p in passes(shape) if p["n"] in (64, 256))
    assert not split((251, 64, 251)) and split((127, 64, 129)) and split((256, 64, 250))
    assert not split((255, 256, 511)) and split((127, 256, 129)) and split((256, 256, 500))
    assert passes((251, 251, 64), "slab")[0]["split"] == [8, 8]


def test_auto_with_one_misaligned_axis_beside_a_longer_one():
    """From 2^25 points up such shapes keep the rotation, whose wide tiles are
    ahead of the slab where the slab's column segments are off the 64-byte halves
    of the lines too (n2 no multiple of 8); the others take the slab."""
    def sched(shape):
        return dft3d.describe(shape, "auto")["schedule"]
    assert sched((400, 875, 300)) == "pencil" and sched((400, 945, 300)) == "pencil"
    assert sched((640, 343, 675)) == "pencil" and sched((378, 432, 660)) == "pencil"
    assert sched((275, 750, 504)) == "slab" and sched((756, 275, 432)) == "slab"
    assert sched((1053, 210, 936)) == "slab"
    assert sched((400, 539, 300)) == "slab"
    assert sched((56, 700, 275)) == "slab" and sched((308, 169, 630)) == "slab"
    assert sched((468, 392, 735)) == "slab"


SHORT = [48, 49, 56, 60, 72, 80, 90, 96, 98, 100, 104, 105, 112, 117, 120, 125, 126]


@pytest.mark.parametrize("n", SHORT)
def test_short_lengths_on_large_grids_take_wide_tiles(n):
    """From 2^17 pencils up the two-step passes of 48..127 points take 32 or 64
    pencils, in every order, so that row segments span several lines."""
    b = passes((1, 1, n))[0]["split"][1]
    for k, want in (((2040, 64), 16), ((2048, 64), 64 if b <= 12 else 32),
                    ((2048, 256), 64 if b <= 16 else 32)):
        for shape, schedule, at in ((k + (n,), "pencil", 0), (k + (n,), "slab", 0),
                                    ((n,) + k, "slab", -1)):
            p = passes(shape, schedule, fused_plane=0)[at]
            assert p["split"] and p["pencils"] == k[0] * k[1]
            assert p["tile"] == want, (shape, schedule, p["tile"], want)
            assert p["threads"] <= 1024 and p["lds_bytes"] <= 160 * 1024
    assert passes((2048, 2048, 45))[0]["tile"] == 16


@pytest.mark.parametrize("n", [640, 768, 896, 1000])
def test_long_misaligned_rotations_on_small_grids_take_tiles_of_8(n):
    """From 640 points up 8 pencils, to 1344 tiles of 16 where rotated rows do
    not start on 128-byte lines, to 544 where they do."""
    def tile(a, b):
        return passes((a, b, n))[0]["tile"]
    assert tile(101, 203) == 8 and tile(151, 263) == 16
    assert tile(104, 200) == 16 and tile(64, 136) == 8


def bar(shape):
    """log2(n) + 1 rounding levels an axis at the tol(N) rate of 1e-6 / 18 a level."""
    return 1e-6 * sum(np.log2(n) + 1 for n in shape if n > 1) / 18.0


def check_sampled(shape, schedule, seed):
    """Sampled output pencils, the last of each axis among them, against the
    oracle's direct sums, and the round trip."""
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    x = inputs.uniform_c64(shape, seed)
    xt = torch.from_numpy(x).cuda()
    y = dft3d.fftn(xt, schedule=schedule)
    torch.cuda.synchronize()
    g = np.random.default_rng(seed)
    k0 = np.concatenate([[0, shape[0] - 1], g.integers(0, shape[0], 4)])
    k1 = np.concatenate([[0, shape[1] - 1], g.integers(0, shape[1], 4)])
    got = y[torch.from_numpy(k0).cuda(), torch.from_numpy(k1).cuda(), :].cpu().numpy()
    assert oracle.rel_l2(got, oracle.sample_pencils(x, k0, k1, -1)) <= bar(shape)
    back = dft3d.ifftn(y, schedule=schedule) / x.size
    rt = (torch.linalg.vector_norm(back - xt) / torch.linalg.vector_norm(xt)).item()
    assert rt <= 2 * bar(shape)


@pytest.mark.parametrize("n", [130, 144, 192, 240, 300, 375, 384, 500, 600, 625])
def test_misaligned_rotation_takes_wider_tiles(n):
    """From 2^16 pencils up the rotating passes whose rows do not start on
    128-byte lines take 32 pencils, from 2^18 48 where they fit; aligned rows,
    fewer pencils and the orders that keep the layout take 16."""
    def tile(shape, schedule="pencil", at=0):
        p = passes(shape, schedule, fused_plane=0)[at]
        assert p["mixed"] and p["lds_bytes"] <= 160 * 1024
        return p["tile"]
    assert tile((257, 257, n)) == 32 and tile((256, 256, n)) == 16
    assert tile((257, 253, n)) == 16
    a, b = passes((1, 1, n))[0]["split"]
    fits = 48 * b <= 1024 and 48 * (a * (b | 1) | 1) * 8 <= 160 * 1024
    assert tile((513, 513, n)) == (48 if fits else 32) and tile((512, 528, n)) == 16
    assert tile((257, 257, n), "slab") == 16 and tile((n, 257, 257), "slab", -1) == 16


@pytest.mark.gpu
@pytest.mark.parametrize("shape", [(363, 362, 60), (363, 96, 362), (105, 363, 362),
                                   (363, 362, 125), (725, 112, 724), (48, 363, 362)])
@pytest.mark.parametrize("schedule", ["pencil", "slab"])
def test_wide_tiles_on_the_gpu(shape, schedule):
    """Tiles of 64 and 32 pencils in every order, with a ragged last tile."""
    print("case wide tiles", shape, schedule, flush=True)
    short = min(shape)
    assert any(p["pencils"] * short == np.prod(shape) and p["tile"] in (32, 64)
               for p in passes(shape, schedule))
    check_sampled(shape, schedule, 81)


@pytest.mark.gpu
@pytest.mark.parametrize("shape", [(257, 257, 130), (257, 192, 259), (375, 259, 257),
                                   (257, 257, 625), (515, 130, 513), (300, 513, 513)])
def test_misaligned_tiles_of_32_on_the_gpu(shape):
    """Tiles of 32 pencils with rows off the 128-byte lines and a ragged last
    tile."""
    print("case misaligned tiles", shape, flush=True)
    assert any(p["tile"] in (32, 48) and p["split"] for p in passes(shape))
    check_sampled(shape, "pencil", 82)
