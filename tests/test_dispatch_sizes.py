"""Which form of a pass large, misaligned and long shapes take, where the form
measured fastest depends on more than the pass length."""
import pytest

from paper_1904_10119_amd import dft3d


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
