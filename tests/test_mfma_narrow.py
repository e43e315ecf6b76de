"""Split-precision passes of small grids in tiles below the default (more
workgroups): which sizes take them, and GPU parity with whole and ragged
tiles in every order.  The split forms meet the FP32 tolerance tol(N); the
single-term forms the bounds of one rounded operand term."""
import numpy as np
import pytest

import oracle
from paper_1904_10119_amd import dft3d, inputs


def tiles(shape, **kw):
    kw.setdefault("precision", "bf16x6")
    return [(p["n"], p["tile"] * p["n"], p["mfma_leaf"])
            for p in dft3d.describe(shape, "pencil", pencil_order=0, **kw)["passes"]]


def test_which_sizes_take_small_tiles():
    assert tiles((64, 64, 64)) == [(64, 1024, 16)] * 3
    assert tiles((256, 16, 128)) == [(128, 1024, 32), (16, 1024, 16), (256, 2048, 32)]
    assert tiles((16, 512, 1024))[0:2] == [(1024, 8192, 16), (512, 8192, 16)]
    assert tiles((2, 512, 1024))[0:2] == [(1024, 4096, 16), (512, 4096, 16)]
    assert tiles((128, 128, 256)) == [(256, 4096, 32), (128, 4096, 32), (128, 4096, 32)]
    assert tiles((256, 256, 256)) == [(256, 8192, 32)] * 3
    assert tiles((16, 16, 2048))[0] == (2048, 16384, 16)
    # an asked-for tile, leaf or persistent form keeps the default tiles
    for kw in ({"tile": 16}, {"mfma_leaf": 16}, {"persistent": 1, "nontemporal": 1}):
        assert all(t == 8192 for _, t, _ in tiles((64, 64, 64), **kw)), kw


@pytest.mark.gpu
@pytest.mark.parametrize("precision", ["bf16x6", "bf16x9", "fp16x3", "bf16x1", "fp16x1"])
@pytest.mark.parametrize("schedule", ["pencil", "slab"])
def test_small_tiles_against_oracle(precision, schedule):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    for shape in ((16, 32, 64), (2, 2, 16), (128, 2, 256), (512, 4, 2), (2, 1024, 4),
                  (64, 128, 128), (16, 256, 256), (32, 1024, 32), (16, 512, 128)):
        print("case mfma narrow", precision, schedule, shape, flush=True)
        x = inputs.uniform_c64(shape, 32)
        for sign in (-1, 1):
            y = dft3d.fftn(torch.from_numpy(x).cuda(), schedule=schedule, precision=precision,
                           inverse=sign == 1)
            torch.cuda.synchronize()
            ref = oracle.dft3d(x.astype(np.complex128), sign, "fft")
            err = oracle.rel_l2(y.cpu().numpy(), ref)
            bound = {"bf16x1": 2e-2, "fp16x1": 3e-3}.get(precision, oracle.tol(x.size))
            assert err <= bound, (precision, schedule, shape, sign, err)
