"""Tiles of the 1D items of a batched call: the one-launch form, which pays a
device-scope release and acquire per tile, keeps the large tiles of the pass
kernel in every order."""
import pytest

from paper_1904_10119_amd import dft3d, inputs

SETS = {"96 problems": inputs.batch_shapes(96, 104),
        "16 and 32": [(a, b, c) for a in (16, 32) for b in (16, 32) for c in (16, 32)],
        "all lengths": [(1, 2, 4), (8, 16, 32), (64, 128, 256), (256, 1, 128), (2, 64, 8)]}


def tiles(shapes, schedule, launch):
    d = dft3d.describe_batch(shapes, schedule, launch)
    out = {}
    for it in d["items"]:
        if not it["n1"]:
            out.setdefault(it["n"], set()).add(it["tile"])
    return d["total"], out


@pytest.mark.parametrize("name", sorted(SETS))
@pytest.mark.parametrize("schedule", ["pencil", "slab", "auto"])
def test_one_launch_tiles(name, schedule):
    total, one = tiles(SETS[name], schedule, "persistent")
    _, lev = tiles(SETS[name], schedule, "levels")
    for n, t in one.items():
        assert len(t) == 1, (n, t)                  # one tile a length, whatever the order
        assert min(t) >= max(lev.get(n, {1})), (n, t, lev[n])
        assert min(t) * n >= 2048 or n < 8, (n, t)  # 8 points a thread or more, 256 threads


def test_one_launch_tickets_of_the_96_problems():
    assert tiles(SETS["96 problems"], "pencil", "persistent")[0] <= 30644
    assert tiles(SETS["96 problems"], "auto", "persistent")[0] <= 27580


def test_level_form_rotates_128_points_in_rows_of_two_lines():
    assert tiles(SETS["96 problems"], "pencil", "levels")[1][128] == {32}
    assert tiles(SETS["all lengths"], "pencil", "levels")[1][256] == {16}
