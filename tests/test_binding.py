"""The Python binding's plan cache and workspace handling, against a stand-in
for the library (no device needed)."""
import ctypes

import numpy as np
import pytest

from paper_1904_10119_amd import dft3d

torch = pytest.importorskip("torch")


@pytest.fixture
def plan_count(monkeypatch):
    made = []

    class Made:
        def __init__(self, shape, *a, **kw):
            made.append(tuple(int(s) for s in shape))
    monkeypatch.setattr(dft3d, "Plan", Made)
    monkeypatch.setattr(dft3d, "_plans", {})
    return made


def test_sides_of_any_integer_type_share_a_plan(plan_count):
    """Sides count by value: 0-d tensors, which hash by identity, and numpy
    integers find the plan of the same ints."""
    sides = [(8, 6, 4), [8, 6, 4], torch.Size((8, 6, 4)), np.array([8, 6, 4]),
             tuple(torch.tensor(v) for v in (8, 6, 4)), torch.tensor([8, 6, 4])]
    plans = {id(dft3d.get_plan(s)) for s in sides for _ in range(2)}
    dft3d._load_torch()  # a torch.Size is then taken as it is
    plans |= {id(dft3d.get_plan(s)) for s in sides}
    assert len(plans) == 1 and plan_count == [(8, 6, 4)]
