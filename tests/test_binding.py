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


OPT = 2


class StandInLibrary:
    """The workspace rules of libdft3d.so: a plan needs `need[h]` bytes, an
    option change sets them, a bound workspace that has become too small is an
    error, and a plan without one gets memory of the library's own."""

    def __init__(self, epoch):
        self.epoch, self.need, self.ws, self.own, self.runs = epoch, {}, {}, 0, 0
        self.handles = []

    def dft3d_plan(self, n0, n1, n2, schedule, layout, out):
        h = len(self.need) + 1
        self.need[h] = 0
        out._obj.value = h
        self.handles.append(out._obj)
        return dft3d.OK

    def dft3d_destroy(self, h):
        return dft3d.OK

    def dft3d_status_string(self, st):
        return b"status"

    def dft3d_plan_set_option(self, h, key, value):
        self.need[h.value] = value
        self.epoch.value += 1
        return dft3d.OK

    def dft3d_workspace_size(self, h, out):
        out._obj.value = self.need[h.value]
        return dft3d.OK

    def dft3d_set_workspace(self, h, ptr, size):
        self.ws[h.value] = size
        return dft3d.OK

    def _run(self, h):
        if self.need[h] > 0 and self.ws.get(h, 0) < self.need[h]:
            if h in self.ws:
                return dft3d.ERR_WORKSPACE_TOO_SMALL
            self.own += 1
        self.runs += 1
        return dft3d.OK

    def dft3d_execute(self, h, x, y, sign, stream):
        return self._run(h.value)

    def dft3d_execute_batched(self, plans, xs, ys, n, sign, stream):
        for i in range(n):
            st = self._run(plans[i])
            if st != dft3d.OK:
                return st
        return dft3d.OK


class Tensor:
    dtype, is_cuda, shape, device = torch.complex64, True, (4, 4, 4), torch.device("cpu")

    def is_contiguous(self):
        return True

    def data_ptr(self):
        return 4096


@pytest.fixture
def library(monkeypatch):
    epoch = ctypes.c_int64(0)
    L = StandInLibrary(epoch)
    dft3d._load_torch()
    monkeypatch.setattr(dft3d, "_lib", L)
    monkeypatch.setattr(dft3d, "_epoch", epoch, raising=False)
    monkeypatch.setattr(dft3d, "_plans", {})
    monkeypatch.setattr(dft3d, "_raw_stream", lambda device: 0)
    yield L
    for h in L.handles:  # plans that outlive the test must not reach the library
        h.value = None


@pytest.mark.parametrize("first,second", [(0, 512), (64, 512), (512, 64), (64, 0)])
def test_options_set_through_the_c_abi_reach_the_bound_workspace(library, first, second):
    """execute() and fftn_batched() bind torch memory for the options a plan
    has now, also when they were changed behind the object: the library never
    reports a small workspace nor allocates its own."""
    x = Tensor()
    p = dft3d.Plan((4, 4, 4))
    p.set_option(OPT, first)
    p.execute(x, x)
    assert library.dft3d_plan_set_option(p.handle, OPT, second) == dft3d.OK
    p.execute(x, x)
    assert library.own == 0 and library.runs == 2
    dft3d.fftn_batched([x, x], outs=[x, x])
    q = dft3d.get_plan((4, 4, 4))
    for need in (first, second):
        assert library.dft3d_plan_set_option(q.handle, OPT, need) == dft3d.OK
        dft3d.fftn_batched([x, x], outs=[x, x])
    assert library.own == 0 and library.runs == 8


def test_workspace_size_is_asked_once_per_option_change(library, monkeypatch):
    x = Tensor()
    p = dft3d.Plan((4, 4, 4))
    asked = []
    real = library.dft3d_workspace_size
    monkeypatch.setattr(library, "dft3d_workspace_size",
                        lambda h, out: asked.append(1) or real(h, out))
    for _ in range(5):
        p.execute(x, x)
    assert len(asked) == 1
    p.set_option(OPT, 64)
    for _ in range(5):
        p.execute(x, x)
    assert len(asked) == 2


def test_a_device_without_streams_is_refused_by_torch(monkeypatch):
    """CPU tensors in a batched call end in torch's ValueError, as from
    torch.cuda.current_stream."""
    def refuse(device):
        raise ValueError(f"Expected a cuda device, but got: {device}")
    dft3d._load_torch()
    monkeypatch.setattr(torch.cuda, "current_stream", refuse)
    with pytest.raises(ValueError, match="cuda device"):
        dft3d._raw_stream(torch.device("cpu"))
