"""Native objects are destroyed children first, each once, however the Python objects die: closed by hand, dropped one
by one, or collected in a cycle, where the collector clears weak references before it runs finalisers and may finalise
the context first.  The library is a recorder here, so the order is checked without a GPU."""
import ctypes
import gc
import types

import pytest
import torch

import paper_2411_08461_amd as q


class Recorder:
    """Hands out handles and notes every destroy call; a destroyed object's owner must still be there."""

    def __init__(self):
        self.next, self.live, self.calls = 1, {}, []

    def __getattr__(self, name):
        if name.endswith("_create"):
            return lambda *args: self._create(name, args)
        if name.endswith("_destroy"):
            return lambda h: self._destroy(name, h.value)
        return lambda *args: 0

    def qcdw_net_bind(self, net, op):
        self.live[net.value] = ("net", [op.value])
        return 0

    def _create(self, name, args):
        kind = name.split("_")[1]
        out = args[0] if kind == "ctx" else args[-1]
        owners = [a.value for a in args if isinstance(a, ctypes.c_void_p) and a.value in self.live]
        if kind == "batch":
            owners += list(args[2])
        out._obj.value = self.next
        self.live[self.next] = (kind, owners)
        self.next += 1
        return 0

    def _destroy(self, name, h):
        kind, owners = self.live.pop(h)  # a second call has no entry
        assert name == f"qcdw_{kind}_destroy"
        assert all(o in self.live for o in owners), f"{kind} outlived an object that it uses"
        self.calls.append(kind)


@pytest.fixture
def lib(monkeypatch):
    r = Recorder()
    monkeypatch.setattr(q, "load_library", lambda: r)
    monkeypatch.setattr(torch.cuda, "is_available", lambda: True)
    monkeypatch.setattr(q, "_ptr", lambda t, dtype=None, name="": None)
    monkeypatch.setattr(q, "_need", lambda t, n, name: None)
    yield r
    gc.collect()


def _family():
    ctx = q.Context(0, stream=types.SimpleNamespace(cuda_stream=0))
    lat = q.make_lattice((4, 4, 4, 4))
    ops = [q.Operator(ctx, lat, None, 0.12, 1.0) for _ in range(2)]
    return [ctx, *ops, q.Batch(ctx, [*ops, ops[0]]), q.Net(ops[0]), q.Multigrid(ops[1], object())]


@pytest.fixture(autouse=True)
def _params(monkeypatch):
    monkeypatch.setattr(ctypes, "byref", lambda o: types.SimpleNamespace(_obj=o))


@pytest.mark.parametrize("order", [(0, 1, 2, 3, 4, 5), (5, 4, 3, 2, 1, 0), (3, 0, 5, 1, 4, 2)])
def test_collected_in_a_cycle(lib, order):
    family = _family()
    gc.collect()
    gc.disable()
    try:
        cycle = [family[k] for k in order]
        cycle.append(cycle)
        del family, cycle
    finally:
        gc.enable()
    gc.collect()
    assert not lib.live and sorted(lib.calls) == ["batch", "ctx", "mg", "net", "op", "op"]
    assert lib.calls[-1] == "ctx"


@pytest.mark.parametrize("order", [(0,), (1, 2, 0), (4, 5, 3, 1, 2, 0), (5, 5, 2, 2, 1, 0)])
def test_closed_by_hand(lib, order):
    family = _family()
    for k in order:
        family[k].close()
        assert family[k].handle is None
    assert not lib.live and len(lib.calls) == 6
    assert all(f.handle is None for f in family)


def test_dropped_one_by_one(lib):
    family = _family()
    for _ in range(6):
        family.pop()
    del family
    gc.collect()
    assert not lib.live and lib.calls[-1] == "ctx"


def test_a_net_follows_its_operator(lib):
    ctx, a, b, batch, net, mg = _family()
    batch.close()
    q.qcdw_net_bind(net, b)
    a.close()
    assert net.handle is not None
    b.close()
    assert net.handle is None and mg.handle is None
    ctx.close()
    assert not lib.live
