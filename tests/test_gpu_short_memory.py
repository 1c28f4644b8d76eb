"""Calls that keep copies or extra vectors for speed, on a device with too little memory left for them: they give the
result of the call with memory to spare.  The rest of the device is held by one allocation that is never touched."""
import contextlib
import gc

import pytest
import torch

import paper_2411_08461_amd as q

pytestmark = pytest.mark.gpu

L = (32, 32, 32, 32)
V = 32 ** 4
LINKS = 36 * V * 16  # bytes of the gauge field


@pytest.fixture(scope="module", autouse=True)
def most_of_the_device():
    """All but 16 GiB held for the module (one allocation of that size takes seconds)."""
    torch.cuda.empty_cache()
    left, _ = torch.cuda.mem_get_info()
    held = torch.empty(left - (16 << 30), dtype=torch.uint8, device="cuda")
    yield
    del held
    torch.cuda.empty_cache()


@contextlib.contextmanager
def only(free):
    """About `free` bytes of device memory left."""
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    left, _ = torch.cuda.mem_get_info()
    held = torch.empty(left - free, dtype=torch.uint8, device="cuda")
    try:
        yield
    finally:
        torch.cuda.synchronize()
        del held
        torch.cuda.empty_cache()


@contextlib.contextmanager
def context():
    """A context whose end gives the library's idle blocks back, so that the next call finds none."""
    gc.collect()
    c = q.Context(0)
    try:
        yield c
    finally:
        torch.cuda.synchronize()
        c.close()


def _field(seed, *shape):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return torch.view_as_complex(torch.randn(*shape, 2, dtype=torch.float64, device="cuda", generator=g))


def _links(seed, spread):
    """Near-unit links (the kernels compared here use nothing of unitarity)."""
    U = spread * _field(seed, 4, 2, V // 2, 3, 3)
    U += torch.eye(3, dtype=torch.complex128, device="cuda")
    return U


def _same(a, b):
    return float((a - b).abs().max()) <= 1e-13 * float(b.abs().max())


def test_clover_build():
    """Its plane-major links take as much as the gauge field."""
    U, lat = _links(1, 0.1), q.make_lattice(L)
    want = torch.empty(2, V // 2, 2, 36, dtype=torch.float64, device="cuda")
    got = torch.full_like(want, float("nan"))
    with context() as ctx:
        q.qcdw_clover_build(ctx, lat, U, want)
    with context() as ctx, only(LINKS * 2 // 3):
        q.qcdw_clover_build(ctx, lat, U, got)
    assert _same(got, want)


def test_clover_force():
    """Copies of the links and spinors take 960 bytes a site beside Gam's 384."""
    U, X, Y = _links(2, 0.1), _field(3, 2, V // 2, 4, 3), _field(4, 2, V // 2, 4, 3)
    lat = q.make_lattice(L, -1)
    want = torch.empty_like(U)
    got = torch.full_like(want, float("nan"))
    with context() as ctx:
        q.qcdw_clover_force(ctx, lat, U, X, Y, 0.12, 1.1, want)
    with context() as ctx, only(860 * V):
        q.qcdw_clover_force(ctx, lat, U, X, Y, 0.12, 1.1, got)
    assert _same(got, want)


@pytest.mark.parametrize("maxiter", [1000, 7])
def test_multishift(maxiter):
    """The residuals of a group of iterations take four fields more; a run cut off in the middle of a group included."""
    field = 6 * V * 16
    b = _field(5, V // 2, 4, 3)
    shifts = [0.3, 1e-2]
    U = _links(6, 0.02)
    want = [torch.empty_like(b) for _ in shifts]
    got = [torch.full_like(b, float("nan")) for _ in shifts]

    def solve(op, x):
        try:
            return q.qcdw_invert_multishift(op, b, x, shifts, maxiter=maxiter)[0]
        except q.QcdwError as e:
            assert maxiter == 7 and "within 7 iterations" in str(e)
            return maxiter

    with context() as ctx:
        n = solve(q.Operator(ctx, q.make_lattice(L), U, 0.11, 1.0, "f64", 18), want)
    with context() as ctx:
        op = q.Operator(ctx, q.make_lattice(L), U, 0.11, 1.0, "f64", 18)
        with only((9 + 4 + 2) * field):  # of the 17 fields with a group's residuals, 13 without
            assert solve(op, got) == n
    for g, w in zip(got, want):
        assert bool(torch.isfinite(torch.view_as_real(w)).all()) and _same(g, w)
