"""The operator and the hop on the paper's layouts (one kernel for both parities) against the oracle, where the
tile order or the site count of a block changes: slices of whole tiles (groups swept along t) and ragged ones,
extents of 2, both time boundaries; and inputs that share memory with the output.  Tolerance: 1e-13 relative,
the FP64 bar of the other operator tests (each output is a sum of about 300 products of order one)."""
import numpy as np
import pytest
import torch

import lattice_inputs as li
import oracle
import paper_2411_08461_amd as q

pytestmark = pytest.mark.gpu

# sites per time slice and parity: 256 (4 whole tiles, grouped), 320 (5), 64 (one tile), 24, 4 (ragged)
LATTICES = [(8, 8, 8, 4), (8, 8, 10, 2), (8, 4, 4, 6), (6, 4, 2, 6), (2, 2, 2, 2)]


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda")


def rel(a, b):
    a = a.cpu().numpy()
    return np.abs(a - b).max() / np.abs(b).max()


@pytest.fixture(scope="module")
def ctx():
    c = q.Context(0)
    yield c
    torch.cuda.synchronize()
    c.close()


@pytest.mark.parametrize("t_bc", [1, -1])
@pytest.mark.parametrize("L", LATTICES)
def test_operator_and_hop_match_oracle(ctx, L, t_bc):
    U, psi = li.random_gauge(L, 0.4, 31), li.gaussian_source(L, 32)
    C = oracle.clover_build(L, U)
    lat = q.make_lattice(L, t_bc)
    out = torch.full(li.fermion_shape(L), float("nan"), dtype=torch.complex128, device="cuda")
    q.qcdw_dslash(ctx, lat, dev(U), dev(C), dev(psi), out, 0.123, 1.2)
    assert rel(out, oracle.dirac(L, U, C, psi, 0.123, 1.2, t_bc)) < 1e-13
    for p in (0, 1):
        out.fill_(float("nan"))
        q.qcdw_hop(ctx, lat, dev(U), dev(psi), out, p)
        expect = np.array(oracle.hop(L, U, psi, t_bc)).reshape(li.fermion_shape(L))
        expect[1 - p] = 0.0
        assert rel(out, expect) < 1e-13


def test_inputs_that_share_memory_with_the_output(ctx):
    """An output field that overlaps psi, the links or the clover field gives the result of separate buffers."""
    L = (4, 4, 4, 4)
    V = 256
    U, psi = li.random_gauge(L, 0.4, 33), li.gaussian_source(L, 34)
    C = oracle.clover_build(L, U)
    lat = q.make_lattice(L)
    ref = torch.empty(12 * V, dtype=torch.complex128, device="cuda")
    q.qcdw_dslash(ctx, lat, dev(U), dev(C), dev(psi), ref, 0.12, 1.0)
    for call in (q.qcdw_dslash, q.qcdw_dslash_noalloc):
        buf = torch.empty(13 * V, dtype=torch.complex128, device="cuda")
        buf[V:] = dev(psi).reshape(-1)
        call(ctx, lat, dev(U), dev(C), buf[V:], buf[: 12 * V], 0.12, 1.0)
        assert torch.equal(buf[: 12 * V], ref)
        buf = dev(U).reshape(-1).clone()
        call(ctx, lat, buf, dev(C), dev(psi), buf[5 * V: 17 * V], 0.12, 1.0)
        assert torch.equal(buf[5 * V: 17 * V], ref)
        both = torch.empty(2 * 36 * V, dtype=torch.float64, device="cuda")
        both[:] = dev(C).reshape(-1)
        call(ctx, lat, dev(U), both, dev(psi), torch.view_as_complex(both[: 24 * V].view(-1, 2)), 0.12, 1.0)
        assert torch.equal(torch.view_as_complex(both[: 24 * V].view(-1, 2)), ref)
