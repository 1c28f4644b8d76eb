"""The kernels on the paper's layouts where their tiles are swept group by group along t: a slice of 36 whole tiles in
two groups of 18 (16x16x18), and one of 33 tiles in three groups of 11 (6x8x88), both time boundaries.  The operator,
the hop into both parities and the clover field against the oracle on every site (1e-13 relative, the FP64 bar of the
other operator tests); the force by every link being written, and on a link of each group and parity by the oracle
(1e-12, the bar of the other force tests)."""
import numpy as np
import pytest
import torch

import lattice_inputs as li
import oracle
import paper_2411_08461_amd as q
from oracle import force as of

pytestmark = pytest.mark.gpu

LATTICES = [((16, 16, 18, 4), -1, 18), ((6, 8, 88, 2), 1, 11)]


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


@pytest.mark.parametrize("L,t_bc,G", LATTICES)
def test_operator_hop_and_clover(ctx, L, t_bc, G):
    U, psi = li.random_gauge(L, 0.4, 121), li.gaussian_source(L, 122)
    lat = q.make_lattice(L, t_bc)
    C = oracle.clover_build(L, U)
    got = torch.full(oracle.packed_shape(L), float("nan"), dtype=torch.float64, device="cuda")
    q.qcdw_clover_build(ctx, lat, dev(U), got)
    assert rel(got, C) < 1e-13
    out = torch.full(li.fermion_shape(L), float("nan"), dtype=torch.complex128, device="cuda")
    q.qcdw_dslash(ctx, lat, dev(U), dev(C), dev(psi), out, 0.123, 1.2)
    assert rel(out, oracle.dirac(L, U, C, psi, 0.123, 1.2, t_bc)) < 1e-13
    full = np.array(oracle.hop(L, U, psi, t_bc)).reshape(li.fermion_shape(L))
    for p in (0, 1):
        out.fill_(float("nan"))
        q.qcdw_hop(ctx, lat, dev(U), dev(psi), out, p)
        expect = full.copy()
        expect[1 - p] = 0.0
        assert rel(out, expect) < 1e-13


@pytest.mark.parametrize("L,t_bc,G", LATTICES)
def test_force(ctx, L, t_bc, G):
    U = li.random_gauge(L, 0.4, 123)
    X, Y = li.gaussian_source(L, 124), li.gaussian_source(L, 125)
    V = int(np.prod(L))
    Vh, nct = V // 2, L[0] // 2 * L[1] * L[2] // 64
    # one site of each parity and group, in different tiles, slices and lanes (a tile that is left out stays NaN)
    links = []
    for grp in range(nct // G):
        for p in range(2):
            tile = (2 * grp + p) % L[3] * nct + grp * G + (G - 1 if p else grp)
            links.append(((2 * p + grp) % 4, p * Vh + 64 * tile + 63 * p))
    H = torch.full(li.gauge_shape(L), float("nan"), dtype=torch.complex128, device="cuda")
    q.qcdw_clover_force(ctx, q.make_lattice(L, t_bc), dev(U), dev(X), dev(Y), 0.122, 1.3, H)
    assert bool(torch.isfinite(torch.view_as_real(H)).all())
    got = H.cpu().numpy().reshape(4, V, 3, 3)
    expect = of.force(L, U, X, Y, 0.122, 1.3, t_bc, links).reshape(4, V, 3, 3)
    for mu, i in links:
        assert np.abs(got[mu, i] - expect[mu, i]).max() < 1e-12 * np.abs(expect[mu, i]).max(), (mu, i)
