"""The clover force where its blocks end: slices of whole 64-site tiles (swept in groups), one site more or less
than a tile, extents of 2 in every direction, both time boundaries.  Against the oracle's exact link derivative on
sampled links, 1e-12 relative (the bar of the other force tests)."""
import numpy as np
import pytest
import torch

import lattice_inputs as li
import paper_2411_08461_amd as q
from oracle import force as of

pytestmark = pytest.mark.gpu


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda")


@pytest.fixture(scope="module")
def ctx():
    c = q.Context(0)
    yield c
    torch.cuda.synchronize()
    c.close()


# sites per parity 1024 (four tiles a slice), 66, 60, 8
@pytest.mark.parametrize("L,t_bc", [((8, 8, 8, 4), -1), ((2, 6, 2, 11 * 2), 1), ((2, 2, 10, 6), -1), ((2, 2, 2, 2), -1)])
def test_force_at_tile_edges(ctx, L, t_bc):
    U = li.random_gauge(L, 0.4, 51)
    X, Y = li.gaussian_source(L, 52), li.gaussian_source(L, 53)
    V = int(np.prod(L))
    Vh = V // 2
    sites = sorted({0, Vh - 1, Vh, V - 1, min(63, Vh - 1), min(64, Vh - 1), Vh + min(63, Vh - 1), Vh + min(64, Vh - 1)})
    links = [(mu, i) for mu in range(4) for i in sites]
    H = torch.full(li.gauge_shape(L), float("nan"), dtype=torch.complex128, device="cuda")
    q.qcdw_clover_force(ctx, q.make_lattice(L, t_bc), dev(U), dev(X), dev(Y), 0.122, 1.3, H)
    assert bool(torch.isfinite(torch.view_as_real(H)).all())
    got = H.cpu().numpy().reshape(4, V, 3, 3)
    expect = of.force(L, U, X, Y, 0.122, 1.3, t_bc, links).reshape(4, V, 3, 3)
    for mu, i in links:
        assert np.abs(got[mu, i] - expect[mu, i]).max() < 1e-12 * np.abs(expect[mu, i]).max(), (mu, i)
