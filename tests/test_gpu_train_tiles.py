"""Loss and weight gradients of the learned layers where the training kernels' tiles end: sites per parity below, at
and above a 64-site tile, more tiles than blocks, both widths, one and several pairs (the partial sums carry over),
against the oracle's FP64 definition.  Tolerance: the fields are FP32; an entry of a gradient sums products of values
that have gone through at most 9 x 12 x 3 x 2 FP32 multiply-adds each, so a worst-case linear growth of the 2^-24
rounding is 4e-5 of the gradient's norm; 2e-5 is asked of the norm."""
import numpy as np
import pytest
import torch

import lattice_inputs as li
import paper_2411_08461_amd as q
from oracle import learned as ol

pytestmark = pytest.mark.gpu


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda")


@pytest.fixture(scope="module")
def ctx():
    c = q.Context(0)
    yield c
    torch.cuda.synchronize()
    c.close()


def _pairs(L, n, seed):
    Vh = int(np.prod(L)) // 2
    rng = np.random.default_rng(seed)

    def field():
        return rng.standard_normal((Vh, 4, 3)) + 1j * rng.standard_normal((Vh, 4, 3))

    return [(field(), field()) for _ in range(n)]


# sites per parity: 8, 64, 66, 25600 (400 tiles, above the 384 blocks of a part)
@pytest.mark.parametrize("hidden", [4, 12])
@pytest.mark.parametrize("L,n", [((2, 2, 2, 2), 2), ((4, 4, 4, 2), 1), ((2, 6, 2, 11 * 2), 3), ((8, 16, 20, 20), 1)])
def test_gradients_at_tile_edges(ctx, L, n, hidden):
    U = li.random_gauge(L, 0.3, 61)
    op = q.Operator(ctx, q.make_lattice(L), dev(U), 0.12, 1.0)
    net = q.qcdw_net_create(op, hidden)
    rng = np.random.default_rng(62)
    W1 = 0.2 * (rng.standard_normal((9, hidden, 4)) + 1j * rng.standard_normal((9, hidden, 4)))
    W2 = 0.2 * (rng.standard_normal((9, 4, hidden)) + 1j * rng.standard_normal((9, 4, hidden)))
    q.qcdw_net_set_weights(net, W1, W2)
    W1, W2 = q.qcdw_net_get_weights(net)  # as rounded to FP32
    pairs = _pairs(L, n, 63)
    args = [dev(r) for r, _ in pairs], [dev(e) for _, e in pairs]
    loss, g1, g2 = q.qcdw_net_loss_grad(net, *args)
    eloss, e1, e2 = ol.net_loss_and_grad(ol.Transport(L, U), W1, W2, pairs)
    assert abs(loss - eloss) < 2e-5 * eloss
    for g, e in ((g1, e1), (g2, e2)):
        assert np.linalg.norm(g - e) < 2e-5 * np.linalg.norm(e)
        assert np.abs(g - e).max() < 1e-4 * np.sqrt(np.mean(np.abs(e) ** 2))
    again = q.qcdw_net_loss_grad(net, *args)
    assert again[0] == loss and np.array_equal(again[1], g1) and np.array_equal(again[2], g2)
    net.close()
    op.close()


def test_zero_error_field_is_refused_and_leaves_the_weights(ctx):
    L = (4, 4, 4, 2)
    op = q.Operator(ctx, q.make_lattice(L), dev(li.random_gauge(L, 0.3, 64)), 0.12, 1.0)
    net = q.qcdw_net_create(op, 12)
    before = q.qcdw_net_get_weights(net)
    (r, e), = _pairs(L, 1, 65)
    rs, es = [dev(r), dev(r)], [dev(e), dev(0 * e)]
    with pytest.raises(q.QcdwError, match="zero error field"):
        q.qcdw_net_loss_grad(net, rs, es)
    with pytest.raises(q.QcdwError, match="zero error field"):
        q.qcdw_net_train(net, rs, es, steps=1, batch=2)
    after = q.qcdw_net_get_weights(net)
    assert all(np.array_equal(a, b) for a, b in zip(before, after))
    net.close()
    op.close()
