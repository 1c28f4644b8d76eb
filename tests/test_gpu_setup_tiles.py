"""The operator set-up (link packing, clover field, A and its inverse in one kernel) where its tiles end: sites
per parity below, at and above the 64-site tile and the 256-link block, slices that are whole tiles (swept in
groups) and not, every inner precision and both reconstructions.  The clover field and M_hat against the oracle at
the FP64 bar (1e-13 relative); the low-precision copies through M_hat in that precision, against the FP64 oracle
within the storage rounding (each of the ~300 products of a site carries at most three roundings of 2^-9 for BF16,
2^-11 for FP16, 2^-24 for FP32; the bounds of the existing operator tests)."""
import numpy as np
import pytest
import torch

import lattice_inputs as li
import oracle
import paper_2411_08461_amd as q

pytestmark = pytest.mark.gpu

# sites per parity: 8, 36, 64, 256 (whole tiles per slice: 64), 264, 1024 (256 a slice)
LATTICES = [(2, 2, 2, 2), (6, 2, 2, 3 * 2), (4, 4, 4, 2), (8, 4, 4, 4), (4, 2, 6, 22), (8, 8, 8, 4)]
BOUND = {"f64": 1e-13, "f32": 2e-6, "bf16": 2e-2, "f16": 4e-3}


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


@pytest.mark.parametrize("inner,recon", [("f64", 12), ("f64", 18), ("f32", 12), ("f32", 18), ("bf16", 12),
                                         ("bf16", 18), ("f16", 12), ("f16", 18)])
@pytest.mark.parametrize("L", LATTICES)
def test_operator_setup_matches_oracle(ctx, L, inner, recon):
    U = li.random_gauge(L, 0.35, 41)
    lat = q.make_lattice(L, -1)
    C = oracle.clover_build(L, U)
    got = torch.full(oracle.packed_shape(L), float("nan"), dtype=torch.float64, device="cuda")
    q.qcdw_clover_build(ctx, lat, dev(U), got)
    assert rel(got, C) < 1e-13
    Ainv, bad = oracle.clover_invert(L, C, 0.121, 1.1)
    assert bad == 0
    Vh = int(np.prod(L)) // 2
    x = li.gaussian_source(L, 42).reshape(-1, 4, 3)[:Vh].copy()
    expect = oracle.schur_matpc(L, U, Ainv, x, 0.121, -1)
    op = q.Operator(ctx, lat, dev(U), 0.121, 1.1, inner, recon)
    for prec in dict.fromkeys(("f64", inner)):
        out = torch.full((Vh, 4, 3), float("nan"), dtype=torch.complex128, device="cuda")
        q.qcdw_op_matpc(op, prec, dev(x), out)
        assert rel(out, expect) < BOUND[prec], prec
    op.close()


def test_operator_setup_reports_blocks_that_are_not_positive_definite(ctx):
    """A strong clover term makes some A indefinite; the padding lanes of the last tile are not counted."""
    L = (6, 2, 2, 6)
    U = li.random_gauge(L, 1.5, 43)
    C = oracle.clover_build(L, U).reshape(-1, 36)
    A = np.zeros((len(C), 6, 6), dtype=np.complex128)
    low = [(j, k) for j in range(6) for k in range(j)]
    for s, (j, k) in enumerate(low):
        A[:, j, k] = -0.13 * 30.0 * (C[:, 6 + 2 * s] + 1j * C[:, 7 + 2 * s])
    for j in range(6):
        A[:, j, j] = 1.0 - 0.13 * 30.0 * C[:, j]
    bad = int(np.sum(np.linalg.eigvalsh(A, UPLO="L")[:, 0] <= 0.0))
    assert bad > 0
    with pytest.raises(q.QcdwError, match=f"^ENOTPD: {bad} clover"):
        q.Operator(ctx, q.make_lattice(L), dev(U), 0.13, 30.0)
