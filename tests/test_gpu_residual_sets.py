"""FP64 source preparation and residuals of all problems of a solve in one launch: the true residual that a solve
reports against the oracle's for its returned x, for converged problems and for ones stopped early (their residual is
of order 1e-2, so the two agree to rounding), right-hand-side counts around a thread group's four, both
reconstructions, whole, ragged and grouped tiles, and a batch of unequal lattices of which one is finished at once.
Tolerance: |difference| <= 1e-12, a residual norm relative to ||b|| formed in FP64 twice."""
import numpy as np
import pytest
import torch

import lattice_inputs as li
import oracle
import paper_2411_08461_amd as q

pytestmark = pytest.mark.gpu


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda")


def _res(L, U, C, x, b, kappa, csw, t_bc):
    r = b - oracle.dirac(L, U, C, x, kappa, csw, t_bc)
    return np.linalg.norm(r) / np.linalg.norm(b)


# 8x8x8x4: four tiles a slice, so the FP64 hops run in groups; 6x4x2x4: slices of 24 sites
@pytest.mark.parametrize("L,t_bc", [((8, 8, 8, 4), -1), ((6, 4, 2, 4), 1)])
@pytest.mark.parametrize("recon", [12, 18])
@pytest.mark.parametrize("maxiter", [3, 1000])
def test_multi_reports_the_residual(L, t_bc, recon, maxiter):
    c = q.Context(0)
    U = li.random_gauge(L, 0.25, 91)
    C = oracle.clover_build(L, U)
    kappa, csw = 0.121, 1.0
    op = q.Operator(c, q.make_lattice(L, t_bc), dev(U), kappa, csw, "bf16", recon)
    for n in (2, 4, 5, 9):
        bs = np.stack([li.gaussian_source(L, 92 + k) for k in range(n)])
        bs[1] = li.point_source(L)
        x = torch.zeros(bs.shape, dtype=torch.complex128, device="cuda")
        infos = q.qcdw_invert_multi(op, dev(bs), x, q.make_params(inner="bf16", maxiter=maxiter))
        for k in range(n):
            want = _res(L, U, C, x[k].cpu().numpy(), bs[k], kappa, csw, t_bc)
            assert abs(infos[k].true_res - want) <= 1e-12, (n, k, infos[k], want)
            assert infos[k].status == (q.QCDW_OK if maxiter > 3 else q.QCDW_ENOCONV)


@pytest.mark.parametrize("inner", ["f64", "bf16"])
@pytest.mark.parametrize("maxiter", [3, 1000])
def test_batch_reports_the_residual(inner, maxiter):
    c = q.Context(0)
    Ls = [(4, 4, 4, 4), (6, 4, 2, 8), (8, 8, 4, 4), (2, 2, 2, 2)]
    kappas, csw = [0.118, 0.121, 0.123, 0.11], 1.0
    Us = [li.random_gauge(L, 0.25, 95 + k) for k, L in enumerate(Ls)]
    Cs = [oracle.clover_build(L, U) for L, U in zip(Ls, Us)]
    bs = [li.gaussian_source(L, 97 + k) for k, L in enumerate(Ls)]
    ops = [q.Operator(c, q.make_lattice(L, -1), dev(U), k, csw, inner, 12) for L, U, k in zip(Ls, Us, kappas)]
    xs = [torch.zeros(b.shape, dtype=torch.complex128, device="cuda") for b in bs]
    q.qcdw_invert(ops[1], dev(bs[1]), xs[1], q.make_params(inner=inner))
    batch = q.Batch(c, ops)
    infos = q.qcdw_invert_batch(batch, [dev(b) for b in bs], xs, q.make_params(inner=inner, maxiter=maxiter))
    for k, L in enumerate(Ls):
        want = _res(L, Us[k], Cs[k], xs[k].cpu().numpy(), bs[k], kappas[k], csw, -1)
        assert abs(infos[k].true_res - want) <= 1e-12, (k, infos[k], want)
    assert infos[1].status == q.QCDW_OK and infos[1].iters == 0
    if maxiter > 3:
        assert all(i.status == q.QCDW_OK for i in infos)
