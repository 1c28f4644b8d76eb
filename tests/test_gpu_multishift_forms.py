"""The normal operator's two hop epilogues (M_hat with g5 A^-1 of its result; the last hop with the shift term and
the dot product) in every form of the single-RHS hop that the tuner may pick, forced through the tuning cache, both
reconstructions and both time boundaries, on a lattice of two tiles a slice and on a ragged one; shifts that
converge in different groups of iterations.  Each solution against its shifted system applied by the oracle:
||b - (N + sigma) x|| <= 1e-9 ||b||, the asked tolerance of 1e-10 with room for the oracle's own rounding."""
import numpy as np
import pytest
import torch

import lattice_inputs as li
import oracle
import paper_2411_08461_amd as q

pytestmark = pytest.mark.gpu

G5 = np.array([1.0, 1.0, -1.0, -1.0])[:, None]


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda")


def _normal(L, U, C, Ainv, x, kappa, t_bc):
    """M_hat^+ M_hat x with M_hat^+ = g5 A_ee M_hat g5 A_ee^-1."""
    Vh = len(x)

    def even(op, v):
        full = np.zeros(li.fermion_shape(L), dtype=np.complex128)
        full[0] = v.reshape(full[0].shape)
        return np.asarray(op(full)).reshape(2, Vh, 4, 3)[0]
    w = oracle.schur_matpc(L, U, Ainv, x, kappa, t_bc)
    u = G5 * even(lambda f: oracle.packed_apply(L, Ainv, f), w)
    u = oracle.schur_matpc(L, U, Ainv, u, kappa, t_bc)
    return G5 * even(lambda f: oracle.clover_apply(L, C, f, kappa, 1.0), u)


@pytest.mark.parametrize("nt,cg,fma,recon", [(1, 0, 0, 12), (1, 0, 1, 18), (1, 2, 1, 12), (1, 2, 2, 12), (1, 1, 3, 18),
                                             (2, 0, 0, 12), (2, 1, 1, 18), (4, 0, 1, 12), (4, 2, 0, 12)])
@pytest.mark.parametrize("L,t_bc", [((8, 8, 4, 8), -1), ((6, 4, 2, 8), 1)])
def test_multishift_in_every_hop_form(tmp_path, monkeypatch, L, t_bc, nt, cg, fma, recon):
    nct = (L[0] // 2 * L[1] * L[2] + 63) // 64
    if cg and nct % cg:
        pytest.skip("group does not divide the tiles of a slice")
    cache = tmp_path / "tune.txt"
    cache.write_text(f"hop_nt/p0/L{L[0]}x{L[1]}x{L[2]}x{L[3]} {nt + 16 * cg + 4096 * fma}\n")
    monkeypatch.setenv("QCDW_TUNE_CACHE", str(cache))
    c = q.Context(0)
    U = li.random_gauge(L, 0.25, 71)
    kappa = 0.122
    Vh = int(np.prod(L)) // 2
    b = li.gaussian_source(L, 72).reshape(-1, 4, 3)[:Vh].copy()
    op = q.Operator(c, q.make_lattice(L, t_bc), dev(U), kappa, 1.0, "f64", recon)
    assert q.qcdw_op_hop_form(op) == (nt, cg, fma)
    shifts = [0.7, 1e-3, 20.0]
    xs = [torch.full((Vh, 4, 3), float("nan"), dtype=torch.complex128, device="cuda") for _ in shifts]
    q.qcdw_invert_multishift(op, dev(b), xs, shifts)
    C = oracle.clover_build(L, U)
    Ainv, _ = oracle.clover_invert(L, C, kappa, 1.0)
    for x, s in zip(xs, shifts):
        x = x.cpu().numpy()
        r = b - _normal(L, U, C, Ainv, x, kappa, t_bc) - s * x
        assert np.linalg.norm(r) <= 1e-9 * np.linalg.norm(b), s
    op.close()
    c.close()
