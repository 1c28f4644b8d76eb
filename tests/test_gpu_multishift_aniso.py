"""The normal operator's hop epilogues (M_hat with g5 A^-1 of its result; the last hop with the shift term and the dot
product) with the weights of the anisotropic action, both reconstructions and time boundaries, in a form of each kind of
the single-RHS hop.  Each solution against its shifted system applied by the oracle: ||b - (N + sigma) x|| <= 1e-9 ||b||,
the asked tolerance of 1e-10 with room for the oracle's own rounding."""
import numpy as np
import pytest
import torch

import lattice_inputs as li
import oracle
import paper_2411_08461_amd as q

pytestmark = pytest.mark.gpu

G5 = np.array([1.0, 1.0, -1.0, -1.0])[:, None]
XI0, NU, M0, CT, CR = 2.464, 0.95, 0.3, 0.91, 1.07  # the paper's example action
KAPPA = oracle.aniso_kappa(M0, XI0, NU)
W = oracle.aniso_weights(XI0, NU)


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda")


def _normal(L, U, C, Ainv, x, t_bc):
    """M_hat^+ M_hat x with M_hat^+ = g5 A_ee M_hat g5 A_ee^-1."""
    Vh = len(x)

    def even(op, v):
        full = np.zeros(li.fermion_shape(L), dtype=np.complex128)
        full[0] = v.reshape(full[0].shape)
        return np.asarray(op(full)).reshape(2, Vh, 4, 3)[0]
    w = oracle.schur_matpc(L, U, Ainv, x, KAPPA, t_bc, weights=W)
    u = G5 * even(lambda f: oracle.packed_apply(L, Ainv, f), w)
    u = oracle.schur_matpc(L, U, Ainv, u, KAPPA, t_bc, weights=W)
    return G5 * even(lambda f: oracle.clover_apply(L, C, f, KAPPA, 1.0), u)


@pytest.mark.parametrize("nt,cg,fma", [(1, 0, 0), (1, 2, 1), (2, 0, 0)])
@pytest.mark.parametrize("recon", [12, 18])
@pytest.mark.parametrize("L,t_bc", [((8, 8, 4, 8), -1), ((6, 4, 2, 8), 1)])
def test_multishift_of_the_anisotropic_operator(tmp_path, monkeypatch, L, t_bc, recon, nt, cg, fma):
    nct = (L[0] // 2 * L[1] * L[2] + 63) // 64
    if cg and nct % cg:
        pytest.skip("group does not divide the tiles of a slice")
    cache = tmp_path / "tune.txt"
    cache.write_text(f"hop_nt/p0/L{L[0]}x{L[1]}x{L[2]}x{L[3]} {nt + 16 * cg + 4096 * fma}\n")
    monkeypatch.setenv("QCDW_TUNE_CACHE", str(cache))
    c = q.Context(0)
    U = li.random_gauge(L, 0.25, 141)
    Vh = int(np.prod(L)) // 2
    b = li.gaussian_source(L, 142).reshape(-1, 4, 3)[:Vh].copy()
    op = q.Operator(c, q.make_lattice(L, t_bc), dev(U), KAPPA, 0.0, "f64", recon, aniso=(XI0, NU, CT, CR))
    assert q.qcdw_op_hop_form(op) == (nt, cg, fma)
    shifts = [0.7, 1e-3, 20.0]
    xs = [torch.full((Vh, 4, 3), float("nan"), dtype=torch.complex128, device="cuda") for _ in shifts]
    q.qcdw_invert_multishift(op, dev(b), xs, shifts)
    C = oracle.clover_build(L, U, plane_weights=(CT, CR / XI0))
    Ainv, bad = oracle.clover_invert(L, C, KAPPA, 1.0)
    assert bad == 0
    for x, s in zip(xs, shifts):
        x = x.cpu().numpy()
        r = b - _normal(L, U, C, Ainv, x, t_bc) - s * x
        assert np.linalg.norm(r) <= 1e-9 * np.linalg.norm(b), s
    op.close()
    c.close()
