"""FGMRES without a preconditioner over restart lengths around the eight vectors of a wave of the orthogonalisation
(1, 7, 8, 9, 33 and the most, 64) on lattices whose half field is no multiple of a block's 64 elements: true residual
<= 1e-10 by the oracle, and the recurrence's last residual estimate agrees with the recomputed one (an orthogonality
lost in the update would part them; at 5e-11 an FP64 recurrence of up to 64 steps is good to 1e-14 / 5e-11 = 2e-4)."""
import numpy as np
import pytest
import torch

import lattice_inputs as li
import oracle
import paper_2411_08461_amd as q

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L", [(6, 4, 2, 6), (2, 2, 2, 6), (8, 8, 8, 4)])
@pytest.mark.parametrize("m", [1, 7, 8, 9, 33, 64])
def test_restart_lengths(L, m):
    c = q.Context(0)
    U = li.random_gauge(L, 0.25, 101)
    kappa, csw = 0.118, 1.0
    b = li.gaussian_source(L, 102)
    op = q.Operator(c, q.make_lattice(L), torch.from_numpy(U).to("cuda"), kappa, csw, "f64", 12)
    x = torch.zeros(b.shape, dtype=torch.complex128, device="cuda")
    info = q.qcdw_invert_fgmres(op, None, torch.from_numpy(b).to("cuda"), x,
                                q.make_params(gmres_restart=m, gmres_fallback=False))
    r = b - oracle.dirac(L, U, oracle.clover_build(L, U), x.cpu().numpy(), kappa, csw, 1)
    want = np.linalg.norm(r) / np.linalg.norm(b)
    assert info.status == q.QCDW_OK and want <= 1e-10, (info, want)
    assert abs(info.true_res - want) <= 1e-13
    assert abs(info.res_hist[-1] - info.iter_res) <= 1e-14 + 1e-3 * info.iter_res
