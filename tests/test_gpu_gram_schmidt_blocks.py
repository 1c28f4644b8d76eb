"""The combined update and dot product of the orthogonalisation on half fields around 768 tiles of 64 elements, from
which its blocks take more than one tile each: 756 tiles (the last of them whole), 768, and 864 (blocks of one and of
two tiles).  FGMRES without a preconditioner, restart lengths of one wave of vectors and of several: true residual
<= 1e-10 by the oracle, and the recurrence's last estimate agrees with the recomputed residual (an orthogonality lost in
the update would part them; at 5e-11 an FP64 recurrence of up to 64 steps is good to 1e-14 / 5e-11 = 2e-4)."""
import numpy as np
import pytest
import torch

import lattice_inputs as li
import oracle
import paper_2411_08461_amd as q

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L", [(6, 6, 8, 28), (8, 8, 8, 16), (8, 8, 8, 18)])
@pytest.mark.parametrize("m", [8, 33])
def test_blocks_of_one_and_more_tiles(L, m):
    c = q.Context(0)
    U = li.random_gauge(L, 0.25, 103)
    kappa, csw = 0.118, 1.0
    b = li.gaussian_source(L, 104)
    op = q.Operator(c, q.make_lattice(L), torch.from_numpy(U).to("cuda"), kappa, csw, "f64", 12)
    x = torch.zeros(b.shape, dtype=torch.complex128, device="cuda")
    info = q.qcdw_invert_fgmres(op, None, torch.from_numpy(b).to("cuda"), x,
                                q.make_params(gmres_restart=m, gmres_fallback=False))
    r = b - oracle.dirac(L, U, oracle.clover_build(L, U), x.cpu().numpy(), kappa, csw, 1)
    want = np.linalg.norm(r) / np.linalg.norm(b)
    assert info.status == q.QCDW_OK and want <= 1e-10, (info, want)
    assert abs(info.true_res - want) <= 1e-13
    assert abs(info.res_hist[-1] - info.iter_res) <= 1e-14 + 1e-3 * info.iter_res
    op.close()
    c.close()
