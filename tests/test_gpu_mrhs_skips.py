"""The multi-RHS hop's register loop with finished right-hand sides at the front, in the middle, side by side and at the
end of nine, in whole solves (skips and both fused dot products): the form is forced through the tuning cache, in site
order and in slice groups, every storage precision, whole tiles and padded ones.  Each unfinished solution against the
oracle's operator: a true residual within the asked 1e-10; the finished ones keep their answer."""
import numpy as np
import pytest
import torch

import lattice_inputs as li
import oracle
import paper_2411_08461_amd as q

pytestmark = pytest.mark.gpu


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda")


# tiles per slice: 4 (whole), 2 (36 sites in the second)
@pytest.mark.parametrize("L,t_bc,variant", [((8, 8, 8, 4), -1, 0), ((8, 8, 8, 4), -1, 4), ((10, 10, 2, 6), 1, 0),
                                            ((10, 10, 2, 6), 1, 2)])
@pytest.mark.parametrize("inner", ["f64", "f32", "bf16", "f16"])
def test_forced_form(tmp_path, monkeypatch, L, t_bc, variant, inner):
    n, zero, solved = 9, (0, 3, 4, 8), 5
    cache = tmp_path / "tune.txt"
    keys = [f"mrhs_hop/p{q.PREC[p]}/L{L[0]}x{L[1]}x{L[2]}x{L[3]}/n{n}" for p in dict.fromkeys(("f64", inner))]
    cache.write_text("".join(f"{k} {variant}\n" for k in keys))
    monkeypatch.setenv("QCDW_TUNE_CACHE", str(cache))
    c = q.Context(0)
    U = li.random_gauge(L, 0.25, 131)
    kappa, csw = 0.121, 1.0
    bs = np.stack([li.gaussian_source(L, 132 + k) for k in range(n)])
    for k in zero:
        bs[k] = 0
    op = q.Operator(c, q.make_lattice(L, t_bc), dev(U), kappa, csw, inner, 12)
    x = torch.zeros(bs.shape, dtype=torch.complex128, device="cuda")
    q.qcdw_invert_multi(op, dev(bs[solved:solved + 1]), x[solved:solved + 1], q.make_params(inner=inner))
    infos = q.qcdw_invert_multi(op, dev(bs), x, q.make_params(inner=inner))
    C = oracle.clover_build(L, U)
    for k in range(n):
        assert infos[k].status == q.QCDW_OK and infos[k].fallback == 0, (k, infos[k])
        xk = x[k].cpu().numpy()
        if k in zero:
            assert not xk.any()
            continue
        r = bs[k] - oracle.dirac(L, U, C, xk, kappa, csw, t_bc)
        assert np.linalg.norm(r) <= 1.01e-10 * np.linalg.norm(bs[k]), k
    assert infos[solved].iters == 0
    assert all(q.qcdw_ctx_tuned(c, k) == variant for k in keys)
    op.close()
    c.close()
