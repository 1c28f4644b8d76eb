"""The multi-RHS hop's pipeline over right-hand sides: counts around the two that it keeps in flight (1 .. 5, and the
most, 16), every storage precision, ragged and whole tiles, both tile orders; finished ones in between skipped.
Bounds: the single-RHS ones of the storage precision; 1e-13 for FP64 (a few hundred operations of rounding 1.1e-16)."""
import numpy as np
import pytest
import torch

import lattice_inputs as li
import oracle
import paper_2411_08461_amd as q

pytestmark = pytest.mark.gpu

BOUND = {"f64": 1e-13, "f32": 2e-6, "bf16": 2e-2, "f16": 4e-3}


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda")


@pytest.mark.parametrize("prec", ["f64", "f32", "bf16", "f16"])
@pytest.mark.parametrize("L,t_bc,cg", [((6, 4, 2, 6), -1, 0), ((8, 8, 4, 4), 1, 0), ((8, 8, 4, 4), -1, 1)])
def test_every_count(tmp_path, monkeypatch, prec, L, t_bc, cg):
    counts = (1, 2, 3, 4, 5, 16)
    cache = tmp_path / "tune.txt"
    cache.write_text("".join(f"mrhs_hop/p{q.PREC[prec]}/L{L[0]}x{L[1]}x{L[2]}x{L[3]}/n{n} {2 * cg}\n" for n in counts))
    monkeypatch.setenv("QCDW_TUNE_CACHE", str(cache))
    c = q.Context(0)
    U = li.random_gauge(L, 0.3, 81)
    kappa = 0.124
    Vh = int(np.prod(L)) // 2
    xs = np.stack([li.gaussian_source(L, 82 + k).reshape(-1, 4, 3)[:Vh] for k in range(max(counts))])
    Ainv, _ = oracle.clover_invert(L, oracle.clover_build(L, U), kappa, 1.0)
    expect = [np.asarray(oracle.schur_matpc(L, U, Ainv, x, kappa, t_bc)).reshape(Vh, 4, 3) for x in xs]
    op = q.Operator(c, q.make_lattice(L, t_bc), dev(U), kappa, 1.0, prec, 12)
    for n in counts:
        out = torch.full((n, Vh, 4, 3), float("nan"), dtype=torch.complex128, device="cuda")
        q.qcdw_op_matpc_multi(op, prec, dev(xs[:n]), out)
        out = out.cpu().numpy()
        for k in range(n):
            err = np.linalg.norm(out[k] - expect[k]) / np.linalg.norm(expect[k])
            assert err <= BOUND[prec], (n, k, err)


@pytest.mark.parametrize("inner", ["f64", "f32", "bf16", "f16"])
def test_finished_ones_between(inner):
    """Zero sources (finished from the start) at the front, in the middle and side by side, and a starting point that
    is already the solution: the others converge, these keep their answer."""
    L = (6, 4, 4, 6)
    c = q.Context(0)
    U = li.random_gauge(L, 0.25, 83)
    kappa, csw = 0.121, 1.0
    bs = np.stack([li.gaussian_source(L, 84 + k) for k in range(9)])
    for k in (0, 3, 4, 8):
        bs[k] = 0
    op = q.Operator(c, q.make_lattice(L), dev(U), kappa, csw, inner, 12)
    x = torch.zeros(bs.shape, dtype=torch.complex128, device="cuda")
    q.qcdw_invert_multi(op, dev(bs[5:6]), x[5:6], q.make_params(inner=inner))
    infos = q.qcdw_invert_multi(op, dev(bs), x, q.make_params(inner=inner))
    C = oracle.clover_build(L, U)
    for k in range(9):
        assert infos[k].status == q.QCDW_OK, (k, infos[k])
        xk = x[k].cpu().numpy()
        if k in (0, 3, 4, 8):
            assert not xk.any()
            continue
        r = bs[k] - oracle.dirac(L, U, C, xk, kappa, csw, 1)
        assert np.linalg.norm(r) <= 1e-10 * np.linalg.norm(bs[k]), k
    assert infos[5].iters == 0
