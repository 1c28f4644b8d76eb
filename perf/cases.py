"""Performance cases of the Wilson-clover framework: the calls of a propagator or HMC program, through
the public Python entry points, from the smallest lattice to the largest.

Each case is one call (or the few calls that belong together) on lattices of this repository's
workloads: 4^4, 8^3x16, 12^3x24, 16^3x32 and 24^3x64, with links exp(i eps H) of random Hermitian
traceless H.  ``draw`` varies every extent (ragged tiles among them), the hopping parameter, the inner
precision, the time boundary and the numbers of right-hand sides, problems, shifts and pairs.

``exact`` computes the same outputs in plain torch, 64 bits, from the definitions: sites in eo order with
neighbour tables, full 4x4 spin matrices, dense 6x6 clover blocks inverted by Gauss-Jordan.
"""
from __future__ import annotations

import math

import torch

import paper_2411_08461_amd as q

C128 = torch.complex128
DEV = "cuda"


# ---------------------------------------------------------------------------
# the cases
# ---------------------------------------------------------------------------
def listed():
    return [
        # the smallest call: one operator application on a test lattice (latency, launches)
        dict(name="dslash_4x4", kind="dslash", L="4x4x4x4", kappa=0.12, csw=1.0, eps=0.3, t_bc=1),
        # one full-lattice operator application on the production lattice, FP64
        dict(name="dslash_24x64", kind="dslash", L="24x24x24x64", kappa=0.125, csw=1.1, eps=0.2, t_bc=1),
        # a new gauge field arrives (each HMC or valence configuration): operator set-up for mixed-precision
        # solves (clover build and inverse, link packing in both precisions) and one use of it
        dict(name="setup_16x32", kind="setup", L="16x16x16x32", kappa=0.124, csw=1.0, eps=0.2, t_bc=1,
             inner="bf16"),
        # one FP64 solve on a cache-resident lattice
        dict(name="solve_f64_16x32", kind="solve", L="16x16x16x32", kappa=0.124, csw=1.0, eps=0.2, t_bc=1,
             inner="f64", source="z2"),
        # one mixed-precision solve on the production lattice
        dict(name="solve_bf16_24x64", kind="solve", L="24x24x24x64", kappa=0.125, csw=1.1, eps=0.2, t_bc=1,
             inner="bf16", source="point"),
        # a whole propagator: 12 spin-colour sources in one lockstep solve
        dict(name="propagator_24x64", kind="propagator", L="24x24x24x64", kappa=0.125, csw=1.1, eps=0.2, t_bc=1,
             inner="bf16", nrhs=12),
        # many uneven problems (small ensembles, mass scans) solved as one batch
        dict(name="batch_24", kind="batch", L="8x8x8x16 12x12x12x24 16x16x16x32", csw=1.0, eps=0.25, t_bc=1,
             inner="bf16", problems=24, kappa_lo=0.115, kappa_hi=0.124),
        # the poles of a rational approximation (RHMC): shifted normal-operator systems in one Krylov space
        dict(name="multishift_16x32", kind="multishift", L="16x16x16x32", kappa=0.124, csw=1.0, eps=0.2, t_bc=1,
             shifts=8, first=1e-4, ratio=4.0),
        # the clover fermion force of one HMC step (the backward pass of the action)
        dict(name="force_16x32", kind="force", L="16x16x16x32", kappa=0.124, csw=1.0, eps=0.2, t_bc=-1),
        # one gradient of the learned preconditioner's training: forward and backward over a batch of pairs
        dict(name="net_grad_16x32", kind="net_grad", L="16x16x16x32", kappa=0.124, csw=1.0, eps=0.2, t_bc=1,
             hidden=12, pairs=8),
        # the pion (or another meson) two-point function of a finished propagator
        dict(name="meson_24x64", kind="meson", L="24x24x24x64", gamma_snk=15, gamma_src=15, px=0, py=0, pz=0),
        # a multigrid-preconditioned solve with the set-up already made for the gauge field
        dict(name="mg_solve_16x32", kind="mg_solve", L="16x16x16x32", kappa=0.1255, csw=1.0, eps=0.2, t_bc=1,
             inner="bf16", block="4x4x4x4", nvec=12),
    ]


def _extents(text):
    return tuple(int(v) for v in text.split("x"))


def _volume(L):
    return L[0] * L[1] * L[2] * L[3]


def _lattice(rng, lo, hi, step=1):
    """Even extents, volume log-uniform in [lo, hi]; step: every extent a multiple of it."""
    want = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    unit = max(2, step)
    while True:
        L = [unit * max(1, round(math.exp(rng.uniform(math.log(2), math.log(32))) / unit)) for _ in range(3)]
        lt = unit * max(1, round(want / (L[0] * L[1] * L[2]) / unit))
        if 2 <= lt <= 96 and max(L) <= 32 and lo <= L[0] * L[1] * L[2] * lt <= hi:
            return "x".join(str(v) for v in (*L, lt))


def draw(rng):
    kind = rng.choice(["dslash", "dslash", "setup", "solve", "solve", "propagator", "batch", "multishift", "force",
                       "net_grad", "meson", "mg_solve"])
    big, mid = 24 ** 3 * 64, 16 ** 3 * 32
    case = dict(kind=kind, kappa=round(rng.uniform(0.115, 0.1245), 4), csw=round(rng.uniform(0.8, 1.2), 3),
                eps=round(rng.uniform(0.15, 0.25), 3), t_bc=rng.choice([1, -1]))
    inner = rng.choice(["f64", "f32", "bf16", "f16"])
    if kind == "dslash":
        case.update(L=_lattice(rng, 256, big))
    elif kind == "setup":
        case.update(L=_lattice(rng, 2048, 2 * mid), inner=inner)
    elif kind == "solve":
        case.update(L=_lattice(rng, 2048, big // 2), inner=inner, source=rng.choice(["z2", "point", "gaussian"]))
    elif kind == "propagator":
        case.update(L=_lattice(rng, 4096, big // 4), inner=rng.choice(["bf16", "f16"]), nrhs=rng.choice([3, 4, 12, 12, 16]))
    elif kind == "batch":
        hi = rng.uniform(0.118, 0.124)
        case.update(L=" ".join(_lattice(rng, 1024, mid) for _ in range(3)), inner=inner,
                    problems=rng.randint(2, 24), kappa_lo=0.115, kappa_hi=round(hi, 4))
        del case["kappa"]
    elif kind == "multishift":
        case.update(L=_lattice(rng, 2048, mid), shifts=rng.randint(1, 12), first=1e-4 * rng.randint(1, 9),
                    ratio=round(rng.uniform(2.0, 5.0), 2))
    elif kind == "force":
        case.update(L=_lattice(rng, 256, 4 * mid))
    elif kind == "net_grad":
        case.update(L=_lattice(rng, 1024, mid), hidden=rng.choice([4, 12, 12]), pairs=rng.randint(1, 8))
    elif kind == "meson":
        case = dict(kind=kind, L=_lattice(rng, 1024, big), gamma_snk=rng.randrange(16), gamma_src=rng.randrange(16),
                    px=rng.randint(0, 1), py=rng.randint(-1, 1), pz=rng.randint(0, 2))
    else:
        case.update(L=_lattice(rng, 4096, mid, step=4), kappa=round(rng.uniform(0.12, 0.1255), 4),
                    inner=rng.choice(["f64", "f32", "bf16"]), block="4x4x4x4", nvec=rng.choice([6, 8, 12]))
    return case


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
_CTX = []


def _ctx():
    """The one context that a program keeps."""
    if not _CTX:
        _CTX.append(q.Context(0))
    return _CTX[0]


def _generator(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    return g


def _normal(g, *shape):
    v = torch.randn(*shape, 2, dtype=torch.float64, device=DEV, generator=g)
    return torch.view_as_complex(v)


def _mm(a, b):
    """Products of 3x3 matrices over the leading axes."""
    out = a[..., :, 0, None] * b[..., 0, None, :]
    out += a[..., :, 1, None] * b[..., 1, None, :]
    out += a[..., :, 2, None] * b[..., 2, None, :]
    return out


def _dag(a):
    return a.conj().transpose(-1, -2).resolve_conj()


def _gauge(g, L, eps):
    """exp(i eps H), H Hermitian and traceless from complex Gaussian entries, eo layout [4, 2, Lt, Lz, Ly, Lx/2, 3, 3]."""
    V = _volume(L)
    out = torch.empty(4, V, 3, 3, dtype=C128, device=DEV)
    eye = torch.eye(3, dtype=C128, device=DEV)
    for mu in range(4):
        a = _normal(g, V, 3, 3)
        h = 0.5 * (a + _dag(a))
        tr = (h[:, 0, 0] + h[:, 1, 1] + h[:, 2, 2]) / 3
        h = (1j * eps / 16) * (h - tr[:, None, None] * eye)
        u = eye + h / 12
        for k in range(11, 0, -1):  # Taylor series of exp(h), nested; then squared four times
            u = eye + _mm(h, u) / k
        for _ in range(4):
            u = _mm(u, u)
        # rows orthonormalised, the third from the first two: SU(3) to the last bits
        r0 = u[:, 0] / torch.linalg.vector_norm(u[:, 0], dim=-1, keepdim=True)
        r1 = u[:, 1] - (r0.conj() * u[:, 1]).sum(-1, keepdim=True) * r0
        r1 = r1 / torch.linalg.vector_norm(r1, dim=-1, keepdim=True)
        r2 = torch.stack([r0[:, 1] * r1[:, 2] - r0[:, 2] * r1[:, 1], r0[:, 2] * r1[:, 0] - r0[:, 0] * r1[:, 2],
                          r0[:, 0] * r1[:, 1] - r0[:, 1] * r1[:, 0]], dim=-1).conj()
        out[mu] = torch.stack([r0, r1, r2], dim=1)
    Lx, Ly, Lz, Lt = L
    return out.reshape(4, 2, Lt, Lz, Ly, Lx // 2, 3, 3)


def _fermion_shape(L):
    return (2, L[3], L[2], L[1], L[0] // 2, 4, 3)


def _source(g, L, kind):
    shape = _fermion_shape(L)
    if kind == "gaussian":
        return _normal(g, *shape)
    if kind == "z2":
        bits = torch.randint(0, 2, (*shape, 2), device=DEV, generator=g).to(torch.float64) * 2 - 1
        return torch.view_as_complex(bits / math.sqrt(2.0))
    b = torch.zeros(shape, dtype=C128, device=DEV)
    b[0, 0, 0, 0, 0, 0, 0] = 1.0
    return b


def _inputs(case, seed):
    """Every input tensor of a case, from the seed alone (the exact values are computed from these too)."""
    g = _generator(seed)
    kind = case["kind"]
    if kind == "batch":
        Ls = [_extents(t) for t in case["L"].split()]
        probs = []
        lo, hi, n = case["kappa_lo"], case["kappa_hi"], case["problems"]
        for k in range(n):
            L = Ls[k % len(Ls)]
            U = _gauge(g, L, case["eps"])
            probs.append(dict(L=L, U=U, b=_source(g, L, "gaussian"), kappa=lo + (hi - lo) * ((7 * k) % n) / n))
        return dict(problems=probs)
    L = _extents(case["L"])
    V = _volume(L)
    if kind == "meson":
        # a propagator falls off with the distance from its source
        S = _normal(g, 12, 2, L[3], L[2], L[1], L[0] // 2, 4, 3)
        t = torch.arange(L[3], device=DEV)
        S *= torch.exp(-0.2 * torch.minimum(t, L[3] - t).to(torch.float64))[None, None, :, None, None, None, None, None]
        return dict(L=L, S=S)
    d = dict(L=L, U=_gauge(g, L, case["eps"]))
    if kind in ("dslash", "setup"):
        d["psi"] = _source(g, L, "gaussian")
        if kind == "setup":
            d["psi"] = d["psi"][0].contiguous()
    elif kind in ("solve", "mg_solve"):
        d["b"] = _source(g, L, case.get("source", "gaussian"))
    elif kind == "propagator":
        n = case["nrhs"]
        b = torch.zeros((n, *_fermion_shape(L)), dtype=C128, device=DEV)
        for k in range(n):  # the 12 spin-colour point sources at the origin, then the same at a neighbour site
            b[k, k // 12, 0, 0, 0, 0, (k % 12) // 3, k % 3] = 1.0
        d["b"] = b
    elif kind == "multishift":
        d["b"] = _normal(g, V // 2, 4, 3)
    elif kind == "force":
        d["X"], d["Y"] = _source(g, L, "gaussian"), _source(g, L, "gaussian")
    elif kind == "net_grad":
        h = case["hidden"]
        # weights as after some training: of the size of a preconditioner near the identity
        d["W1"] = (0.2 * _normal(g, 9, h, 4)).cpu()
        d["W2"] = (0.2 * _normal(g, 9, 4, h)).cpu()
        d["e"] = [_normal(g, V // 2, 4, 3) for _ in range(case["pairs"])]
        d["r"] = [e + 0.3 * _normal(g, V // 2, 4, 3) for e in d["e"]]
    return d


class _State(dict):
    """What a program holds between calls; its library objects are closed before the operator they use."""

    def __del__(self):
        for key in ("mg", "net", "batch"):
            if key in self:
                self[key].close()


TOL = 1e-11  # solves: an order below the default, so that solutions agree to about 1e-10
TOL_HARD = 1e-12  # the smallest shifts and the multigrid case are the worst conditioned


def prepare(case, seed):
    ctx, kind = _ctx(), case["kind"]
    d = _inputs(case, seed)
    st = _State(case=dict(case), ctx=ctx)
    if kind == "batch":
        ops, st["b"], st["x"] = [], [], []
        for p in d["problems"]:
            ops.append(q.Operator(ctx, q.make_lattice(p["L"], case["t_bc"]), p["U"], p["kappa"], case["csw"], case["inner"]))
            st["b"].append(p["b"])
            st["x"].append(torch.zeros_like(p["b"]))
        st["batch"] = q.Batch(ctx, ops)
        st["prm"] = q.make_params(tol=TOL, inner=case["inner"])
        return st
    L = d["L"]
    st["lat"] = lat = q.make_lattice(L, case.get("t_bc", 1))
    if kind == "meson":
        st["S"] = d["S"]
        st["out"] = torch.empty(L[3], dtype=C128, device=DEV)
        return st
    kappa, csw, U = case["kappa"], case["csw"], d["U"]
    if kind == "dslash":
        # the clover field belongs to the gauge field: built once, used by every application
        clover = torch.empty(2, L[3], L[2], L[1], L[0] // 2, 2, 36, dtype=torch.float64, device=DEV)
        q.qcdw_clover_build(ctx, lat, U, clover)
        st.update(U=U, clover=clover, psi=d["psi"], out=torch.empty_like(d["psi"]))
    elif kind == "setup":
        st.update(U=U, psi=d["psi"], out=torch.empty_like(d["psi"]))
        # the kernel forms of a lattice are timed once in a program, not for each gauge field
        q.Operator(ctx, lat, U, kappa, csw, case["inner"]).close()
    elif kind in ("solve", "propagator"):
        st.update(op=q.Operator(ctx, lat, U, kappa, csw, case["inner"]), b=d["b"], x=torch.zeros_like(d["b"]),
                  prm=q.make_params(tol=TOL, inner=case["inner"]))
    elif kind == "multishift":
        st.update(op=q.Operator(ctx, lat, U, kappa, csw), b=d["b"], x=[torch.empty_like(d["b"]) for _ in range(case["shifts"])],
                  shifts=[case["first"] * case["ratio"] ** k for k in range(case["shifts"])])
    elif kind == "force":
        st.update(U=U, X=d["X"], Y=d["Y"], H=torch.empty_like(U))
    elif kind == "net_grad":
        op = q.Operator(ctx, lat, U, kappa, csw)
        net = q.qcdw_net_create(op, case["hidden"])
        q.qcdw_net_set_weights(net, d["W1"].numpy(), d["W2"].numpy())
        st.update(net=net, r=d["r"], e=d["e"])
    else:
        op = q.Operator(ctx, lat, U, kappa, csw, case["inner"])
        mg = q.Multigrid(op, q.make_mg_params(block=_extents(case["block"]), nvec=case["nvec"]))
        st.update(mg=mg, op=op, b=d["b"], x=torch.zeros_like(d["b"]), prm=q.make_params(tol=TOL_HARD, inner=case["inner"]))
    return st


def run(st):
    case, ctx = st["case"], st["ctx"]
    kind = case["kind"]
    if kind == "dslash":
        q.qcdw_dslash(ctx, st["lat"], st["U"], st["clover"], st["psi"], st["out"], case["kappa"], case["csw"])
        return st["out"]
    if kind == "setup":
        op = q.qcdw_op_create(ctx, st["lat"], st["U"], case["kappa"], case["csw"], case["inner"])
        q.qcdw_op_matpc(op, "f64", st["psi"], st["out"])
        q.qcdw_op_destroy(op)
        return st["out"]
    if kind == "solve":
        st["x"].zero_()
        q.qcdw_invert(st["op"], st["b"], st["x"], st["prm"], raise_on_error=True)
        return st["x"]
    if kind == "propagator":
        st["x"].zero_()
        q.qcdw_invert_multi(st["op"], st["b"], st["x"], st["prm"])
        return st["x"]
    if kind == "batch":
        for x in st["x"]:
            x.zero_()
        q.qcdw_invert_batch(st["batch"], st["b"], st["x"], st["prm"])
        return st["x"]
    if kind == "multishift":
        q.qcdw_invert_multishift(st["op"], st["b"], st["x"], st["shifts"], tol=TOL_HARD)
        return st["x"]
    if kind == "force":
        q.qcdw_clover_force(ctx, st["lat"], st["U"], st["X"], st["Y"], case["kappa"], case["csw"], st["H"])
        return st["H"]
    if kind == "net_grad":
        loss, g1, g2 = q.qcdw_net_loss_grad(st["net"], st["r"], st["e"])
        # weights, activations and gradients of the net are FP32: the gradients as the optimiser takes them
        return {"loss": torch.tensor(loss, dtype=torch.float32), "g1": g1.astype("complex64"), "g2": g2.astype("complex64")}
    if kind == "meson":
        q.qcdw_meson_2pt(ctx, st["lat"], st["S"], case["gamma_snk"], case["gamma_src"], (case["px"], case["py"], case["pz"]),
                         st["out"])
        return st["out"]
    st["x"].zero_()
    q.qcdw_invert_mg(st["op"], st["mg"], st["b"], st["x"], st["prm"])
    return st["x"]


# ---------------------------------------------------------------------------
# work
# ---------------------------------------------------------------------------
# Krylov iterations that a solve of the listed kind takes (TOL, FP64 recurrence); they grow with kappa
def _iterations(kappa):
    return 60.0 if kappa <= 0.1245 else 75.0


_FP = {"f64": 16, "f32": 8, "bf16": 4, "f16": 4}  # bytes of a stored complex number


def _iteration_bytes(cb, nrhs=1):
    """Bytes per even site of one BiCGStab iteration on the even-odd operator with cb bytes per complex:
    4 hops (8 links of 6 entries and 36 clover complex, shared by the right-hand sides; one spinor in, one
    out, the xpay operand in half of them) and 14 vector passes."""
    return cb * (4 * (48 + 36) + nrhs * (4 * 24 + 2 * 12 + 14 * 12))


def work(case):
    kind = case["kind"]
    if kind == "batch":
        Ls = [_extents(t) for t in case["L"].split()]
        half = sum(_volume(Ls[k % len(Ls)]) // 2 for k in range(case["problems"]))
        it = _iterations(case["kappa_hi"])
        return {"bytes": half * it * _iteration_bytes(_FP[case["inner"]]), "flops": half * it * 4 * 1900.0}
    V = _volume(_extents(case["L"]))
    half = V // 2
    if kind == "dslash":  # links, clover and spinor in, spinor out
        return {"bytes": V * 1536.0, "flops": V * 1900.0}
    if kind == "setup":  # links in; links, A and its inverse out in FP64 and the inner precision; one M_hat
        cb = _FP[case["inner"]]
        lo = 0 if cb == 16 else cb * (24 + 36)
        return {"bytes": V * (576.0 + 384 + 2 * 576 + lo) + half * (2 * 1728.0 + 384), "flops": V * (6 * 4 * 600.0 + 3000)}
    if kind == "solve":
        it = _iterations(case["kappa"])
        return {"bytes": half * it * _iteration_bytes(_FP[case["inner"]]), "flops": half * it * 4 * 1900.0}
    if kind == "propagator":
        it, n = _iterations(case["kappa"]), case["nrhs"]
        return {"bytes": half * it * _iteration_bytes(_FP[case["inner"]], n), "flops": half * n * it * 4 * 1900.0}
    if kind == "multishift":  # per iteration four hops and two clover products; every live shift's x and p
        it = 130.0
        return {"bytes": half * it * (16 * (6 * 36 + 4 * 48 + 4 * 36) + 0.5 * case["shifts"] * 768.0), "flops": half * it * 8000.0}
    if kind == "force":  # links, X and Y in, H out
        return {"bytes": V * (576.0 + 2 * 192 + 576), "flops": V * 4 * (6 * 9 * 198.0 + 2000)}
    if kind == "net_grad":  # forward and backward of both layers: six channel mixings of 9 hops
        h = case["hidden"]
        return {"bytes": case["pairs"] * V * (2 * 192.0 + 3 * 192 + 4 * 24 * h), "flops": case["pairs"] * V * 6 * 9 * 3 * 4 * h * 8.0}
    if kind == "meson":
        return {"bytes": V * 2304.0, "flops": V * 2000.0}
    return {"bytes": half * 20 * (4 * _iteration_bytes(_FP[case["inner"]]) + 4 * case["nvec"] * 48.0), "flops": half * 20 * 30000.0}


# ---------------------------------------------------------------------------
# exact values
# ---------------------------------------------------------------------------
# DeGrand-Rossi gammas: gamma_mu has one nonzero per row, (gamma_mu)[s][PERM[mu][s]] = PHASE[mu][s]
PERM = [[3, 2, 1, 0], [3, 2, 1, 0], [2, 3, 0, 1], [2, 3, 0, 1]]
PHASE = [[1j, 1j, -1j, -1j], [-1, 1, 1, -1], [1j, -1j, -1j, 1j], [1, 1, 1, 1]]


def _gamma(mu):
    m = torch.zeros(4, 4, dtype=C128)
    for s in range(4):
        m[s, PERM[mu][s]] = PHASE[mu][s]
    return m


def _gamma_mask(n):
    m = torch.eye(4, dtype=C128)
    for mu in range(4):
        if (n >> mu) & 1:
            m = m @ _gamma(mu)
    return m


def _coords(L):
    """Coordinates [V] of the sites in eo order."""
    Lx, Ly, Lz, Lt = L
    p, t, z, y, xh = torch.meshgrid(torch.arange(2), torch.arange(Lt), torch.arange(Lz), torch.arange(Ly),
                                    torch.arange(Lx // 2), indexing="ij")
    x = 2 * xh + ((p + y + z + t) % 2)
    return [v.reshape(-1).to(DEV) for v in (x, y, z, t)]


class _Lattice:
    """Neighbour tables in eo order."""

    def __init__(self, L):
        self.L, self.V = L, _volume(L)
        self.c = _coords(L)
        self.fwd = [self.shift(mu, 1) for mu in range(4)]
        self.bwd = [self.shift(mu, -1) for mu in range(4)]

    def shift(self, mu, d):
        c = list(self.c)
        c[mu] = (c[mu] + d) % self.L[mu]
        x, y, z, t = c
        Lx, Ly, Lz, _ = self.L
        return ((x + y + z + t) % 2) * (self.V // 2) + ((t * Lz + z) * Ly + y) * (Lx // 2) + x // 2


def _colour(U, psi):
    """U psi for links [n, 3, 3] and spinors [n, S, 3]."""
    out = U[:, None, :, 0] * psi[:, :, 0, None]
    out += U[:, None, :, 1] * psi[:, :, 1, None]
    out += U[:, None, :, 2] * psi[:, :, 2, None]
    return out


class _Dirac:
    """M = A - kappa H in 64 bits, on the sites of each parity."""

    def __init__(self, L, U, kappa, csw, t_bc, invert=True):
        lat = self.lat = _Lattice(L)
        self.kappa, self.V, self.h = kappa, lat.V, lat.V // 2
        U = U.reshape(4, lat.V, 3, 3)
        self.perm = [torch.tensor(p, device=DEV) for p in PERM]
        self.ph = [torch.tensor(p, dtype=C128, device=DEV)[:, None] for p in PHASE]
        self.hops = []  # per parity and direction: links and neighbours (indices within the other parity)
        for p in range(2):
            own, other = slice(p * self.h, (p + 1) * self.h), (1 - p) * self.h
            rows = []
            for mu in range(4):
                uf, b = U[mu, own], lat.bwd[mu][own]
                ub = _dag(U[mu, b])
                if mu == 3 and t_bc < 0:
                    t = lat.c[3][own]
                    uf = uf * torch.where(t == L[3] - 1, -1.0, 1.0)[:, None, None]
                    ub = ub * torch.where(t == 0, -1.0, 1.0)[:, None, None]
                rows.append((uf, lat.fwd[mu][own] - other, ub, b - other))
            self.hops.append(rows)
        self.A = self.blocks(U, kappa, csw)
        self.Ainv = _invert6(self.A) if invert else None

    def blocks(self, U, kappa, csw):
        """A = 1 - kappa csw sum sigma F as [V, 2, 6, 6] chirality blocks."""
        lat = self.lat
        A = torch.zeros(lat.V, 2, 6, 6, dtype=C128, device=DEV)
        for k in range(6):
            A[:, :, k, k] = 1.0
        eye = torch.eye(3, dtype=C128, device=DEV)
        for mu in range(4):
            for nu in range(mu + 1, 4):
                def at(rho, *steps):
                    i = None
                    for m, d in steps:
                        s = (lat.fwd if d > 0 else lat.bwd)[m]
                        i = s if i is None else s[i]
                    return U[rho] if i is None else U[rho][i]
                Um, Un = U[mu], U[nu]
                Q = _mm(_mm(_mm(Um, at(nu, (mu, 1))), _dag(at(mu, (nu, 1)))), _dag(Un))
                Q += _mm(_mm(_mm(Un, _dag(at(mu, (mu, -1), (nu, 1)))), _dag(at(nu, (mu, -1)))), at(mu, (mu, -1)))
                Q += _mm(_mm(_mm(_dag(at(mu, (mu, -1))), _dag(at(nu, (mu, -1), (nu, -1)))), at(mu, (mu, -1), (nu, -1))),
                         at(nu, (nu, -1)))
                Q += _mm(_mm(_mm(_dag(at(nu, (nu, -1))), at(mu, (nu, -1))), at(nu, (mu, 1), (nu, -1))), _dag(Um))
                F = (Q - _dag(Q)) / 8
                F = F - ((F[:, 0, 0] + F[:, 1, 1] + F[:, 2, 2]) / 3)[:, None, None] * eye
                sigma = _gamma(mu) @ _gamma(nu)
                for s in range(4):
                    for r in range(4):
                        w = complex(sigma[s, r])
                        if w:
                            i, j = 3 * (s % 2), 3 * (r % 2)
                            A[:, s // 2, i:i + 3, j:j + 3] -= (kappa * csw * w) * F
        return A

    def hop(self, p, psi):
        """H psi on the sites of parity p from the field [h, 4, 3] of the other parity."""
        out = torch.zeros_like(psi)
        for mu in range(4):
            uf, f, ub, b = self.hops[p][mu]
            w = _colour(uf, psi[f])
            out += w
            out -= self.ph[mu] * w[:, self.perm[mu]]
            w = _colour(ub, psi[b])
            out += w
            out += self.ph[mu] * w[:, self.perm[mu]]
        return out

    def site(self, M, p, psi):
        """The 6x6 blocks of parity p times a field."""
        own = M[p * self.h:(p + 1) * self.h]
        v = psi.reshape(self.h, 2, 6)
        out = own[..., 0] * v[:, :, 0, None]
        for k in range(1, 6):
            out += own[..., k] * v[:, :, k, None]
        return out.reshape(self.h, 4, 3)

    def matpc(self, v):
        t = self.site(self.Ainv, 1, self.hop(1, v))
        return v - self.kappa ** 2 * self.site(self.Ainv, 0, self.hop(0, t))

    def matpc_dag(self, v):
        """M_hat^+ = 1 - kappa^2 g5 H_eo A_oo^-1 H_oe g5 A_ee^-1 (g5 M g5 = M^+, and g5 commutes with A)."""
        g5 = self.g5
        t = self.site(self.Ainv, 1, self.hop(1, g5 * self.site(self.Ainv, 0, v)))
        return v - self.kappa ** 2 * g5 * self.hop(0, t)

    @property
    def g5(self):
        return torch.diagonal(_gamma_mask(15)).to(DEV)[:, None]

    def full(self, psi):
        v = psi.reshape(2, self.h, 4, 3)
        return torch.stack([self.site(self.A, p, v[p]) - self.kappa * self.hop(p, v[1 - p]) for p in range(2)])

    def solve(self, b):
        """x = M^-1 b by BiCGStab on the even sites, restarted from the true residual, to about 1e-15."""
        v = b.reshape(2, self.h, 4, 3)
        ye, yo = self.site(self.Ainv, 0, v[0]), self.site(self.Ainv, 1, v[1])
        rhs = ye + self.kappa * self.site(self.Ainv, 0, self.hop(0, yo))
        x = torch.zeros_like(rhs)
        stop = 1e-15 * float(torch.linalg.vector_norm(rhs))
        for _ in range(8):
            r = rhs - self.matpc(x)
            rn = float(torch.linalg.vector_norm(r))
            if rn <= 2 * stop:
                break
            x = x + _bicgstab(self.matpc, r, max(stop, 1e-9 * rn))
        xo = yo + self.kappa * self.site(self.Ainv, 1, self.hop(1, x))
        return torch.stack([x, xo]).reshape(b.shape)


def _dot(a, b):
    return torch.sum(a.conj() * b)


def _bicgstab(op, b, stop):
    x, r = torch.zeros_like(b), b.clone()
    r0, p = b.clone(), b.clone()
    rho = _dot(r0, r)
    for it in range(5000):
        v = op(p)
        alpha = rho / _dot(r0, v)
        s = r - alpha * v
        t = op(s)
        omega = _dot(t, s) / _dot(t, t)
        x += alpha * p + omega * s
        r = s - omega * t
        if it % 4 == 3 and not float(torch.linalg.vector_norm(r)) > stop:
            break
        new = _dot(r0, r)
        p = r + (new / rho) * (alpha / omega) * (p - omega * v)
        rho = new
    return x


def _cg(op, b, stop):
    x, r, p = torch.zeros_like(b), b.clone(), b.clone()
    rr = _dot(r, r).real
    for it in range(5000):
        v = op(p)
        a = rr / _dot(p, v).real
        x += a * p
        r -= a * v
        new = _dot(r, r).real
        if it % 4 == 3 and not math.sqrt(float(new)) > stop:
            break
        p = r + (new / rr) * p
        rr = new
    return x


def _invert6(A):
    """Inverse of Hermitian positive blocks by Gauss-Jordan elimination on the diagonal."""
    M = torch.cat([A, torch.eye(6, dtype=C128, device=DEV).expand_as(A)], dim=-1)
    for k in range(6):
        row = M[..., k, :] / M[..., k, k, None]
        M = M - M[..., :, k, None] * row[..., None, :]
        M[..., k, :] = row
    return M[..., 6:].contiguous()


def _transport(lat, U, a, phi):
    """T_a phi of channels [V, C, 3]: 1, then U_mu(x) phi(x+mu) and U_mu(x-mu)^+ phi(x-mu)."""
    if a == 0:
        return phi
    mu, back = (a - 1) // 2, (a - 1) % 2
    if back == 0:
        return _colour(U[mu], phi[lat.fwd[mu]])
    return _colour(_dag(U[mu][lat.bwd[mu]]), phi[lat.bwd[mu]])


def _net_grad(d):
    lat = _Lattice(d["L"])
    U = d["U"].reshape(4, lat.V, 3, 3)
    W1, W2 = d["W1"].to(DEV), d["W2"].to(DEV)
    h = lat.V // 2

    def mix(w, phi):  # [out, in] x [V, in, 3]
        out = torch.zeros(lat.V, w.shape[0], 3, dtype=C128, device=DEV)
        for c in range(w.shape[1]):
            out += w[None, :, c, None] * phi[:, None, c]
        return out

    def layer(W, phi):
        return sum(mix(W[a], _transport(lat, U, a, phi)) for a in range(9))

    def adjoint(W, g):
        return sum(_transport(lat, U, 0 if a == 0 else (a + 1 if a % 2 else a - 1), mix(W[a].conj().T.contiguous(), g))
                   for a in range(9))

    def flat(v):
        return v.transpose(0, 1).reshape(v.shape[1], -1)

    def weight_grad(phi, g):
        return torch.stack([flat(g) @ flat(_transport(lat, U, a, phi)).conj().T.contiguous() for a in range(9)])

    def embed(e):
        return torch.cat([e, torch.zeros_like(e)])

    loss, g1, g2 = 0.0, torch.zeros_like(W1), torch.zeros_like(W2)
    for r, e in zip(d["r"], d["e"]):
        phi = embed(r)
        hid = layer(W1, phi)
        diff = layer(W2, hid)[:h] - e
        en = float(torch.sum(e.abs() ** 2))
        loss += float(torch.sum(diff.abs() ** 2)) / en
        gz = embed(2.0 * diff / en)
        g2 += weight_grad(hid, gz)
        g1 += weight_grad(phi, adjoint(W2, gz))
    return {"loss": torch.tensor(loss, dtype=torch.float64), "g1": g1, "g2": g2}


def _force(case, d):
    """H = sum_a T^a d/dw [2 Re Y^+ M X] along exp(i w T^a) U: minus half of the traceless Hermitian part of
    U g^+ / i, g the gradient of the bilinear with respect to the link's real and imaginary parts."""
    U = d["U"].clone().requires_grad_(True)
    with torch.enable_grad():
        D = _Dirac(d["L"], U, case["kappa"], case["csw"], case["t_bc"], invert=False)
        S = 2.0 * torch.sum(d["Y"].reshape(-1).conj() * D.full(d["X"]).reshape(-1)).real
        g, = torch.autograd.grad(S, U)
    B = _mm(d["U"], _dag(g))
    K = (B - _dag(B)) / 2j
    tr = (K[..., 0, 0] + K[..., 1, 1] + K[..., 2, 2]) / 3
    return -0.5 * (K - tr[..., None, None] * torch.eye(3, dtype=C128, device=DEV))


def exact(case, seed):
    kind = case["kind"]
    size = sum(_volume(_extents(t)) for t in case["L"].split())
    if kind == "propagator" and size * case["nrhs"] > 8_000_000:
        return None  # 12 solves of the largest lattice take over 20 seconds
    d = _inputs(case, seed)
    with torch.no_grad():
        if kind == "batch":
            return [_Dirac(p["L"], p["U"], p["kappa"], case["csw"], case["t_bc"]).solve(p["b"]) for p in d["problems"]]
        if kind == "net_grad":
            return _net_grad(d)
        if kind == "force":
            return _force(case, d)
        if kind == "meson":
            return _meson(case, d)
        D = _Dirac(d["L"], d["U"], case["kappa"], case["csw"], case["t_bc"], invert=kind != "dslash")
        if kind == "dslash":
            return D.full(d["psi"]).reshape(d["psi"].shape)
        if kind == "setup":
            return D.matpc(d["psi"].reshape(-1, 4, 3)).reshape(d["psi"].shape)
        if kind == "propagator":
            return torch.stack([D.solve(b) for b in d["b"]])
        if kind == "multishift":
            out, norm = [], float(torch.linalg.vector_norm(d["b"]))
            for k in range(case["shifts"]):
                sigma = case["first"] * case["ratio"] ** k

                def normal(v):
                    return D.matpc_dag(D.matpc(v)) + sigma * v
                x = _cg(normal, d["b"], 1e-13 * norm)
                out.append(x + _cg(normal, d["b"] - normal(x), 1e-15 * norm))
            return out
        return D.solve(d["b"])


def _meson(case, d):
    """C(t) = sum_x e^{-ip.x} Tr[G_snk S(x) G_src g5 S(x)^+ g5], S(x)[3 s + c, 3 s0 + c0] = field 3 s0 + c0."""
    L = d["L"]
    x, y, z, t = _coords(L)
    x, y, z = (v.to(torch.float64) for v in (x, y, z))
    phase = torch.exp(-2j * math.pi * (case["px"] * x / L[0] + case["py"] * y / L[1] + case["pz"] * z / L[2]))
    g5 = _gamma_mask(15)
    left, right = g5 @ _gamma_mask(case["gamma_snk"]), _gamma_mask(case["gamma_src"]) @ g5
    S = d["S"].reshape(4, 3, -1, 4, 3)  # [s0, c0, x, s, c]
    site = torch.zeros(S.shape[2], dtype=C128, device=DEV)
    for a in range(4):
        for b in range(4):
            for s in range(4):
                for r in range(4):  # left[a, b] S[b, s] right[s, r] conj(S[a, r])
                    w = complex(left[a, b] * right[s, r])
                    if w:
                        for c0 in range(3):
                            site += w * torch.sum(S[s, c0, :, b] * S[r, c0, :, a].conj(), dim=-1)
    out = torch.zeros(L[3], dtype=C128, device=DEV)
    v = (phase * site).reshape(2, L[3], -1)
    for k in range(L[3]):
        out[k] = v[:, k].sum()
    return out
