// Clover fermion force: the derivative of the bilinear 2 Re(Y^+ M X) with respect to every link.
//
// HMC with clover fermions (paper Sec. IV) moves the links along the derivative of the pseudo-fermion
// action; for S = phi^+ (M^+ M)^-1 phi with X = (M^+ M)^-1 phi and Y = M X the change of S is
// -2 Re(Y^+ dM X).  For a link variation U_mu(x) -> exp(i w T^a) U_mu(x) the derivative of
// 2 Re(Y^+ M X) is F^a = 2 Tr(T^a H_mu(x)), and this file computes the Hermitian traceless H_mu(x):
//
//   hop term (M = A - kappa H):  K = kappa s (B - B^+) / (2i),  B = U A1 - A2 U^+,
//     A1 = sum_s [(1 - g_mu) X(x+mu)]_s Y(x)_s^+,  A2 = sum_s [(1 + g_mu) X(x)]_s Y(x+mu)_s^+,
//     s the time-boundary sign of the link;
//   clover term (A = 1 - kappa csw sum_{mu<nu} sigma_{mu nu} F_{mu nu}, F = traceless (Q - Q^+)/8):
//     with Gam_{mu nu}(x) = the traceless part of (L - L^+), L = sum_s (sigma_{mu nu} X(x))_s Y(x)_s^+,
//     every leaf through the link contributes +-(kappa csw / 8)(G - G^+)/(2i), G the leaf's loop started
//     at x along the link (leaves that run the link forward, +) or ended along it backward (-), with
//     Gam inserted at the leaf's base corner.  For the link in direction rho and a plane (rho, sig), the
//     forward leaves are the four corners of the plaquette on the +sig side when rho is the plane's first
//     direction (on the -sig side when it is the second), the backward leaves the four corners of the
//     other plaquette.
// Gam is anti-Hermitian, so the two kinds of leaves are one: with S = U2 U3 U4 the staple from x+rho round a
// plaquette to x and d = +-sig its side, both are +-U_rho(x) T,
//   T = Gam(x+rho) S + U2 (Gam(x+rho+d) U3 U4 + U3 (Gam(x+d) U4 + U4 Gam(x))),
// a backward leaf as the adjoint of the same expression; likewise -A2 U^+ gives the part of U A2^+.  A link's
// six plaquettes and its hop term are summed before the one product with U: 8 products a plaquette instead of 12.
//
// Three kernels.  The links go to plane-major copies (launch_pack_links, 9 entries).  k_force_gamma takes 64 sites
// per block, stages X and Y in LDS, writes Gam as 8 real planes per lattice plane and X and Y as 12 complex
// planes each.  k_force_link takes 64 sites of one parity per block, a wave per link direction and a lane per site,
// so every load is a whole run; H leaves through LDS.  From the paper's records (144 and 192 bytes, a cache line
// per lane and load) with Gam in full matrices the link kernel took 574 us at 16^3x32, bound by the address path.
// Measured at 16^3x32, one call: 606 -> 238 us (link copies 32, Gam 30, links 170 us).  The link kernel's multiply-adds
// need 88 us at the full FP64 rate; two waves per SIMD (256 VGPRs) hide the loads better than one (215 us) and than
// three, which spill (395 us).
#include "host.h"

namespace qcdw {

namespace {

using c3 = cx<double>[3][3];

// DeGrand-Rossi gamma_mu: one nonzero per row, gamma_mu[s][perm] = ph
__device__ __forceinline__ constexpr int gperm(int mu, int s) { return mu < 2 ? 3 - s : (s + 2) & 3; }
__device__ __forceinline__ cx<double> gph(int mu, int s)
{
    switch (mu) {
    case 0: return s < 2 ? cx<double>{0.0, 1.0} : cx<double>{0.0, -1.0};
    case 1: return (s == 0 || s == 3) ? cx<double>{-1.0, 0.0} : cx<double>{1.0, 0.0};
    case 2: return (s == 0 || s == 3) ? cx<double>{0.0, 1.0} : cx<double>{0.0, -1.0};
    default: return {1.0, 0.0};
    }
}

// plane index of (mu, nu), mu < nu: (0,1) (0,2) (0,3) (1,2) (1,3) (2,3)
__device__ __forceinline__ int plane_of(int mu, int nu)
{
    return mu == 0 ? nu - 1 : (mu == 1 ? nu + 1 : 5);
}

// t = u t, in place column by column
__device__ __forceinline__ void left_mul(const c3& u, c3& t)
{
#pragma unroll
    for (int j = 0; j < 3; j++) {
        const cx<double> a = t[0][j], b = t[1][j], c = t[2][j];
#pragma unroll
        for (int i = 0; i < 3; i++) {
            cx<double> s = u[i][0] * a;
            cmac(s, u[i][1], b);
            cmac(s, u[i][2], c);
            t[i][j] = s;
        }
    }
}

// A traceless anti-Hermitian matrix by its 8 reals: Im of entries 00 and 11, then entries 01, 02, 12
struct Anti {
    double r[8];
    __device__ __forceinline__ double diag(int i) const { return i < 2 ? r[i] : -(r[0] + r[1]); }
    __device__ __forceinline__ cx<double> at(int i, int j) const  // i != j
    {
        const int k = 2 * (i + j);
        return i < j ? cx<double>{r[k], r[k + 1]} : cx<double>{-r[k], r[k + 1]};
    }
};

// t += G m, and t += m G
__device__ __forceinline__ void add_gm(c3& t, const Anti& G, const c3& m)
{
#pragma unroll
    for (int i = 0; i < 3; i++)
#pragma unroll
        for (int j = 0; j < 3; j++) {
#pragma unroll
            for (int k = 0; k < 3; k++) {
                if (k == i) {
                    t[i][j].re -= G.diag(i) * m[i][j].im;
                    t[i][j].im += G.diag(i) * m[i][j].re;
                } else {
                    cmac(t[i][j], G.at(i, k), m[k][j]);
                }
            }
        }
}
__device__ __forceinline__ void add_mg(c3& t, const c3& m, const Anti& G)
{
#pragma unroll
    for (int i = 0; i < 3; i++)
#pragma unroll
        for (int j = 0; j < 3; j++) {
#pragma unroll
            for (int k = 0; k < 3; k++) {
                if (k == j) {
                    t[i][j].re -= G.diag(j) * m[i][j].im;
                    t[i][j].im += G.diag(j) * m[i][j].re;
                } else {
                    cmac(t[i][j], G.at(k, j), m[i][k]);
                }
            }
        }
}

constexpr int FS = 64;  // sites per block

// Gam of plane (MU, NU) at a site: the traceless part of L - L^+, L = sum_s (sigma X)_s Y_s^+, sigma_{mu nu} = g_mu g_nu
// (mu != nu, the DeGrand-Rossi gammas anticommute)
template <int MU, int NU>
__device__ __forceinline__ Anti gamma_plane(const double2* x, const double2* y)
{
    c3 L;
#pragma unroll
    for (int i = 0; i < 3; i++)
#pragma unroll
        for (int j = 0; j < 3; j++) L[i][j] = {0.0, 0.0};
#pragma unroll
    for (int s = 0; s < 4; s++) {
        const int s1 = gperm(MU, s), s2 = gperm(NU, s1);
        const cx<double> ph = gph(MU, s) * gph(NU, s1);  // (g_mu g_nu)[s][s2]
#pragma unroll
        for (int i = 0; i < 3; i++) {
            const double2 v = x[3 * s2 + i];
            const cx<double> sx = ph * cx<double>{v.x, v.y};
#pragma unroll
            for (int j = 0; j < 3; j++) {
                const double2 w = y[3 * s + j];
                cmac_conj(L[i][j], {w.x, w.y}, sx);
            }
        }
    }
    const double tr = (L[0][0].im + L[1][1].im + L[2][2].im) * (2.0 / 3.0);
    Anti G;
    G.r[0] = 2.0 * L[0][0].im - tr;
    G.r[1] = 2.0 * L[1][1].im - tr;
#pragma unroll
    for (int k = 0; k < 3; k++) {
        const int i = k == 2 ? 1 : 0, j = k == 0 ? 1 : 2;
        G.r[2 + 2 * k] = L[i][j].re - L[j][i].re;
        G.r[3 + 2 * k] = L[i][j].im + L[j][i].im;
    }
    return G;
}

}  // namespace

// Gam[(8 plane + k) V + e] (6 planes, V sites in eo order) and, unless it is null, XY[c V + e]: the 12 components of X,
// then of Y
__global__ __launch_bounds__(384) void k_force_gamma(int V, const double2* __restrict__ X,
                                                     const double2* __restrict__ Y, double* __restrict__ Gam,
                                                     double2* __restrict__ XY)
{
    constexpr int ROW = 13;  // 12 complex padded: a lane's row starts in another bank than its neighbours'
    __shared__ double2 sx[FS * ROW], sy[FS * ROW];
    const int e0 = blockIdx.x * FS, n = V - e0 < FS ? V - e0 : FS;
    for (int k = threadIdx.x; k < n * 12; k += 384) {
        sx[k / 12 * ROW + k % 12] = X[(long)e0 * 12 + k];
        sy[k / 12 * ROW + k % 12] = Y[(long)e0 * 12 + k];
    }
    __syncthreads();
    const int lane = threadIdx.x & 63, plane = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (lane >= n) return;
    const double2 *x = sx + lane * ROW, *y = sy + lane * ROW;
    if (XY)
        for (int c = plane; c < 24; c += 6) XY[(long)c * V + e0 + lane] = c < 12 ? x[c] : y[c - 12];
    Anti G;
    switch (plane) {
    case 0: G = gamma_plane<0, 1>(x, y); break;
    case 1: G = gamma_plane<0, 2>(x, y); break;
    case 2: G = gamma_plane<0, 3>(x, y); break;
    case 3: G = gamma_plane<1, 2>(x, y); break;
    case 4: G = gamma_plane<1, 3>(x, y); break;
    default: G = gamma_plane<2, 3>(x, y); break;
    }
#pragma unroll
    for (int k = 0; k < 8; k++) Gam[(long)(8 * plane + k) * V + e0 + lane] = G.r[k];
}

namespace {

// What a lane of k_force_link reads: Gam's planes, and the links and spinors from F, a source of the numbers of one
// link and of one component of X (0 .. 11) or Y (12 .. 23) at an eo site
struct PlaneFields {
    LinkPlanes U;
    const double2* XY;
    struct Link {
        const double2 *p, *q;
        long Vh;
        __device__ __forceinline__ double2 operator[](int e) const { return e < 6 ? p[e * Vh] : q[(e - 6) * Vh]; }
    };
    __device__ __forceinline__ long Vh() const { return U.Vh; }
    __device__ __forceinline__ Link link(int mu, Site s) const
    {
        return {U.top + (long)(mu * 2 + s.parity) * U.top_rec * U.Vh + s.cb,
                U.low + (long)(mu * 2 + s.parity) * U.low_rec * U.Vh + s.cb, U.Vh};
    }
    __device__ __forceinline__ double2 spinor(int c, long e) const { return XY[c * 2 * U.Vh + e]; }
};
// the caller's records, for a call that finds no memory for copies
struct RecordFields {
    const double2 *U, *X, *Y;
    long nVh;
    __device__ __forceinline__ long Vh() const { return nVh; }
    __device__ __forceinline__ const double2* link(int mu, Site s) const
    {
        return U + ((long)(mu * 2 + s.parity) * nVh + s.cb) * 9;
    }
    __device__ __forceinline__ double2 spinor(int c, long e) const { return c < 12 ? X[e * 12 + c] : Y[e * 12 + c - 12]; }
};
template <class F>
struct ForceFields : F {
    const double* Gam;
    // link (mu, site), adjoint if DAG
    template <bool DAG>
    __device__ __forceinline__ void link(int mu, Site s, c3& m) const
    {
        const auto u = F::link(mu, s);
#pragma unroll
        for (int e = 0; e < 9; e++) {
            const double2 v = u[e];
            if (DAG)
                m[e % 3][e / 3] = {v.x, -v.y};
            else
                m[e / 3][e % 3] = {v.x, v.y};
        }
    }
    __device__ __forceinline__ Anti gam(int p, Site s) const
    {
        Anti G;
#pragma unroll
        for (int k = 0; k < 8; k++) G.r[k] = Gam[(long)(8 * p + k) * 2 * F::Vh() + s.parity * F::Vh() + s.cb];
        return G;
    }
    // row k of the half-spinor (1 + sg gamma_mu) projects a spinor on (X: first = 0, Y: first = 12), see hop_common.h
    __device__ __forceinline__ void half(int first, Site s, int mu, int k, double sg, cx<double> (&h)[3]) const
    {
        const long e = s.parity * F::Vh() + s.cb;
        const int l = gperm(mu, k);
        const cx<double> c = gph(mu, k);
#pragma unroll
        for (int i = 0; i < 3; i++) {
            const double2 a = F::spinor(first + 3 * k + i, e), b = F::spinor(first + 3 * l + i, e);
            const cx<double> w = c * cx<double>{b.x, b.y};
            h[i] = {a.x + sg * w.re, a.y + sg * w.im};
        }
    }
};

// acc += sgn T for the plaquette of (rho, sig) on side D = +-1 (file header)
template <int D, class F>
__device__ __forceinline__ void add_plaquette(const ForceFields<F>& f, const Geom& g, const int (&c)[4], int rho, int sig,
                                              int p, double sgn, Site y, Site yr, c3& acc)
{
    const Site yd = site_step(g, c, sig, D, sig, 0), yrd = site_step(g, c, rho, 1, sig, D);
    c3 S, t, u;
    f.template link<(D > 0)>(sig, D > 0 ? y : yd, S);  // U4: from x+d to x
#pragma unroll
    for (int i = 0; i < 3; i++)
#pragma unroll
        for (int j = 0; j < 3; j++) t[i][j] = {0.0, 0.0};
    add_gm(t, f.gam(p, yd), S);
    add_mg(t, S, f.gam(p, y));
    f.template link<true>(rho, yd, u);  // U3: from x+rho+d to x+d
    left_mul(u, t);
    left_mul(u, S);
    add_gm(t, f.gam(p, yrd), S);
    f.template link<(D < 0)>(sig, D > 0 ? yr : yrd, u);  // U2: from x+rho to x+rho+d
    left_mul(u, t);
    left_mul(u, S);
    add_gm(t, f.gam(p, yr), S);
#pragma unroll
    for (int i = 0; i < 3; i++)
#pragma unroll
        for (int j = 0; j < 3; j++) {
            acc[i][j].re += sgn * t[i][j].re;
            acc[i][j].im += sgn * t[i][j].im;
        }
}

}  // namespace

// H (paper gauge layout [4][2][Vh][3][3]): a block takes 64 sites of one parity, wave rho their links rho
template <class F>
__global__ __launch_bounds__(256, 2) void k_force_link(Geom g, ForceFields<F> f, double kappa, double csw,
                                                       double2* __restrict__ H, int G)
{
    __shared__ double2 stage[4][FS * 9];
    const int blk = xcd_tile(blockIdx.x, gridDim.x);
    const int parity = blk & 1, tile = grouped_tile(g, blk >> 1, G);
    const int lane = threadIdx.x & 63, rho = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int site = tile * FS + lane;
    int c[4];
    site_coords(g, site < g.Vh ? site : g.Vh - 1, parity, c[0], c[1], c[2], c[3]);
    const Site y = site_step(g, c, 0, 0, 0, 0), yr = site_step(g, c, rho, 1, rho, 0);
    c3 acc;
#pragma unroll
    for (int i = 0; i < 3; i++)
#pragma unroll
        for (int j = 0; j < 3; j++) acc[i][j] = {0.0, 0.0};
    // clover term: the two plaquettes through the link in each plane (rho, sig)
    const double wcl = kappa * csw / 8.0;
#pragma unroll 1
    for (int sig = 0; sig < 4; sig++) {
        if (sig == rho) continue;
        const int p = rho < sig ? plane_of(rho, sig) : plane_of(sig, rho);
        const double w = rho < sig ? wcl : -wcl;  // the side whose plaquette runs the link forward
        add_plaquette<1>(f, g, c, rho, sig, p, w, y, yr, acc);
        add_plaquette<-1>(f, g, c, rho, sig, p, -w, y, yr, acc);
    }
    // hop term: kappa s (A1 + A2^+), A1 = sum_s [(1 - g) X(x+rho)]_s Y(x)_s^+ = sum_k h_k(X(x+rho)) h_k(Y(x))^+ over
    // the two rows of the half-spinors, A2^+ = sum_k h_k(Y(x+rho)) h_k(X(x))^+ with 1 + g
    const double sk = (rho == 3 && g.t_bc < 0 && c[3] == g.Lt - 1) ? -kappa : kappa;
#pragma unroll 1
    for (int k = 0; k < 2; k++) {
        cx<double> a[3], b[3];
        f.half(0, yr, rho, k, -1.0, a);
        f.half(12, y, rho, k, -1.0, b);
#pragma unroll
        for (int i = 0; i < 3; i++)
#pragma unroll
            for (int j = 0; j < 3; j++) cmac_conj(acc[i][j], {sk * b[j].re, sk * b[j].im}, a[i]);
        f.half(12, yr, rho, k, 1.0, a);
        f.half(0, y, rho, k, 1.0, b);
#pragma unroll
        for (int i = 0; i < 3; i++)
#pragma unroll
            for (int j = 0; j < 3; j++) cmac_conj(acc[i][j], {sk * b[j].re, sk * b[j].im}, a[i]);
    }
    // H = the traceless Hermitian part (B - B^+) / (2i) of B = U acc
    c3 u;
    f.template link<false>(rho, y, u);
    left_mul(u, acc);
    double2* o = stage[rho] + lane * 9;
    const double tr = (acc[0][0].im + acc[1][1].im + acc[2][2].im) / 3.0;
#pragma unroll
    for (int i = 0; i < 3; i++)
#pragma unroll
        for (int j = 0; j < 3; j++)
            o[3 * i + j] = i == j ? make_double2(acc[i][i].im - tr, 0.0)
                                  : make_double2(0.5 * (acc[i][j].im + acc[j][i].im),
                                                 -0.5 * (acc[i][j].re - acc[j][i].re));
    __syncthreads();
    const int left = g.Vh - tile * FS, n = (left < FS ? left : FS) * 9;
    double2* h = H + ((long)(2 * rho + parity) * g.Vh + (long)tile * FS) * 9;
    for (int e = lane; e < n; e += 64) h[e] = stage[rho][e];
}

template <class F>
static hipError_t force_links(hipStream_t s, const Geom& g, const F& fields, const double* Gam, double kappa, double csw,
                              void* H)
{
    const ForceFields<F> f{fields, Gam};
    hipLaunchKernelGGL(k_force_link<F>, dim3(2 * ((g.Vh + FS - 1) / FS)), dim3(256), 0, s, g, f, kappa, csw, (double2*)H,
                       grouped_order(g));
    return hipGetLastError();
}

hipError_t launch_clover_force(hipStream_t s, const Geom& g, const void* U, const void* X, const void* Y,
                               double kappa, double csw, void* scratch, bool copies, void* H)
{
    const long V = 2L * g.Vh;
    double2* planes = (double2*)scratch;  // links [4][2][9][Vh], X and Y [24][V], Gam [48][V] reals
    double2* XY = copies ? planes + 36 * V : nullptr;
    double* Gam = copies ? (double*)(XY + 24 * V) : (double*)scratch;
    if (copies) {
        const hipError_t e = launch_pack_links(s, g, U, 18, planes, nullptr, F64, 18, nullptr);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(k_force_gamma, dim3((unsigned)((V + FS - 1) / FS)), dim3(384), 0, s, (int)V, (const double2*)X,
                       (const double2*)Y, Gam, XY);
    if (copies)
        return force_links(s, g, PlaneFields{link_planes(planes, 18, nullptr, g.Vh), XY}, Gam, kappa, csw, H);
    return force_links(s, g, RecordFields{(const double2*)U, (const double2*)X, (const double2*)Y, g.Vh}, Gam, kappa, csw,
                       H);
}

}  // namespace qcdw

extern "C" qcdw_status qcdw_clover_force(qcdw_ctx* ctx, const qcdw_lattice* lat, const void* U, const void* X,
                                         const void* Y, double kappa, double csw, void* H)
{
    if (!ctx) return QCDW_EINVAL;
    DeviceGuard dg(ctx->device);
    Geom g;
    CHK(check_lattice(ctx, lat, g));
    CHK(check_dev(ctx, U, "U"));
    CHK(check_dev(ctx, X, "X"));
    CHK(check_dev(ctx, Y, "Y"));
    CHK(check_dev(ctx, H, "H"));
    if (H == U || H == X || H == Y) return fail(ctx, QCDW_EINVAL, "H must not alias U, X or Y");
    if (!std::isfinite(kappa) || !std::isfinite(csw)) return fail(ctx, QCDW_EINVAL, "kappa and csw must be finite");
    CallScratch scratch(ctx->stream);
    void* work = scratch(2UL * g.Vh * FORCE_SITE_BYTES);
    const bool copies = work != nullptr;
    if (!work) work = scratch(2UL * g.Vh * FORCE_GAMMA_BYTES);
    if (!work) return fail(ctx, QCDW_ENOMEM, "out of device memory for the force's workspace");
    HIPCHK(ctx, launch_clover_force(ctx->stream, g, U, X, Y, kappa, csw, work, copies, H));
    HIPCHK(ctx, hipStreamSynchronize(ctx->stream));
    return QCDW_OK;
}
