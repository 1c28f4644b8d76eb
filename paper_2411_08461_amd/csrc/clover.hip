// Clover term kernels (FP64):
//   build  : C(x) = sum_{mu<nu} sigma_{mu nu} F_{mu nu}(x)     (Sec. III.B, Eq. "clover"), paper layout
//   apply  : out = (1 - kappa csw C) psi, paper layouts
//   invert : (1 - kappa csw C)^-1 per chirality block, by Cholesky, paper layout
//            or, for an operator, A = 1 - kappa csw C and A^-1 in the internal packings
// Packed clover per site and chirality (Sec. II.A): 6 real diagonal entries,
// then the 15 strictly-lower complex entries in row-major order; block index
// j = 3 * (spin % 2) + colour, chirality 0 = spins {0,1}, 1 = spins {2,3}.
#include "internal.h"

namespace qcdw {

using cd = cx<double>;

struct M3 {
    cd m[9];
};

__device__ __forceinline__ M3 mul(const M3& a, const M3& b)
{
    M3 r;
#pragma unroll
    for (int i = 0; i < 3; i++)
#pragma unroll
        for (int j = 0; j < 3; j++) {
            cd s = a.m[3 * i] * b.m[j];
            cmac(s, a.m[3 * i + 1], b.m[3 + j]);
            cmac(s, a.m[3 * i + 2], b.m[6 + j]);
            r.m[3 * i + j] = s;
        }
    return r;
}

// a * b^+
__device__ __forceinline__ M3 mul_nd(const M3& a, const M3& b)
{
    M3 r;
#pragma unroll
    for (int i = 0; i < 3; i++)
#pragma unroll
        for (int j = 0; j < 3; j++) {
            cd s = cmul_conj(b.m[3 * j], a.m[3 * i]);
            cmac_conj(s, b.m[3 * j + 1], a.m[3 * i + 1]);
            cmac_conj(s, b.m[3 * j + 2], a.m[3 * i + 2]);
            r.m[3 * i + j] = s;
        }
    return r;
}

// a^+ * b
__device__ __forceinline__ M3 mul_dn(const M3& a, const M3& b)
{
    M3 r;
#pragma unroll
    for (int i = 0; i < 3; i++)
#pragma unroll
        for (int j = 0; j < 3; j++) {
            cd s = cmul_conj(a.m[i], b.m[j]);
            cmac_conj(s, a.m[3 + i], b.m[3 + j]);
            cmac_conj(s, a.m[6 + i], b.m[6 + j]);
            r.m[3 * i + j] = s;
        }
    return r;
}

// f += the anti-Hermitian part of p r^+ (nd) or p^+ r (dn): imaginary diagonal / 2 and m - m^+ above it
__device__ __forceinline__ void add_antiherm_nd(double (&f)[9], const M3& p, const M3& r)
{
#pragma unroll
    for (int i = 0; i < 3; i++)
#pragma unroll
        for (int k = 0; k < 3; k++) {  // Im p_ik conj(r_ik)
            f[i] += p.m[3 * i + k].im * r.m[3 * i + k].re;
            f[i] -= p.m[3 * i + k].re * r.m[3 * i + k].im;
        }
#pragma unroll
    for (int e = 0; e < 3; e++) {
        const int i = e == 2 ? 1 : 0, j = e == 0 ? 1 : 2;
        cd v = {f[3 + 2 * e], f[4 + 2 * e]};
#pragma unroll
        for (int k = 0; k < 3; k++) {  // p_ik conj(r_jk) - r_ik conj(p_jk)
            cmac_conj(v, r.m[3 * j + k], p.m[3 * i + k]);
            cmac_conj(v, p.m[3 * j + k], {-r.m[3 * i + k].re, -r.m[3 * i + k].im});
        }
        f[3 + 2 * e] = v.re;
        f[4 + 2 * e] = v.im;
    }
}

__device__ __forceinline__ void add_antiherm_dn(double (&f)[9], const M3& p, const M3& r)
{
#pragma unroll
    for (int i = 0; i < 3; i++)
#pragma unroll
        for (int k = 0; k < 3; k++) {  // Im conj(p_ki) r_ki
            f[i] += p.m[3 * k + i].re * r.m[3 * k + i].im;
            f[i] -= p.m[3 * k + i].im * r.m[3 * k + i].re;
        }
#pragma unroll
    for (int e = 0; e < 3; e++) {
        const int i = e == 2 ? 1 : 0, j = e == 0 ? 1 : 2;
        cd v = {f[3 + 2 * e], f[4 + 2 * e]};
#pragma unroll
        for (int k = 0; k < 3; k++) {  // conj(p_ki) r_kj - conj(r_ki) p_kj
            cmac_conj(v, p.m[3 * k + i], r.m[3 * k + j]);
            cmac_conj(v, r.m[3 * k + i], {-p.m[3 * k + j].re, -p.m[3 * k + j].im});
        }
        f[3 + 2 * e] = v.re;
        f[4 + 2 * e] = v.im;
    }
}

__device__ __forceinline__ M3 ld_link(const LinkPlanes& U, int mu, Site s)
{
    M3 r;
    const double2* p = U.top + (long)(mu * 2 + s.parity) * U.top_rec * U.Vh + s.cb;
    const double2* q = U.low + (long)(mu * 2 + s.parity) * U.low_rec * U.Vh + s.cb;
#pragma unroll
    for (int e = 0; e < 6; e++) {
        const double2 v = p[e * U.Vh];
        r.m[e] = {v.x, v.y};
    }
#pragma unroll
    for (int e = 0; e < 3; e++) {
        const double2 v = q[e * U.Vh];
        r.m[6 + e] = {v.x, v.y};
    }
    return r;
}

// the paper's links as they are, for a call that finds no memory for a plane-major copy
struct LinkRecords {
    const double2* U;
    long Vh;
};
__device__ __forceinline__ M3 ld_link(const LinkRecords& U, int mu, Site s)
{
    M3 r;
    const double2* p = U.U + ((long)(mu * 2 + s.parity) * U.Vh + s.cb) * 9;
#pragma unroll
    for (int e = 0; e < 9; e++) r.m[e] = {p[e].x, p[e].y};
    return r;
}

// F_{mu nu}(x): traceless part of (Q - Q^+)/8, Q = sum of the four
// counter-clockwise plaquettes in the (mu, nu) plane that touch x, times w.  F is
// anti-Hermitian: out gets the imaginary diagonal and the three entries above it.
template <class Links>
__device__ __forceinline__ void field_strength(const Links& U, const Geom& g, const int (&c)[4], int mu, int nu,
                                               double w, double (&out)[8])
{
    const Site x = site_step(g, c, mu, 0, nu, 0);
    double f[9];  // Q - Q^+: imaginary diagonal / 2, then the entries above it
#pragma unroll
    for (int i = 0; i < 9; i++) f[i] = 0.0;
    // each leaf as a product of two half-leaves, the first two links in one order and the last two in the other:
    // two matrices are live, and only the anti-Hermitian part of their product is formed
    {  // upper-right: U_mu(x) U_nu(x+mu) [U_nu(x) U_mu(x+nu)]^+
        const M3 p = mul(ld_link(U, mu, x), ld_link(U, nu, site_step(g, c, mu, 1, nu, 0)));
        const M3 r = mul(ld_link(U, nu, x), ld_link(U, mu, site_step(g, c, mu, 0, nu, 1)));
        add_antiherm_nd(f, p, r);
    }
    {  // upper-left: U_nu(x) U_mu(x-mu+nu)^+ [U_mu(x-mu)^+ U_nu(x-mu)]^+
        const Site xm = site_step(g, c, mu, -1, nu, 0);
        const M3 p = mul_nd(ld_link(U, nu, x), ld_link(U, mu, site_step(g, c, mu, -1, nu, 1)));
        const M3 r = mul_dn(ld_link(U, mu, xm), ld_link(U, nu, xm));
        add_antiherm_nd(f, p, r);
    }
    {  // lower-left: [U_nu(x-mu-nu) U_mu(x-mu)]^+ U_mu(x-mu-nu) U_nu(x-nu)
        const Site xmn = site_step(g, c, mu, -1, nu, -1);
        const M3 p = mul(ld_link(U, nu, xmn), ld_link(U, mu, site_step(g, c, mu, -1, nu, 0)));
        const M3 r = mul(ld_link(U, mu, xmn), ld_link(U, nu, site_step(g, c, mu, 0, nu, -1)));
        add_antiherm_dn(f, p, r);
    }
    {  // lower-right: U_nu(x-nu)^+ U_mu(x-nu) [U_mu(x) U_nu(x+mu-nu)^+]^+
        const Site xn = site_step(g, c, mu, 0, nu, -1);
        const M3 p = mul_dn(ld_link(U, nu, xn), ld_link(U, mu, xn));
        const M3 r = mul_nd(ld_link(U, mu, x), ld_link(U, nu, site_step(g, c, mu, 1, nu, -1)));
        add_antiherm_nd(f, p, r);
    }
    const double tr = (1.0 / 3.0) * (f[0] + f[1] + f[2]);
#pragma unroll
    for (int i = 0; i < 2; i++) out[i] = w * (0.25 * (f[i] - tr));
#pragma unroll
    for (int i = 2; i < 8; i++) out[i] = w * (0.125 * f[i + 1]);
}

__device__ __forceinline__ void unpack6(const double* p, cd (&B)[6][6])
{
#pragma unroll
    for (int j = 0; j < 6; j++) B[j][j] = {p[j], 0.0};
    int slot = 0;
#pragma unroll
    for (int j = 1; j < 6; j++)
#pragma unroll
        for (int k = 0; k < j; k++) {
            B[j][k] = {p[6 + 2 * slot], p[7 + 2 * slot]};
            B[k][j] = conj(B[j][k]);
            slot++;
        }
}

// A = 1 - kc C = L L^+ (Cholesky), A^-1 = L^-+ L^-1 of one packed block p into o (o may be p); false if A is not
// positive definite
__device__ __forceinline__ bool invert_block(const double* p, double* o, double kc)
{
    cd A[6][6];
    unpack6(p, A);
#pragma unroll
    for (int j = 0; j < 6; j++)
#pragma unroll
        for (int k = 0; k < 6; k++) A[j][k] = (j == k ? 1.0 : 0.0) * cd{1.0, 0.0} - kc * A[j][k];
    cd Lm[6][6];
    double dinv[6];
    bool ok = true;
#pragma unroll
    for (int j = 0; j < 6; j++) {
        double d = A[j][j].re;
#pragma unroll
        for (int k = 0; k < j; k++) d -= norm2(Lm[j][k]);
        if (!(d > 0.0)) ok = false;
        const double lj = sqrt(d > 0.0 ? d : 1.0);
        dinv[j] = 1.0 / lj;
        Lm[j][j] = {lj, 0.0};
#pragma unroll
        for (int i = j + 1; i < 6; i++) {
            cd s = A[i][j];
#pragma unroll
            for (int k = 0; k < j; k++) s = s - Lm[i][k] * conj(Lm[j][k]);
            Lm[i][j] = dinv[j] * s;
        }
    }
    // W = L^-1 (lower triangular) by forward substitution
    cd W[6][6];
#pragma unroll
    for (int j = 0; j < 6; j++) {
#pragma unroll
        for (int i = 0; i < 6; i++) W[i][j] = {0.0, 0.0};
        W[j][j] = {dinv[j], 0.0};
#pragma unroll
        for (int i = j + 1; i < 6; i++) {
            cd s = {0.0, 0.0};
#pragma unroll
            for (int k = j; k < i; k++) s = s + Lm[i][k] * W[k][j];
            W[i][j] = (-dinv[i]) * s;
        }
    }
    // A^-1 = W^+ W ; entry (j,k) = sum_{m >= max(j,k)} conj(W[m][j]) W[m][k]
#pragma unroll
    for (int j = 0; j < 6; j++) {
        double s = 0.0;
#pragma unroll
        for (int m = j; m < 6; m++) s += norm2(W[m][j]);
        o[j] = s;
    }
    int slot = 0;
#pragma unroll
    for (int j = 1; j < 6; j++)
#pragma unroll
        for (int k = 0; k < j; k++) {
            cd s = {0.0, 0.0};
#pragma unroll
            for (int m = j; m < 6; m++) s = s + cmul_conj(W[m][j], W[m][k]);
            o[6 + 2 * slot] = s.re;
            o[7 + 2 * slot] = s.im;
            slot++;
        }
    return ok;
}

// In the DeGrand-Rossi basis sigma_{mu nu} = [g_mu, g_nu]/2 is block-diagonal
// in chirality; its 2x2 spin blocks give, with F_{mu nu} (mu, nu = 0..3):
//   upper (spins 0,1): B00 = -iF01 + iF23   B11 = iF01 - iF23
//                      B01 = -F02 + iF03 - iF12 - F13   B10 = F02 + iF03 - iF12 + F13
//   lower (spins 2,3): B00 = -iF01 - iF23   B11 = iF01 + iF23
//                      B01 = -F02 - iF03 - iF12 + F13   B10 = F02 - iF03 - iF12 - F13
// and the 6x6 chirality block is [[B00, B01], [B10, B11]] in colour-inner order.
// wt weights the planes (i, t) and ws the spatial planes (the anisotropic action of Sec. III.B:
// wt = c_SW^t, ws = c_SW^r / xi_0; 1 and 1 for the isotropic C).
//
//
// A block of two waves takes 64 sites of one parity: each wave forms three planes, a lane per site, so that a
// wave's links are whole runs of the plane-major copy (LinkPlanes) and a thread holds a few 3x3 matrices.  F goes
// to LDS (eight reals per plane: anti-Hermitian, traceless), then each thread forms one chirality block from it,
// and the packed blocks leave through LDS in contiguous runs.  A thread per site with all six planes spilled
// 1.8 kB per lane and read the paper's 144-byte records, a cache line per lane and load.
// With 210 VGPRs two waves fit a SIMD; three (168 VGPRs) spill and are slower (252 against 179 us a call at
// 16^3x32).  What bounds it is the links that miss the XCD's 4 MB L2 (each is read by 24 leaves): the two parities
// of a tile next to each other took 179 to 137 us there, and on larger lattices the tiles of a group are swept along t
// (grouped_order: 24^3x64 827 to 768 us).
// Measured per call, with the plane-major copy: 16^3x32 130 us, 24^3x64 768 us (385 us and 2.92 ms with a thread per
// site).
// OP: the operator's form; instead of C it writes, per parity and in the internal packing, A and A^-1 in FP64 and
// A^-1 in the inner precision PL (lo nullptr: none).  C, the inverse and five repackings of whole fields as
// kernels of their own moved 7.5 kB per site and took 570 us at 16^3x32 with the build; this form writes 1.3 kB and
// takes 114 us.
constexpr int CB_SITES = 64, CB_ROW = 37;  // CB_ROW: a packed block in LDS, padded off the bank period

// place in the internal packing
//   [d0 d1 d2 | L10 L20 L21 | L30 L31 L32 L40 L41 L42 L50 L51 L52 | d3 d4 d5 | L43 L53 L54]
// of entry m of the paper packing [d0..d5 | L10 L20 L21 L30 L31 L32 L40 L41 L42 L43 L50 .. L54]
__device__ __forceinline__ constexpr int clover_dst_pos(int m)
{
    if (m < 3) return m;
    if (m < 6) return 27 + (m - 3);
    const int s = (m - 6) >> 1, ri = (m - 6) & 1;  // lower slot: L3x 3..5, L4x 6..8, L43 9, L5x 10..12, L53 13, L54 14
    if (s < 9) return 3 + 2 * s + ri;
    if (s == 9) return 30 + ri;
    if (s < 13) return 21 + 2 * (s - 10) + ri;
    return 32 + 2 * (s - 13) + ri;
}

struct CloverOut {
    double* C;                   // paper layout (not OP)
    double *A[2], *inv[2];       // internal packing per parity (OP)
    void* lo[2];                 // A^-1 in the inner precision, or nullptr
    double kc;                   // kappa csw
    int* notpd;                  // raised by the blocks whose A is not positive definite
};

// n reals in rows of 36 in LDS to consecutive places, f(index, value)
template <class F>
__device__ __forceinline__ void copy_rows(const double* stage, int n, F&& f)
{
    int row = threadIdx.x / 36, m = threadIdx.x % 36;
    for (int e = threadIdx.x; e < n; e += 128) {
        f(e, stage[row * CB_ROW + m]);
        m += 128 - 3 * 36;  // 128 entries on: three rows and 20
        row += 3;
        if (m >= 36) {
            m -= 36;
            row++;
        }
    }
}

template <class Links, class PL, bool OP>
__global__ __launch_bounds__(128) void k_clover_build(Links U, Geom g, double wt, double ws, int G,
                                                      CloverOut out)
{
    __shared__ double sh[6 * 8 * CB_SITES];  // F, then the packed blocks of half of the sites at a time
    static_assert(CB_SITES * CB_ROW <= 6 * 8 * CB_SITES, "half of the blocks fit where F was");
    const int blk = xcd_tile(blockIdx.x, gridDim.x);
    const int parity = blk & 1, tile = grouped_tile(g, blk >> 1, G);
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    {
        const int site = tile * CB_SITES + lane;
        int c[4];
        site_coords(g, site < g.Vh ? site : g.Vh - 1, parity, c[0], c[1], c[2], c[3]);
#pragma unroll 1
        for (int plane = w; plane < 6; plane += 2) {
            // planes (0,1) (0,2) (0,3) (1,2) (1,3) (2,3), one code for all: six inlined copies (100 kB) miss the
            // instruction cache
            const int mu = plane < 3 ? 0 : (plane < 5 ? 1 : 2), nu = plane < 3 ? plane + 1 : (plane < 5 ? plane - 1 : 3);
            double o[8];
            field_strength(U, g, c, mu, nu, nu == 3 ? wt : ws, o);
#pragma unroll
            for (int e = 0; e < 8; e++) sh[(plane * 8 + e) * CB_SITES + lane] = o[e];
        }
    }
    __syncthreads();
    double C[36];  // the packed block of (site lane, chirality w)
    {
        const double s = w == 0 ? 1.0 : -1.0;  // sign of the time-plane terms
        // entry (a, b) of F in plane p
        const auto F = [&](int p, int a, int b) -> cd {
            const double* r = sh + p * 8 * CB_SITES + lane;
            if (a == b) return {0.0, a < 2 ? r[a * CB_SITES] : -(r[0] + r[CB_SITES])};
            const int k = a + b - 1;  // (0,1) 0, (0,2) 1, (1,2) 2
            const double re = r[(2 + 2 * k) * CB_SITES], im = r[(3 + 2 * k) * CB_SITES];
            return a < b ? cd{re, im} : cd{-re, im};
        };
        const cd I = {0.0, 1.0};
        // the diagonal of B00 and B11, and their strictly lower entries: rows 0..2 and 3..5
#pragma unroll
        for (int a = 0; a < 3; a++)
#pragma unroll
            for (int b = 0; b <= a; b++) {
                const cd f01 = F(0, a, b), f23 = F(5, a, b);
                const cd u = I * (s * f23 - f01), v = I * (f01 - s * f23);
                if (a == b) {
                    C[a] = u.re;
                    C[3 + a] = v.re;
                } else {
                    const int s0 = a * (a - 1) / 2 + b, s1 = (3 + a) * (2 + a) / 2 + 3 + b;
                    C[6 + 2 * s0] = u.re;
                    C[7 + 2 * s0] = u.im;
                    C[6 + 2 * s1] = v.re;
                    C[7 + 2 * s1] = v.im;
                }
            }
        // B10: rows 3..5, columns 0..2
#pragma unroll
        for (int a = 0; a < 3; a++)
#pragma unroll
            for (int b = 0; b < 3; b++) {
                const cd f02 = F(1, a, b), f03 = F(2, a, b), f12 = F(3, a, b), f13 = F(4, a, b);
                const cd v = (f02 + s * f13) + I * (s * f03 - f12);
                const int slot = (3 + a) * (2 + a) / 2 + b;
                C[6 + 2 * slot] = v.re;
                C[7 + 2 * slot] = v.im;
            }
    }
    const int left = g.Vh - tile * CB_SITES;
    const long first = (long)tile * CB_SITES * 72;
    // every thread's 36 values (place(m) of its row) to consecutive reals, f(index, value)
    const auto emit = [&](const double(&v)[36], auto place, auto f) {
        constexpr int HALF = CB_SITES / 2;
#pragma unroll
        for (int h = 0; h < 2; h++) {
            __syncthreads();
            if (lane / HALF == h) {
                double* mine = sh + (2 * (lane - h * HALF) + w) * CB_ROW;
#pragma unroll
                for (int m = 0; m < 36; m++) mine[place(m)] = v[m];
            }
            __syncthreads();
            const int rest = left - h * HALF;
            copy_rows(sh, (rest < HALF ? rest : HALF) * 72, [&](int e, double x) { f(first + h * HALF * 72 + e, x); });
        }
    };
    if constexpr (!OP) {
        double* o = out.C + (long)parity * g.Vh * 72;
        emit(C, [](int m) { return m; }, [&](long e, double x) { o[e] = x; });
    } else {
        const double kc = out.kc;
        double r[36];
#pragma unroll
        for (int m = 0; m < 36; m++) r[m] = (m < 6 ? 1.0 : 0.0) - kc * C[m];
        double* a = parity ? out.A[1] : out.A[0];
        emit(r, [](int m) { return clover_dst_pos(m); }, [&](long e, double x) { a[e] = x; });
        if (!invert_block(C, r, kc) && lane < left) atomicAdd(out.notpd, 1);
        double* o = parity ? out.inv[1] : out.inv[0];
        void* lo = parity ? out.lo[1] : out.lo[0];
        using T = typename PL::real;
        emit(r, [](int m) { return clover_dst_pos(m); }, [&](long e, double x) {
            o[e] = x;
            if (lo) PL::str(lo, e, (T)x);
        });
    }
}

__global__ void k_clover_apply(const double* __restrict__ clover, const double2* __restrict__ psi,
                               double2* __restrict__ out, long V, double kc)
{
    const long blk = (long)blockIdx.x * blockDim.x + threadIdx.x;  // site*2 + chirality
    if (blk >= 2 * V) return;
    cd B[6][6];
    unpack6(clover + blk * 36, B);
    cd v[6];
#pragma unroll
    for (int j = 0; j < 6; j++) v[j] = {psi[blk * 6 + j].x, psi[blk * 6 + j].y};
#pragma unroll
    for (int j = 0; j < 6; j++) {
        cd s = {0.0, 0.0};
#pragma unroll
        for (int k = 0; k < 6; k++) s = s + B[j][k] * v[k];
        out[blk * 6 + j] = make_double2(v[j].re - kc * s.re, v[j].im - kc * s.im);
    }
}

__global__ void k_clover_invert(const double* __restrict__ clover, double* __restrict__ inv, long V, double kc,
                                int* notpd)
{
    const long blk = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (blk >= 2 * V) return;
    if (!invert_block(clover + blk * 36, inv + blk * 36, kc)) atomicAdd(notpd, 1);
}

static inline dim3 grid_for(long n) { return dim3((unsigned)((n + 255) / 256)); }

template <class Links>
static hipError_t clover_build(hipStream_t s, const Geom& g, const Links& U, void* clover)
{
    if (g.Vh == 0) return hipSuccess;
    const int tiles = (g.Vh + CB_SITES - 1) / CB_SITES;
    CloverOut o{};
    o.C = (double*)clover;
    hipLaunchKernelGGL((k_clover_build<Links, P64, false>), dim3(2 * tiles), dim3(128), 0, s, U, g, 1.0, 1.0,
                       grouped_order(g), o);
    return hipGetLastError();
}

hipError_t launch_clover_build(hipStream_t s, const Geom& g, const LinkPlanes& U, void* clover)
{
    return clover_build(s, g, U, clover);
}

hipError_t launch_clover_build_records(hipStream_t s, const Geom& g, const void* U, void* clover)
{
    return clover_build(s, g, LinkRecords{(const double2*)U, g.Vh}, clover);
}

hipError_t launch_clover_op(hipStream_t s, const Geom& g, const LinkPlanes& U, double wt, double ws, double kappa,
                            double csw, void* const A[2], void* const inv[2], int prec_lo, void* const lo[2],
                            int* notpd_count)
{
    if (g.Vh == 0) return hipSuccess;
    const int tiles = (g.Vh + CB_SITES - 1) / CB_SITES;
    CloverOut o{};
    for (int p = 0; p < 2; p++) {
        o.A[p] = (double*)A[p];
        o.inv[p] = (double*)inv[p];
        o.lo[p] = prec_lo == F64 ? nullptr : lo[p];
    }
    o.kc = kappa * csw;
    o.notpd = notpd_count;
#define QCDW_CLOVER_OP(P)                                                                                              \
    hipLaunchKernelGGL((k_clover_build<LinkPlanes, P, true>), dim3(2 * tiles), dim3(128), 0, s, U, g, wt, ws,          \
                       grouped_order(g), o)
    switch (prec_lo) {
    case F64: QCDW_CLOVER_OP(P64); break;
    case F32: QCDW_CLOVER_OP(P32); break;
    case BF16: QCDW_CLOVER_OP(PBF16); break;
    case F16: QCDW_CLOVER_OP(PF16); break;
    default: return hipErrorInvalidValue;
    }
#undef QCDW_CLOVER_OP
    return hipGetLastError();
}

hipError_t launch_clover_apply(hipStream_t s, const Geom& g, const void* clover, const void* psi, void* out,
                               double kappa, double csw)
{
    const long V = 2L * g.Vh;
    if (V == 0) return hipSuccess;
    hipLaunchKernelGGL(k_clover_apply, grid_for(2 * V), dim3(256), 0, s, (const double*)clover, (const double2*)psi,
                       (double2*)out, V, kappa * csw);
    return hipGetLastError();
}

hipError_t launch_clover_invert(hipStream_t s, const Geom& g, const void* clover, double kappa, double csw, void* inv,
                                int* notpd_count)
{
    const long V = 2L * g.Vh;
    if (V == 0) return hipSuccess;
    hipLaunchKernelGGL(k_clover_invert, grid_for(2 * V), dim3(256), 0, s, (const double*)clover, (double*)inv, V,
                       kappa * csw, notpd_count);
    return hipGetLastError();
}

}  // namespace qcdw
