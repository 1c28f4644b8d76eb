// Kernels of the learned gauge-covariant preconditioner (the published idea of
// gauge-equivariant convolutions: Favoni et al. 2022, Lehner and Wettig 2023;
// the paper's own accelerator for clover solves is multigrid, Sec. II.E).
//
// A layer maps CIN channels phi_c (colour 3-vector fields on the full lattice)
// to COUT channels:  out_{c'}(x) = sum_a sum_c W_a[c', c] (T_a phi_c)(x),
// a in {0, +-mu}: T_0 = 1, (T_{+mu} phi)(x) = U_mu(x) phi(x+mu),
// (T_{-mu} phi)(x) = U_mu(x-mu)^+ phi(x-mu).  Hop index a = 1 + 2 mu + back.
// Activation layout [parity][channel][Vh][3] complex: with 4 channels it is two
// internal spinor fields (even, odd), so spins are the input/output channels.
// Links: the operator's reconstruct-12 internal layout, FP32.  Arithmetic FP32.
#include <algorithm>

#include "internal.h"

namespace qcdw {

struct NetArgs {
    const void* in;
    void* out;
    const void* gauge;  // reconstruct-12 links in FP32, in the layout of the FP64 links (link_base, link_stride)
    const float2* W;    // [9][COUT][CIN]
    Geom g;
};

// link (mu, p, site) of an FP32 reconstruct-12 internal gauge field (two rows stored)
__device__ __forceinline__ void su3_row3(const void* gauge, int mu, int p, int site, long Vh, cx<float> (&u)[9])
{
    constexpr bool soa = link_soa_for(P64::cbytes);  // an element-wise FP32 copy of the operator's FP64 links
    const long off = link_base(mu, p, site, Vh, 6, soa), st = link_stride(Vh, soa);
#pragma unroll
    for (int e = 0; e < 6; e++) u[e] = P32::ld(gauge, off + e * st);
    u[6] = conj(u[1] * u[5] - u[2] * u[4]);
    u[7] = conj(u[2] * u[3] - u[0] * u[5]);
    u[8] = conj(u[0] * u[4] - u[1] * u[3]);
}

// neighbour (parity 1 - p) of site i of parity p one step along mu (dir 0 forward, 1 backward)
__device__ __forceinline__ int nbr_index(const Geom& g, int i, int x, int y, int z, int t, int mu, int dir)
{
    const int xh = i % g.Lxh;
    switch (mu) {
    case 0: {
        const int row = i - xh;
        const int xn = dir == 0 ? ((x + 1 == g.Lx) ? 0 : x + 1) : ((x == 0) ? g.Lx - 1 : x - 1);
        return row + (xn >> 1);
    }
    case 1: {
        const int S = g.Lxh;
        return dir == 0 ? ((y + 1 == g.Ly) ? i - (g.Ly - 1) * S : i + S) : ((y == 0) ? i + (g.Ly - 1) * S : i - S);
    }
    case 2: {
        const int S = g.Lxh * g.Ly;
        return dir == 0 ? ((z + 1 == g.Lz) ? i - (g.Lz - 1) * S : i + S) : ((z == 0) ? i + (g.Lz - 1) * S : i - S);
    }
    default: {
        const int S = g.Lxh * g.Ly * g.Lz;
        return dir == 0 ? ((t + 1 == g.Lt) ? i - (g.Lt - 1) * S : i + S) : ((t == 0) ? i + (g.Lt - 1) * S : i - S);
    }
    }
}

// Y[c] = (T_a phi_c)(x) for the site (p, i)
template <class PI, int CIN>
__device__ __forceinline__ void transport(const void* in, const void* gauge, const Geom& g, int p, int i, int x,
                                          int y, int z, int t, int a, cx<float> (&Y)[CIN][3])
{
    const long Vh = g.Vh;
    if (a == 0) {
#pragma unroll
        for (int c = 0; c < CIN; c++)
#pragma unroll
            for (int k = 0; k < 3; k++) {
                const auto v = PI::ld(in, sp_idx((long)p * CIN + c, i, k, Vh));
                Y[c][k] = {(float)v.re, (float)v.im};
            }
        return;
    }
    const int mu = (a - 1) >> 1, back = (a - 1) & 1;
    const int j = nbr_index(g, i, x, y, z, t, mu, back);
    cx<float> u[9];
    su3_row3(gauge, mu, back == 0 ? p : 1 - p, back == 0 ? i : j, Vh, u);
#pragma unroll
    for (int c = 0; c < CIN; c++) {
        cx<float> v[3];
#pragma unroll
        for (int k = 0; k < 3; k++) {
            const auto w = PI::ld(in, sp_idx((long)(1 - p) * CIN + c, j, k, Vh));
            v[k] = {(float)w.re, (float)w.im};
        }
#pragma unroll
        for (int r = 0; r < 3; r++) {
            cx<float> s = {0.f, 0.f};
#pragma unroll
            for (int k = 0; k < 3; k++) s = back == 0 ? s + u[3 * r + k] * v[k] : s + cmul_conj(u[3 * k + r], v[k]);
            Y[c][r] = s;
        }
    }
}

typedef float mfma_f4 __attribute__((ext_vector_type(4)));
typedef short mfma_s4 __attribute__((ext_vector_type(4)));

// two floats rounded to BF16 (nearest even) and packed low, high
__device__ __forceinline__ uint32_t pk_bf16(float lo, float hi)
{
    return __builtin_bit_cast(uint32_t, f2bf2(lo, hi));
}
__device__ __forceinline__ mfma_s4 s4_of(uint32_t lo, uint32_t hi) { return __builtin_bit_cast(mfma_s4, make_uint2(lo, hi)); }

// The layers with their channel mixing on the matrix cores in BF16 (v_mfma_f32_16x16x16_bf16, FP32
// accumulation): the application path of the preconditioner.  For each colour k the mixing of hop a is the
// real product  D[m][n] = sum_kk A[m][kk] B[kk][n]  with the weights as A (rows m = 2 d + re/im of output
// channel d; K: kk = 2 c + re/im of input channel c; the real form [[Re W, -Im W], [Im W, Re W]]) and the
// sites of a wave as the 16 columns n.  The instruction takes A[m][kk] from lane m + 16 (kk / 4) and B[kk][n]
// from lane n + 16 (kk / 4), elements kk % 4, 16 kk per step, and leaves D[m][n] in lane n + 16 (m / 4),
// element m % 4: lane L = n + 16 g supplies input channels 2 g, 2 g + 1 (+ 8 per step) of site n and
// receives output channels 2 g, 2 g + 1 (+ 8 per row tile) of the same site, as whole complex numbers.
// Two orders of the same sum, chosen by the cheaper transport: CIN <= COUT transports the CIN inputs first
// (B = T_a phi, one accumulator over all hops); CIN > COUT mixes the neighbour's raw inputs first
// (B = phi(x + a), the 16-bit inputs taken as they are stored) and transports the COUT mixed channels.

// A operand of hop a, row tile t, K step s for this lane
template <int CIN, int COUT>
__device__ __forceinline__ mfma_s4 net_wop(const float2* __restrict__ W, int a, int t, int s, int lane)
{
    const int m = 16 * t + (lane & 15), d = m >> 1, rho = m & 1, grp = lane >> 4;
    uint32_t v[2];
#pragma unroll
    for (int h = 0; h < 2; h++) {
        const int c = 8 * s + 2 * grp + h;
        float x = 0.f, y = 0.f;
        if (d < COUT && c < CIN) {
            const float2 w = W[((long)a * COUT + d) * CIN + c];
            x = rho ? w.y : w.x;   // row re: (Re W, -Im W); row im: (Im W, Re W)
            y = rho ? w.x : -w.y;
        }
        v[h] = pk_bf16(x, y);
    }
    return s4_of(v[0], v[1]);
}

// B operand dword of input channel c (colour k) of site (p, i): a 16-bit complex as stored, or FP32 rounded
template <class PI>
__device__ __forceinline__ uint32_t net_in_bits(const void* in, long idx)
{
    if constexpr (PI::cbytes == 4) {
        return reinterpret_cast<const uint32_t*>(in)[idx];
    } else {
        const auto v = PI::ld(in, idx);
        return pk_bf16((float)v.re, (float)v.im);
    }
}

// W v with W = U (forward hop) or U^+ (backward hop)
__device__ __forceinline__ void net_link_mul(const cx<float> (&u)[9], int back, const cx<float> (&v)[3],
                                             cx<float> (&y)[3])
{
#pragma unroll
    for (int r = 0; r < 3; r++) {
        cx<float> sacc = {0.f, 0.f};
#pragma unroll
        for (int k = 0; k < 3; k++) sacc = back == 0 ? sacc + u[3 * r + k] * v[k] : sacc + cmul_conj(u[3 * k + r], v[k]);
        y[r] = sacc;
    }
}

template <class PI, class PO, int CIN, int COUT>
__global__ __launch_bounds__(256) void k_net_layer_mfma(NetArgs n)
{
    constexpr int NT = (2 * COUT + 15) / 16;  // row tiles of the output channels
    constexpr int NS = (2 * CIN + 15) / 16;   // K steps over the input channels
    constexpr bool TFIRST = CIN <= COUT;
    const Geom g = n.g;
    const long Vh = g.Vh;
    const int lane = threadIdx.x & 63, grp = lane >> 4;
    // the weight operands of every (hop, row tile, K step) for the 64 lane positions, built once per block
    __shared__ uint2 wop[9 * NT * NS][64];
    for (int e = threadIdx.x; e < 9 * NT * NS * 64; e += 256) {
        const int l = e & 63, q = e >> 6, s2 = q % NS, tl = (q / NS) % NT, a = q / (NS * NT);
        wop[q][l] = __builtin_bit_cast(uint2, net_wop<CIN, COUT>(n.W, a, tl, s2, l));
    }
    __syncthreads();
    const long wave = ((long)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
    const long gsite = wave * 16 + (lane & 15);
    const bool valid = gsite < 2 * Vh;  // other lanes compute on site 0 and store nothing
    const int p = valid ? (int)(gsite / Vh) : 0, i = valid ? (int)(gsite % Vh) : 0;
    int x, y, z, t;
    site_coords(g, i, p, x, y, z, t);
    using TO = typename PO::real;
    if constexpr (TFIRST) {
        mfma_f4 acc[3][NT];
#pragma unroll
        for (int k = 0; k < 3; k++)
#pragma unroll
            for (int tl = 0; tl < NT; tl++) acc[k][tl] = mfma_f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int a = 0; a < 9; a++) {
            const int mu = (a - 1) >> 1, back = (a - 1) & 1;
            const int j = a == 0 ? i : nbr_index(g, i, x, y, z, t, mu, back);
            const int pj = a == 0 ? p : 1 - p;
            cx<float> u[9];
            const bool link = a > 0 && 2 * grp < CIN;
            if (link) su3_row3(n.gauge, mu, back == 0 ? p : 1 - p, back == 0 ? i : j, Vh, u);
            mfma_s4 B[NS][3];
#pragma unroll
            for (int s2 = 0; s2 < NS; s2++) {
                const int c0 = 8 * s2 + 2 * grp;
                uint32_t bw[2][3];
#pragma unroll
                for (int h = 0; h < 2; h++) {
                    const int c = c0 + h;
                    cx<float> v[3], yv[3] = {{0.f, 0.f}, {0.f, 0.f}, {0.f, 0.f}};
                    if (c < CIN) {  // (u is loaded only by lanes with input channels)
#pragma unroll
                        for (int k = 0; k < 3; k++) {
                            const auto w = PI::ld(n.in, sp_idx((long)pj * CIN + c, j, k, Vh));
                            v[k] = {(float)w.re, (float)w.im};
                        }
                        if (a > 0)
                            net_link_mul(u, back, v, yv);
                        else
#pragma unroll
                            for (int k = 0; k < 3; k++) yv[k] = v[k];
                    }
#pragma unroll
                    for (int k = 0; k < 3; k++) bw[h][k] = pk_bf16(yv[k].re, yv[k].im);
                }
#pragma unroll
                for (int k = 0; k < 3; k++) B[s2][k] = s4_of(bw[0][k], bw[1][k]);
            }
#pragma unroll
            for (int tl = 0; tl < NT; tl++)
#pragma unroll
                for (int s2 = 0; s2 < NS; s2++) {
                    const mfma_s4 A = __builtin_bit_cast(mfma_s4, wop[(a * NT + tl) * NS + s2][lane]);
#pragma unroll
                    for (int k = 0; k < 3; k++)
                        acc[k][tl] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(A, B[s2][k], acc[k][tl], 0, 0, 0);
                }
        }
#pragma unroll
        for (int tl = 0; tl < NT; tl++)
#pragma unroll
            for (int h = 0; h < 2; h++) {
                const int d = 8 * tl + 2 * grp + h;
                if (valid && d < COUT) {
#pragma unroll
                    for (int k = 0; k < 3; k++)
                        PO::st(n.out, sp_idx((long)p * COUT + d, i, k, Vh),
                               cx<TO>{(TO)acc[k][tl][2 * h], (TO)acc[k][tl][2 * h + 1]});
                }
            }
    } else {
        static_assert(NT == 1, "the mix-first order keeps one row tile");
        cx<float> o[2][3];
#pragma unroll
        for (int h = 0; h < 2; h++)
#pragma unroll
            for (int k = 0; k < 3; k++) o[h][k] = {0.f, 0.f};
#pragma unroll
        for (int a = 0; a < 9; a++) {
            const int mu = (a - 1) >> 1, back = (a - 1) & 1;
            const int j = a == 0 ? i : nbr_index(g, i, x, y, z, t, mu, back);
            const int pj = a == 0 ? p : 1 - p;
            cx<float> u[9];
            if (a > 0 && 2 * grp < COUT) su3_row3(n.gauge, mu, back == 0 ? p : 1 - p, back == 0 ? i : j, Vh, u);
            mfma_f4 acc[3];
#pragma unroll
            for (int k = 0; k < 3; k++) acc[k] = mfma_f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int s2 = 0; s2 < NS; s2++) {
                const int c0 = 8 * s2 + 2 * grp;
                mfma_s4 B[3];
#pragma unroll
                for (int k = 0; k < 3; k++) {
                    const uint32_t b0 = c0 < CIN ? net_in_bits<PI>(n.in, sp_idx((long)pj * CIN + c0, j, k, Vh)) : 0u;
                    const uint32_t b1 =
                        c0 + 1 < CIN ? net_in_bits<PI>(n.in, sp_idx((long)pj * CIN + c0 + 1, j, k, Vh)) : 0u;
                    B[k] = s4_of(b0, b1);
                }
                const mfma_s4 A = __builtin_bit_cast(mfma_s4, wop[a * NS + s2][lane]);
#pragma unroll
                for (int k = 0; k < 3; k++) acc[k] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(A, B[k], acc[k], 0, 0, 0);
            }
            // this lane's mixed channels d = 2 grp + h of the neighbour, then their transport
            if (2 * grp < COUT) {
#pragma unroll
                for (int h = 0; h < 2; h++) {
                    cx<float> v[3], yv[3];
#pragma unroll
                    for (int k = 0; k < 3; k++) v[k] = {acc[k][2 * h], acc[k][2 * h + 1]};
                    if (a > 0)
                        net_link_mul(u, back, v, yv);
                    else
#pragma unroll
                        for (int k = 0; k < 3; k++) yv[k] = v[k];
#pragma unroll
                    for (int k = 0; k < 3; k++) o[h][k] = o[h][k] + yv[k];
                }
            }
        }
#pragma unroll
        for (int h = 0; h < 2; h++) {
            const int d = 2 * grp + h;
            if (valid && d < COUT) {
#pragma unroll
                for (int k = 0; k < 3; k++)
                    PO::st(n.out, sp_idx((long)p * COUT + d, i, k, Vh), cx<TO>{(TO)o[h][k].re, (TO)o[h][k].im});
            }
        }
    }
}

template <class PI, class PO, int CIN, int COUT>
__global__ __launch_bounds__(256) void k_net_layer(NetArgs n)
{
    const Geom g = n.g;
    const long gid = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (gid >= 2L * g.Vh) return;
    const int p = (int)(gid / g.Vh), i = (int)(gid % g.Vh);
    int x, y, z, t;
    site_coords(g, i, p, x, y, z, t);
    cx<float> acc[COUT][3];
#pragma unroll
    for (int d = 0; d < COUT; d++)
#pragma unroll
        for (int k = 0; k < 3; k++) acc[d][k] = {0.f, 0.f};
    for (int a = 0; a < 9; a++) {
        cx<float> Y[CIN][3];
        transport<PI, CIN>(n.in, n.gauge, g, p, i, x, y, z, t, a, Y);
        const float2* Wa = n.W + (long)a * COUT * CIN;
#pragma unroll
        for (int d = 0; d < COUT; d++)
#pragma unroll
            for (int c = 0; c < CIN; c++) {
                const float2 w = Wa[d * CIN + c];
                const cx<float> wc = {w.x, w.y};
#pragma unroll
                for (int k = 0; k < 3; k++) acc[d][k] = acc[d][k] + wc * Y[c][k];
            }
    }
    using TO = typename PO::real;
#pragma unroll
    for (int d = 0; d < COUT; d++)
#pragma unroll
        for (int k = 0; k < 3; k++)
            PO::st(n.out, sp_idx((long)p * COUT + d, i, k, g.Vh), cx<TO>{(TO)acc[d][k].re, (TO)acc[d][k].im});
}

// ---------------------------------------------------------------------------
// Training: loss and weight gradients of one pair (r, e), FP32 fields and products, FP64 sums.
//
// The residual r lives on even sites and only even sites of the output enter the loss, so half of every layer is
// zero or unused: hid = layer 1 of r is W1_0 r on even sites and the eight hops on odd ones, z = layer 2 is formed
// on even sites only, and gz = dL/dz is zero on odd ones.  The weight gradients are
//   G1_a[d][c] = sum_x gh_d(x) conj((T_a r_c)(x)),   gh = layer 2's adjoint of gz,
//   G2_a[d][c] = sum_x gz_d(x) conj((T_a hid_c)(x)) = sum_x (T_a^+ gz_d)(x) conj(hid_c(x)),  T_a^+ = T_a',
// so both need only the transports of a four-channel field living on even sites: to odd sites for the eight
// hops, to themselves for a = 0.  Both are real products of 16 rows (two hops of four complex channels) with the
// 2 H columns of the other field over sites and colours; they run on v_mfma_f64_16x16x4 (the FP32 factors and their
// products are exact there), with the accumulators of all hops kept in registers over the tiles of a block and
// the partial sums of the blocks kept over the pairs of a batch.
//
// Blocks take 64 sites, a lane per site; wave w transports channel w, the four waves share the result through
// LDS (rows R[k][16], k = 64 colour + site) and each forms a quarter of the hidden channels from it.
// One thread per site with a block reduction of every gradient entry, a launch per hop, full lattices and a host
// round trip per pair took 955 us a pair at 16^3x32; this takes 168 us (hid and gh 24 each, output 30, products
// 69), where the products' FP64 matrix work needs 20 us and the layers' multiply-adds 60 us at the full rates: the
// transports wait on their gathers.
// ---------------------------------------------------------------------------
struct TrainArgs {
    Geom g;
    const void* gauge;  // FP32 reconstruct-12 links (su3_row3)
    const void* r;      // FP32 residual, even sites, [4][Vh][3]
    const void* gz;     // FP32 dL/dz, even sites
    void* hid;          // FP32 hidden field [2][H][Vh][3]
    void* gh;           // FP32 gradient of the hidden field [2][H][Vh][3]
    const float2* W;    // layer 1 (hidden), layer 2 (output) or the adjoint of layer 2 (gradient)
    double* partials;
    int tiles, accumulate;
};

constexpr int TR_ROW = 18;  // floats per row of R: 16 and a pad that spreads the lanes of a store over the banks
constexpr int TR_R = 192 * TR_ROW;
static_assert(TR_ROW % 2 == 0 && TR_R % 4 == 0, "rows are read in pairs of floats, arrays of R stay 16-byte aligned");

// this wave's channel of the two hops (forward, backward) along mu into R; site odd
__device__ __forceinline__ void train_transport(const Geom& g, const void* gauge, const void* field, int mu, int w,
                                                int i, bool valid, int x, int y, int z, int t, float* R)
{
    const int lane = threadIdx.x & 63;
    // opaque here, so that the addresses of all eight hops are not formed ahead and held (they would spill)
    asm volatile("" : "+v"(i), "+v"(x), "+v"(y), "+v"(z), "+v"(t));
#pragma unroll
    for (int back = 0; back < 2; back++) {
        const int j = nbr_index(g, i, x, y, z, t, mu, back);
        cx<float> u[9], v[3], o[3];
        su3_row3(gauge, mu, back == 0 ? 1 : 0, back == 0 ? i : j, g.Vh, u);
#pragma unroll
        for (int k = 0; k < 3; k++) v[k] = P32::ld(field, sp_idx(w, j, k, g.Vh));
#pragma unroll
        for (int k = 0; k < 3; k++) {
            cx<float> s = back == 0 ? u[3 * k] * v[0] : cmul_conj(u[k], v[0]);
#pragma unroll
            for (int l = 1; l < 3; l++) {
                if (back == 0)
                    cmac(s, u[3 * k + l], v[l]);
                else
                    cmac_conj(s, u[3 * l + k], v[l]);
            }
            o[k] = s;
        }
#pragma unroll
        for (int k = 0; k < 3; k++)
            *reinterpret_cast<float2*>(R + (64 * k + lane) * TR_ROW + 8 * back + 2 * w) =
                valid ? make_float2(o[k].re, o[k].im) : make_float2(0.f, 0.f);
    }
}

// acc_d += sum_c W[d][c] R_c for this wave's H / 4 channels d and one half of the rows
template <int H>
__device__ __forceinline__ void train_mix(const float* R, int half, const float2* __restrict__ W, int w,
                                          cx<float> (&acc)[H / 4][3])
{
    const int lane = threadIdx.x & 63;
    // the weights are uniform over the wave: scalar loads (constant address space), through a pointer that is opaque
    // per call, or all hops' weights would be loaded ahead of the tile loop and held in vector registers
    typedef const __attribute__((address_space(4))) float* sptr;
    sptr p = (sptr)(uintptr_t)(W + w * H);
    asm volatile("" : "+s"(p));
#pragma unroll
    for (int k = 0; k < 3; k++) {
        const float* row = R + (64 * k + lane) * TR_ROW + 8 * half;
#pragma unroll
        for (int c = 0; c < 4; c++) {
            const float2 v = *reinterpret_cast<const float2*>(row + 2 * c);
#pragma unroll
            for (int d = 0; d < H / 4; d++) cmac(acc[d][k], {p[2 * (4 * d + c)], p[2 * (4 * d + c) + 1]}, {v.x, v.y});
        }
    }
}

// the four channels of an even field at its own sites into one half of R
__device__ __forceinline__ void train_own(const void* field, long Vh, int w, int i, bool valid, int half, float* R)
{
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int k = 0; k < 3; k++) {
        const cx<float> v = P32::ld(field, sp_idx(w, i, k, Vh));
        *reinterpret_cast<float2*>(R + (64 * k + lane) * TR_ROW + 8 * half + 2 * w) =
            valid ? make_float2(v.re, v.im) : make_float2(0.f, 0.f);
    }
}

// hid = layer 1 of r: odd tiles first (eight hops), then the even ones (a = 0)
template <int H>
__global__ __launch_bounds__(256) void k_train_hidden(TrainArgs n)
{
    __shared__ alignas(16) float R[2][TR_R];
    const Geom& g = n.g;
    const int odd = (int)blockIdx.x < n.tiles, tile = odd ? blockIdx.x : blockIdx.x - n.tiles;
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const bool valid = tile * 64 + lane < g.Vh;
    const int i = valid ? tile * 64 + lane : g.Vh - 1;
    cx<float> acc[H / 4][3];
#pragma unroll
    for (int d = 0; d < H / 4; d++)
#pragma unroll
        for (int k = 0; k < 3; k++) acc[d][k] = {0.f, 0.f};
    if (odd) {
        int x, y, z, t;
        site_coords(g, i, 1, x, y, z, t);
        for (int mu = 0; mu < 4; mu++) {
            float* r = R[mu & 1];  // the other half is still being read
            train_transport(g, n.gauge, n.r, mu, w, i, valid, x, y, z, t, r);
            __syncthreads();
            train_mix<H>(r, 0, n.W + (1 + 2 * mu) * 4 * H, w, acc);
            train_mix<H>(r, 1, n.W + (2 + 2 * mu) * 4 * H, w, acc);
        }
    } else {
        train_own(n.r, g.Vh, w, i, valid, 0, R[0]);
        __syncthreads();
        train_mix<H>(R[0], 0, n.W, w, acc);
    }
    if (valid) {
#pragma unroll
        for (int d = 0; d < H / 4; d++)
#pragma unroll
            for (int k = 0; k < 3; k++) P32::st(n.hid, sp_idx((long)odd * H + w * (H / 4) + d, i, k, g.Vh), acc[d][k]);
    }
}

// z = layer 2 of hid on even sites; gz = 2 (z - e) / ||e||^2 and the partial sums of ||z - e||^2 per block.  Wave mu
// takes the two hops along mu (wave 0 also a = 0): the neighbour's H channels are mixed first, then the four
// results are transported.  e: the paper's even-site field; en: ||e||^2.
template <int H>
__global__ __launch_bounds__(256) void k_train_output(TrainArgs n, const double2* __restrict__ e,
                                                      const double* __restrict__ en, void* gz)
{
    __shared__ float2 part[4][12][64];
    const Geom& g = n.g;
    const int tile = blockIdx.x, lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const bool valid = tile * 64 + lane < g.Vh;
    const int i = valid ? tile * 64 + lane : g.Vh - 1;
    int x, y, z, t;
    site_coords(g, i, 0, x, y, z, t);
    cx<float> acc[4][3];
    const auto mixed = [&](int a, int p, int j, cx<float>(&m)[4][3]) {
#pragma unroll
        for (int d = 0; d < 4; d++)
#pragma unroll
            for (int k = 0; k < 3; k++) m[d][k] = {0.f, 0.f};
#pragma unroll
        for (int c = 0; c < H; c++) {
            cx<float> v[3];
#pragma unroll
            for (int k = 0; k < 3; k++) v[k] = P32::ld(n.hid, sp_idx((long)p * H + c, j, k, g.Vh));
#pragma unroll
            for (int d = 0; d < 4; d++) {
                const float2 q = n.W[((long)a * 4 + d) * H + c];
#pragma unroll
                for (int k = 0; k < 3; k++) cmac(m[d][k], {q.x, q.y}, v[k]);
            }
        }
    };
    if (w == 0) {
        mixed(0, 0, i, acc);
    } else {
#pragma unroll
        for (int d = 0; d < 4; d++)
#pragma unroll
            for (int k = 0; k < 3; k++) acc[d][k] = {0.f, 0.f};
    }
#pragma unroll
    for (int back = 0; back < 2; back++) {
        const int j = nbr_index(g, i, x, y, z, t, w, back);
        cx<float> u[9], m[4][3];
        su3_row3(n.gauge, w, back, back == 0 ? i : j, g.Vh, u);
        mixed(1 + 2 * w + back, 1, j, m);
#pragma unroll
        for (int d = 0; d < 4; d++)
#pragma unroll
            for (int k = 0; k < 3; k++)
#pragma unroll
                for (int l = 0; l < 3; l++) {
                    if (back == 0)
                        cmac(acc[d][k], u[3 * k + l], m[d][l]);
                    else
                        cmac_conj(acc[d][k], u[3 * l + k], m[d][l]);
                }
    }
#pragma unroll
    for (int d = 0; d < 4; d++)
#pragma unroll
        for (int k = 0; k < 3; k++) part[w][3 * d + k][lane] = make_float2(acc[d][k].re, acc[d][k].im);
    __syncthreads();
    // wave w finishes channel w
    const double coef = 2.0 / en[0];
    double v[1] = {0.0};
#pragma unroll
    for (int k = 0; k < 3; k++) {
        const float2 a = part[0][3 * w + k][lane], b = part[1][3 * w + k][lane], c = part[2][3 * w + k][lane],
                     d = part[3][3 * w + k][lane];
        const double2 ee = e[(long)i * 12 + 3 * w + k];
        const double re = (double)((a.x + b.x) + (c.x + d.x)) - ee.x, im = (double)((a.y + b.y) + (c.y + d.y)) - ee.y;
        if (valid) {
            v[0] += re * re + im * im;
            P32::st(gz, sp_idx(w, i, k, g.Vh), cx<float>{(float)(coef * re), (float)(coef * im)});
        }
    }
    block_sum_store<1>(v, n.partials + blockIdx.x);
}

typedef double mfma_d4 __attribute__((ext_vector_type(4)));

// Weight-gradient products.  Accumulator tile of 16 rows x 16 columns: v_mfma_f64_16x16x4 takes A[row][k] from lane
// row + 16 k, B[k][column] from lane column + 16 k and leaves D[row][column] in element row / 4 of lane
// column + 16 (row % 4).
//   odd tiles, the eight hops:  accumulators [product][mu][column tile], rows 8 back + 2 c + re/im.
//   even tiles, a = 0: rows gz (0..7) and r (8..15); accumulators [product][column tile].
// Product 0: rows of transported gz, columns hid (G2); product 1: rows of transported r, columns gh (G1).
template <int H>
__host__ __device__ constexpr int train_ct() { return (2 * H + 15) / 16; }
template <int H, bool ODD>
__host__ __device__ constexpr int train_entries() { return 2 * (ODD ? 4 : 1) * train_ct<H>() * 256; }

// columns of a tile into C[k][2 H]: this wave's quarter of the H channels of a field at its sites
template <int H>
__device__ __forceinline__ void train_columns(const void* field, long plane0, long Vh, int w, int i, bool valid, float* C)
{
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int d = 0; d < H / 4; d++)
#pragma unroll
        for (int k = 0; k < 3; k++) {
            const int c = w * (H / 4) + d;
            const cx<float> v = P32::ld(field, sp_idx(plane0 + c, i, k, Vh));
            *reinterpret_cast<float2*>(C + (64 * k + lane) * (2 * H + 2) + 2 * c) =
                valid ? make_float2(v.re, v.im) : make_float2(0.f, 0.f);
        }
}

// o += rows^T columns over this wave's quarter of the 192 (site, colour) entries
template <int H>
__device__ __forceinline__ void train_product(const float* rows, const float* C, int w, mfma_d4 (&o)[train_ct<H>()])
{
    const int lane = threadIdx.x & 63;
#pragma unroll 4
    for (int kk = 12 * w; kk < 12 * w + 12; kk++) {
        const int k = 4 * kk + (lane >> 4);
        const double A = (double)rows[k * TR_ROW + (lane & 15)];
#pragma unroll
        for (int t = 0; t < train_ct<H>(); t++)
            o[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(A, (double)C[k * (2 * H + 2) + 16 * t + (lane & 15)], o[t], 0,
                                                        0, 0);
    }
}

// the four waves' accumulators of one tile summed into (or added to) a block's partial sums; red: the bits of
// [4][256] doubles, in LDS that held floats
typedef float bits64 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ void train_store(bits64* red, double* out, int accumulate, const mfma_d4& acc, int w)
{
    const int lane = threadIdx.x & 63, e = threadIdx.x;
    __syncthreads();
#pragma unroll
    for (int r = 0; r < 4; r++) red[w * 256 + 64 * r + lane] = __builtin_bit_cast(bits64, (double)acc[r]);
    __syncthreads();
    const auto part = [&](int k) { return __builtin_bit_cast(double, red[256 * k + e]); };
    const double s = ((part(0) + part(1)) + part(2)) + part(3);
    out[e] = accumulate ? out[e] + s : s;
}

// Blocks [0, nb): odd tiles' product 0; [nb, 2 nb): their product 1; [2 nb, 3 nb): both products of the even tiles.
// With gh formed here as well (it needs the same transports as product 0) the accumulators and the mixing took
// 217-298 VGPRs and the launch waited on its loads: 81 us and 33 us for the products (16^3x32) against 69 us,
// and 24 us for gh from k_train_hidden, with the three parts in one launch.
template <int H>
__global__ __launch_bounds__(256) void k_train_grad(TrainArgs n, int nb)
{
    constexpr int CT = train_ct<H>(), CROW = 2 * H + 2;
    __shared__ alignas(16) float R[TR_R];
    __shared__ alignas(16) float C[192 * CROW + 16];  // columns: C[k][2 H]; the last tile reads up to 16 floats past a row
    const Geom& g = n.g;
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int part = blockIdx.x / nb, b0 = blockIdx.x - part * nb;
    if (threadIdx.x < 16) C[192 * CROW + threadIdx.x] = 0.f;
    if (threadIdx.x < 192) {
#pragma unroll
        for (int j = 2 * H; j < CROW; j++) C[threadIdx.x * CROW + j] = 0.f;
    }
    bits64* red = reinterpret_cast<bits64*>(R);  // [4][256]
    static_assert(TR_R * 4 >= 4 * 256 * 8, "the reduction buffer fits in R");
    if (part < 2) {
        const void* rows = part == 0 ? n.gz : n.r;
        const void* cols = part == 0 ? n.hid : n.gh;
        mfma_d4 acc[4][CT];
#pragma unroll
        for (int q = 0; q < 4; q++)
#pragma unroll
            for (int t = 0; t < CT; t++) acc[q][t] = mfma_d4{0.0, 0.0, 0.0, 0.0};
        for (int tile = b0; tile < n.tiles; tile += nb) {
            const bool valid = tile * 64 + lane < g.Vh;
            const int i = valid ? tile * 64 + lane : g.Vh - 1;
            int x, y, z, t;
            site_coords(g, i, 1, x, y, z, t);
            __syncthreads();  // the last tile's columns and rows are no longer read
            train_columns<H>(cols, H, g.Vh, w, i, valid, C);
            // not unrolled: the four copies' addresses would be formed ahead of the tile loop
#pragma unroll 1
            for (int mu = 0; mu < 4; mu++) {
                if (mu > 0) __syncthreads();
                train_transport(g, n.gauge, rows, mu, w, i, valid, x, y, z, t, R);
                __syncthreads();
                switch (mu) {  // registers are indexed statically
                case 0: train_product<H>(R, C, w, acc[0]); break;
                case 1: train_product<H>(R, C, w, acc[1]); break;
                case 2: train_product<H>(R, C, w, acc[2]); break;
                default: train_product<H>(R, C, w, acc[3]); break;
                }
            }
        }
        double* out = n.partials + (long)b0 * train_entries<H, true>() + part * 4 * CT * 256;
#pragma unroll
        for (int q = 0; q < 4; q++)
#pragma unroll
            for (int t = 0; t < CT; t++) train_store(red, out + (q * CT + t) * 256, n.accumulate, acc[q][t], w);
    } else {
        mfma_d4 acc[2][CT];
#pragma unroll
        for (int m = 0; m < 2; m++)
#pragma unroll
            for (int t = 0; t < CT; t++) acc[m][t] = mfma_d4{0.0, 0.0, 0.0, 0.0};
        for (int tile = b0; tile < n.tiles; tile += nb) {
            const bool valid = tile * 64 + lane < g.Vh;
            const int i = valid ? tile * 64 + lane : g.Vh - 1;
            __syncthreads();
            train_own(n.gz, g.Vh, w, i, valid, 0, R);
            train_own(n.r, g.Vh, w, i, valid, 1, R);
            train_columns<H>(n.hid, 0, g.Vh, w, i, valid, C);
            __syncthreads();
            train_product<H>(R, C, w, acc[0]);
            __syncthreads();
            train_columns<H>(n.gh, 0, g.Vh, w, i, valid, C);
            __syncthreads();
            train_product<H>(R, C, w, acc[1]);
        }
        double* out = n.partials + (long)nb * train_entries<H, true>() + (long)b0 * train_entries<H, false>();
#pragma unroll
        for (int m = 0; m < 2; m++)
#pragma unroll
            for (int t = 0; t < CT; t++) train_store(red, out + (m * CT + t) * 256, n.accumulate, acc[m][t], w);
    }
}

// sums over the blocks of both kernels, [odd entries | even entries]
__global__ __launch_bounds__(256) void k_train_sum(const double* odd, int nb_odd, int n_odd, const double* even,
                                                   int nb_even, int n_even, double* out)
{
    __shared__ double red[4][64];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int e = blockIdx.x * 64 + lane;  // n_odd and n_even are multiples of 64
    const bool is_odd = e < n_odd;
    const double* p = is_odd ? odd + e : even + (e - n_odd);
    const int nb = is_odd ? nb_odd : nb_even, stride = is_odd ? n_odd : n_even;
    double s = 0.0;
#pragma unroll 8
    for (int b = w; b < nb; b += 4) s += p[(long)b * stride];
    red[w][lane] = s;
    __syncthreads();
    if (w == 0) out[e] = ((red[0][lane] + red[1][lane]) + red[2][lane]) + red[3][lane];
}

// the complex gradients from the real sums (k_train_grad): G1 [9][H][4], G2 [9][4][H]
template <int H>
__global__ void k_train_gather(const double* __restrict__ S, double2* __restrict__ G1, double2* __restrict__ G2)
{
    constexpr int CT = train_ct<H>(), N_ODD = train_entries<H, true>();
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= 2 * 9 * 4 * H) return;
    const int m = e / (9 * 4 * H), q = e % (9 * 4 * H), a = q / (4 * H);
    // c: the four-channel index (row), h: the hidden index (column)
    const int c = m == 0 ? (q / H) % 4 : q % 4, h = m == 0 ? q % H : (q / 4) % H;
    // product 0 pairs hid with gz transported by the reversed hop
    const int hop = a == 0 ? 0 : (m == 0 ? (((a - 1) & 1) ? a - 1 : a + 1) : a);
    const int row0 = a == 0 ? 8 * m + 2 * c : 8 * ((hop - 1) & 1) + 2 * c;
    const long base = a == 0 ? N_ODD + (long)m * CT * 256 : (long)((m * 4 + ((hop - 1) >> 1)) * CT) * 256;
    const auto D = [&](int row, int col) {
        return S[base + (col >> 4) * 256 + 64 * (row >> 2) + (col & 15) + 16 * (row & 3)];
    };
    const double rr = D(row0, 2 * h), ri = D(row0, 2 * h + 1), ir = D(row0 + 1, 2 * h), ii = D(row0 + 1, 2 * h + 1);
    // product 0: row conj(column); product 1: column conj(row)
    const double2 v = make_double2(rr + ii, m == 0 ? ir - ri : ri - ir);
    if (m == 0)
        G2[q] = v;
    else
        G1[q] = v;
}

// Wt[a'][c][d] = conj(W[a][d][c]), a' the reversed hop (T_a^+ = T_a'), for the adjoint layer
__global__ void k_net_adjoint_w(const float2* W, float2* Wt, int cout, int cin)
{
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= 9 * cout * cin) return;
    const int a = e / (cout * cin), r = e % (cout * cin), d = r / cin, c = r % cin;
    const int at = a == 0 ? 0 : (((a - 1) & 1) ? a - 1 : a + 1);
    const float2 w = W[e];
    Wt[(long)at * cin * cout + c * cout + d] = make_float2(w.x, -w.y);
}

// Adam (Kingma and Ba 2015) on the real and imaginary parts of the weights
__global__ void k_adam(float* W, const double* G, double* m, double* v, int n, double lr, double b1, double b2,
                       double eps, int step, double gscale)
{
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= n) return;
    const double g = G[e] * gscale;
    m[e] = b1 * m[e] + (1.0 - b1) * g;
    v[e] = b2 * v[e] + (1.0 - b2) * g * g;
    const double mh = m[e] / (1.0 - pow(b1, (double)step));
    const double vh = v[e] / (1.0 - pow(b2, (double)step));
    W[e] = (float)((double)W[e] - lr * mh / (sqrt(vh) + eps));
}

// Gaussian complex entries (re, im ~ N(0,1)) from a counter-based generator:
// splitmix64 of (seed, stream, element) feeds a Box-Muller transform, so the
// field depends only on (seed, stream), not on the launch shape.
__device__ __forceinline__ uint64_t splitmix64(uint64_t z)
{
    z += 0x9e3779b97f4a7c15ull;
    z = (z ^ (z >> 30)) * 0xbf58476d1ce4e5b9ull;
    z = (z ^ (z >> 27)) * 0x94d049bb133111ebull;
    return z ^ (z >> 31);
}

__global__ void k_gaussian(double2* out, long n, uint64_t seed, uint64_t stream)
{
    const long e = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= n) return;
    const uint64_t k = splitmix64(seed ^ splitmix64(stream ^ splitmix64((uint64_t)e)));
    const uint64_t k2 = splitmix64(k);
    const double u1 = ((k >> 11) + 1.0) * (1.0 / 9007199254740993.0);  // (0, 1]
    const double u2 = (k2 >> 11) * (1.0 / 9007199254740992.0);          // [0, 1)
    const double rad = sqrt(-2.0 * log(u1)), th = 6.283185307179586 * u2;
    out[e] = make_double2(rad * cos(th), rad * sin(th));
}

static inline dim3 g256(long n) { return dim3((unsigned)((n + 255) / 256)); }

hipError_t launch_gaussian(hipStream_t s, void* out, long n, uint64_t seed, uint64_t stream)
{
    hipLaunchKernelGGL(k_gaussian, g256(n), dim3(256), 0, s, (double2*)out, n, seed, stream);
    return hipGetLastError();
}

hipError_t launch_net_layer(hipStream_t s, int pin, int pout, int cin, int cout, const void* in, void* out,
                            const void* gauge32, const void* W, const Geom& g, int mfma)
{
    NetArgs n{in, out, gauge32, (const float2*)W, g};
    const dim3 grid = g256(2L * g.Vh);
    const dim3 grid_mfma((unsigned)((2L * g.Vh + 63) / 64));  // 16 sites per wave, 4 waves per block
    // layers with a BF16 end (the preconditioner's application) mix channels on the matrix cores
#define QCDW_NET_MFMA_CASE(PI, PO, CI, CO, pi, po)                                                \
    if (pin == pi && pout == po && cin == CI && cout == CO) {                                     \
        hipLaunchKernelGGL((k_net_layer_mfma<PI, PO, CI, CO>), grid_mfma, dim3(256), 0, s, n);     \
        return hipGetLastError();                                                                 \
    }
#define QCDW_NET_CASE(PI, PO, CI, CO, pi, po)                                              \
    if (pin == pi && pout == po && cin == CI && cout == CO) {                              \
        hipLaunchKernelGGL((k_net_layer<PI, PO, CI, CO>), grid, dim3(256), 0, s, n);        \
        return hipGetLastError();                                                          \
    }
    if (mfma) {
        QCDW_NET_MFMA_CASE(P32, PBF16, 4, 12, F32, BF16)
        QCDW_NET_MFMA_CASE(PBF16, P32, 12, 4, BF16, F32)
        QCDW_NET_MFMA_CASE(P32, PBF16, 4, 4, F32, BF16)
        QCDW_NET_MFMA_CASE(PBF16, P32, 4, 4, BF16, F32)
    }
    QCDW_NET_CASE(P32, P32, 4, 12, F32, F32)
    QCDW_NET_CASE(P32, P32, 12, 4, F32, F32)
    QCDW_NET_CASE(P32, PBF16, 4, 12, F32, BF16)
    QCDW_NET_CASE(PBF16, P32, 12, 4, BF16, F32)
    QCDW_NET_CASE(P32, P32, 4, 4, F32, F32)
    QCDW_NET_CASE(P32, PBF16, 4, 4, F32, BF16)
    QCDW_NET_CASE(PBF16, P32, 4, 4, BF16, F32)
#undef QCDW_NET_CASE
#undef QCDW_NET_MFMA_CASE
    return hipErrorInvalidValue;
}

static int train_tiles(const Geom& g) { return (g.Vh + 63) / 64; }
// blocks of each part of the gradient kernel; each keeps its own partial sums.  At 16^3x32 (1024 tiles) 256, 384
// and 512 take 1.40, 1.34 and 1.36 ms for eight pairs
static int train_blocks(const Geom& g) { return std::min(train_tiles(g), 384); }

size_t train_partials(const Geom& g, int hidden)
{
    const size_t per = hidden == 12 ? train_entries<12, true>() + train_entries<12, false>()
                                    : train_entries<4, true>() + train_entries<4, false>();
    return (size_t)(train_blocks(g) + 1) * per + train_tiles(g);
}

template <int H>
static hipError_t train_pair(hipStream_t s, const Geom& g, const TrainFields& f, const void* e, const double* en,
                             double* dn, bool first)
{
    const int tiles = train_tiles(g), nb = train_blocks(g);
    double* odd = f.partials;
    double* even = odd + (size_t)nb * train_entries<H, true>();
    double* loss = even + (size_t)(nb + 1) * train_entries<H, false>() + train_entries<H, true>();
    TrainArgs n{g, f.gauge32, f.r, f.gz, f.hid, f.gh, (const float2*)f.W1, nullptr, tiles, first ? 0 : 1};
    hipLaunchKernelGGL(k_train_hidden<H>, dim3(2 * tiles), dim3(256), 0, s, n);
    n.W = (const float2*)f.W2;
    n.partials = loss;
    hipLaunchKernelGGL(k_train_output<H>, dim3(tiles), dim3(256), 0, s, n, (const double2*)e, en, f.gz);
    if (const hipError_t e1 = launch_sum_partials(s, loss, tiles, dn); e1 != hipSuccess) return e1;
    // gh: the adjoint of layer 2 is a layer from even sites like layer 1
    TrainArgs adj{g, f.gauge32, f.gz, nullptr, f.gh, nullptr, (const float2*)f.Wt, nullptr, tiles, 0};
    hipLaunchKernelGGL(k_train_hidden<H>, dim3(2 * tiles), dim3(256), 0, s, adj);
    n.partials = odd;
    hipLaunchKernelGGL(k_train_grad<H>, dim3(3 * nb), dim3(256), 0, s, n, nb);
    return hipGetLastError();
}

template <int H>
static hipError_t train_finish(hipStream_t s, const Geom& g, double* partials, void* G1, void* G2)
{
    constexpr int NO = train_entries<H, true>(), NE = train_entries<H, false>();
    const int nb = train_blocks(g);
    double* even = partials + (size_t)nb * NO;
    double* S = even + (size_t)nb * NE;
    hipLaunchKernelGGL(k_train_sum, dim3((NO + NE) / 64), dim3(256), 0, s, partials, nb, NO, even, nb, NE, S);
    hipLaunchKernelGGL(k_train_gather<H>, g256(2L * 9 * 4 * H), dim3(256), 0, s, S, (double2*)G1, (double2*)G2);
    return hipGetLastError();
}

hipError_t launch_train_pair(hipStream_t s, int hidden, const Geom& g, const TrainFields& f, const void* e,
                             const double* en, double* dn, bool first)
{
    if (hidden == 12) return train_pair<12>(s, g, f, e, en, dn, first);
    if (hidden == 4) return train_pair<4>(s, g, f, e, en, dn, first);
    return hipErrorInvalidValue;
}

hipError_t launch_train_finish(hipStream_t s, int hidden, const Geom& g, double* partials, void* G1, void* G2)
{
    if (hidden == 12) return train_finish<12>(s, g, partials, G1, G2);
    if (hidden == 4) return train_finish<4>(s, g, partials, G1, G2);
    return hipErrorInvalidValue;
}

hipError_t launch_net_adjoint_w(hipStream_t s, const void* W, void* Wt, int cout, int cin)
{
    hipLaunchKernelGGL(k_net_adjoint_w, g256(9L * cout * cin), dim3(256), 0, s, (const float2*)W, (float2*)Wt, cout,
                       cin);
    return hipGetLastError();
}

hipError_t launch_adam(hipStream_t s, void* W, const double* G, double* m, double* v, int n, double lr, double b1,
                       double b2, double eps, int step, double gscale)
{
    hipLaunchKernelGGL(k_adam, g256(n), dim3(256), 0, s, (float*)W, G, m, v, n, lr, b1, b2, eps, step, gscale);
    return hipGetLastError();
}

}  // namespace qcdw
