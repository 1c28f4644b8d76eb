// Multi-right-hand-side parity hop (a propagator is 12 solves, paper Sec. III.B;
// the paper names a multi-source solve as the next step).  Four lanes per site as
// in hop.hip, but each lane loads its four reconstruct-12 links and its clover
// window once and applies them to every right-hand side in a register-resident
// loop, so link and clover bytes are paid once per site for all RHS.  RHS k of a
// field lives at offset k * 12 * Vh complex (a stack of single-RHS fields), and RHS
// whose solver flag is set are skipped.  With cgroup > 0 the tiles follow the
// slice-group order of the single-RHS hop.
//
// The lanes of a wave are ordered spin by spin, 16 sites each: a load of one spin's
// three colours then reads a run of consecutive sites in neighbouring lanes, and the
// first cache counts 2.5 times fewer accesses.  With the four spins of a site in
// neighbouring lanes (the order of hop.hip) the loop ran at the rate of one access
// per lane and load: 0.31 ms for 12 BF16 right-hand sides at 24^3x64, all active.
// The two exchanges between a site's lanes go through ds_bpermute.
#include <hip/hip_ext.h>

#include <type_traits>

#include "hop_common.h"

namespace qcdw {

// whether every right-hand side is finished (uniform; the launches enqueued after the end of a cycle return here,
// before they load links: 47 us each at 24^3x64)
__device__ __forceinline__ bool all_finished(const Scal* S, int nrhs)
{
    if (!S) return false;
    for (int r = 0; r < nrhs; r++)
        if (!S[r].flags) return false;
    return true;
}

// Reduction partials of a block, right-hand side by right-hand side: each wave leaves its sums in LDS, and the block
// adds the four waves' once at the end (a barrier pair per right-hand side held the loop's loads up).
constexpr int MRHS_MAX = 16;
struct MrhsSums {
    double v[MRHS_MAX][4][3];
};
__device__ __forceinline__ void mrhs_sum_wave(MrhsSums& m, int r, double (&v)[3], int n)
{
#pragma unroll
    for (int k = 0; k < 3; k++) {
        if (k >= n) break;
        const double s = wave_sum(v[k]);
        if ((threadIdx.x & 63) == 0) m.v[r][threadIdx.x >> 6][k] = s;
    }
}
// partials [r][nblk][3] of this block; finished right-hand sides keep theirs
__device__ __forceinline__ void mrhs_sum_store(const MrhsSums& m, const Scal* S, int nrhs, int n, double* partials,
                                               int tile, int nblk)
{
    __syncthreads();
    const int r = threadIdx.x >> 2, k = threadIdx.x & 3;
    if (r < nrhs && k < 3 && !(S && S[r].flags))
        partials[3 * ((long)r * nblk + tile) + k] =
            k < n ? ((m.v[r][0][k] + m.v[r][1][k]) + m.v[r][2][k]) + m.v[r][3][k] : 0.0;
}

// v of the lane at byte address `at` (ds_bpermute: the exchange between rows of 16 lanes, on the idle LDS pipe)
__device__ __forceinline__ float lane_val(float v, int at)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_ds_bpermute(at, __builtin_bit_cast(int, v)));
}
__device__ __forceinline__ double lane_val(double v, int at)
{
    const uint2 u = __builtin_bit_cast(uint2, v);
    return __builtin_bit_cast(double, make_uint2((unsigned)__builtin_amdgcn_ds_bpermute(at, (int)u.x),
                                                 (unsigned)__builtin_amdgcn_ds_bpermute(at, (int)u.y)));
}
template <typename T>
__device__ __forceinline__ cx<T> lane_cx(cx<T> v, int at)
{
    return {lane_val(v.re, at), lane_val(v.im, at)};
}

// complex number c of a run of words as they were loaded (a bit copy: the words are no object of P's storage type)
template <class P>
__device__ __forceinline__ cx<typename P::real> words_cx(const uint32_t* w, int c)
{
    if constexpr (P::cbytes == 16)
        return {__builtin_bit_cast(double, make_uint2(w[4 * c], w[4 * c + 1])),
                __builtin_bit_cast(double, make_uint2(w[4 * c + 2], w[4 * c + 3]))};
    else if constexpr (P::cbytes == 8)
        return {__builtin_bit_cast(float, w[2 * c]), __builtin_bit_cast(float, w[2 * c + 1])};
    else if constexpr (std::is_same_v<P, PBF16>)
        return {bf_bits2f(w[c] & 0xffffu), bf_bits2f(w[c] >> 16)};
    else
        return {(float)__builtin_bit_cast(_Float16, (uint16_t)(w[c] & 0xffffu)),
                (float)__builtin_bit_cast(_Float16, (uint16_t)(w[c] >> 16))};
}

template <class P, int EPI, int RED>
__global__ __launch_bounds__(256, P::cbytes == 16 ? 1 : 2) void hop_mrhs_kernel(HopArgs a, const Scal* S)
{
    if (all_finished(S, a.nrhs)) return;
    __shared__ MrhsSums sums;
    constexpr int NSUM = RED == RED_WDOT ? 2 : 3;
    using T = typename P::real;
    const Geom g = a.g;
    const int tile = xcd_tile(blockIdx.x, gridDim.x);
    const int nblk = gridDim.x;
    const int q = (threadIdx.x >> 4) & 3, ts = (threadIdx.x >> 6) * 16 + (threadIdx.x & 15);
    // lanes (byte addresses) of this site's partner half and of the chirality block's other spin
    const int at_partner = 4 * ((threadIdx.x & 15) + 16 * (q < 2 ? q + 2 : 3 - q)),
              at_xor1 = 4 * ((threadIdx.x & 63) ^ 16);
    int site;
    bool valid;
    if (a.cgroup > 0) {  // slice-group order, as in the single-RHS hop_kernel
        const int St = g.Lxh * g.Ly * g.Lz;
        int t;
        const int c = group_ctile(g, tile, a.cgroup, t) * HOP_SITES_PER_BLOCK + ts;
        site = t * St + c;
        valid = c < St;
    } else {
        site = tile * HOP_SITES_PER_BLOCK + ts;
        valid = site < g.Vh;
    }
    const int gq = q >> 1;
    const long Vh = g.Vh;
    const long field = 12L * Vh;  // complex per RHS
    // this lane's own spin and the one that its directions couple to it: row q of (1 -/+ gamma) psi, so that the sum
    // for spin q collects in acc_u in every lane (for z and t that is the row l of hop_common.h, with the
    // conjugate coefficient)
    const int su = q, sl = gq == 0 ? 3 - q : q - 2;

    // per-lane hop geometry, links (row 2 rebuilt once) and clover window, shared by all RHS
    LaneHops<T, 6> L;
    cx<T> ur[4][9];
    T win[27];
#pragma unroll
    for (int h = 0; h < 4; h++) {
        L.nbh[h] = 0;
        L.loff[h] = 0;
        L.cs[h] = T(0);
        L.fsg[h] = T(1);
#pragma unroll
        for (int e = 0; e < 9; e++) ur[h][e] = {T(0), T(0)};
    }
#pragma unroll
    for (int e = 0; e < 27; e++) win[e] = T(0);
    if (valid) lane_hops<T, 6, link_soa_for(P::cbytes)>(g, site, a.parity, q, L);
    if (gq == 1) L.cs[0] = -L.cs[0], L.cs[1] = -L.cs[1];
    // Right-hand sides in flight ahead of the one that is computed: two in BF16 (a hop's words are replaced as soon
    // as they are read; 24 registers each, 30 with the epilogue's operands), one in FP16 (whose conversions take the
    // registers) and, without the epilogue's operands, in FP32; none in FP64.  The links leave room for two waves per
    // SIMD, which do not cover the loads' latency.  24^3x64, 12 BF16 right-hand sides, a solve's mean per launch (first
    // hop / r0 dot / t dot; the launches enqueued past the end of a cycle count): a site's lanes side by side
    // 207 / 426 / 296 us; this order, three waves, none ahead 170 / 385 / 351; one 189 / 220 / 213; two 165 / 213 / 209.
    constexpr int AHEAD = std::is_same_v<P, PBF16> ? 2 : P::cbytes <= 8 ? 1 : 0;
    constexpr bool OWN_AHEAD = P::cbytes == 4;
    constexpr bool HAS_Y = EPI == EPI_CLOV_XPAY || RED == RED_TS, HAS_W = RED == RED_WDOT;
    // byte offsets within a right-hand side: 32-bit beside a scalar base in 16-bit storage
    using Off = std::conditional_t<P::cbytes == 4, uint32_t, long>;
    const long own = sp_idx(q, valid ? site : 0, 0, Vh);
    const Off own_at = (Off)(own * P::cbytes);
    Off at_u[4], at_l[4];
#pragma unroll
    for (int h = 0; h < 4; h++) {
        at_u[h] = (Off)(sp_idx(su, L.nbh[h], 0, Vh) * P::cbytes);
        at_l[h] = (Off)(sp_idx(sl, L.nbh[h], 0, Vh) * P::cbytes);
    }
    struct Raw {
        uint32_t u[3 * P::cbytes / 4];
    };
    auto fetch = [&](const void* base, int r, Off at) {
        Raw v;
        uint64_t b = (uint64_t)base + __builtin_amdgcn_readfirstlane(r) * field * P::cbytes;
        asm volatile("" : "+s"(b));  // kept scalar: an address takes one 32-bit register, not a 64-bit pair
        const auto* src = (const __attribute__((address_space(1))) uint32_t*)(
            (const __attribute__((address_space(1))) char*)b + at);
#pragma unroll
        for (int e = 0; e < 3 * P::cbytes / 4; e++) v.u[e] = src[e];
        return v;
    };
    auto next_rhs = [&](int r) {  // uniform: every thread reads the same flags
        while (r < a.nrhs && S && S[r].flags) r++;
        return r;
    };
    struct Flight {
        Raw u[4], l[4], y, w;
    } fl[AHEAD == 2 ? 2 : 1];
    auto fetch_hop = [&](Flight& f, int h, int r) {
        f.u[h] = fetch(a.psi, r, at_u[h]);
        f.l[h] = fetch(a.psi, r, at_l[h]);
    };
    auto fetch_own = [&](Flight& f, int r) {
        if constexpr (HAS_Y) f.y = fetch(a.y, r, own_at);
        if constexpr (HAS_W) f.w = fetch(a.w, r, own_at);
    };
    auto fetch_all = [&](Flight& f, int r) {
#pragma unroll
        for (int h = 0; h < 4; h++) fetch_hop(f, h, r);
        if constexpr (OWN_AHEAD) fetch_own(f, r);
    };
    // the first right-hand side's loads go out before the links'
    int r = next_rhs(0), r1 = next_rhs(r + 1);
    if constexpr (AHEAD > 0)
        if (r < a.nrhs) fetch_all(fl[0], r);
    if constexpr (AHEAD > 1)
        if (r1 < a.nrhs) fetch_all(fl[1], r1);
    if (valid) {
#pragma unroll
        for (int h = 0; h < 4; h++) {
            load_link<P, 6>(a.gauge, L.loff[h], L.lstr, ur[h]);
#pragma unroll
            for (int e = 0; e < 9; e++) ur[h][e] = L.fsg[h] * ur[h][e];
        }
        T raw[27];
        load_window<P>(a.clov, Vh, site, q, raw);
        herm_coef(raw, q & 1, win);
    }
    auto clov_row = [&](const T (&m)[27], int i, T (&row)[11]) {
        // own entries (1,0), (2,0), (2,1) at 3, 5, 7; (i, j) and (j, i) are conjugates
        const int f0 = i == 2 ? 5 : 3, f1 = i == 0 ? 5 : 7;
        const T s0 = i == 0 ? T(-1) : T(1), s1 = i == 2 ? T(1) : T(-1);
        row[0] = m[i];
        row[1] = m[f0];
        row[2] = s0 * m[f0 + 1];
        row[3] = m[f1];
        row[4] = s1 * m[f1 + 1];
#pragma unroll
        for (int e = 0; e < 6; e++) row[5 + e] = m[9 + 6 * i + e];
    };
    auto one_rhs = [&](Flight& f, int r, int rn, auto more) {
        constexpr bool MORE = decltype(more)::value;
        if constexpr (AHEAD == 0) fetch_all(f, r);
        if constexpr (!OWN_AHEAD) fetch_own(f, r);
        cx<T> acc_u[3], acc_l[3];
#pragma unroll
        for (int c = 0; c < 3; c++) acc_u[c] = acc_l[c] = {T(0), T(0)};
#pragma unroll
        for (int h = 0; h < 4; h++) {
            cx<T> pu[3], pl[3], hv[3];
#pragma unroll
            for (int c = 0; c < 3; c++) {
                pu[c] = words_cx<P>(f.u[h].u, c);
                pl[c] = words_cx<P>(f.l[h].u, c);
            }
            project<true>(pu, pl, L.cs[h], h < 2, hv);
            if constexpr (MORE) fetch_hop(f, h, rn);
            hop_rows<true>(ur[h], h & 1, h < 2, T(1), L.cs[h], hv, acc_u, acc_l);
        }
        cx<T> res[3], outv[3], yv[3], wv[3];
#pragma unroll
        for (int c = 0; c < 3; c++) {
            res[c] = acc_u[c] + lane_cx(acc_l[c], at_partner);
            if constexpr (HAS_Y) yv[c] = words_cx<P>(f.y.u, c);
            if constexpr (HAS_W) wv[c] = words_cx<P>(f.w.u, c);
        }
        cx<T> ox[3], br[3];
#pragma unroll
        for (int c = 0; c < 3; c++) ox[c] = lane_cx(res[c], at_xor1);
#pragma unroll
        for (int i = 0; i < 3; i++) {
            T m[11];
            clov_row(win, i, m);
            const int j0 = i == 0 ? 1 : 0, j1 = i == 2 ? 1 : 2;
            cx<T> s = {m[0] * res[i].re, m[0] * res[i].im};
            cmac(s, cx<T>{m[1], m[2]}, res[j0]);
            cmac(s, cx<T>{m[3], m[4]}, res[j1]);
#pragma unroll
            for (int b = 0; b < 3; b++) cmac(s, cx<T>{m[5 + 2 * b], m[6 + 2 * b]}, ox[b]);
            br[i] = s;
        }
        const T aa = (T)a.a;
#pragma unroll
        for (int c = 0; c < 3; c++) outv[c] = (EPI == EPI_CLOV) ? br[c] : yv[c] - aa * br[c];
        if constexpr (MORE && OWN_AHEAD) fetch_own(f, rn);
#pragma unroll
        for (int c = 0; c < 3; c++) outv[c] = P::rt(outv[c]);
        if (valid) {
#pragma unroll
            for (int c = 0; c < 3; c++) P::st(a.out, r * field + own + c, outv[c]);
        }
        if constexpr (RED != RED_NONE) {
            double v[3] = {0.0, 0.0, 0.0};
            if (valid) {
#pragma unroll
                for (int c = 0; c < 3; c++) {
                    const cx<T> o = outv[c];
                    if constexpr (RED == RED_WDOT) {
                        v[0] += (double)wv[c].re * o.re + (double)wv[c].im * o.im;
                        v[1] += (double)wv[c].re * o.im - (double)wv[c].im * o.re;
                    } else {
                        v[0] += (double)o.re * yv[c].re + (double)o.im * yv[c].im;
                        v[1] += (double)o.re * yv[c].im - (double)o.im * yv[c].re;
                        v[2] += (double)o.re * o.re + (double)o.im * o.im;
                    }
                }
            }
            mrhs_sum_wave(sums, r, v, NSUM);
        }
    };
    if constexpr (AHEAD == 2) {
        while (r1 < a.nrhs) {
            const int r2 = next_rhs(r1 + 1), r3 = next_rhs(r2 + 1);
            if (r3 >= a.nrhs) {  // two or three left
                one_rhs(fl[0], r, r2 < a.nrhs ? r2 : r, std::true_type{});
                one_rhs(fl[1], r1, r1, std::false_type{});
                r = r2;
                break;
            }
            one_rhs(fl[0], r, r2, std::true_type{});
            one_rhs(fl[1], r1, r3, std::true_type{});
            r = r2;
            r1 = r3;
        }
        if (r < a.nrhs) one_rhs(fl[0], r, r, std::false_type{});
    } else if constexpr (AHEAD == 1) {
        for (; r1 < a.nrhs; r = r1, r1 = next_rhs(r + 1)) one_rhs(fl[0], r, r1, std::true_type{});
        if (r < a.nrhs) one_rhs(fl[0], r, r, std::false_type{});
    } else {
        for (; r < a.nrhs; r = next_rhs(r + 1)) one_rhs(fl[0], r, r, std::false_type{});
    }
    if constexpr (RED != RED_NONE) mrhs_sum_store(sums, S, a.nrhs, NSUM, a.partials, tile, nblk);
}

template <class P>
static hipError_t launch_mrhs_p(hipStream_t s, int epi, int red, const HopArgs& a, const Scal* S, hipEvent_t e0,
                                hipEvent_t e1)
{
    dim3 grid(a.cgroup > 0 ? hop_ctiles(a.g) * a.g.Lt : hop_blocks(a.g.Vh)), block(256);
#define QCDW_MRHS_CASE(E, D)                                                                     \
    if (epi == E && red == D) {                                                                 \
        if (e0)                                                                                 \
            hipExtLaunchKernelGGL((hop_mrhs_kernel<P, E, D>), grid, block, 0, s, e0, e1, 0, a, S); \
        else                                                                                    \
            hipLaunchKernelGGL((hop_mrhs_kernel<P, E, D>), grid, block, 0, s, a, S);             \
        return hipGetLastError();                                                               \
    }
    QCDW_MRHS_CASE(EPI_CLOV, RED_NONE)
    QCDW_MRHS_CASE(EPI_CLOV_XPAY, RED_NONE)
    QCDW_MRHS_CASE(EPI_CLOV_XPAY, RED_WDOT)
    QCDW_MRHS_CASE(EPI_CLOV_XPAY, RED_TS)
#undef QCDW_MRHS_CASE
    return hipErrorInvalidValue;
}

hipError_t launch_hop_mrhs(hipStream_t s, int prec, int epi, int red, const HopArgs& a, const Scal* S,
                           hipEvent_t e0, hipEvent_t e1)
{
    if (a.g.Vh <= 0 || a.nrhs <= 0) return hipSuccess;
    if (a.nrhs > MRHS_MAX || !mrhs_offsets_fit(prec, a.g.Vh)) return hipErrorInvalidValue;
    switch (prec) {
    case F64: return launch_mrhs_p<P64>(s, epi, red, a, S, e0, e1);
    case F32: return launch_mrhs_p<P32>(s, epi, red, a, S, e0, e1);
    case BF16: return launch_mrhs_p<PBF16>(s, epi, red, a, S, e0, e1);
    case F16: return launch_mrhs_p<PF16>(s, epi, red, a, S, e0, e1);
    }
    return hipErrorInvalidValue;
}

// ---------------------------------------------------------------------------
// Matrix-core form (16-bit storage): the SU(3) products of the hop on v_mfma_f32_4x4x4 (16 blocks of
// 4x4x4 per wave, FP32 accumulation).  Block b of an instruction is the quad of lanes 4b..4b+3, one site:
// lane 4b+i supplies row i of the A operand (K = 4 entries), lane 4b+j column j of B, and receives column j
// of D = A B in its four accumulator elements.  With A the hop's link W (rows: colour i, K: colour k, row and
// column 3 zero) and column j of B the neighbour's spin j, D holds (W psi_j)[i] in lane j: the lane of the
// output spin.  The spin projector is not formed: (1 -/+ gamma_mu) psi = psi_j + e_j psi_perm(j) with e_j a
// unit number (+-1 or +-i), so each direction adds W psi_j and W (e_j psi_perm(j)); the partner's spin comes
// from the quad by a DPP permutation, e_j by swapping re/im and flipping sign bits, both exact in 16 bits.
// Complex products take four real instructions (Re: Wr Br - Wi Bi, Im: Wr Bi + Wi Br).  Row 2 of the link
// is rebuilt in FP32 and rounded to 16 bits once per site (the only rounding the vector form does not have);
// the products are exact in FP32 and all eight directions accumulate there (the spatial ones first, their sum
// then scaled by the spatial weight).  Link operands are built once per site and kept in registers for all
// right-hand sides; the clover epilogue is the vector form's.  Measured at 24^3x64 with 12 RHS (BF16), a solve's
// mean per launch (first hop / r0 dot / t dot): 232 / 347 / 312 us against 165 / 213 / 209 us for the vector register
// loop: the quad of a site must be neighbouring lanes here, so its loads cost an access per lane, and it keeps
// nothing in flight for the next right-hand side.  The multi-RHS tuner times this form beside the others.
// ---------------------------------------------------------------------------
typedef float mf4 __attribute__((ext_vector_type(4)));
typedef short ms4 __attribute__((ext_vector_type(4)));
typedef _Float16 mh4 __attribute__((ext_vector_type(4)));

template <class P>
struct Mfma16;
template <>
struct Mfma16<PBF16> {
    __device__ static uint32_t bits(float f) { return __builtin_bit_cast(uint16_t, (__bf16)f); }
    __device__ static float val(uint32_t b) { return bf_bits2f(b & 0xffffu); }
    __device__ static mf4 mma(ms4 a, ms4 b, mf4 c) { return __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(a, b, c, 0, 0, 0); }
};
template <>
struct Mfma16<PF16> {
    __device__ static uint32_t bits(float f) { return __builtin_bit_cast(uint16_t, (_Float16)f); }
    __device__ static float val(uint32_t b) { return (float)__builtin_bit_cast(_Float16, (uint16_t)(b & 0xffffu)); }
    __device__ static mf4 mma(ms4 a, ms4 b, mf4 c)
    {
        return __builtin_amdgcn_mfma_f32_4x4x4f16(__builtin_bit_cast(mh4, a), __builtin_bit_cast(mh4, b), c, 0, 0, 0);
    }
};

__device__ __forceinline__ ms4 ms4_of(uint32_t lo, uint32_t hi) { return __builtin_bit_cast(ms4, make_uint2(lo, hi)); }

// quad permutations of the partner spin: 3 - s (x, y) and s + 2 mod 4 (z, t)
template <int CTRL>
__device__ __forceinline__ uint32_t quad_dpp(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, CTRL, 0xf, 0xf, true);
}

template <class P, int EPI, int RED>
__global__ __launch_bounds__(256) void hop_mrhs_mfma_kernel(HopArgs a, const Scal* S)
{
    static_assert(QCDW_SPINOR_SOA == 0, "the matrix-core form reads a spin's three colours as one run");
    if (all_finished(S, a.nrhs)) return;
    __shared__ MrhsSums sums;
    constexpr int NSUM = RED == RED_WDOT ? 2 : 3;
    using M = Mfma16<P>;
    constexpr uint32_t SGN = 0x80008000u;
    const Geom g = a.g;
    const int tile = xcd_tile(blockIdx.x, gridDim.x);
    const int nblk = gridDim.x;
    const int q = threadIdx.x & 3;
    int site;
    bool valid;
    if (a.cgroup > 0) {
        const int St = g.Lxh * g.Ly * g.Lz;
        int t;
        const int c = group_ctile(g, tile, a.cgroup, t) * HOP_SITES_PER_BLOCK + (threadIdx.x >> 2);
        site = t * St + c;
        valid = c < St;
    } else {
        site = tile * HOP_SITES_PER_BLOCK + (threadIdx.x >> 2);
        valid = site < g.Vh;
    }
    const long Vh = g.Vh;
    const long field = 12L * Vh;

    // the eight hops of the site: group G = 0 (x, y) and 1 (z, t), hop h = 2 j + dir (mu = 2 G + j);
    // nb: the lane's spin of each neighbour (complex offset within one right-hand side)
    int nb[8];
    ms4 Ar[8], Ai[8];
#pragma unroll
    for (int G = 0; G < 2; G++) {
        LaneHops<float, 6> L;
        L.lstr = 1;
#pragma unroll
        for (int h = 0; h < 4; h++) {
            L.nbh[h] = 0;
            L.loff[h] = 0;
            L.fsg[h] = 1.f;
        }
        if (valid) lane_hops<float, 6, link_soa_for(P::cbytes)>(g, site, a.parity, 2 * G, L);
#pragma unroll
        for (int h = 0; h < 4; h++) {
            nb[4 * G + h] = (int)sp_idx(q, L.nbh[h], 0, Vh);  // site 0 when invalid: read, results dropped
            cx<float> u[9];
#pragma unroll
            for (int e = 0; e < 6; e++) u[e] = P::ld(a.gauge, L.loff[h] + e * L.lstr);
            u[6] = conj(u[1] * u[5] - u[2] * u[4]);
            u[7] = conj(u[2] * u[3] - u[0] * u[5]);
            u[8] = conj(u[0] * u[4] - u[1] * u[3]);
            // row q of W = U (forward) or U^+ (backward), times the time-boundary sign; the spatial weight
            // is applied to the accumulated sum
            const float sg = (G == 1 && (h >> 1) == 1) ? L.fsg[h] : 1.f;
            uint32_t wr[3], wi[3];
#pragma unroll
            for (int k = 0; k < 3; k++) {
                // entries selected as scalars (a select of whole structs would select their addresses and
                // keep u in scratch memory)
                const int e0 = (h & 1) == 0 ? k : 3 * k, e1 = (h & 1) == 0 ? 3 + k : 3 * k + 1,
                          e2 = (h & 1) == 0 ? 6 + k : 3 * k + 2;
                const float re = q == 0 ? u[e0].re : q == 1 ? u[e1].re : u[e2].re;
                const float im = q == 0 ? u[e0].im : q == 1 ? u[e1].im : u[e2].im;
                wr[k] = q == 3 ? 0u : M::bits(sg * re);
                wi[k] = q == 3 ? 0u : M::bits((h & 1) == 0 ? sg * im : -sg * im);
            }
            Ar[4 * G + h] = ms4_of(wr[0] | (wr[1] << 16), wr[2]);
            Ai[4 * G + h] = ms4_of(wi[0] | (wi[1] << 16), wi[2]);
        }
    }
    float win[27];
#pragma unroll
    for (int e = 0; e < 27; e++) win[e] = 0.f;
    if (valid) load_window<P>(a.clov, Vh, site, q, win);

    // sign bits of e_j psi_perm(j) per direction (forward hop; the backward hop has the opposite sign):
    // x: e = -i, -i, +i, +i;  y: +1, -1, -1, +1;  z: -i, +i, +i, -i;  t: -1 for every spin
    const uint32_t sx = q < 2 ? SGN : 0u;                // sigma = -1 where e = -i (x)
    const uint32_t sy = (q == 1 || q == 2) ? SGN : 0u;  // sigma = -1 where e = -1 (y)
    const uint32_t sz = (q == 0 || q == 3) ? SGN : 0u;  // sigma = -1 where e = -i (z)
    const float xs = (float)g.xs;
    const uint32_t* psi = reinterpret_cast<const uint32_t*>(a.psi);

    // the lane's spin of the eight neighbours of right-hand side r (three colours, re/im interleaved)
    auto fetch = [&](int r, uint32_t (&d)[8][3]) {
        const uint32_t* base = psi + (long)r * field;
#pragma unroll
        for (int k = 0; k < 8; k++) {
            const uint32_t* pp = base + nb[k];
            d[k][0] = pp[0];
            d[k][1] = pp[1];
            d[k][2] = pp[2];
        }
    };
    auto next_rhs = [&](int r) {  // uniform: every thread reads the same flags
        while (r < a.nrhs && S && S[r].flags) r++;
        return r;
    };
    auto compute = [&](int r, const uint32_t (&d)[8][3]) {
        const long off = (long)r * field;
        mf4 dr = {0.f, 0.f, 0.f, 0.f}, di = dr;
        // spatial directions first (x, y, then z), the sum scaled by the spatial weight, then t
#pragma unroll
        for (int k = 0; k < 8; k++) {
            const int G = k >> 2, h = k & 3;
            if (k == 6) {
                dr *= xs;
                di *= xs;
            }
            const uint32_t d0 = d[k][0], d1 = d[k][1], d2 = d[k][2];
            // own spin: re and im planes of the three colours
            const uint32_t br0 = __builtin_amdgcn_perm(d1, d0, 0x05040100u), br1 = d2 & 0xffffu;
            const uint32_t bi0 = __builtin_amdgcn_perm(d1, d0, 0x07060302u), bi1 = d2 >> 16;
            // partner spin from the quad
            uint32_t pr0, pr1, pi0, pi1;
            if (G == 0) {
                pr0 = quad_dpp<0x1b>(br0);
                pr1 = quad_dpp<0x1b>(br1);
                pi0 = quad_dpp<0x1b>(bi0);
                pi1 = quad_dpp<0x1b>(bi1);
            } else {
                pr0 = quad_dpp<0x4e>(br0);
                pr1 = quad_dpp<0x4e>(br1);
                pi0 = quad_dpp<0x4e>(bi0);
                pi1 = quad_dpp<0x4e>(bi1);
            }
            const uint32_t flip = (h & 1) ? SGN : 0u;  // backward hop: -e
            ms4 b2r, b2i;
            if ((h >> 1) == 0) {  // x or z: e = i sigma, e psi = (-sigma psi_i, sigma psi_r)
                const uint32_t m = (G == 0 ? sx : sz) ^ flip;
                b2r = ms4_of(pi0 ^ m ^ SGN, pi1 ^ ((m ^ SGN) & 0xffffu));
                b2i = ms4_of(pr0 ^ m, pr1 ^ (m & 0xffffu));
            } else {  // y or t: e = sigma
                const uint32_t m = (G == 0 ? sy : SGN) ^ flip;
                b2r = ms4_of(pr0 ^ m, pr1 ^ (m & 0xffffu));
                b2i = ms4_of(pi0 ^ m, pi1 ^ (m & 0xffffu));
            }
            const ms4 b1r = ms4_of(br0, br1), b1i = ms4_of(bi0, bi1);
            const uint2 ai = __builtin_bit_cast(uint2, Ai[k]);
            const ms4 nai = ms4_of(ai.x ^ SGN, ai.y ^ SGN);
            dr = M::mma(Ar[k], b1r, dr);
            dr = M::mma(nai, b1i, dr);
            di = M::mma(Ar[k], b1i, di);
            di = M::mma(Ai[k], b1r, di);
            dr = M::mma(Ar[k], b2r, dr);
            dr = M::mma(nai, b2i, dr);
            di = M::mma(Ar[k], b2i, di);
            di = M::mma(Ai[k], b2r, di);
        }
        cx<float> res[3];
#pragma unroll
        for (int c = 0; c < 3; c++) res[c] = {dr[c], di[c]};
        cx<float> outv[3], yv[3];
        if constexpr (EPI == EPI_CLOV_XPAY || RED == RED_TS) {
#pragma unroll
            for (int c = 0; c < 3; c++) yv[c] = valid ? P::ld(a.y, off + sp_idx(q, site, c, Vh)) : cx<float>{0.f, 0.f};
        }
        cx<float> ox[3], br[3];
#pragma unroll
        for (int c = 0; c < 3; c++) ox[c] = quad_dpp_cx<QUAD_XOR1>(res[c]);
        herm_rows<true>(win, q & 1, res, ox, br);
        const float aa = (float)a.a;
#pragma unroll
        for (int c = 0; c < 3; c++) outv[c] = (EPI == EPI_CLOV) ? br[c] : yv[c] - aa * br[c];
#pragma unroll
        for (int c = 0; c < 3; c++) outv[c] = P::rt(outv[c]);
        if (valid) {
#pragma unroll
            for (int c = 0; c < 3; c++) P::st(a.out, off + sp_idx(q, site, c, Vh), outv[c]);
        }
        if constexpr (RED != RED_NONE) {
            double v[3] = {0.0, 0.0, 0.0};
            if (valid) {
#pragma unroll
                for (int c = 0; c < 3; c++) {
                    const cx<float> o = outv[c];
                    if constexpr (RED == RED_WDOT) {
                        const cx<float> wv = P::ld(a.w, off + sp_idx(q, site, c, Vh));
                        v[0] += (double)wv.re * o.re + (double)wv.im * o.im;
                        v[1] += (double)wv.re * o.im - (double)wv.im * o.re;
                    } else {
                        v[0] += (double)o.re * yv[c].re + (double)o.im * yv[c].im;
                        v[1] += (double)o.re * yv[c].im - (double)o.im * yv[c].re;
                        v[2] += (double)o.re * o.re + (double)o.im * o.im;
                    }
                }
            }
            mrhs_sum_wave(sums, r, v, NSUM);
        }
    };

    // right-hand sides in a register double buffer: the neighbours of the next active RHS are in flight
    // while the current one is computed
    // (a register double buffer that fetches the next RHS during the current one was measured slower: the
    // extra 24 VGPRs cost a wave per SIMD)
    uint32_t da[8][3];
    for (int r = next_rhs(0); r < a.nrhs; r = next_rhs(r + 1)) {
        fetch(r, da);
        compute(r, da);
    }
    if constexpr (RED != RED_NONE) mrhs_sum_store(sums, S, a.nrhs, NSUM, a.partials, tile, nblk);
}

template <class P>
static hipError_t launch_mrhs_mfma_p(hipStream_t s, int epi, int red, const HopArgs& a, const Scal* S, hipEvent_t e0,
                                     hipEvent_t e1)
{
    dim3 grid(a.cgroup > 0 ? hop_ctiles(a.g) * a.g.Lt : hop_blocks(a.g.Vh)), block(256);
#define QCDW_MRHS_CASE(E, D)                                                                          \
    if (epi == E && red == D) {                                                                      \
        if (e0)                                                                                      \
            hipExtLaunchKernelGGL((hop_mrhs_mfma_kernel<P, E, D>), grid, block, 0, s, e0, e1, 0, a, S); \
        else                                                                                         \
            hipLaunchKernelGGL((hop_mrhs_mfma_kernel<P, E, D>), grid, block, 0, s, a, S);             \
        return hipGetLastError();                                                                    \
    }
    QCDW_MRHS_CASE(EPI_CLOV, RED_NONE)
    QCDW_MRHS_CASE(EPI_CLOV_XPAY, RED_NONE)
    QCDW_MRHS_CASE(EPI_CLOV_XPAY, RED_WDOT)
    QCDW_MRHS_CASE(EPI_CLOV_XPAY, RED_TS)
#undef QCDW_MRHS_CASE
    return hipErrorInvalidValue;
}

hipError_t launch_hop_mrhs_mfma(hipStream_t s, int prec, int epi, int red, const HopArgs& a, const Scal* S,
                                hipEvent_t e0, hipEvent_t e1)
{
    if (a.g.Vh <= 0 || a.nrhs <= 0) return hipSuccess;
    if (a.nrhs > MRHS_MAX || 12L * a.g.Vh > 0x7fffffffL) return hipErrorInvalidValue;  // 32-bit neighbour offsets
    switch (prec) {
    case BF16: return launch_mrhs_mfma_p<PBF16>(s, epi, red, a, S, e0, e1);
    case F16: return launch_mrhs_mfma_p<PF16>(s, epi, red, a, S, e0, e1);
    }
    return hipErrorInvalidValue;  // FP64 and FP32 storage use the vector forms
}

}  // namespace qcdw
