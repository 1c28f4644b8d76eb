// The full Wilson-clover operator and the parity hop applied directly on the paper's layouts (Sec. II.A,
// FP64), in one kernel: nothing is packed, converted or kept.
//
//   M psi = A psi - kappa H psi,  A = 1 - kappa csw C,
//   (H psi)(x) = sum_mu (1 - g_mu) U_mu(x) psi(x+mu) + (1 + g_mu) U_mu(x-mu)^+ psi(x-mu)   (Sec. III.B)
//
// A caller that applies the operator a few times to one gauge field (standalone calls, residual checks) hands
// over links, clover and spinor as they are, so the work is one pass over 1536 B per site; packing them first
// moved 5.6 kB per site and needed 3 kB per site of workspace.
//
// Work split: that of the packed hop (hop_common.h), four lanes per site, lane q = 2 gq + k with row k of the
// projections of directions 2 gq and 2 gq + 1, so a site's four lanes share its loads and 4 V threads hide the
// latency.  A block takes 64 sites of one parity; the blocks of the two parities of a tile run next to each
// other, so that a link read as the forward link of one is still in the XCD's L2 as the backward link of the
// other, and large slices of whole tiles are swept along t group by group (grouped_order).
//
// Measured, one call with its synchronisation: 24^3x64 390 us = 3.5 TB/s of the 1536 B per site (a device copy of
// this part reaches 5.2 TB/s), 16^3x32 59 us, 4^4 18 us.  The pack-then-hop form took 1.6 ms of kernels at
// 24^3x64, and 50 ms with the allocation and release of its workspace.  What bounds it is the vector-memory
// address path: the paper's records (144 B links, 192 B spinors) put the lanes of a load on as many cache lines
// as there are sites, so the two lanes that need a link share its load (load_link_shared: 490 -> 437 us).  Four
// waves per SIMD (124 VGPRs instead of 134) were slower, 449 against 400 us.
#include "host.h"
#include "hop_common.h"

namespace qcdw {

namespace {

// lane h = q & 1 of a chirality block: its 27-entry window (herm_rows) of A = 1 - kc C read from the paper
// packing [d0..d5 | L10 L20 L21 L30..L32 L40..L43 L50..L54].  Each lane reads 18 contiguous reals, forms A and
// exchanges what the other one needs by DPP (half 0: L40..L42, L50..L52; half 1: d3..d5, L30..L32).
__device__ __forceinline__ void load_window_paper(const double* blk, int h, double kc, bool valid, double (&win)[27])
{
    double own[18];
#pragma unroll
    for (int e = 0; e < 18; e++) own[e] = 0.0;
    if (valid) {
#pragma unroll
        for (int e = 0; e < 18; e++) own[e] = ((h == 0 && e < 6) ? 1.0 : 0.0) - kc * blk[18 * h + e];
    }
    double rcv[12];
#pragma unroll
    for (int j = 0; j < 12; j++) {
        const double s0 = j < 3 ? own[3 + j] : (j < 9 ? own[9 + j] : 0.0);
        const double s1 = j < 6 ? own[j] : own[2 + j];
        rcv[j] = quad_dpp<QUAD_XOR1>(h ? s1 : s0);
    }
#pragma unroll
    for (int e = 0; e < 27; e++) {
        const double w0 = e < 3 ? own[e] : (e < 15 ? own[e + 3] : rcv[e - 15]);
        const double w1 = e < 6    ? rcv[3 + e]     // L30 L31 L32
                          : e < 12 ? own[e - 6]     // L40 L41 L42
                          : e < 18 ? own[e - 4]     // L50 L51 L52
                          : e < 21 ? rcv[e - 18]    // d3 d4 d5
                          : e < 23 ? own[e - 15]    // L43
                                   : own[e - 9];    // L53 L54
        win[e] = h ? w1 : w0;
    }
}

// The link that lanes k = 0 and 1 of a direction pair both use: lane k loads entries 4 k .. 4 k + 4 and takes the
// other four from its partner by DPP.  Both lanes are active (they belong to one site).  Entries are selected
// as scalars: a select of whole structs selects addresses and moves them to memory.
__device__ __forceinline__ void load_link_shared(const double2* link, int k, cx<double> (&u)[9])
{
    const auto sel = [&](cx<double> a, cx<double> b) { return cx<double>{k ? a.re : b.re, k ? a.im : b.im}; };
    cx<double> own[5];
#pragma unroll
    for (int e = 0; e < 5; e++) own[e] = P64::ld(link, 4 * k + e);
#pragma unroll
    for (int e = 0; e < 4; e++) {
        const cx<double> rc = quad_dpp_cx<QUAD_XOR1>(sel(own[1 + e], own[e]));
        u[e] = sel(rc, own[e]);
        u[5 + e] = sel(own[1 + e], rc);
    }
    u[4] = sel(own[0], own[4]);
}

}  // namespace

// CLOV: out = A psi - kappa H psi on both parities.  Else out = H psi on the sites of parity hop_p and zero on
// the others.  out overlaps no input (the host sees to it).
template <bool CLOV>
__global__ __launch_bounds__(256) void k_dslash_paper(Geom g, const double2* __restrict__ U,
                                                      const double* __restrict__ clover,
                                                      const double2* __restrict__ psi, double2* __restrict__ out,
                                                      double kappa, double kc, int hop_p, int G)
{
    const int b = xcd_tile(blockIdx.x, gridDim.x);
    const int p = b & 1, site = grouped_tile(g, b >> 1, G) * HOP_SITES_PER_BLOCK + (threadIdx.x >> 2);
    const long Vh = g.Vh;
    const int q = threadIdx.x & 3, gq = q >> 1, k = q & 1;
    const bool valid = site < g.Vh;
    double2* o = out + ((long)p * Vh + site) * 12 + 3 * q;
    if (!CLOV && p != hop_p) {
        if (valid) {
#pragma unroll
            for (int c = 0; c < 3; c++) o[c] = make_double2(0.0, 0.0);
        }
        return;
    }
    const int su = k, sl = gq == 0 ? 3 - k : 2 + k;
    const double2* other = psi + (long)(1 - p) * Vh * 12;
    cx<double> acc_u[3], acc_l[3];
#pragma unroll
    for (int c = 0; c < 3; c++) acc_u[c] = acc_l[c] = {0.0, 0.0};
    if (valid) {
        LaneHops<double, 9> L;
        lane_hops<double, 9, false>(g, site, p, q, L);  // link-major R = 9: the paper's gauge layout
#pragma unroll
        for (int h = 0; h < 4; h++) {
            cx<double> pu[3], pl[3], hv[3];
            const double2* n = other + (long)L.nbh[h] * 12;
#pragma unroll
            for (int c = 0; c < 3; c++) {
                pu[c] = P64::ld(n, 3 * su + c);
                pl[c] = P64::ld(n, 3 * sl + c);
            }
            project<true>(pu, pl, L.cs[h], h < 2, hv);
            cx<double> u[9];
            load_link_shared(U + L.loff[h], k, u);
            hop_rows<true>(u, h & 1, h < 2, L.fsg[h], L.cs[h], hv, acc_u, acc_l);
        }
    }
    cx<double> res[3];
#pragma unroll
    for (int c = 0; c < 3; c++) {  // lane q finishes spin q (partner lane: q < 2 ? q + 2 : 3 - q)
        const cx<double> mine = gq == 0 ? acc_u[c] : acc_l[c];
        const cx<double> theirs = gq == 0 ? acc_l[c] : acc_u[c];
        res[c] = mine + quad_dpp_cx<QUAD_PARTNER>(theirs);
    }
    if constexpr (CLOV) {
        cx<double> y[3], ox[3], by[3];
        double win[27];
        const long e = (long)p * Vh + site;
#pragma unroll
        for (int c = 0; c < 3; c++) y[c] = valid ? P64::ld(psi, e * 12 + 3 * q + c) : cx<double>{0.0, 0.0};
        load_window_paper(clover + (2 * e + gq) * 36, k, kc, valid, win);
#pragma unroll
        for (int c = 0; c < 3; c++) ox[c] = quad_dpp_cx<QUAD_XOR1>(y[c]);
        herm_rows<true>(win, k, y, ox, by);
#pragma unroll
        for (int c = 0; c < 3; c++) res[c] = by[c] - kappa * res[c];
    }
    if (valid) {
#pragma unroll
        for (int c = 0; c < 3; c++) o[c] = make_double2(res[c].re, res[c].im);
    }
}

hipError_t launch_dslash_paper(hipStream_t s, const Geom& g, const void* U, const void* clover, const void* psi,
                               void* out, double kappa, double csw)
{
    // Groups in tile order: 24^3x64 takes 27 of 108 tiles (groups of 12, 18, 36, 54: 421, 416, 412, 404 against 400 us)
    hipLaunchKernelGGL(k_dslash_paper<true>, dim3(2 * hop_blocks(g.Vh)), dim3(256), 0, s, g, (const double2*)U,
                       (const double*)clover, (const double2*)psi, (double2*)out, kappa, kappa * csw, 0,
                       grouped_order(g));
    return hipGetLastError();
}

hipError_t launch_hop_paper(hipStream_t s, const Geom& g, const void* U, const void* psi, void* out, int parity)
{
    hipLaunchKernelGGL(k_dslash_paper<false>, dim3(2 * hop_blocks(g.Vh)), dim3(256), 0, s, g, (const double2*)U,
                       (const double*)nullptr, (const double2*)psi, (double2*)out, 1.0, 0.0, parity,
                       grouped_order(g));
    return hipGetLastError();
}

}  // namespace qcdw

extern "C" qcdw_status qcdw_hop(qcdw_ctx* ctx, const qcdw_lattice* lat, const void* U, const void* psi, void* out,
                                int out_parity)
{
    if (!ctx) return QCDW_EINVAL;
    DeviceGuard dg(ctx->device);
    Geom g;
    CHK(check_lattice(ctx, lat, g));
    CHK(check_dev(ctx, U, "U"));
    CHK(check_dev(ctx, psi, "psi"));
    CHK(check_dev(ctx, out, "out"));
    if (out_parity != 0 && out_parity != 1) return fail(ctx, QCDW_EINVAL, "out_parity must be 0 or 1");
    if (psi == out) return fail(ctx, QCDW_EINVAL, "out must not alias psi");
    CallScratch scratch(ctx->stream);
    OperatorInputs in{U, nullptr, psi};
    CHK(detach(ctx, g, in, out, scratch));
    HIPCHK(ctx, launch_hop_paper(ctx->stream, g, in.U, in.psi, out, out_parity));
    HIPCHK(ctx, hipStreamSynchronize(ctx->stream));
    return QCDW_OK;
}

extern "C" qcdw_status qcdw_dslash(qcdw_ctx* ctx, const qcdw_lattice* lat, const void* U, const void* clover,
                                   const void* psi, void* out, double kappa, double csw)
{
    if (!ctx) return QCDW_EINVAL;
    DeviceGuard dg(ctx->device);
    Geom g;
    CHK(check_lattice(ctx, lat, g));
    CHK(check_dev(ctx, U, "U"));
    if (clover) CHK(check_dev(ctx, clover, "clover"));
    CHK(check_dev(ctx, psi, "psi"));
    CHK(check_dev(ctx, out, "out"));
    if (psi == out) return fail(ctx, QCDW_EINVAL, "out must not alias psi");
    CallScratch scratch(ctx->stream);
    OperatorInputs in{U, clover, psi};
    CHK(detach(ctx, g, in, out, scratch));
    if (!clover) {
        void* c = scratch(144UL * g.Vh * 8);
        if (!c) return fail(ctx, QCDW_ENOMEM, "out of device memory for the clover field");
        HIPCHK(ctx, clover_from_paper(ctx->stream, g, in.U, c, scratch(8UL * g.Vh * 9 * 16)));
        in.clover = c;
    }
    HIPCHK(ctx, launch_dslash_paper(ctx->stream, g, in.U, in.clover, in.psi, out, kappa, csw));
    HIPCHK(ctx, hipStreamSynchronize(ctx->stream));
    return QCDW_OK;
}
