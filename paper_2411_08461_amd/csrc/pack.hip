// Conversion between the paper's field layouts (Sec. II.A, FP64) and the
// library's internal site-major layouts, with optional down-conversion to
// FP32 / BF16 / FP16 storage (round to nearest even) and a scale factor.
#include "internal.h"

namespace qcdw {

// spinor: paper [2][Vh][4][3] complex f64  <->  internal spinor (sp_idx order) complex P
template <class P>
__global__ void k_pack_spinor(const double2* __restrict__ paper, void* out, int Vh, int parity, double scale)
{
    const long e = (long)blockIdx.x * blockDim.x + threadIdx.x;  // internal element
    if (e >= 12L * Vh) return;
    long s, site;
    int c;
    sp_coords(e, Vh, s, site, c);
    const double2 v = paper[((long)parity * Vh + site) * 12 + s * 3 + c];
    using T = typename P::real;
    P::st(out, e, cx<T>{(T)(scale * v.x), (T)(scale * v.y)});
}

template <class P>
__global__ void k_unpack_spinor(const void* in, double2* __restrict__ paper, int Vh, int parity, double scale)
{
    const long e = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= 12L * Vh) return;
    long s, site;
    int c;
    sp_coords(e, Vh, s, site, c);
    const auto v = P::ld(in, e);
    paper[((long)parity * Vh + site) * 12 + s * 3 + c] = make_double2(scale * (double)v.re, scale * (double)v.im);
}

// Links: paper [4][2][Vh][3][3] into everything that is kept of them, in one pass.  A block stages 256 links of
// one direction and parity in LDS (36 kB, whole runs in), then writes
//   top: entries 0 .. R-1 plane-major in FP64 ([mu][p][R][Vh], the FP64 hop's layout), or nothing (nullptr);
//   low: entries 6 .. 8 plane-major ([mu][p][3][Vh]; for the clover build when R = 6), or nothing;
//   lo:  the inner precision's RL entries at link_base, or nothing.
// At 16^3x32 with FP64 and BF16 links 36 us = 4.5 TB/s; a pass over the paper's field for each output took 45 us
// and left out the third rows.
template <int R, class PL, int RL>
__global__ __launch_bounds__(256) void k_pack_links(const double2* __restrict__ paper, double2* __restrict__ top,
                                                    double2* __restrict__ low, void* lo, int Vh)
{
    __shared__ double2 u[256 * 9];
    const int mp = blockIdx.y, s0 = blockIdx.x * 256;
    const int n = Vh - s0 < 256 ? Vh - s0 : 256;
    const double2* in = paper + ((long)mp * Vh + s0) * 9;
    for (int e = threadIdx.x; e < n * 9; e += 256) u[e] = in[e];
    __syncthreads();
    if ((int)threadIdx.x < n) {
        const double2* mine = u + threadIdx.x * 9;
        const int site = s0 + threadIdx.x;
        if (top) {
#pragma unroll
            for (int e = 0; e < R; e++) top[((long)mp * R + e) * Vh + site] = mine[e];
        }
        if (low) {
#pragma unroll
            for (int e = 0; e < 3; e++) low[((long)mp * 3 + e) * Vh + site] = mine[6 + e];
        }
    }
    if (lo) {
        using T = typename PL::real;
        constexpr bool soa = link_soa_for(PL::cbytes);
        for (int e = threadIdx.x; e < n * RL; e += 256) {
            const int k = e / RL, j = e - k * RL;
            const double2 v = u[k * 9 + j];
            PL::st(lo, link_base(mp >> 1, mp & 1, s0 + k, Vh, RL, soa) + j * link_stride(Vh, soa),
                   cx<T>{(T)v.x, (T)v.y});
        }
    }
}

static inline dim3 grid_for(long n) { return dim3((unsigned)((n + 255) / 256)); }

hipError_t launch_pack_spinor(hipStream_t s, int prec, const Geom& g, const void* paper, int parity, void* internal,
                              double scale)
{
    const long n = 12L * g.Vh;
    if (n == 0) return hipSuccess;
    const double2* pp = (const double2*)paper;
    switch (prec) {
    case F64: hipLaunchKernelGGL(k_pack_spinor<P64>, grid_for(n), dim3(256), 0, s, pp, internal, g.Vh, parity, scale); break;
    case F32: hipLaunchKernelGGL(k_pack_spinor<P32>, grid_for(n), dim3(256), 0, s, pp, internal, g.Vh, parity, scale); break;
    case BF16: hipLaunchKernelGGL(k_pack_spinor<PBF16>, grid_for(n), dim3(256), 0, s, pp, internal, g.Vh, parity, scale); break;
    case F16: hipLaunchKernelGGL(k_pack_spinor<PF16>, grid_for(n), dim3(256), 0, s, pp, internal, g.Vh, parity, scale); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_unpack_spinor(hipStream_t s, int prec, const Geom& g, const void* internal, int parity, void* paper,
                                double scale)
{
    const long n = 12L * g.Vh;
    if (n == 0) return hipSuccess;
    double2* pp = (double2*)paper;
    switch (prec) {
    case F64: hipLaunchKernelGGL(k_unpack_spinor<P64>, grid_for(n), dim3(256), 0, s, internal, pp, g.Vh, parity, scale); break;
    case F32: hipLaunchKernelGGL(k_unpack_spinor<P32>, grid_for(n), dim3(256), 0, s, internal, pp, g.Vh, parity, scale); break;
    case BF16: hipLaunchKernelGGL(k_unpack_spinor<PBF16>, grid_for(n), dim3(256), 0, s, internal, pp, g.Vh, parity, scale); break;
    case F16: hipLaunchKernelGGL(k_unpack_spinor<PF16>, grid_for(n), dim3(256), 0, s, internal, pp, g.Vh, parity, scale); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_pack_links(hipStream_t s, const Geom& g, const void* paper, int recon, void* top, void* low,
                             int prec_lo, int recon_lo, void* lo)
{
    static_assert(link_soa_for(P64::cbytes), "the FP64 links are written plane-major");
    if (g.Vh == 0) return hipSuccess;
    const dim3 grid((unsigned)((g.Vh + 255) / 256), 8), block(256);
#define QCDW_PACK(R, P, RL)                                                                                  \
    hipLaunchKernelGGL((k_pack_links<R, P, RL>), grid, block, 0, s, (const double2*)paper, (double2*)top,    \
                       (double2*)low, lo, g.Vh)
    if (!lo) {
        if (recon == 18)
            QCDW_PACK(9, P32, 6);
        else
            QCDW_PACK(6, P32, 6);
    } else if (recon_lo == 18) {
        if (prec_lo != F32 || recon != 18) return hipErrorInvalidValue;
        QCDW_PACK(9, P32, 9);
    } else if (recon == 18) {
        switch (prec_lo) {
        case BF16: QCDW_PACK(9, PBF16, 6); break;
        case F16: QCDW_PACK(9, PF16, 6); break;
        default: return hipErrorInvalidValue;
        }
    } else {
        switch (prec_lo) {
        case F32: QCDW_PACK(6, P32, 6); break;
        case BF16: QCDW_PACK(6, PBF16, 6); break;
        case F16: QCDW_PACK(6, PF16, 6); break;
        default: return hipErrorInvalidValue;
        }
    }
#undef QCDW_PACK
    return hipGetLastError();
}

}  // namespace qcdw
