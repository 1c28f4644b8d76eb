// Block Gram-Schmidt kernels for flexible GMRES (Saad 1993): several dot
// products against one vector in a single pass, and a combined update
// w += sign * sum_i c_i V_i.  Vectors are FP64 complex; V_i = V + i * stride.
// Reductions use a fixed order, so results are bitwise reproducible.
#include "internal.h"

namespace qcdw {

constexpr int MDOT_GROUP = 8;  // vectors per pass

// partials[(group * nb + block) * 16 + 2 j + {0,1}] = partial sum of conj(V_{8 group + j}) w
__global__ __launch_bounds__(256) void k_multidot(const double2* V, long stride, int nvec, const double2* w, long n,
                                                  double* partials)
{
    const int i0 = blockIdx.y * MDOT_GROUP;
    const int cnt = min(MDOT_GROUP, nvec - i0);
    double acc[2 * MDOT_GROUP];
#pragma unroll
    for (int j = 0; j < 2 * MDOT_GROUP; j++) acc[j] = 0.0;
    for (long e = (long)blockIdx.x * 256 + threadIdx.x; e < n; e += (long)gridDim.x * 256) {
        const double2 we = w[e];
#pragma unroll
        for (int j = 0; j < MDOT_GROUP; j++) {
            if (j < cnt) {
                const double2 v = V[(long)(i0 + j) * stride + e];
                acc[2 * j] += v.x * we.x + v.y * we.y;
                acc[2 * j + 1] += v.x * we.y - v.y * we.x;
            }
        }
    }
    block_sum_store<2 * MDOT_GROUP>(acc, partials + ((long)blockIdx.y * gridDim.x + blockIdx.x) * 2 * MDOT_GROUP);
}

// out[2 i + {0,1}] = sum over blocks, i < nvec
__global__ __launch_bounds__(256) void k_multidot_sum(const double* partials, int nb, int nvec, double* out)
{
    const int e = blockIdx.x;  // 0 .. 2*8-1 within the group
    const int group = blockIdx.y;
    const int i = group * MDOT_GROUP + e / 2;
    double v[1] = {0.0};
    for (int b = threadIdx.x; b < nb; b += 256) v[0] += partials[((long)group * nb + b) * 2 * MDOT_GROUP + e];
    __shared__ double res[1];
    block_sum_store<1>(v, res);
    __syncthreads();
    if (threadIdx.x == 0 && i < nvec) out[2 * i + (e & 1)] = res[0];
}

// The step between the two orthogonalisations in one pass over V: w -= sum_i c_i V_i, then the dots of the new w.
// A block takes 64 elements at a time; wave k holds those of vectors 8 k .. 8 k + 7 in registers, the waves add their
// shares of the sum in LDS, and each forms its own vectors' dots.  Bound by the reads of V: at 16^3x32 (12.6 MB a
// vector, 17 on average over a 33-iteration solve) 46 us = 4.7 TB/s, where the update and the dots took 38 + 41 us.
__global__ __launch_bounds__(512) void k_multiaxpy_dot(const double2* V, long stride, int nvec, const double* c,
                                                       double2* w, long n, double* partials)
{
    __shared__ double2 share[8][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, waves = blockDim.x >> 6;
    const int i0 = wave * MDOT_GROUP, cnt = min(MDOT_GROUP, nvec - i0);
    double acc[2 * MDOT_GROUP];
#pragma unroll
    for (int j = 0; j < 2 * MDOT_GROUP; j++) acc[j] = 0.0;
    for (long e0 = (long)blockIdx.x * 64; e0 < n; e0 += (long)gridDim.x * 64) {
        const long e = e0 + lane;
        const bool valid = e < n;
        double2 v[MDOT_GROUP], s = make_double2(0.0, 0.0), we = s;
        if (valid) we = w[e];
#pragma unroll
        for (int j = 0; j < MDOT_GROUP; j++)
            v[j] = valid && j < cnt ? V[(long)(i0 + j) * stride + e] : make_double2(0.0, 0.0);
#pragma unroll
        for (int j = 0; j < MDOT_GROUP; j++) {
            if (j >= cnt) continue;
            const double cr = c[2 * (i0 + j)], ci = c[2 * (i0 + j) + 1];
            s.x += cr * v[j].x - ci * v[j].y;
            s.y += cr * v[j].y + ci * v[j].x;
        }
        __syncthreads();  // the last tile's shares have been read
        share[wave][lane] = s;
        __syncthreads();
        for (int k = 0; k < waves; k++) {
            we.x -= share[k][lane].x;
            we.y -= share[k][lane].y;
        }
        if (valid && wave == 0) w[e] = we;
#pragma unroll
        for (int j = 0; j < MDOT_GROUP; j++) {
            acc[2 * j] += v[j].x * we.x + v[j].y * we.y;
            acc[2 * j + 1] += v[j].x * we.y - v[j].y * we.x;
        }
    }
#pragma unroll
    for (int j = 0; j < 2 * MDOT_GROUP; j++) {
        const double t = wave_sum(acc[j]);
        if (lane == 0) partials[((long)wave * gridDim.x + blockIdx.x) * 2 * MDOT_GROUP + j] = t;
    }
}

// w += sign * sum_i c_i V_i; partials (unless null): the blocks' sums of |w|^2
__global__ __launch_bounds__(256) void k_multiaxpy(const double2* V, long stride, int nvec, const double* c,
                                                   double2* w, long n, double sign, double* partials)
{
    double nrm[1] = {0.0};
    for (long e = (long)blockIdx.x * 256 + threadIdx.x; e < n; e += (long)gridDim.x * 256) {
        double2 acc = w[e];
        for (int i = 0; i < nvec; i++) {
            const double2 v = V[(long)i * stride + e];
            const double cr = sign * c[2 * i], ci = sign * c[2 * i + 1];
            acc.x += cr * v.x - ci * v.y;
            acc.y += cr * v.y + ci * v.x;
        }
        w[e] = acc;
        nrm[0] += acc.x * acc.x + acc.y * acc.y;
    }
    if (partials) block_sum_store<1>(nrm, partials + blockIdx.x);
}

// out = w / sqrt(*nrm2) (out = 0 if the norm is zero)
__global__ __launch_bounds__(256) void k_scale_inv_norm(const double2* w, double2* out, long n, const double* nrm2)
{
    const double q = *nrm2;
    const double sc = q > 0.0 ? 1.0 / sqrt(q) : 0.0;
    for (long e = (long)blockIdx.x * 256 + threadIdx.x; e < n; e += (long)gridDim.x * 256) {
        const double2 v = w[e];
        out[e] = make_double2(sc * v.x, sc * v.y);
    }
}

hipError_t launch_scale_inv_norm(hipStream_t s, const void* w, void* out, long n, const double* nrm2)
{
    hipLaunchKernelGGL(k_scale_inv_norm, dim3(blas_blocks(n)), dim3(256), 0, s, (const double2*)w, (double2*)out, n,
                       nrm2);
    return hipGetLastError();
}

hipError_t launch_multidot(hipStream_t s, const void* V, long stride, int nvec, const void* w, long n,
                           double* partials, double* out)
{
    if (nvec <= 0) return hipSuccess;
    const int ng = (nvec + MDOT_GROUP - 1) / MDOT_GROUP;
    const int nb = blas_blocks(n);
    hipLaunchKernelGGL(k_multidot, dim3(nb, ng), dim3(256), 0, s, (const double2*)V, stride, nvec, (const double2*)w,
                       n, partials);
    hipLaunchKernelGGL(k_multidot_sum, dim3(2 * MDOT_GROUP, ng), dim3(256), 0, s, partials, nb, nvec, out);
    return hipGetLastError();
}

hipError_t launch_multiaxpy_dot(hipStream_t s, const void* V, long stride, int nvec, const double* c, void* w, long n,
                                double* partials, double* out)
{
    if (nvec <= 0 || nvec > 8 * MDOT_GROUP) return hipErrorInvalidValue;
    const int ng = (nvec + MDOT_GROUP - 1) / MDOT_GROUP;
    const int nb = multiaxpy_dot_blocks(n);
    hipLaunchKernelGGL(k_multiaxpy_dot, dim3(nb), dim3(64 * ng), 0, s, (const double2*)V, stride, nvec, c, (double2*)w,
                       n, partials);
    hipLaunchKernelGGL(k_multidot_sum, dim3(2 * MDOT_GROUP, ng), dim3(256), 0, s, partials, nb, nvec, out);
    return hipGetLastError();
}

hipError_t launch_multiaxpy(hipStream_t s, const void* V, long stride, int nvec, const double* c, void* w, long n,
                            double sign, double* partials, double* nrm2)
{
    if (nvec <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_multiaxpy, dim3(blas_blocks(n)), dim3(256), 0, s, (const double2*)V, stride, nvec, c,
                       (double2*)w, n, sign, partials);
    if (partials) return launch_sum_partials(s, partials, blas_blocks(n), nrm2);
    return hipGetLastError();
}

}  // namespace qcdw
