// Host-side internal interfaces of libqcdw: launch descriptors and launcher
// declarations shared between the kernel files and the C-ABI layer.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "dev.h"

namespace qcdw {

struct Scal;  // BiCGStab scalars, below

enum Prec { F64 = 0, F32 = 1, BF16 = 2, F16 = 3 };

inline int cplx_bytes(int prec) { return prec == F64 ? 16 : prec == F32 ? 8 : 4; }
inline int real_bytes(int prec) { return prec == F64 ? 8 : prec == F32 ? 4 : 2; }

// hop epilogues
enum Epi {
    EPI_CLOV = 1,       // out = B (H psi)
    EPI_CLOV_XPAY = 2,  // out = y - a B (H psi)
    EPI_XPAY_CLOVY = 3,  // out = B y - a (H psi)
    // the normal operator's (FP64): M_hat with g5 A^-1 of its result, and the adjoint's last hop
    EPI_CLOV_XPAY_G5CLOV = 4,  // out = y - a B (H psi), out2 = g5 B out
    EPI_XPAY_G5_SHIFT = 5,     // out = y - a g5 (H psi) + shift w
    EPI_CLOV_RESID = 6         // out = w - (y - a C H psi)   (with RED_NORM)
};
// hop fused reductions (per-block partials)
enum Red {
    RED_NONE = 0,
    RED_WDOT = 1,  // (w, out)              -> 2 doubles
    RED_TS = 2,    // (out, y), ||out||^2   -> 3 doubles
    // FP64 residuals:
    RED_NORM = 3,  // ||out||^2             -> 1 double
    RED_DIST = 4   // ||w - out||^2, out is not stored -> 1 double
};

struct HopArgs {
    const void* psi;    // input spinor, parity 1 - parity
    void* out;          // output spinor, parity `parity`
    const void* gauge;  // R entries per link at link_base / link_stride (dev.h)
    const void* clov;   // clover-type matrix of the output parity, [Vh][2][36] reordered
    const void* y;      // xpay / dot operand on the output parity
    const void* w;      // dot operand on the output parity
    double a;           // xpay coefficient
    void* out2;         // second output (EPI_CLOV_XPAY_G5CLOV)
    double shift;       // coefficient of w (EPI_XPAY_G5_SHIFT)
    double* partials;   // [nblocks][3]
    Geom g;
    int parity;
    int nrhs;           // right-hand sides interleaved per site (1 or more)
    const int* active;  // multi-RHS: per-RHS active flag (nullptr: all active)
    const int* stop;    // if non-null and *stop != 0 the launch does nothing
    int nt;             // single-RHS hop: output sites per thread along t (1, 2, 4 or 8; 0 means 1)
    int cgroup;         // single-RHS hop: c-tiles per group swept along t (0: no grouping)
    int fma;            // single-RHS hop: bit 0 the multiply-add form of the hop arithmetic, bit 1 the
                        // t-neighbours staged in LDS (slice groups with one site per thread group only)
};

// one problem of a batched solve (device table entry); reconstruct-12 operators
struct BatchEntry {
    Geom g;
    double kappa, kappa2;  // kappa and kappa^2 of this problem
    const void* a64[2];   // A per parity in FP64
    const void* gauge;    // links in the batch's Krylov precision
    const void* clov[2];  // A^-1 per parity, same precision
    long off;             // element offset (complex) of this problem in the concatenated vectors
    long n;               // 12 Vh
    int tile0;            // first global hop tile of this problem
    int ntiles;           // hop tiles of this problem
};

struct BatchHopArgs {
    const BatchEntry* tab;
    int nprob;
    int total_tiles;
    int parity;
    int nbmax;           // partials stride per problem (tiles)
    int kpow;            // xpay coefficient: 2 kappa^2 of each problem, 1 `a` kappa, 0 `a`
    double a;
    const void* psi;     // concatenated vectors, problem k at element offset tab[k].off
    void* out;
    const void* y;
    const void* w;
    double* partials;    // [problem][nbmax][3]
    const Scal* S;       // per-problem solver scalars (flags) or nullptr
};

constexpr int HOP_SITES_PER_BLOCK = 64;  // 4 lanes per site, 256 threads
__host__ __device__ inline int hop_blocks(int Vh) { return (Vh + HOP_SITES_PER_BLOCK - 1) / HOP_SITES_PER_BLOCK; }
// the t-stepping hop (nt sites per thread along t) needs Lt % (2 nt) == 0
__host__ __device__ inline bool hop_nt_fits(const Geom& g, int nt)
{
    return nt <= 1 || ((nt == 2 || nt == 4 || nt == 8) && g.Lt % (2 * nt) == 0);
}
// tiles of 64 consecutive sites within one t-slice (eo index c in [0, Lxh Ly Lz))
__host__ __device__ inline int hop_ctiles(const Geom& g) { return (g.Lxh * g.Ly * g.Lz + 63) / 64; }
// a c-tile group size is valid if it divides the c-tiles of a slice
__host__ __device__ inline bool hop_cgroup_fits(const Geom& g, int cg)
{
    return cg == 0 || (cg > 0 && hop_ctiles(g) % cg == 0);
}
// Order of the 64-site tiles in kernels that run the two parities of a tile next to each other: 0 the eo order,
// else the tiles of a group of G < tiles of a slice swept along t, so that what slice t shares with t - 1 and t + 1 is
// G tiles apart and still in the XCD's L2.  Only for slices that are whole tiles (padded ones would leave lanes idle),
// and of more than 32 of them: in the eo order neighbours along t are a slice apart, and up to 32 tiles of it stay in
// L2 anyway.  In groups against the eo order: 32^4 (256 tiles, groups of 32) operator 461 and 535 us, clover build 940
// and 1025; 24^3x64 (108, 27) 390 and 410, 768 and 827, force 1607 and 1666; 16x16x18x32 (36, 18) 62 and 64, 137 and
// 141; 16^3x32 (32, groups of 16 to try) 57 and 59, but 153 and 130.
inline int grouped_order(const Geom& g)
{
    const int nct = hop_ctiles(g);
    if (nct <= 32 || (g.Lxh * g.Ly * g.Lz) % 64) return 0;
    for (int d = 32; d >= 4; d--)
        if (nct % d == 0) return d;
    return 0;
}
// place k of a launch whose c-tiles are swept along t in groups of G: slice t and c-tile
__device__ __forceinline__ int group_ctile(const Geom& g, int k, int G, int& t)
{
    const int grp = k / (G * g.Lt), r = k - grp * G * g.Lt;
    t = r / G;
    return grp * G + (r - t * G);
}
// the eo tile of place k in that order
__device__ __forceinline__ int grouped_tile(const Geom& g, int k, int G)
{
    if (G == 0) return k;
    int t;
    const int ct = group_ctile(g, k, G, t);
    return t * hop_ctiles(g) + ct;
}
// blocks (and reduction partials) of one single-RHS hop launch
__host__ __device__ inline int hop_blocks_nt(const Geom& g, int nt, int cg)
{
    if (nt <= 1) return cg > 0 ? hop_ctiles(g) * g.Lt : hop_blocks(g.Vh);
    return hop_ctiles(g) * (g.Lt / nt);
}

// e0/e1: optional events recorded by the kernel dispatch itself (timing)
hipError_t launch_hop(hipStream_t s, int prec, int recon, int epi, int red, const HopArgs& a,
                      hipEvent_t e0 = nullptr, hipEvent_t e1 = nullptr);

// the full operator A psi - kappa H psi, and H psi on one parity (zeros on the other), on the paper's layouts
// (dslash.hip); out must not share memory with an input
hipError_t launch_dslash_paper(hipStream_t s, const Geom& g, const void* U, const void* clover, const void* psi,
                               void* out, double kappa, double csw);
hipError_t launch_hop_paper(hipStream_t s, const Geom& g, const void* U, const void* psi, void* out, int parity);

// BiCGStab scalars kept on the device (complex values as re, im pairs)
hipError_t launch_hop_batch(hipStream_t s, int prec, int epi, int red, const BatchHopArgs& b, int grid,
                            hipEvent_t e0 = nullptr, hipEvent_t e1 = nullptr);

struct Scal {
    double rho[2];    // (r0, r)
    double rho_prev[2];  // rho of the iteration in progress (the beta step's denominator)
    double alpha[2];
    double omega[2];
    double beta[2];
    double rr;        // ||r||^2 of the iterated residual
    double r0n2;      // ||r0||^2 (breakdown thresholds)
    double stop_rr;   // convergence when rr <= stop_rr
    double hist_norm; // history entry = sqrt(rr) * hist_norm
    int iter;         // iterations completed
    int flags;        // FLAG_* below
    int fault_iter;   // > 0: force a breakdown when iter reaches this value; < 0: flag an overflow at -value
    int hist_len;     // capacity of the device history
};
enum { FLAG_CONV = 1, FLAG_BREAK = 2, FLAG_NAN = 4, FLAG_STOP = 8 /* cycle ended by the host */ };

constexpr int BLAS_THREADS = 256;
// number of blocks used by the BLAS reductions on n complex elements
inline int blas_blocks(long n)
{
    long b = (n + BLAS_THREADS * 4 - 1) / (BLAS_THREADS * 4);
    if (b < 1) b = 1;
    if (b > 2048) b = 2048;
    return (int)b;
}

// Vector kernels act on nrhs stacked fields of n complex elements each; RHS y uses
// elements [y n, (y+1) n), scalars S[y] and partials [y][blocks][..].  With a map
// (device array of (offset, length) per vector, problems of different sizes) the
// ranges come from the map and nmax is the longest length.
hipError_t launch_norm2(hipStream_t s, int prec, const void* x, long n, double* partials, double* out, int nrhs = 1,
                        const long2* map = nullptr, long nmax = 0);
// out[k] = sum over b < nbs[k] (nb if nbs is null) of p0[k][b][0], plus the same of p1 unless null; the hops'
// one-double partials, [problem][stride][3]
hipError_t launch_sum_hop_norms(hipStream_t s, const double* p0, const double* p1, int nb, int stride, const int* nbs,
                                double* out, int nprob);
hipError_t launch_xmy_norm2(hipStream_t s, const void* b, const void* y, void* r, long n, double* partials,
                            double* out);  // r = b - y (FP64; r may be null), out = ||r||^2
hipError_t launch_convert(hipStream_t s, int prec_in, int prec_out, const void* in, void* out, long n, double scale);
// y_k += a_k x_k (y FP64, x FP32) for the problems of a solve; coefs: a per problem on the device
hipError_t launch_axpy_hi(hipStream_t s, const double* coefs, const void* x, void* y, long n, int nrhs,
                          const long2* map, long nmax);
hipError_t launch_clov_apply_internal(hipStream_t s, int prec, const Geom& g, const void* clov, const void* in,
                                      void* out);

// BiCGStab iteration pieces
// start of a Krylov cycle from the FP64 residuals rhi: r = scales[y] rhi in precision prec; unless
// resume, r0 = p = r and the scalars S are initialised from ||r||^2 (rho = ||r||^2, flags from
// stop_rr); xlo (FP32 complex, may be nullptr) is cleared.  partials: nrhs x blas_blocks doubles.
hipError_t launch_cycle_start(hipStream_t s, int prec, const void* rhi, void* r, void* r0, void* p, void* xlo, long n,
                              const double* scales, Scal* S, double* partials, int nrhs, const long2* map, long nmax,
                              bool resume);
// rho' = (r0, r), beta from the previous step's scalars, for a cycle that continues the recurrence
hipError_t launch_bicg_resume(hipStream_t s, int prec, const void* r0, const void* r, long n, Scal* S,
                              double* partials, int nrhs, const long2* map, long nmax);
// The BiCGStab vector updates.  Each takes its scalar (beta, alpha, omega) from S, recorded there by
// the matching launch_fin_* kernel, or, with fin != nullptr, forms it itself from the reduction
// partials fin [RHS][fin_nb][3] (fin_nbs: per-RHS counts, or nullptr) and records it in S: one
// launch fewer per scalar.  hist: the residual history of the beta step (fused form only).
hipError_t launch_bicg_p(hipStream_t s, int prec, void* p, const void* r, const void* v, long n, Scal* S,
                         int nrhs = 1, const long2* map = nullptr, long nmax = 0, const double* fin = nullptr,
                         int fin_nb = 0, double* hist = nullptr);
hipError_t launch_bicg_s(hipStream_t s, int prec, void* sv, const void* r, const void* v, long n, Scal* S,
                         int nrhs = 1, const long2* map = nullptr, long nmax = 0, const double* fin = nullptr,
                         int fin_nb = 0, const int* fin_nbs = nullptr);
// partials (its own output) must not overlap fin
hipError_t launch_bicg_xr(hipStream_t s, int prec, int prec_x, void* x, const void* p, const void* sv, void* r,
                          const void* t, const void* r0, long n, Scal* S, double* partials, int nrhs = 1,
                          const long2* map = nullptr, long nmax = 0, const double* fin = nullptr, int fin_nb = 0,
                          const int* fin_nbs = nullptr);
// nb: partials stride per RHS; nbs (optional, per RHS) the count actually written
hipError_t launch_fin_alpha(hipStream_t s, Scal* S, const double* partials, int nb, int nrhs = 1,
                            const int* nbs = nullptr);
hipError_t launch_fin_omega(hipStream_t s, Scal* S, const double* partials, int nb, int nrhs = 1,
                            const int* nbs = nullptr);
hipError_t launch_fin_beta(hipStream_t s, Scal* S, const double* partials, int nb, double* hist, int nrhs = 1);

// multi-RHS hop forms (tuning-cache value of "mrhs_hop/..."): bit 0 set: one block per (tile, RHS), links
// re-read from L2; else the register loop, in slice-group order of (v & 1023) / 2 c-tiles when nonzero, on
// the matrix cores when MRHS_MFMA is set (16-bit storage)
constexpr int MRHS_MFMA = 1024;
// in 16-bit storage the register loop's byte offsets within a right-hand side (12 Vh complex of 4 bytes) are 32-bit
inline bool mrhs_offsets_fit(int prec, long Vh) { return (prec != BF16 && prec != F16) || 48 * Vh <= 1L << 32; }
inline bool mrhs_variant_fits(const Geom& g, int prec, int v)
{
    if (v == 1) return true;
    if ((v & 1) || (v & ~(MRHS_MFMA | 1023))) return false;
    // the matrix-core form keeps its neighbour offsets (complex index within one RHS) in 32 bits
    if ((v & MRHS_MFMA) && ((prec != BF16 && prec != F16) || 12L * g.Vh > 0x7fffffffL)) return false;
    if (!(v & MRHS_MFMA) && !mrhs_offsets_fit(prec, g.Vh)) return false;
    const int cg = (v & 1023) >> 1;
    return cg == 0 || hop_cgroup_fits(g, cg);
}
inline int mrhs_blocks(const Geom& g, int v)
{
    const int cg = (v & 1) ? 0 : (v & 1023) >> 1;
    return cg > 0 ? hop_ctiles(g) * g.Lt : hop_blocks(g.Vh);
}
// multi-RHS hop (reconstruct-12): a.nrhs stacked fields; RHS y skipped when S[y].flags != 0;
// partials [y][hop_blocks][3]
hipError_t launch_hop_mrhs(hipStream_t s, int prec, int epi, int red, const HopArgs& a, const Scal* S,
                           hipEvent_t e0 = nullptr, hipEvent_t e1 = nullptr);
// the same with the link products on the matrix cores (BF16 / FP16 storage only; hipErrorInvalidValue
// otherwise); same grid and partials as launch_hop_mrhs
hipError_t launch_hop_mrhs_mfma(hipStream_t s, int prec, int epi, int red, const HopArgs& a, const Scal* S,
                                hipEvent_t e0 = nullptr, hipEvent_t e1 = nullptr);
// the same operation with one block per (tile, rhs), rhs fastest (links and clover re-read from L2)
hipError_t launch_hop_rhs(hipStream_t s, int prec, int epi, int red, const HopArgs& a, const Scal* S,
                          hipEvent_t e0 = nullptr, hipEvent_t e1 = nullptr);
// the FP64 hop of source preparation and residuals, several RHS per thread group (either reconstruction; EPI_CLOV, EPI_CLOV_XPAY,
// EPI_CLOV_RESID with RED_NORM, EPI_XPAY_CLOVY with RED_DIST)
hipError_t launch_hop_rhs64(hipStream_t s, int recon, int epi, int red, const HopArgs& a, const Scal* S);
// c-tiles per group of that hop: the largest divisor of a slice's tiles with tiles x right-hand sides <= 216, so that
// neighbours along t (and most along z) are still in the XCD's L2; none where the padding of a slice to whole tiles is
// more than 1/32 of its sites, which costs more lanes than the order gives.  Source preparation and residual of 12
// right-hand sides in groups against none: 24^3x32 7.55 and 7.94 ms (two hops of 24^3x64 in groups of 18 / 9 / 6 / none
// 2.90 / 2.98 / 3.03 / 3.15), 22^3x32 (1 % of padding) 6.08 and 6.33, 16^3x32 2.22 and 2.24; 14^3x32 (2.6 %) 1.79 and
// 1.76, 14^2x2x64 (31 %) 0.69 and 0.67; four and sixteen of them alike.
inline int rhs64_cgroup(const Geom& g, int nrhs)
{
    const int sites = g.Lxh * g.Ly * g.Lz, nct = hop_ctiles(g), m = 216 / nrhs;
    if ((64L * nct - sites) * 32 > sites) return 0;
    for (int d = m < nct - 1 ? m : nct - 1; d >= 2; d--)
        if (nct % d == 0) return d;
    return 0;
}

// learned preconditioner layers (activations [parity][channel][Vh][3], FP32/BF16 storage)
// mfma: layers with a BF16 end mix channels on the BF16 matrix cores (k_net_layer_mfma)
hipError_t launch_net_layer(hipStream_t s, int pin, int pout, int cin, int cout, const void* in, void* out,
                            const void* gauge32, const void* W, const Geom& g,
                            int mfma = 0);
// training (net.hip): what a pair's loss and gradients are formed from.  r: FP32 residual on even sites; gz, hid,
// gh: scratch; W1, W2 the layers, Wt the adjoint of layer 2; partials: train_partials() doubles, kept over the pairs of
// a batch
struct TrainFields {
    const void *gauge32, *r;
    void *gz, *hid, *gh;
    const void *W1, *W2, *Wt;
    double* partials;
};
size_t train_partials(const Geom& g, int hidden);
// adds a pair's gradients to the partial sums (first: starts them) and writes dn = ||P(r) - e||^2; e: paper field of
// the even sites, en: its squared norm on the device
hipError_t launch_train_pair(hipStream_t s, int hidden, const Geom& g, const TrainFields& f, const void* e,
                             const double* en, double* dn, bool first);
// the sums of the pairs since the first one into G1 [9][hidden][4] and G2 [9][4][hidden] (FP64 complex)
hipError_t launch_train_finish(hipStream_t s, int hidden, const Geom& g, double* partials, void* G1, void* G2);
hipError_t launch_net_adjoint_w(hipStream_t s, const void* W, void* Wt, int cout, int cin);
hipError_t launch_gaussian(hipStream_t s, void* out, long n, uint64_t seed, uint64_t stream);  // FP64 complex
hipError_t launch_adam(hipStream_t s, void* W, const double* G, double* m, double* v, int n, double lr, double b1,
                       double b2, double eps, int step, double gscale);

// FGMRES block Gram-Schmidt on FP64 vectors V_i = V + i stride (complex elements)
hipError_t launch_scale_inv_norm(hipStream_t s, const void* w, void* out, long n, const double* nrm2);
hipError_t launch_multidot(hipStream_t s, const void* V, long stride, int nvec, const void* w, long n,
                           double* partials, double* out);  // out[2i..] = (V_i, w); partials: 16 ceil(nvec/8) blocks
hipError_t launch_multiaxpy(hipStream_t s, const void* V, long stride, int nvec, const double* c, void* w, long n,
                            double sign, double* partials = nullptr,
                            double* nrm2 = nullptr);  // w += sign sum_i c_i V_i [, nrm2 = ||w||^2]
// Blocks (and groups of partials) of launch_multiaxpy_dot, whose blocks take 64 elements at a time where those of the
// other vector kernels take 1024: small fields get a block per tile, up to three per CU.  With blas_blocks(n) alone
// FGMRES(32) at 8^3x16 (48 blocks) took 5.24 ms for its 58 iterations, 4.64 so; 12^3x24 7.40 and 7.07; from 16^3x32 on
// the count is the same.
inline int multiaxpy_dot_blocks(long n)
{
    const long tiles = (n + 63) / 64, few = tiles < 768 ? tiles : 768, b = blas_blocks(n);
    return (int)(b > few ? b : few);
}
// w -= sum_i c_i V_i and out[2i..] = (V_i, w) of the result in one pass; at most 64 vectors
hipError_t launch_multiaxpy_dot(hipStream_t s, const void* V, long stride, int nvec, const double* c, void* w, long n,
                                double* partials, double* out);
hipError_t launch_sum_partials(hipStream_t s, const double* partials, int nb, double* out);  // one double per block

// pack / unpack between the paper layouts and the internal ones
hipError_t launch_pack_spinor(hipStream_t s, int prec, const Geom& g, const void* paper, int parity, void* internal,
                              double scale);
hipError_t launch_unpack_spinor(hipStream_t s, int prec, const Geom& g, const void* internal, int parity, void* paper,
                                double scale);
// the paper's links into plane-major FP64 entries 0 .. R-1 (top; R = 6 or 9 for recon 12 or 18), plane-major
// entries 6 .. 8 (low) and the inner precision's links (lo); each may be nullptr
hipError_t launch_pack_links(hipStream_t s, const Geom& g, const void* paper, int recon, void* top, void* low,
                             int prec_lo, int recon_lo, void* lo);

// FP64 links, one plane of Vh sites per entry: entry e < 6 of (mu, p) at top + ((2 mu + p) top_rec + e) Vh + site,
// entry e >= 6 at low + ((2 mu + p) low_rec + e - 6) Vh + site
struct LinkPlanes {
    const double2 *top, *low;
    int top_rec, low_rec;
    long Vh;
};
inline LinkPlanes link_planes(const void* top, int recon, const void* low, long Vh)
{
    if (recon == 18) return {(const double2*)top, (const double2*)top + 6 * Vh, 9, 9, Vh};
    return {(const double2*)top, (const double2*)low, 6, 3, Vh};
}

// clover kernels on the paper layouts (FP64)
// the 12 wall sources on slice t0 with spatial momentum mom (12 paper-layout fields into out)
hipError_t launch_wall_sources(hipStream_t s, const Geom& g, int t0, const int mom[3], void* out);
// meson contraction of the 12-field propagators S and T (T = S: the two-point function) into out[Lt]
// (complex FP64); site_scratch: V complex
hipError_t launch_meson_2pt(hipStream_t s, const Geom& g, const void* S, const void* T, int g_snk, int g_src,
                            const int mom[3], void* site_scratch, void* out);
// sequential sources through the sink slice t_f from the propagator S (12 fields into out)
hipError_t launch_seq_sources(hipStream_t s, const Geom& g, const void* S, int t_f, int g_f, const int mom[3],
                              void* out);
// the isotropic clover field C = sum_{mu<nu} sigma_{mu nu} F_{mu nu}, from plane-major links or from the paper's
hipError_t launch_clover_build(hipStream_t s, const Geom& g, const LinkPlanes& U, void* clover);
hipError_t launch_clover_build_records(hipStream_t s, const Geom& g, const void* U, void* clover);
// A = 1 - kappa csw C, C = wt sum_i sigma_i4 F_i4 + ws sum_{i<j} sigma_ij F_ij (wt = ws = 1: the isotropic field), and
// its inverse per parity in the internal packing, the inverse also in prec_lo (F64: not); notpd_count is raised by the
// blocks that are not positive definite
hipError_t launch_clover_op(hipStream_t s, const Geom& g, const LinkPlanes& U, double wt, double ws, double kappa,
                            double csw, void* const A[2], void* const inv[2], int prec_lo, void* const lo[2],
                            int* notpd_count);
hipError_t launch_clover_apply(hipStream_t s, const Geom& g, const void* clover, const void* psi, void* out,
                               double kappa, double csw);
hipError_t launch_clover_invert(hipStream_t s, const Geom& g, const void* clover, double kappa, double csw,
                                void* inv, int* notpd_count);
// clover fermion force of the bilinear 2 Re(Y^+ M X) (force.hip); scratch: FORCE_SITE_BYTES per site for plane-major
// copies of the fields and Gam (copies), or FORCE_GAMMA_BYTES for Gam alone (slower)
constexpr size_t FORCE_GAMMA_BYTES = 48 * 8, FORCE_SITE_BYTES = (36 + 24) * 16 + FORCE_GAMMA_BYTES;
hipError_t launch_clover_force(hipStream_t s, const Geom& g, const void* U, const void* X, const void* Y,
                               double kappa, double csw, void* scratch, bool copies, void* H);

}  // namespace qcdw
