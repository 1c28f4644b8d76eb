// Rules by which the library's host code lays out its launches, checked where they change.  Prints "ok" at the end.
#include "internal.h"

#include <cstdio>

using namespace qcdw;

#define EXPECT(c)                                                \
    do {                                                         \
        if (!(c)) {                                              \
            std::fprintf(stderr, "line %d: %s\n", __LINE__, #c); \
            return 1;                                            \
        }                                                        \
    } while (0)

// blocks of the combined update and dot product: never more than tiles of 64 elements (but one), enough to fill the
// device on small fields, and as many partials as the other vector kernels' blocks need
static int vector_blocks()
{
    EXPECT(multiaxpy_dot_blocks(1) == 1 && multiaxpy_dot_blocks(64) == 1 && multiaxpy_dot_blocks(65) == 2);
    EXPECT(multiaxpy_dot_blocks(12L * 128) == 24);
    EXPECT(multiaxpy_dot_blocks(12L * 4096) == 768);
    for (long n = 1; n < 1L << 36; n += n / 3 + 1) {
        const long b = multiaxpy_dot_blocks(n);
        EXPECT(b >= blas_blocks(n) && b <= (n + 63) / 64 && b <= 2048);
        EXPECT(b >= 512 || b == (n + 63) / 64);
    }
    return 0;
}

static Geom lattice(int x, int y, int z, int t)
{
    Geom g{};
    g.Lx = x, g.Ly = y, g.Lz = z, g.Lt = t, g.Lxh = x / 2, g.Vh = x / 2 * y * z * t, g.t_bc = 1;
    return g;
}

// groups of the FP64 hop of several right-hand sides: whole groups, none on slices that are mostly padding, and never
// many more lanes than sites
static int rhs64_groups()
{
    EXPECT(rhs64_cgroup(lattice(24, 24, 24, 64), 12) == 18);
    EXPECT(rhs64_cgroup(lattice(14, 14, 2, 32), 12) == 0);  // 196 of 256 lanes
    EXPECT(rhs64_cgroup(lattice(12, 10, 10, 32), 12) == 0);  // 600 of 640
    EXPECT(rhs64_cgroup(lattice(14, 6, 6, 4), 9) == 2);      // 252 of 256
    for (int x = 2; x <= 32; x += 2)
        for (int y = 2; y <= 32; y += 2)
            for (int z = 2; z <= 32; z += 2)
                for (int n = 1; n <= 16; n++) {
                    const Geom g = lattice(x, y, z, 16);
                    const int c = rhs64_cgroup(g, n);
                    EXPECT(hop_cgroup_fits(g, c) && c * n <= 216);
                    EXPECT(64L * hop_blocks_nt(g, 1, c) <= g.Vh + g.Vh / 32 + 63);
                }
    return 0;
}

// tile orders of the kernels on the paper's layouts: groups are proper ones of whole tiles, and every tile has one place
static int tile_orders()
{
    EXPECT(grouped_order(lattice(24, 24, 24, 64)) == 27 && grouped_order(lattice(16, 16, 18, 4)) == 18);
    EXPECT(grouped_order(lattice(16, 16, 16, 32)) == 0);  // one group would be the eo order
    EXPECT(grouped_order(lattice(14, 14, 14, 32)) == 0);  // no whole tiles
    for (int x = 2; x <= 32; x += 2)
        for (int y = 2; y <= 32; y += 2)
            for (int z = 2; z <= 32; z += 2) {
                const Geom g = lattice(x, y, z, 4);
                const int G = grouped_order(g), nct = hop_ctiles(g);
                EXPECT(G == 0 || (G >= 4 && G < nct && nct % G == 0 && x / 2 * y * z == 64 * nct));
            }
    return 0;
}

// forms of the multi-RHS hop on lattices whose right-hand side does not fit the 32-bit byte offsets of 16-bit storage:
// the forms with wider offsets are left, so that every call still has one
static int mrhs_forms()
{
    const Geom fits = lattice(256, 128, 64, 84), big = lattice(256, 128, 64, 86);
    EXPECT(48L * fits.Vh <= 1L << 32 && 48L * big.Vh > 1L << 32);
    for (int prec : {F64, F32, BF16, F16}) {
        const bool narrow = prec == BF16 || prec == F16;
        for (int v : {0, 8}) {
            EXPECT(mrhs_variant_fits(fits, prec, v));
            EXPECT(mrhs_variant_fits(big, prec, v) == !narrow);
        }
        EXPECT(mrhs_offsets_fit(prec, fits.Vh) && mrhs_offsets_fit(prec, big.Vh) == !narrow);
        EXPECT(mrhs_variant_fits(big, prec, 1));
        EXPECT(!mrhs_variant_fits(fits, prec, 3) && !mrhs_variant_fits(fits, prec, 2 * 7));
        EXPECT(mrhs_variant_fits(fits, prec, MRHS_MFMA) == narrow);
    }
    return 0;
}

int main()
{
    if (vector_blocks() || rhs64_groups() || tile_orders() || mrhs_forms()) return 1;
    std::puts("ok");
    return 0;
}
