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

int main()
{
    if (vector_blocks()) return 1;
    std::puts("ok");
    return 0;
}
