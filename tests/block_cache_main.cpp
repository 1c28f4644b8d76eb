// The library's device buffers (DevBuf, PoolBuf and the block cache behind them) on a device of fixed capacity whose
// runtime calls are answered here.  One scenario per run, named by the first argument; prints "ok" at the end.
#include "host.h"

constexpr size_t MB = 1 << 20;
static size_t capacity, used, mallocs, frees;
static std::map<void*, size_t> blocks;
static hipError_t last_error = hipSuccess;
static char* next_address = (char*)(1UL << 40);

hipError_t hipGetDevice(int* d)
{
    *d = 0;
    return hipSuccess;
}
hipError_t hipGetDeviceProperties(hipDeviceProp_t* p, int)
{
    std::memset(p, 0, sizeof *p);
    p->totalGlobalMem = 4000 * MB;  // the cache keeps at most 1000 MB
    return hipSuccess;
}
hipError_t hipMalloc(void** p, size_t n)
{
    if (used + n > capacity) return last_error = hipErrorOutOfMemory;
    mallocs++;
    used += n;
    *p = next_address;
    next_address += n;
    blocks[*p] = n;
    return hipSuccess;
}
hipError_t hipFree(void* p)
{
    auto it = blocks.find(p);
    if (it == blocks.end()) abort();  // never handed out, or freed twice
    used -= it->second;
    frees++;
    blocks.erase(it);
    return hipSuccess;
}
hipError_t hipGetLastError()
{
    const hipError_t e = last_error;
    last_error = hipSuccess;
    return e;
}

#define EXPECT(c)                                                    \
    do {                                                             \
        if (!(c)) {                                                  \
            std::fprintf(stderr, "line %d: %s\n", __LINE__, #c);     \
            return 1;                                                \
        }                                                            \
    } while (0)

static void use(size_t n)
{
    PoolBuf b;
    (void)b.alloc(n);
}

// memory that only the cache holds is there for every buffer, pooled or not
static int out_of_memory()
{
    capacity = 1000 * MB;
    for (int pooled = 0; pooled < 2; pooled++) {
        use(700 * MB);
        EXPECT(used == 700 * MB);
        DevBuf b;
        b.pooled = pooled;
        EXPECT(b.alloc(500 * MB) == hipSuccess && b.n == 500 * MB);
        EXPECT(used == 500 * MB);
    }
    DevBuf big;
    EXPECT(big.alloc(1001 * MB) == hipErrorOutOfMemory && big.p == nullptr && big.n == 0);
    EXPECT(big.alloc(900 * MB) == hipSuccess);
    return 0;
}

// a cache full of sizes that nobody asks for any more makes room for those in use, oldest first
static int full_cache()
{
    capacity = 100000 * MB;
    for (int k = 0; k < 2; k++) {
        use(400 * MB);
        use(250 * MB);
        use(310 * MB);
    }
    EXPECT(used == 960 * MB && mallocs == 3);
    use(120 * MB);
    EXPECT(used <= 1000 * MB);
    const size_t n = mallocs;
    for (int k = 0; k < 5; k++) use(120 * MB);
    EXPECT(mallocs == n);
    use(310 * MB);  // the last one in before the new size
    EXPECT(mallocs == n);
    use(400 * MB);  // the first one in: gone
    EXPECT(mallocs == n + 1 && used <= 1000 * MB);
    use(1001 * MB);  // larger than the cache: returned at once, and nothing else with it
    const size_t held = used;
    use(1001 * MB);
    EXPECT(used == held && mallocs == n + 3);
    return 0;
}

// an allocation that fails is reported once, by the call itself: the next launch's own check finds no error
static int error_left_behind()
{
    capacity = 1000 * MB;
    for (int pooled = 0; pooled < 2; pooled++) {
        DevBuf b;
        b.pooled = pooled;
        EXPECT(b.alloc(1200 * MB) == hipErrorOutOfMemory);
        EXPECT(hipGetLastError() == hipSuccess);
    }
    return 0;
}

int main(int argc, char** argv)
{
    const std::string what = argc > 1 ? argv[1] : "";
    int bad = 1;
    if (what == "out_of_memory") bad = out_of_memory();
    if (what == "full_cache") bad = full_cache();
    if (what == "error_left_behind") bad = error_left_behind();
    if (bad == 0) std::puts("ok");
    return bad;
}
