// Host-only check of the rules that choose launches and kernels by size.
#include <algorithm>
#include <cstdio>

#include "sparse.h"

using namespace lbl;

static int fails = 0;
#define CHECK(c)                                                      \
    do {                                                              \
        if (!(c)) {                                                   \
            ++fails;                                                  \
            std::fprintf(stderr, "FAILED %s:%d %s\n", __FILE__, __LINE__, #c); \
        }                                                             \
    } while (0)

// A planner sweep has threads for its edges and for its vertices' marks and
// outputs, within the bound on workgroups.
static void plan_blocks()
{
    for (uint64_t n : {1ull, 1000ull, 100000ull, 10000000ull, 4000000000ull})
        for (uint64_t e : {0ull, 1ull, 1000ull, 568958ull, 100000000ull}) {
            const uint64_t threads = 256ull * plan_sweep_blocks(n, e);
            CHECK(threads >= 256 && threads <= 256ull * 8192);
            CHECK(threads >= std::min<uint64_t>(e, 256ull * 8192));
            CHECK(threads >= std::min<uint64_t>(n / 16, 256ull * 8192));
        }
}

int main()
{
    plan_blocks();
    if (fails) return 1;
    std::printf("rules OK\n");
    return 0;
}
