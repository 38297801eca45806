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

// One launch for the smallest frames only, by mask width and alignment: (entries,
// segments, propositions, aligned) where it measured faster and slower than two.
static void one_launch()
{
    struct Case {
        uint64_t n_ent, n_seg;
        uint32_t n_props;
        bool aligned, pays;
    };
    for (const Case &c : {Case{7600, 64, 8, true, true}, Case{5612, 96, 24, true, true}, Case{12994, 96, 8, true, true},
                          Case{6562, 325, 16, true, false}, Case{5345, 72, 40, true, true}, Case{7441, 64, 36, true, true},
                          Case{10324, 72, 64, true, false}, Case{11417, 64, 36, true, false}, Case{2988, 96, 10, false, true},
                          Case{12348, 96, 14, false, false}, Case{1595, 72, 17, false, true}, Case{6041, 64, 26, false, false},
                          Case{3811, 64, 41, false, false}, Case{9186, 64, 61, false, false}, Case{64, 1, 33, false, false}}) {
        CHECK(one_launch_pays(c.n_ent, c.n_seg, 1, c.n_props, c.aligned) == c.pays);
        CHECK(!one_launch_pays(c.n_ent, c.n_seg, 2, c.n_props, c.aligned));
    }
}

// Masks from O: as measured with the pack kernel and without.
static void masks_from_frame()
{
    struct Case {
        uint64_t n_ent, n_seg;
        uint32_t n_props;
        bool aligned, pays;
    };
    for (const Case &c : {Case{800000, 7168, 32, true, true}, Case{2300000, 30000, 64, true, false}, Case{183747, 256, 31, false, true},
                          Case{276204, 768, 47, false, true}, Case{204296, 960, 38, false, true}, Case{367339, 864, 30, false, true}, Case{429803, 448, 31, false, false}, Case{438214, 448, 17, false, false},
                          Case{438214, 448, 16, true, true}, Case{1459632, 1408, 13, false, true}, Case{855870, 1224, 47, false, false}})
        CHECK(tiles_pack(c.n_ent, c.n_seg, c.n_props, c.aligned) == c.pays);
}

// The copies of a layout's words: made first, dropped where they fail for want
// of memory or offsets, kept out where memory is short.
static void copies()
{
    CHECK(copies_fit(0, 0) && copies_fit(1000000, 1ull << 30) && !copies_fit(4000000, 1ull << 30));
    CHECK(copies_fit(37000000, 280ull << 30) && !copies_fit(10000000000ull, 288ull << 30));
    for (lbl_status first : {LBL_OK, LBL_ENOMEM, LBL_EINVAL, LBL_EDEVICE})
        for (lbl_status second : {LBL_OK, LBL_ENOMEM}) {
            std::vector<bool> made;
            auto make = [&](bool c) {
                made.push_back(c);
                return c ? first : second;
            };
            const bool again = first == LBL_ENOMEM || first == LBL_EINVAL;
            CHECK(with_copies(true, make) == (again ? second : first));
            CHECK(made == (again ? std::vector<bool>{true, false} : std::vector<bool>{true}));
            made.clear();
            CHECK(with_copies(false, make) == second && made == std::vector<bool>{false});
        }
}

int main()
{
    plan_blocks();
    copies();
    masks_from_frame();
    one_launch();
    if (fails) return 1;
    std::printf("rules OK\n");
    return 0;
}
