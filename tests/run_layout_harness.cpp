// Host-only check of the run encoding of words (runs.h) and of the tilings
// over run entries.  No device memory is touched.
#include <algorithm>
#include <cstdio>
#include <random>

#include "sparse.h"

using namespace lbl;

static int fails = 0;
#define CHECK(c)                                                      \
    do {                                                              \
        if (!(c)) {                                                   \
            if (++fails <= 20) std::fprintf(stderr, "FAILED %s:%d %s\n", __FILE__, __LINE__, #c); \
        }                                                             \
    } while (0)

// The cells a code of a tile row stands for, from the order of the table.
static uint32_t cells_of(uint32_t code)
{
    if (code == 0) return 0;
    for (uint32_t n = 8; n >= 1; --n)
        if (code >= run_off(n) && code < run_off(n) + 9 - n) return ((1u << n) - 1u) << (code - run_off(n));
    CHECK(!"a code outside the table");
    return 0;
}

// The bit of cell (x, y) in a word: x the more significant bit of each pair.
static uint32_t bit_of(uint32_t x, uint32_t y)
{
    uint32_t z = 0;
    for (uint32_t b = 0; b < 3; ++b) z |= ((x >> b) & 1u) << (2 * b + 1) | ((y >> b) & 1u) << (2 * b);
    return z;
}

static void check_word(uint64_t v)
{
    const uint32_t n = word_entries(v);
    CHECK(n <= 4 && (n == 0) == (v == 0));
    uint64_t all = 0;
    for (uint32_t j = 0; j < n; ++j) {
        const uint64_t e = word_codes(v, j);
        uint64_t piece = 0, used = 0;
        for (uint32_t k = 0; k < 8; ++k) {
            const uint32_t b = run_code_bit(k), c = (uint32_t)(e >> b) & 63u;
            used |= 63ull << b;
            CHECK(c < kRunCodes);
            CHECK(k < 5 ? b + 6 <= 32 : b >= 32 && b + 6 <= kRunRowBit);
            for (uint32_t x = 0; x < 8; ++x) piece |= (uint64_t)(cells_of(c) >> x & 1u) << bit_of(x, k);
        }
        CHECK((e & ~used) == 0);
        CHECK(piece != 0);
        all |= piece;
    }
    CHECK(all == v);
}

// Walk a tiling as the run kernel does: every entry is taken by one active
// lane, with the tables of its own segment's word in the slot that its
// segment's parity names, built before use, and no lane (active or not)
// reads further than the padding.
static void check_tiling(const std::vector<uint64_t> &start, const std::vector<uint32_t> &word,
                         const std::vector<uint64_t> &rb_seg, const std::vector<uint32_t> &k)
{
    TilingHost h;
    make_run_tiling(start, word, rb_seg, k, &h);
    const size_t n_rb = rb_seg.size() - 1;
    uint64_t n_tiles = 0;
    for (uint32_t x : k) n_tiles += x;
    CHECK(h.tasks.size() == n_tiles * kTileWaves && h.rb_tile.size() == n_rb + 1 && h.rb_tile[n_rb] == n_tiles);
    std::vector<uint32_t> order = h.block_tile;
    std::sort(order.begin(), order.end());
    CHECK(order.size() == n_tiles);
    for (uint32_t i = 0; i < order.size(); ++i) CHECK(order[i] == i);
    std::vector<uint8_t> seen(start.back(), 0);
    for (size_t rb = 0; rb < n_rb; ++rb) {
        const uint64_t E1 = start[rb_seg[rb + 1]];
        uint64_t next = start[rb_seg[rb]];
        for (uint64_t q = (uint64_t)h.rb_tile[rb] * kTileWaves; q < (uint64_t)h.rb_tile[rb + 1] * kTileWaves; ++q) {
            const SpTask &t = h.tasks[q];
            CHECK(t.lo == next);
            int64_t slot_word[2] = {-1, -1};
            for (uint32_t i = 0; i < t.n_rounds; ++i) {
                const SpRound &r = h.rounds[t.round0 + i];
                const uint32_t n = (r.meta >> 8) & 0xFF, cut = (r.meta >> 16) & 0xFF;
                CHECK((r.meta & 0xFF) == 0 && n >= 1 && n <= 64 && cut >= 1 && cut <= 64 && (r.meta >> 27) == 0);
                CHECK(t.lo + r.e_off == next && t.lo + r.e_off + 64 <= start.back() + kEntryPad);
                const uint32_t s0 = (r.meta & kMetaSlot0) ? 1 : 0;
                CHECK(!((r.meta & kMetaBuild0) && (r.meta & kMetaBuild1)));
                if (r.meta & kMetaBuild0) slot_word[s0] = r.tword;
                if (r.meta & kMetaBuild1) slot_word[s0 ^ 1] = r.tword;
                for (uint32_t l = 0; l < n; ++l) {
                    const uint64_t e = t.lo + r.e_off + l;
                    CHECK(e < E1);
                    if (e >= E1) continue;
                    ++seen[e];
                    const uint64_t s = std::upper_bound(start.begin(), start.end(), e) - start.begin() - 1;
                    CHECK(s >= rb_seg[rb] && s < rb_seg[rb + 1] && (s & 1) == (s0 ^ (l >= cut ? 1 : 0)));
                    CHECK(slot_word[s & 1] == (int64_t)word[s]);
                }
                next = t.lo + r.e_off + n;
            }
        }
        CHECK(next == E1);
    }
    for (uint8_t c : seen) CHECK(c == 1);
}

int main()
{
    std::mt19937_64 rng(3);
    for (uint32_t r = 0; r < 256; ++r)  // every pattern of a row, in every row
        for (uint32_t k = 0; k < 8; ++k) {
            uint64_t v = 0;
            for (uint32_t x = 0; x < 8; ++x) v |= (uint64_t)(r >> x & 1u) << bit_of(x, k);
            CHECK(word_row(v, k) == r);
            check_word(v);
        }
    for (int i = 0; i < 20000; ++i) check_word(i & 1 ? rng() : rng() & rng() & rng());
    check_word(~0ull);
    CHECK(run_off(1) + 8 == kRunCodes && kRunCodes <= kRunRow);
    // the stores of build_runs: what a lane writes outside its row's runs is
    // written again by a later store, with the run's value
    for (uint32_t k = 0; k < 8; ++k) {
        std::vector<int> by(kRunWords + 64, -1);  // length that last wrote an entry, or -2: garbage
        for (uint32_t n = 8; n >= 1; --n)
            for (uint32_t c = 0; c < 8; ++c) by[k * kRunRow + run_off(n) + c] = c + n <= 8 ? (int)n : -2;
        for (uint32_t i = 0; i < by.size(); ++i) {
            const bool mine = i > k * kRunRow && i < k * kRunRow + kRunCodes;
            CHECK(mine ? by[i] >= 1 && i - k * kRunRow >= run_off(by[i]) && i - k * kRunRow < run_off(by[i]) + 9 - by[i]
                       : by[i] == -1);
        }
    }
    // tilings: typical, tiny and huge segments, empty row blocks
    for (int mode = 0; mode < 4; ++mode)
        for (int trial = 0; trial < 4; ++trial) {
            const uint32_t n_rb = 1 + rng() % 5, W = 16 + rng() % 300;
            std::vector<uint64_t> start, rb_seg(n_rb + 1, 0);
            std::vector<uint32_t> word;
            uint64_t e = 0;
            for (uint32_t rb = 0; rb < n_rb; ++rb) {
                rb_seg[rb] = word.size();
                if (mode == 3 && rng() % 2 == 0) continue;
                for (uint32_t w = 0; w < W; ++w) {
                    const uint32_t n = mode == 0 ? (uint32_t)(rng() % 120) : mode == 1 ? (uint32_t)(rng() % 3) :
                                       mode == 2 ? (rng() % 16 == 0 ? (uint32_t)(rng() % 3000) : 0u) : 1u + (uint32_t)(rng() % 90);
                    if (n == 0) continue;
                    start.push_back(e);
                    word.push_back(w);
                    e += n;
                }
            }
            rb_seg[n_rb] = word.size();
            start.push_back(e);
            for (uint32_t target : {1u, 7u, 40u}) check_tiling(start, word, rb_seg, tiles_per_block(run_costs(start, rb_seg), target));
        }
    CHECK(use_runs(100, 100) && !use_runs(100, 400) && !use_runs(0, 0));
    if (fails) return 1;
    std::printf("run layout OK\n");
    return 0;
}
