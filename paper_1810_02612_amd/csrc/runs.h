// The run encoding of T's words, and the device code that reads it.
//
// A swept footprint meets an 8 x 8-cell word in rows of consecutive cells:
// 99.7-99.9% of the words of the 200k x 512^2 and 50k x 256^2 maps have at
// most one run of set cells in each of their eight rows (97% on 0.8 m
// cells).  A row with one run is one of 37 patterns (empty, or one of the 36
// intervals [c, d) of 8 cells), so a word is eight 6-bit codes, and its label
// is the OR of eight table entries, one per row, where nibble tables need
// sixteen.  A word with k runs in some row is stored as k entries (OR is
// idempotent), so any word can be held.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#ifdef __HIPCC__
#include "tables.h"
#endif

namespace lbl {

// A word's run tables: per tile row the 37 entries of its patterns, entry 0
// (no cell) first, then the runs by falling length: length n starting at
// cell c is entry run_off(n) + c.
constexpr uint32_t kRunCodes = 37;
// Entries between tile rows: with 40, the 16 lanes (two rows of cells) that
// an LDS store of 8-byte entries takes at a time meet 16 different bank
// pairs, for every run length.
constexpr uint32_t kRunRow = 40;
constexpr uint32_t kRunWords = 8 * kRunRow;
__host__ __device__ constexpr uint32_t run_off(uint32_t n) { return 1 + (8 - n) * (9 - n) / 2; }

// A run entry: the code of tile row k at bits 6k .. 6k + 5 (rows 0-4 in the
// low dword, 5-7 in the high one after 2 unused bits), the local row at bits
// 50 .. 62, and at bit 63 the parity of its segment's index, which is the
// table slot the segment's tables are built in.
constexpr uint32_t kRunRowBit = 50;
__host__ __device__ constexpr uint32_t run_code_bit(uint32_t k) { return k < 5 ? 6 * k : 32 + 6 * (k - 5); }

// Cells of tile row k of a word in device order (z-order bits, x the odd
// ones): bit x of the result is cell (x, k).
__host__ __device__ inline uint32_t word_row(uint64_t v, uint32_t k)
{
    const uint32_t y = (k & 1u) | ((k & 2u) << 1) | ((k & 4u) << 2);  // k's bits at 0, 2, 4
    uint32_t r = 0;
    for (uint32_t x = 0; x < 8; ++x)
        r |= (uint32_t)(v >> (y + (((x & 1u) << 1) | ((x & 2u) << 2) | ((x & 4u) << 3))) & 1u) << x;
    return r;
}

// Number of runs of set bits in a tile row (0 .. 4).
__host__ __device__ inline uint32_t row_runs(uint32_t r)
{
#ifdef __HIP_DEVICE_COMPILE__
    return __popc(r & ~(r << 1) & 0xFFu);
#else
    return (uint32_t)__builtin_popcount(r & ~(r << 1) & 0xFFu);
#endif
}

// Entries a word value takes: its rows' largest number of runs.
__host__ __device__ inline uint32_t word_entries(uint64_t v)
{
    uint32_t n = 0;
    for (uint32_t k = 0; k < 8; ++k) {
        const uint32_t c = row_runs(word_row(v, k));
        n = c > n ? c : n;
    }
    return n;
}

// Codes of the word's piece number `piece`: run `piece` of every row that has
// that many.
__host__ __device__ inline uint64_t word_codes(uint64_t v, uint32_t piece)
{
    uint64_t e = 0;
    for (uint32_t k = 0; k < 8; ++k) {
        uint32_t r = word_row(v, k);
        for (uint32_t j = 0; j < piece && r; ++j) r &= r + (r & (0u - r));  // drop the lowest run
        if (!r) continue;
        uint32_t c = 0, n = 0;
        while (!((r >> c) & 1u)) ++c;
        while ((r >> (c + n)) & 1u) ++n;
        e |= (uint64_t)(run_off(n) + c) << run_code_bit(k);
    }
    return e;
}

#ifdef __HIPCC__

// Lane i's v from lane i + 1 of its row of 16 lanes.
__device__ __forceinline__ uint32_t from_next(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x101, 0xF, 0xF, true);
}
__device__ __forceinline__ uint64_t from_next(uint64_t v)
{
    return ((uint64_t)from_next((uint32_t)(v >> 32)) << 32) | from_next((uint32_t)v);
}

// The run tables of one word at t (LDS), built by one wavefront: lane 8k + c
// holds the proposition mask of cell (c, k).  Entry 0 of every row is not
// written (it stays zero).  Lane 8k + c ORs its run of every length; lanes
// whose run would leave the row hold garbage, which lands on entries of
// shorter runs of the same row: the stores go from the longest run to the
// shortest, and LDS instructions of a wavefront complete in issue order, so
// those entries are written again with their values (run_off puts longer
// runs first, and length 1 has no garbage).
template <typename M>
__device__ __forceinline__ void build_runs(M m, M *t, uint32_t lane)
{
    M v[8];
    v[0] = m;
#pragma unroll
    for (int j = 1; j < 8; ++j) v[j] = m | from_next(v[j - 1]);
    M *e = t + (lane >> 3) * kRunRow + (lane & 7u);
#pragma unroll
    for (int j = 7; j >= 0; --j) {
        e[run_off(j + 1)] = v[j];
        lds_in_order();  // keeps the stores apart as well
    }
}

#endif  // __HIPCC__

}  // namespace lbl
