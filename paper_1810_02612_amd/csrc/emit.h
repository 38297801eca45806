// Rows of 0/1 bytes from bits, written by one wavefront (device code only).
#pragma once

#include "tables.h"

namespace lbl {

// A native vector type: loads and stores of it through address-space
// qualified pointers compile (HIP's vector structs assign only in the generic
// address space).
typedef unsigned int v4u32 __attribute__((ext_vector_type(4)));

// LDS dwords of one wavefront's staging (emit_block): a bit per byte of 64 rows
// of at most 64 bytes at an offset below 16, and the two dwords a row's last
// bits may reach.
constexpr uint32_t kStageWords = (64 * 64 + 16) / 32 + 2;

// The label bytes of rows [t0, t0 + n) of one job (n <= 64), written as one
// contiguous block L[t0 * np .. (t0 + n) * np): lane r holds the job's bits
// of row t0 + r in v (bit p = proposition p, none above np).  The rows' bits are
// lined up in LDS, bit i standing for byte i of the block counted from the
// 16-byte boundary at or before its start, so that every 16-byte unit of the
// block is 16 aligned bits; the lanes spread them to bytes and write whole
// units.  The units at the block's two ends, which also hold bytes of other
// rows, are written byte by byte, so no byte outside the block is stored.
//
// Lining up bytes instead, eight times the LDS (an atomic for every four label
// bytes), the combine of 25k rows x 128^2 x 4 frames took 8.1 us, not 7.1, and of
// six maps x 16 frames 108, not 103.
__device__ __forceinline__ void emit_block(uint32_t *stage, uint32_t lane, uint32_t n, uint64_t v, uint8_t *dst,
                                           uint32_t np)
{
    const uint32_t mis = (uint32_t)(reinterpret_cast<uintptr_t>(dst) & 15u);
    const uint32_t total = mis + n * np;  // bits, <= 15 + 4096
    const uint32_t n_units = (total + 15) >> 4;
    for (uint32_t w = lane; w < (total + 31) / 32; w += 64) stage[w] = 0;
    lds_in_order();
    if (lane < n) {
        const uint32_t o = mis + lane * np, sh = o & 31u;
        uint32_t *w = stage + (o >> 5);
        const uint32_t lo = (uint32_t)v, hi = (uint32_t)(v >> 32);
        // the row's bits from bit sh of w[0]: zero parts change nothing
        auto put = [&](uint32_t i, uint32_t x) {
            if (x) __hip_atomic_fetch_or(w + i, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
        };
        put(0, lo << sh);
        put(1, (uint32_t)(((uint64_t)hi << 32 | lo) >> (32 - sh)));
        put(2, sh ? hi >> (32 - sh) : 0u);
    }
    lds_in_order();
    // device memory (flat stores would also count on the LDS wait counter)
    __attribute__((address_space(1))) uint8_t *g = (__attribute__((address_space(1))) uint8_t *)(dst - mis);
    const lds_u16 *bits = reinterpret_cast<const lds_u16 *>(stage);
    for (uint32_t u = lane; u < n_units; u += 64) {
        const uint32_t b16 = bits[u];
        const uint32_t lo = 16 * u, hi = lo + 16;
        if (lo >= mis && hi <= total) {
            *(__attribute__((address_space(1))) v4u32 *)(g + lo) =
                v4u32{spread_nib(b16 & 0xFu), spread_nib((b16 >> 4) & 0xFu), spread_nib((b16 >> 8) & 0xFu), spread_nib(b16 >> 12)};
        } else {
            for (uint32_t b = 0; b < 16; ++b)
                if (lo + b >= mis && lo + b < total) g[lo + b] = (uint8_t)((b16 >> b) & 1u);
        }
    }
    lds_in_order();  // the stage is reused by the next block
}

// emit_block for rows of 16 * upr bytes (upr = 1 .. 4) at a 16-byte aligned
// dst, without staging: lane l writes the 16-byte units l, l + 64, ... of the
// block, fetching the bits of each unit's row from the lane that holds them.
__device__ __forceinline__ void emit_units(uint32_t lane, uint32_t n, uint64_t bits, uint8_t *dst, uint32_t upr)
{
    const uint32_t shift = upr == 1 ? 0 : upr == 2 ? 1 : upr == 4 ? 2 : 32;  // 32: not a power of two
    const uint32_t units = n * upr;
    uint4 *d = reinterpret_cast<uint4 *>(dst);
    // uniform trip count: every lane takes part in the shuffles
    for (uint32_t ub = 0; ub < units; ub += 64) {
        const uint32_t u = ub + lane;  // < 64 * upr, so row < 64
        const uint32_t row = min(shift < 32 ? u >> shift : u / upr, 63u);
        const uint32_t c = u - row * upr;
        const uint32_t lo = (uint32_t)__shfl((int)(uint32_t)bits, (int)row);
        const uint32_t hi = (uint32_t)__shfl((int)(uint32_t)(bits >> 32), (int)row);
        const uint32_t b = (uint32_t)((((uint64_t)hi << 32) | lo) >> (16 * c)) & 0xFFFFu;
        if (u < units)
            d[u] = make_uint4(spread_nib(b & 0xFu), spread_nib((b >> 4) & 0xFu), spread_nib((b >> 8) & 0xFu),
                              spread_nib(b >> 12));
    }
}

}  // namespace lbl
