// Rows of 0/1 bytes from bits, written by one wavefront (device code only).
#pragma once

#include "tables.h"

namespace lbl {

// A native vector type: loads and stores of it through address-space
// qualified pointers compile (HIP's vector structs assign only in the generic
// address space).
typedef unsigned int v4u32 __attribute__((ext_vector_type(4)));

// LDS of one wavefront's staging (emit_block): 64 rows of at most 64 bytes
// at an offset below 16, plus the word a row's last bytes may spill into.
constexpr uint32_t kStageWords = (64 * 64 + 32) / 4;

// The label bytes of rows [t0, t0 + n) of one job (n <= 64), written as one
// contiguous block L[t0 * np .. (t0 + n) * np): lane r holds the job's bits
// of row t0 + r in v (bit p = proposition p).  The block is staged in LDS at
// its offset modulo 16 (each lane ORs its row's bytes into 4-byte-aligned
// words; neighbouring rows share the words at their boundary), then written
// with 16-byte stores; the units at the block's two ends, which also hold
// bytes of other rows, are written byte by byte, so no byte outside the
// block is stored.  stage: 64 * 64 + 32 bytes of this wavefront's LDS (the
// last row's words reach at most 2 bytes past the block).
__device__ __forceinline__ void emit_block(uint32_t *stage, uint32_t lane, uint32_t n, uint64_t v, uint8_t *dst,
                                           uint32_t np)
{
    const uintptr_t base = reinterpret_cast<uintptr_t>(dst);
    const uint32_t mis = (uint32_t)(base & 15u);
    const uint32_t total = mis + n * np;  // staged bytes, <= 15 + 4096
    const uint32_t n_units = (total + 15) >> 4;
    v4u32 *st4 = reinterpret_cast<v4u32 *>(stage);
    for (uint32_t u = lane; u < n_units; u += 64) st4[u] = v4u32{0u, 0u, 0u, 0u};
    __builtin_amdgcn_wave_barrier();
    if (lane < n) {
        const uint32_t o = mis + lane * np;
        const uint32_t sh = 8 * (o & 3u);
        uint32_t *w = stage + (o >> 2);
        const uint32_t nq = ((o & 3u) + np + 3) >> 2;
        uint32_t prev = 0;
        for (uint32_t q = 0; q < nq; ++q) {
            const uint32_t cur = 4 * q < np ? spread_nib((uint32_t)(v >> (4 * q)) & 0xFu) : 0u;
            const uint32_t out = sh ? (cur << sh) | (prev >> (32 - sh)) : cur;
            __hip_atomic_fetch_or(w + q, out, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
            prev = cur;
        }
    }
    __builtin_amdgcn_wave_barrier();
    // device memory (flat stores would also count on the LDS wait counter)
    __attribute__((address_space(1))) uint8_t *g = (__attribute__((address_space(1))) uint8_t *)(dst - mis);
    for (uint32_t u = lane; u < n_units; u += 64) {
        const v4u32 x = st4[u];
        const uint32_t lo = 16 * u, hi = lo + 16;
        if (lo >= mis && hi <= total) {
            *(__attribute__((address_space(1))) v4u32 *)(g + lo) = x;
        } else {
            const uint32_t xs[4] = {x.x, x.y, x.z, x.w};
            for (uint32_t b = 0; b < 16; ++b)
                if (lo + b >= mis && lo + b < total) g[lo + b] = (uint8_t)(xs[b >> 2] >> (8 * (b & 3u)));
        }
    }
    __builtin_amdgcn_wave_barrier();  // the stage is reused by the next block
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
