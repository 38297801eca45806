// Nibble tables of a word, built by one wavefront (device code only).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace lbl {

// High bit of each byte of x: the byte is not zero.
__device__ __forceinline__ uint32_t nz_high(uint32_t x) { return (((x & 0x7F7F7F7Fu) + 0x7F7F7F7Fu) | x) & 0x80808080u; }

// Nonzero bytes of a 32-bit word -> 4 bits (bit k for byte k): the bytes'
// flags (0 or 128) weighted 1, 2, 4, 8 and summed in one instruction.
__device__ __forceinline__ uint32_t nz_bytes(uint32_t x) { return __builtin_amdgcn_udot4(nz_high(x), 0x08040201u, 0u, false) >> 7; }

// Nonzero bytes of 8 bytes -> 8 bits.
__device__ __forceinline__ uint32_t nz_bytes8(uint32_t x, uint32_t y)
{
    return __builtin_amdgcn_udot4(nz_high(y), 0x80402010u, __builtin_amdgcn_udot4(nz_high(x), 0x08040201u, 0u, false), false) >> 7;
}

// Four bits -> four bytes 0/1 (bit k to byte k).
__device__ __forceinline__ uint32_t spread_nib(uint32_t x) { return (x * 0x00204081u) & 0x01010101u; }

// Nonzero bytes of 16 bytes -> 16 bits (bit k for byte k).
__device__ __forceinline__ uint32_t nz_bytes16(uint32_t x, uint32_t y, uint32_t z, uint32_t w)
{
    return nz_bytes8(x, y) | (nz_bytes8(z, w) << 8);
}
__device__ __forceinline__ uint32_t nz_bytes16(const uint4 &q) { return nz_bytes16(q.x, q.y, q.z, q.w); }

// Between LDS accesses of one wavefront, whose lanes read what others of it
// wrote: the hardware completes them in issue order, and this keeps the compiler
// from moving any across (the barrier alone is none for memory).
__device__ __forceinline__ void lds_in_order()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");
    __builtin_amdgcn_wave_barrier();
}
// Halves of LDS dwords that are also accessed whole.
typedef uint16_t lds_u16 __attribute__((may_alias));

// Loads from any byte address of device memory.
typedef uint32_t u32x4_any __attribute__((ext_vector_type(4), aligned(1)));
typedef uint32_t u32x2_any __attribute__((ext_vector_type(2), aligned(1)));
typedef uint32_t u32_any __attribute__((aligned(1)));
typedef uint16_t u16_any __attribute__((aligned(1)));
typedef __attribute__((address_space(1))) const uint8_t global_u8;
template <typename T>
__device__ __forceinline__ T load_any(global_u8 *p)
{
    return *reinterpret_cast<__attribute__((address_space(1))) const T *>(p);
}

// byte_mask of 16 C - 15 .. 16 C bytes.
template <uint32_t C>
__device__ __forceinline__ uint64_t byte_mask_16(global_u8 *src, uint32_t n)
{
    u32x4_any q[C];
#pragma unroll
    for (uint32_t k = 0; k < C; ++k) q[k] = load_any<u32x4_any>(src + (k + 1 < C ? 16 * k : n - 16));
    uint64_t m = 0;
#pragma unroll
    for (uint32_t k = 0; k < C; ++k)
        m |= (uint64_t)nz_bytes16(q[k].x, q[k].y, q[k].z, q[k].w) << (k + 1 < C ? 16 * k : n - 16);
    return m;
}

// Bit p set iff byte p of bytes[0 .. n) (device memory, any address) is
// non-zero, 1 <= n <= 64, n the same in every lane.  The bytes are read in
// the widest pieces that fit, all of them before the first is used; the last
// piece ends with the last byte and may read bytes of the one before again,
// so no byte outside is read and no piece is narrower than it need be.  For
// 37 bytes that is three 16-byte loads, where single bytes in groups of four
// took ten waits for memory (packing 75,003 x 328 x 200 x 37: 5.6 -> 3.3 us).
__device__ __forceinline__ uint64_t byte_mask(const uint8_t *bytes, uint32_t n)
{
    global_u8 *src = (global_u8 *)bytes;
    if (n > 48) return byte_mask_16<4>(src, n);
    if (n > 32) return byte_mask_16<3>(src, n);
    if (n > 16) return byte_mask_16<2>(src, n);
    if (n == 16) return byte_mask_16<1>(src, n);
    if (n >= 8) {
        const u32x2_any a = load_any<u32x2_any>(src), b = load_any<u32x2_any>(src + n - 8);
        return nz_bytes8(a.x, a.y) | (nz_bytes8(b.x, b.y) << (n - 8));
    }
    if (n >= 4) {
        const uint32_t a = load_any<u32_any>(src), b = load_any<u32_any>(src + n - 4);
        return nz_bytes(a) | (nz_bytes(b) << (n - 4));
    }
    if (n >= 2) {
        const uint32_t a = load_any<u16_any>(src), b = load_any<u16_any>(src + n - 2);
        return nz_bytes(a) | (nz_bytes(b) << (n - 2));
    }
    return src[0] != 0;
}

// Value of lane C of each group of four lanes (DPP quad permutation).
template <int C>
__device__ __forceinline__ uint64_t quad_bcast(uint64_t v)
{
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)v, C * 0x55, 0xF, 0xF, false);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(v >> 32), C * 0x55, 0xF, 0xF, false);
    return ((uint64_t)hi << 32) | lo;
}

// The 16 x 16 nibble tables of one 64-cell word: entry [n][v] is the OR of
// the proposition masks of the cells 4n + b with bit b of v set, so that
// OR over n of entry [n][nibble n of x] is the label of a word value x.
// Lane l holds the mask of cell l; the four lanes of nibble n share their
// masks and lane 4n + j writes the four consecutive entries [n][4j .. 4j+3]
// (32 bytes) to dst[n * 16 + 4j ..].  Every lane of the wavefront must be
// active.
__device__ __forceinline__ void write_tables(uint64_t cell, uint64_t *dst, uint32_t lane)
{
    const uint64_t o0 = quad_bcast<0>(cell), o1 = quad_bcast<1>(cell);
    const uint64_t o2 = quad_bcast<2>(cell), o3 = quad_bcast<3>(cell);
    const uint32_t j = lane & 3u;
    const uint64_t h = ((j & 1u) ? o2 : 0ull) | ((j & 2u) ? o3 : 0ull);  // bits 2, 3 of v = 4j + m
    ulonglong2 *d = reinterpret_cast<ulonglong2 *>(dst + (lane >> 2) * 16 + 4 * j);
    d[0] = make_ulonglong2(h, h | o0);
    d[1] = make_ulonglong2(h | o1, h | o0 | o1);
}

// 32-bit version of quad_bcast.
template <int C>
__device__ __forceinline__ uint32_t quad_bcast32(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, C * 0x55, 0xF, 0xF, false);
}

// write_tables for 32-bit proposition masks (frames of at most 32
// propositions): the same 16 x 16 tables with 4-byte entries, lane 4n + j
// writing the 16 bytes of entries [n][4j .. 4j+3] to dst[n * 16 + 4j ..].
__device__ __forceinline__ void write_tables32(uint32_t cell, uint32_t *dst, uint32_t lane)
{
    const uint32_t o0 = quad_bcast32<0>(cell), o1 = quad_bcast32<1>(cell);
    const uint32_t o2 = quad_bcast32<2>(cell), o3 = quad_bcast32<3>(cell);
    const uint32_t j = lane & 3u;
    const uint32_t h = ((j & 1u) ? o2 : 0u) | ((j & 2u) ? o3 : 0u);
    *reinterpret_cast<uint4 *>(dst + (lane >> 2) * 16 + 4 * j) = make_uint4(h, h | o0, h | o1, h | o0 | o1);
}

}  // namespace lbl
