// Row tiles: frames of at most 4 propositions in one kernel.
//
// A label needs no table here: bit p of an entry's label is (word value AND
// mask p of its word) != 0, mask p holding a bit for each cell of the word
// that meets proposition p.  The layout is T's entries once more, in tiles of
// 64 to 512 consecutive rows, by word inside a tile: a tile holds every
// entry of its rows, so its workgroup writes their label bytes whole, with no
// other kernel to clear L before or to combine partial labels after, and
// forms the masks of the few words its rows meet itself, straight from O.
//
// Worth it where neighbouring rows meet the same words (a roadmap stores its
// transitions by source vertex) or the layout is small: a mask costs a read of
// 64 cells, so a tile must use each for many entries, or there must be few
// (row_tiles_pay).  Other layouts keep the split of sparse.hip (k_pack_masks,
// k_label_direct).
#include <algorithm>
#include <memory>

#include "emit.h"
#include "rowtiles.h"
#include "sparse.h"

namespace lbl {
namespace {

// First index in rows[lo, hi) (ascending) that is >= key.
__device__ __forceinline__ uint64_t lower_row(const uint16_t *rows, uint64_t lo, uint64_t hi, uint32_t key)
{
    while (lo < hi) {
        const uint64_t mid = lo + (hi - lo) / 2;
        if (rows[mid] < key) lo = mid + 1;
        else hi = mid;
    }
    return lo;
}

// The segments (row block, word) of sparse.hip's layout, as the builders read
// them: segment s holds entries seg[s] .. seg[s + 1], row block rb the
// segments rb_seg[rb] .. rb_seg[rb + 1].
struct Segments {
    const uint64_t *seg, *rb_seg;
    const uint32_t *seg_cell;  // first cell id of the segment's word
    const uint16_t *row;
    const uint64_t *val;
};

// Entries and segments of tile blockIdx.x (the rows of its row block from
// first to last).
__global__ void __launch_bounds__(256)
k_tile_count(Segments g, uint32_t rows_per_tile, uint32_t *__restrict__ n_ent, uint32_t *__restrict__ n_seg)
{
    const uint32_t per_rb = kRowBlock / rows_per_tile, rb = blockIdx.x / per_rb, r0 = blockIdx.x % per_rb * rows_per_tile;
    uint32_t e = 0, n = 0;
    for (uint64_t s = g.rb_seg[rb] + threadIdx.x; s < g.rb_seg[rb + 1]; s += blockDim.x) {
        const uint64_t lo = lower_row(g.row, g.seg[s], g.seg[s + 1], r0);
        const uint32_t c = (uint32_t)(lower_row(g.row, lo, g.seg[s + 1], r0 + rows_per_tile) - lo);
        e += c;
        n += c != 0;
    }
    __shared__ uint32_t sum[2];
    if (threadIdx.x < 2) sum[threadIdx.x] = 0;
    __syncthreads();
    if (e) atomicAdd(&sum[0], e);
    if (n) atomicAdd(&sum[1], n);
    __syncthreads();
    if (threadIdx.x == 0) {
        n_ent[blockIdx.x] = sum[0];
        n_seg[blockIdx.x] = sum[1];
    }
}

// Writes tile blockIdx.x: its entries by word (rows local to the tile), the
// words of its segments and its chunk records (cleared before the launch).
__global__ void __launch_bounds__(256)
k_tile_fill(Segments g, uint32_t rows_per_tile, const RowTile *__restrict__ tiles, uint64_t *__restrict__ val,
            uint8_t *__restrict__ row, uint32_t *__restrict__ seg_cell, RowChunk *__restrict__ chunks)
{
    __shared__ uint32_t upto[2][256];  // inclusive sums of entries and segments over the threads
    const uint32_t per_rb = kRowBlock / rows_per_tile, rb = blockIdx.x / per_rb, r0 = blockIdx.x % per_rb * rows_per_tile;
    const RowTile tile = tiles[blockIdx.x];
    const uint64_t s_end = g.rb_seg[rb + 1];
    uint32_t ent0 = 0, seg0 = 0;  // entries and segments of the tile so far
    for (uint64_t sb = g.rb_seg[rb]; sb < s_end; sb += blockDim.x) {
        const uint64_t s = sb + threadIdx.x;
        uint64_t lo = 0;
        uint32_t c = 0;
        if (s < s_end) {
            lo = lower_row(g.row, g.seg[s], g.seg[s + 1], r0);
            c = (uint32_t)(lower_row(g.row, lo, g.seg[s + 1], r0 + rows_per_tile) - lo);
        }
        upto[0][threadIdx.x] = c;
        upto[1][threadIdx.x] = c != 0;
        __syncthreads();
        for (uint32_t off = 1; off < 256; off <<= 1) {
            uint32_t a = 0, b = 0;
            if (threadIdx.x >= off) {
                a = upto[0][threadIdx.x - off];
                b = upto[1][threadIdx.x - off];
            }
            __syncthreads();
            upto[0][threadIdx.x] += a;
            upto[1][threadIdx.x] += b;
            __syncthreads();
        }
        if (c) {
            const uint32_t o = ent0 + upto[0][threadIdx.x] - c, q = seg0 + upto[1][threadIdx.x] - 1u;
            if (q < tile.n_seg && o + c <= kRowChunk * tile.n_chunks) {  // as counted
                seg_cell[tile.seg_first + q] = g.seg_cell[s];
                for (uint32_t k = 0; k < c; ++k) {
                    const uint64_t at = (uint64_t)kRowChunk * tile.c0 + o + k;
                    val[at] = g.val[lo + k];
                    const uint32_t r = g.row[lo + k] - r0, i = (o + k) % kRowChunk;
                    row[at] = (uint8_t)r;
                    if (r >> 8) {
                        RowChunk &ch = chunks[tile.c0 + (o + k) / kRowChunk];
                        atomicOr(reinterpret_cast<unsigned long long *>(i & 1u ? &ch.up_odd : &ch.up_even), 1ull << (i / 2));
                    }
                }
                // the chunk the segment starts in, and the ones that start in it
                if (const uint32_t i = o % kRowChunk) {
                    RowChunk &ch = chunks[tile.c0 + o / kRowChunk];
                    atomicOr(reinterpret_cast<unsigned long long *>(i & 1u ? &ch.odd : &ch.even), 1ull << ((i - 1) / 2));
                }
                for (uint32_t j = (o + kRowChunk - 1) / kRowChunk; kRowChunk * j < o + c; ++j) chunks[tile.c0 + j].seg0 = q;
            }
        }
        ent0 += upto[0][255];
        seg0 += upto[1][255];
        __syncthreads();
    }
}

// OR of v over each group of 8 lanes (every lane gets it).
__device__ __forceinline__ uint32_t or8(uint32_t v)
{
    v |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xB1, 0xF, 0xF, false);   // lane ^ 1
    v |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x4E, 0xF, 0xF, false);   // lane ^ 2
    return v | (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x141, 0xF, 0xF, false);  // 7 - lane of 8
}

// The word masks of a group of 8 lanes, whose lane y holds 8 consecutive
// cells of the word at src (row y of its 8 x 8 block, or with z-order ids its
// cells 8y ..), P bytes each: mask[p] has a bit for every cell whose byte p is
// not zero.  The cells start at a multiple of 8 bytes from O.  SHIFT: O is not
// dword aligned; the lane reads the 2 P + 1 aligned dwords its cells touch and
// shifts their bits (loads of these lengths from odd addresses made 100,000
// random rows x 128^2, 256 words to a tile, take 36.1 us with 4 propositions and
// 21.2 with 2; so 20.0 and 14.9, dword aligned 18.1 and 12.3; the split of
// sparse.hip 18.7 and 16.3).
template <uint32_t P, bool SHIFT>
__device__ __forceinline__ void word_masks(const uint8_t *src, uint32_t y, uint32_t morton, uint64_t (&mask)[P])
{
    const uint32_t mis = SHIFT ? (uint32_t)(reinterpret_cast<uintptr_t>(src) & 3u) : 0u;  // 1 .. 3 if SHIFT
    constexpr uint32_t N = 2 * P + (SHIFT ? 1 : 0);
    uint32_t d[N];
    __builtin_memcpy(d, __builtin_assume_aligned(src - mis, 4), 4 * N);
    uint32_t bits = 0;  // bit P x + p: byte p of cell x
#pragma unroll
    for (uint32_t k = 0; k < 2 * P; ++k) bits |= nz_bytes(d[k]) << (4 * k);
    if constexpr (SHIFT) {
        const uint32_t last = nz_bytes(d[2 * P]);
        bits = P == 4 ? __builtin_amdgcn_alignbit(last, bits, mis) : (bits | last << (8 * (P & 3u))) >> mis;
    }
#pragma unroll
    for (uint32_t p = 0; p < P; ++p) {
        uint32_t lo = 0, hi = 0;
        if (morton) {
            uint32_t b = 0;
#pragma unroll
            for (uint32_t x = 0; x < 8; ++x) b |= ((bits >> (P * x + p)) & 1u) << x;
            (y < 4 ? lo : hi) = b << (8 * (y & 3u));
        } else {
            // cell (x, y) is bit z of the mask, x taking z's odd bits
#pragma unroll
            for (uint32_t x = 0; x < 4; ++x) {
                lo |= ((bits >> (P * x + p)) & 1u) << (((x & 1u) << 1) | ((x & 2u) << 2));
                hi |= ((bits >> (P * (x + 4) + p)) & 1u) << (((x & 1u) << 1) | ((x & 2u) << 2));
            }
            const uint32_t sh = (y & 1u) | ((y & 2u) << 1) | ((y & 4u) << 2);
            lo <<= sh;
            hi <<= sh;
        }
        mask[p] = ((uint64_t)or8(hi) << 32) | or8(lo);
    }
}

// One workgroup per tile: masks of the tile's words into LDS (eight lanes per
// word, each reading a row of its cells), then the tile's chunks of 128 entries dealt to
// the wavefronts in turn, each lane ORing its entry's label into its row's
// LDS accumulator, then the rows' label bytes.
//
// Bound by the entries, 9 bytes each, read once with the chunk records (40
// bytes per 128 entries) kRowAhead chunks before they are used; every load is
// in bounds, the wavefront's last chunk being read again past its end.  Two
// entries per lane, so that a load takes 16 bytes of each: with 8 (64-entry
// chunks) the largest system took 70 us and not 61.
//
// 1,097,702 transitions, 1 proposition: 61.5 us per frame, 345 MB, 5.6 TB/s; the
// split of sparse.hip took 5.8 us to pack the masks and clear L, then 71.8.
// 154,776, 2 propositions: 15.9 us against 5.6 + 16.6, 21.0 per call.
constexpr int kRowWaves = 8;
constexpr int kRowAhead = 3;

template <uint32_t P, bool SHIFT>
__global__ void __launch_bounds__(64 * kRowWaves, 8)
k_label_row_tiles(const RowTile *__restrict__ tiles, const RowChunk *__restrict__ chunks,
                  const uint32_t *__restrict__ seg_cell, const uint8_t *__restrict__ rows,
                  const uint64_t *__restrict__ vals, const uint8_t *__restrict__ O, uint32_t nx, uint32_t morton,
                  uint32_t rows_per_tile, uint64_t n_traj, uint8_t *__restrict__ L)
{
    constexpr int R = kRowAhead + 1;
    __shared__ uint32_t acc[kRowTileMost];
    extern __shared__ uint64_t msk[];  // [n_seg][P]
    const uint32_t lane = threadIdx.x & 63;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const RowTile t = tiles[blockIdx.x];
    const uint32_t n = t.n_chunks > wave ? (t.n_chunks - wave + kRowWaves - 1) / kRowWaves : 0u;
    const uint32_t c0 = t.c0 + wave;
    struct Stage {
        uint32_t rec;    // lanes 0-8: the chunk's record
        ulonglong2 x;    // this lane's two word values
        uint32_t r;      // their rows in the tile, a byte each
    };
    Stage st[R];
    auto fetch = [&](Stage &q, uint32_t k) {
        const uint64_t c = c0 + (uint64_t)min(k, n - 1) * kRowWaves;
        q.rec = reinterpret_cast<const uint32_t *>(chunks + c)[min(lane, 8u)];
        q.x = reinterpret_cast<const ulonglong2 *>(vals + kRowChunk * c)[lane];
        q.r = reinterpret_cast<const uint16_t *>(rows + kRowChunk * c)[lane];
    };
    if (n > 0) {
#pragma unroll
        for (int k = 0; k < kRowAhead; ++k) fetch(st[k], k);
    }
    for (uint32_t i = threadIdx.x; i < kRowTileMost; i += 64 * kRowWaves) acc[i] = 0;
    {
        const uint32_t y = lane & 7u;
        const uint64_t off = morton ? 8u * y : (uint64_t)y * nx;
        for (uint32_t i = threadIdx.x / 8; i < t.n_seg; i += 8 * kRowWaves) {  // whole groups of lanes
            uint64_t m[P];
            word_masks<P, SHIFT>(O + (seg_cell[t.seg_first + i] + off) * P, y, morton, m);
#pragma unroll
            for (uint32_t p = 0; p < P; ++p)
                if (y == p) msk[i * P + p] = m[p];
        }
    }
    __syncthreads();
    for (uint32_t k0 = 0; k0 < n; k0 += R) {
#pragma unroll
        for (int u = 0; u < R; ++u) {
            const uint32_t k = k0 + u;
            fetch(st[(u + kRowAhead) % R], k + kRowAhead);
            if (k < n) {
                const Stage &q = st[u];
                auto word = [&](int i) { return (uint32_t)__builtin_amdgcn_readlane((int)q.rec, i); };
                auto bits = [&](int i) { return (uint64_t)word(2 * i + 1) << 32 | word(2 * i); };
                const uint64_t even = bits(0), odd = bits(1);
                const uint32_t s = __builtin_amdgcn_mbcnt_hi((uint32_t)(odd >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)odd,
                    __builtin_amdgcn_mbcnt_hi((uint32_t)(even >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)even, word(8)))));
                const uint32_t next = __builtin_amdgcn_inverse_ballot_w64(odd) ? 1u : 0u;
                const uint32_t ra = (q.r & 0xFFu) + (__builtin_amdgcn_inverse_ballot_w64(bits(2)) ? 256u : 0u);
                const uint32_t rb = (q.r >> 8) + (__builtin_amdgcn_inverse_ballot_w64(bits(3)) ? 256u : 0u);
                const uint64_t *m = msk + s * P, *m2 = m + next * P;
                uint32_t a = 0, b = 0;
#pragma unroll
                for (uint32_t p = 0; p < P; ++p) {
                    a |= (uint32_t)((q.x.x & m[p]) != 0ull) << p;
                    b |= (uint32_t)((q.x.y & m2[p]) != 0ull) << p;
                }
                // entries that fill a tile's last chunk are zero
                if (a) __hip_atomic_fetch_or(acc + ra, a, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                if (b) __hip_atomic_fetch_or(acc + rb, b, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            }
        }
    }
    __syncthreads();
    const uint64_t t0 = (uint64_t)blockIdx.x * rows_per_tile;
    static_assert(kRowTileMost <= 64 * kRowWaves, "one thread per row");
    if (threadIdx.x < rows_per_tile && t0 + threadIdx.x < n_traj) {
        const uint32_t v = spread_nib(acc[threadIdx.x]);
        __builtin_memcpy(L + (t0 + threadIdx.x) * P, &v, P);
    }
}

template <uint32_t P>
hipError_t launch(const lbl_abs *a, const RowTiles &t, const uint8_t *O, uint8_t *L, hipStream_t s)
{
    const auto kernel = reinterpret_cast<uintptr_t>(O) & 3u ? &k_label_row_tiles<P, true> : &k_label_row_tiles<P, false>;
    hipLaunchKernelGGL(kernel, dim3(t.n_tiles), dim3(64 * kRowWaves), (size_t)t.max_seg * P * sizeof(uint64_t),
                       s, t.tiles, t.chunks, t.seg_cell, t.row, t.val, O, a->nx, (uint32_t)a->order.morton,
                       t.rows_per_tile, a->n_traj, L);
    return hipGetLastError();
}

}  // namespace

RowTiles::~RowTiles()
{
    (void)hipFree(tiles);
    (void)hipFree(chunks);
    (void)hipFree(seg_cell);
    (void)hipFree(row);
    (void)hipFree(val);
}

// Measured, us per frame at 64, 128 and 256 rows, 2 propositions: 34,639
// transitions 9.2, 14.0, 13.6; 60,000 10.0, 10.5, 12.8; 125,000 16.2, 13.8,
// 13.6; 200,000 21.5, 18.5, 18.5; 154,776 with 256 and 512 16.3, 17.0;
// 1,097,702, 1 proposition, with 128, 256, 512 and 1,024 80.8, 68.9, 61.4, 65.  A tile costs about 5 us of latency (its record,
// its words, O, and only then its entries), so many small ones are slow, and
// fewer than about two per CU leave CUs idle.
uint32_t rows_per_tile(uint64_t n_traj)
{
    return n_traj >= (1u << 18) ? 512 : n_traj >= (1u << 17) ? 256 : n_traj >= (1u << 16) ? 128 : 64;
}

// Measured against the split of sparse.hip, us per frame: segments of 19 entries
// (60,000 transitions, 4 propositions) 14.2 against 15.4; 70,000 segments of
// 4.4 entries, at most 256 to a tile, 9.1 against 12.1; 46,000 of 9 entries, at
// most 359, 9.1 against 13.0; a million of 2.6, up to 962 to a tile, 14.7
// against 12.7 with 1 proposition and 31.5 against 14.3 with 4.
bool row_tiles_pay(uint64_t nnz, uint64_t n_seg, uint32_t max_seg)
{
    return nnz != 0 && ((n_seg <= nnz / 16 && max_seg <= kRowTileSegs) || (n_seg <= (1u << 17) && max_seg <= 384));
}

lbl_status build_row_tiles(const lbl_abs *a, const SparseLayout &sp, const std::vector<uint64_t> &seg_start,
                           const std::vector<uint32_t> &seg_word, const std::vector<uint64_t> &rb_seg,
                           std::unique_ptr<RowTiles> *out)
{
    const uint64_t n_seg = seg_word.size();
    if (sp.nnz == 0 || n_seg >= (1ull << 32)) return LBL_OK;
    std::unique_ptr<RowTiles> t(new RowTiles);
    t->rows_per_tile = rows_per_tile(a->n_traj);
    const uint64_t n_tiles = (a->n_traj + t->rows_per_tile - 1) / t->rows_per_tile;
    if (n_tiles >= (1ull << 31)) return LBL_OK;
    t->n_tiles = (uint32_t)n_tiles;
    std::vector<uint32_t> cell(n_seg);
    for (uint64_t s = 0; s < n_seg; ++s)
        cell[s] = a->order.morton ? seg_word[s] * 64u : a->order.word_cell[(uint64_t)seg_word[s] * 64];
    struct Free {
        void operator()(void *p) const { (void)hipFree(p); }
    };
    std::unique_ptr<void, Free> d_seg, d_rb, d_cell, d_cnt;
    auto up = [](std::unique_ptr<void, Free> &d, const void *src, size_t bytes) -> lbl_status {
        void *p = nullptr;
        LBL_HIP_TRY(hipMalloc(&p, std::max<size_t>(bytes, 1)));
        d.reset(p);
        if (src) LBL_HIP_TRY(hipMemcpy(p, src, bytes, hipMemcpyHostToDevice));
        return LBL_OK;
    };
    lbl_status st = up(d_seg, seg_start.data(), seg_start.size() * sizeof(uint64_t));
    if (st == LBL_OK) st = up(d_rb, rb_seg.data(), rb_seg.size() * sizeof(uint64_t));
    if (st == LBL_OK) st = up(d_cell, cell.data(), n_seg * sizeof(uint32_t));
    if (st == LBL_OK) st = up(d_cnt, nullptr, 2 * n_tiles * sizeof(uint32_t));
    if (st != LBL_OK) return st;
    const Segments g{static_cast<uint64_t *>(d_seg.get()), static_cast<uint64_t *>(d_rb.get()),
                     static_cast<uint32_t *>(d_cell.get()), sp.row, sp.val};
    uint32_t *cnt = static_cast<uint32_t *>(d_cnt.get());
    hipLaunchKernelGGL(k_tile_count, dim3(t->n_tiles), dim3(256), 0, nullptr, g, t->rows_per_tile, cnt, cnt + n_tiles);
    LBL_HIP_TRY(hipGetLastError());
    std::vector<uint32_t> h(2 * n_tiles);
    LBL_HIP_TRY(hipMemcpy(h.data(), cnt, h.size() * sizeof(uint32_t), hipMemcpyDeviceToHost));
    std::vector<RowTile> tiles(n_tiles);
    uint64_t c = 0, q = 0;
    for (uint64_t i = 0; i < n_tiles; ++i) {
        const uint32_t nc = (h[i] + kRowChunk - 1) / kRowChunk;
        tiles[i] = RowTile{(uint32_t)c, nc, (uint32_t)q, h[n_tiles + i]};
        c += nc;
        q += h[n_tiles + i];
        t->max_seg = std::max(t->max_seg, h[n_tiles + i]);
    }
    if (!row_tiles_pay(sp.nnz, q, t->max_seg) || c >= (1ull << 32) || q >= (1ull << 32)) return LBL_OK;
    t->n_chunks = c;
    t->n_seg = q;
    LBL_HIP_TRY(hipMalloc(&t->tiles, n_tiles * sizeof(RowTile)));
    LBL_HIP_TRY(hipMemcpy(t->tiles, tiles.data(), n_tiles * sizeof(RowTile), hipMemcpyHostToDevice));
    LBL_HIP_TRY(hipMalloc(&t->chunks, c * sizeof(RowChunk)));
    LBL_HIP_TRY(hipMemset(t->chunks, 0, c * sizeof(RowChunk)));
    LBL_HIP_TRY(hipMalloc(&t->seg_cell, q * sizeof(uint32_t)));
    LBL_HIP_TRY(hipMalloc(&t->row, kRowChunk * c));
    LBL_HIP_TRY(hipMemset(t->row, 0, kRowChunk * c));
    LBL_HIP_TRY(hipMalloc(&t->val, kRowChunk * c * sizeof(uint64_t)));
    LBL_HIP_TRY(hipMemset(t->val, 0, kRowChunk * c * sizeof(uint64_t)));
    hipLaunchKernelGGL(k_tile_fill, dim3(t->n_tiles), dim3(256), 0, nullptr, g, t->rows_per_tile, t->tiles, t->val, t->row,
                       t->seg_cell, t->chunks);
    LBL_HIP_TRY(hipGetLastError());
    LBL_HIP_TRY(hipDeviceSynchronize());
    *out = std::move(t);
    return LBL_OK;
}

lbl_status run_row_tiles(const lbl_abs *a, const RowTiles &t, const uint8_t *O, uint32_t n_props, uint8_t *L, hipStream_t s)
{
    switch (n_props) {
    case 1: LBL_HIP_TRY(launch<1>(a, t, O, L, s)); break;
    case 2: LBL_HIP_TRY(launch<2>(a, t, O, L, s)); break;
    case 3: LBL_HIP_TRY(launch<3>(a, t, O, L, s)); break;
    case 4: LBL_HIP_TRY(launch<4>(a, t, O, L, s)); break;
    default: LBL_REQUIRE(false, "row tiles label at most 4 propositions");
    }
    return LBL_OK;
}

}  // namespace lbl
