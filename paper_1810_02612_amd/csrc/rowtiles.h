// Row tiles of a sparse layout (frames of at most 4 propositions).
#pragma once

#include <memory>
#include <vector>

#include "lbl_internal.h"

namespace lbl {

struct SparseLayout;

// 128 consecutive entries of a tile, lane l of a wavefront taking entries 2l
// and 2l + 1.  Bit l of odd (even) is set iff entry 2l + 1 (2l + 2) begins a
// new segment; seg0 is the segment of entry 0, counted from the tile's first;
// bit l of up_even (up_odd) is bit 8 of the row of entry 2l (2l + 1).
constexpr uint32_t kRowChunk = 128;
struct RowChunk {
    uint64_t even, odd;
    uint64_t up_even, up_odd;
    uint32_t seg0;
    uint32_t pad;
};

// The entries of rows [tile * rows_per_tile, ...): chunks c0 .. + n_chunks
// (chunk c's entries from kRowChunk * c, zeros filling the last), in segments seg_first .. + n_seg (one per word the rows meet).
struct RowTile {
    uint32_t c0, n_chunks;
    uint32_t seg_first, n_seg;
};

struct RowTiles {
    uint32_t rows_per_tile = 0;   // 64, 128, 256 or 512
    uint32_t n_tiles = 0;
    uint32_t max_seg = 0;         // segments of a tile at most
    uint64_t n_chunks = 0, n_seg = 0;
    RowTile *tiles = nullptr;     // device [n_tiles]
    RowChunk *chunks = nullptr;   // device [n_chunks]
    uint32_t *seg_cell = nullptr; // device [n_seg] the first cell id of the segment's word
    uint8_t *row = nullptr;       // device [kRowChunk * n_chunks] row in the tile (its low 8 bits)
    uint64_t *val = nullptr;      // device [kRowChunk * n_chunks] word value
    RowTiles() = default;
    RowTiles(const RowTiles &) = delete;
    RowTiles &operator=(const RowTiles &) = delete;
    ~RowTiles();
    size_t bytes() const { return n_tiles * sizeof(RowTile) + n_chunks * (sizeof(RowChunk) + kRowChunk * 9) + n_seg * sizeof(uint32_t); }
};

constexpr uint32_t kRowTileMost = 512;  // rows of a tile at most
// Segments of a tile whose masks fit its workgroup's LDS (32 KiB at 4
// propositions).
constexpr uint32_t kRowTileSegs = 1024;

uint32_t rows_per_tile(uint64_t n_traj);
// Whether a layout of nnz entries whose row tiles have n_seg segments, at
// most max_seg in one tile, is labeled by them.
bool row_tiles_pay(uint64_t nnz, uint64_t n_seg, uint32_t max_seg);

// The row tiles of a's sparse layout (sp's entries still in row and val), or
// null where they do not pay.
lbl_status build_row_tiles(const lbl_abs *a, const SparseLayout &sp, const std::vector<uint64_t> &seg_start,
                           const std::vector<uint32_t> &seg_word, const std::vector<uint64_t> &rb_seg,
                           std::unique_ptr<RowTiles> *out);

// Label a frame of at most 4 propositions (device pointers).
lbl_status run_row_tiles(const lbl_abs *a, const RowTiles &t, const uint8_t *O, uint32_t n_props, uint8_t *L, hipStream_t s);

}  // namespace lbl
