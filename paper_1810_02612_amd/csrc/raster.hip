// Proposition regions of a frame rasterized into O on the device (Sec. 4.1
// encoding: a cell's entry is 1 iff the region intersects the cell, read as
// an overlap of positive area with the closed cell square).
//
// One workgroup takes a tile of 512 cells (fewer on small grids, wavefronts then
// sharing the shapes of the same cells): it lists the shapes whose bounding
// box meets the tile, then one lane per cell tests the listed shapes, collects
// its propositions as a bit mask, and the wavefront writes its 64 cells' bytes
// as one block.  Every byte of O is written once.  The tests are exact:
//   rectangle: on both axes the overlap length, min of the upper ends minus
//              max of the lower ends, is positive, that is, each of the two
//              intervals starts before the other ends;
//   disc:      the squared distance from the centre to the square's nearest
//              point is below the squared radius.
// Cell bounds are ix * cell and ix * cell + cell in double precision, and
// products are not fused with sums, so every decision is the one the
// definition gives in IEEE double arithmetic.
//
// At 512 x 512 x 64 with 357 shapes (16.8 MB written, 2.4 us at the rate a
// fill reaches) the kernel takes 10.0 us: 2.5 us of vector instructions, the
// wait for the shapes, and the drain of the writes; 12.5-14 us per call with
// the upload of the shapes (a 3 us copy).  Clearing O and then storing single
// bytes, one workgroup group per shape, took 6.5 + 24 us, the bytes of a cell
// lying 64 apart; 30-31 us per call.  Tiles of 256 cells: 10.3 us.
#include <algorithm>
#include <cmath>

#include "emit.h"
#include "lbl_internal.h"

namespace lbl {
namespace {

constexpr uint32_t kRasterWaves = 8;  // wavefronts per workgroup

// The cell coordinate in a z-order index: every second bit of z from bit 0
// (y) or, of z >> 1, x.
__device__ __forceinline__ uint32_t z_coord(uint32_t z)
{
    z &= 0x55555555u;
    z = (z | (z >> 1)) & 0x33333333u;
    z = (z | (z >> 2)) & 0x0F0F0F0Fu;
    z = (z | (z >> 4)) & 0x00FF00FFu;
    return (z | (z >> 8)) & 0xFFFFu;
}

// A shape as the cells test it: a rectangle's ends on both axes, or a disc's
// centre and squared radius.
struct Listed {
    double a, b, c, d;  // rectangle: x from a to b, y from c to d; disc: centre (a, b), c = radius squared
};

// Tiles of 64 CW cells, CW wavefronts to their cells and 8 / CW to share the
// listed shapes of the same cells: with row-major ids 64 x CW cells, wavefront w
// taking row w % CW of the tile; with z-order ids 64 CW consecutive ids,
// wavefront w taking ids 64 (w % CW) ...
template <uint32_t CW>
__global__ void __launch_bounds__(64 * kRasterWaves)
k_raster_tiles(const lbl_shape *__restrict__ shapes, uint32_t n_shapes, uint32_t nx, uint32_t ny, double cell,
               uint32_t n_props, uint32_t morton, uint32_t n_tiles, uint8_t *__restrict__ O)
{
#pragma clang fp contract(off)
    constexpr uint32_t kMost = 64 * kRasterWaves;  // shapes looked at (and listed) at a time
    constexpr uint32_t kShare = kRasterWaves / CW;
    __shared__ uint64_t part_mask[kShare > 1 ? kShare - 1 : 1][CW][64];
    __shared__ Listed list[kMost];
    __shared__ uint32_t info[kMost];  // proposition, bit 31: rectangle
    __shared__ uint32_t n_listed;
    __shared__ uint32_t stage[kRasterWaves][kStageWords];
    const uint32_t lane = threadIdx.x & 63;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t cw = wave % CW, part = wave / CW;
    for (uint32_t tile = blockIdx.x; tile < n_tiles; tile += gridDim.x) {
        // the tile's cells [tx, tx + tw) x [ty, ty + th), this lane's cell, the
        // id of the wavefront's first cell and its number of cells
        uint32_t tx, ty, tw, th, ix, iy, n;
        uint64_t id0;
        if (morton) {
            const uint32_t z0 = tile * (64 * CW), z = z0 + 64 * cw + lane;
            tx = z_coord(z0 >> 1);
            ty = z_coord(z0);
            tw = CW >= 4 ? 16 : 8;
            th = CW == 8 ? 32 : CW == 1 ? 8 : 16;
            ix = z_coord(z >> 1);
            iy = z_coord(z);
            id0 = z0 + 64u * cw;
            n = id0 < (uint64_t)nx * ny ? 64u : 0u;
        } else {
            const uint32_t across = (nx + 63) / 64;
            tx = tile % across * 64u;
            ty = tile / across * CW;
            tw = 64;
            th = CW;
            ix = tx + lane;
            iy = ty + cw;
            id0 = (uint64_t)iy * nx + tx;
            n = min(64u, nx - tx);  // ny is a multiple of 8
        }
        const double x0 = (double)ix * cell, x1 = x0 + cell;
        const double y0 = (double)iy * cell, y1 = y0 + cell;
        const double tx0 = (double)tx * cell, tx1 = (double)(tx + tw - 1) * cell + cell;
        const double ty0 = (double)ty * cell, ty1 = (double)(ty + th - 1) * cell + cell;
        uint64_t mask = 0;
        for (uint32_t s0 = 0; s0 < n_shapes; s0 += kMost) {
            if (threadIdx.x == 0) n_listed = 0;
            __syncthreads();
            const uint32_t s = s0 + threadIdx.x;
            if (s < n_shapes) {
                const lbl_shape sh = shapes[s];
                const bool rect = sh.kind == LBL_SHAPE_RECT;
                const double hx = sh.a, hy = rect ? sh.b : sh.a;
                const double xl = sh.cx - hx, xh = sh.cx + hx, yl = sh.cy - hy, yh = sh.cy + hy;
                // on both axes the shape must start before the tile's last
                // cell ends and end after its first cell starts: a cell that
                // the tests below accept lies between the same rounded ends
                bool in = xl <= tx1 && tx0 <= xh && yl <= ty1 && ty0 <= yh;
                if (rect) in = in && xl < xh && yl < yh;  // without an inside it overlaps nothing
                if (in) {
                    const uint32_t i = atomicAdd(&n_listed, 1u);  // < kMost: one per thread
                    list[i] = rect ? Listed{xl, xh, yl, yh} : Listed{sh.cx, sh.cy, sh.a * sh.a, 0.0};
                    info[i] = sh.prop | (rect ? 0x80000000u : 0u);
                }
            }
            __syncthreads();
            const uint32_t m = n_listed;
            for (uint32_t i = part; i < m; i += kShare) {
                const uint32_t f = (uint32_t)__builtin_amdgcn_readfirstlane((int)info[i]);
                const Listed q = list[i];
                bool hit;
                if (f >> 31) {
                    hit = q.a < x1 && x0 < q.b && q.c < y1 && y0 < q.d;
                } else {
                    const double ex = q.a - fmin(fmax(q.a, x0), x1), ey = q.b - fmin(fmax(q.b, y0), y1);
                    hit = ex * ex + ey * ey < q.c;
                }
                mask |= hit ? 1ull << (f & 63u) : 0ull;
            }
            __syncthreads();  // the list is filled again
        }
        if constexpr (kShare > 1) {
            if (part) part_mask[part - 1][cw][lane] = mask;
            __syncthreads();
            if (part == 0)
                for (uint32_t k = 0; k + 1 < kShare; ++k) mask |= part_mask[k][cw][lane];
            __syncthreads();  // the next tile's masks go to the same place
            if (part) continue;
        }
        uint8_t *dst = O + id0 * n_props;
        if (n == 0) continue;  // whole wavefronts (every barrier is behind them)
        if ((n_props & 15u) == 0 && (reinterpret_cast<uintptr_t>(O) & 15u) == 0)
            emit_units(lane, n, mask, dst, n_props / 16);
        else
            emit_block(stage[wave], lane, n, mask, dst, n_props);
    }
}

}  // namespace
}  // namespace lbl

using namespace lbl;

lbl_status lbl_raster_frame(const lbl_grid *g, double cell_m, const lbl_shape *shapes, uint64_t n_shapes,
                            uint32_t n_props, uint8_t *O, void *hip_stream)
{
    clear_error();
    LBL_REQUIRE(g != nullptr && O != nullptr, "grid or O is null");
    LBL_REQUIRE(n_shapes == 0 || shapes != nullptr, "shapes is null");
    {
        const lbl_status gst = check_grid(g);
        if (gst != LBL_OK) return gst;
    }
    LBL_REQUIRE(n_props >= 1 && n_props <= 64, "n_props must be in [1, 64]");
    LBL_REQUIRE(std::isfinite(cell_m) && cell_m > 0.0, "cell_m must be finite and positive");
    LBL_REQUIRE(n_shapes < (1ull << 31), "too many shapes");
    for (uint64_t i = 0; i < n_shapes; ++i) {
        const lbl_shape &s = shapes[i];
        LBL_REQUIRE(s.kind == LBL_SHAPE_RECT || s.kind == LBL_SHAPE_DISC, "unknown shape kind");
        LBL_REQUIRE(s.prop < n_props, "shape prop >= n_props");
        LBL_REQUIRE(std::isfinite(s.cx) && std::isfinite(s.cy) && std::isfinite(s.a) && std::isfinite(s.b),
                    "shape coordinates and sizes must be finite");
        LBL_REQUIRE(s.a >= 0.0 && (s.kind == LBL_SHAPE_DISC || s.b >= 0.0), "shape sizes must be non-negative");
    }
    hipStream_t st = reinterpret_cast<hipStream_t>(hip_stream);
    lbl_shape *d_shapes = nullptr;
    if (n_shapes) {
        void *ws = nullptr;
        lbl_status rc = workspace(st, n_shapes * sizeof(lbl_shape), &ws);
        if (rc != LBL_OK) return rc;
        d_shapes = static_cast<lbl_shape *>(ws);
        LBL_HIP_TRY(hipMemcpyAsync(d_shapes, shapes, n_shapes * sizeof(lbl_shape), hipMemcpyHostToDevice, st));
    }
    const bool morton = g->cell_order == LBL_MORTON;
    const uint64_t n_cells = (uint64_t)g->nx * g->ny;
    // the largest tiles that give two workgroups per CU: a tile's shapes are
    // listed once, but testing them is one wavefront's chain.  Us per call with
    // tiles of 512, 256, 128 and 64 cells: 64^2 x 39 15.0, 12.1, 12.2, 12.2;
    // 128^2 x 56 13.5, 11.7, 11.5, 11.9; 392 x 336 x 52 11.7, 11.5, 11.5, 13.0;
    // 512^2 x 64 13.0, 12.7, 14.7, 19.3
    auto tiles_of = [&](uint32_t cw) {
        return morton ? (n_cells + 64 * cw - 1) / (64 * cw) : (uint64_t)((g->nx + 63) / 64) * (g->ny / cw);
    };
    uint32_t cw = kRasterWaves;
    while (cw > 1 && tiles_of(cw) < 512) cw /= 2;
    const auto kernel = cw == 8 ? &k_raster_tiles<8> : cw == 4 ? &k_raster_tiles<4> : cw == 2 ? &k_raster_tiles<2> : &k_raster_tiles<1>;
    const uint64_t tiles = tiles_of(cw);
    hipLaunchKernelGGL(kernel, dim3((unsigned)std::min<uint64_t>(tiles, 1u << 20)), dim3(64 * kRasterWaves), 0,
                       st, d_shapes, (uint32_t)n_shapes, g->nx, g->ny, cell_m, n_props, (uint32_t)morton,
                       (uint32_t)tiles, O);
    LBL_HIP_TRY(hipGetLastError());
    return LBL_OK;
}
