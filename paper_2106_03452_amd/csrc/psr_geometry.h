// Work decomposition shared by the host launch code and the device kernels.
#pragma once

// Threads per workgroup of the column passes and of the row passes.
#ifndef PSR_COL_THREADS
#define PSR_COL_THREADS 256
#endif
#ifndef PSR_ROW_THREADS
#define PSR_ROW_THREADS 512
#endif
#ifndef PSR_J0_THREADS
#define PSR_J0_THREADS 256
#endif
// The j0 passes below 256: smaller workgroups, more of them per CU.
#ifndef PSR_J0_THREADS_SMALL
#define PSR_J0_THREADS_SMALL 128
#endif
// Smallest grid size whose plane passes split each plane into two parts.
#ifndef PSR_PLANE_SPLIT_MIN
#define PSR_PLANE_SPLIT_MIN 256
#endif

namespace psr {

// Work split of a length-L line FFT: plan_TPL(L) threads per line, each
// holding plan_E(L) elements in registers.
__host__ __device__ constexpr int plan_E(int L) { return L < 16 ? L : 16; }
__host__ __device__ constexpr int plan_TPL(int L) { return L / plan_E(L); }
__host__ __device__ constexpr int imin(int a, int b) { return a < b ? a : b; }

// Column passes (FFT along j1 / j0, length res): tile_cols(res) lines per
// workgroup of cols_block(res) threads.
__host__ __device__ constexpr int tile_cols(int res) { return imin(res, PSR_COL_THREADS / plan_TPL(res)); }
__host__ __device__ constexpr int cols_block(int res) { return tile_cols(res) * plan_TPL(res); }

// The fused j0 passes (three transforms per line) may use their own tile.
__host__ __device__ constexpr int tile_j0(int res) {
  return imin(res, (res < 256 ? PSR_J0_THREADS_SMALL : PSR_J0_THREADS) / plan_TPL(res));
}
__host__ __device__ constexpr int j0_block(int res) { return tile_j0(res) * plan_TPL(res); }

// Row passes (splat + r2c and c2r + gather along j2; half-length complex
// lines of res/2): tile_rows(res) consecutive j1 lines of one j0 per
// workgroup of rows_block(res) threads. Points are binned by these tiles,
// two bins per tile (floor column b1 inside the tile, or on its last column,
// which also reaches the next tile): bin = b0 * 2 row_tiles(res) +
// 2 (b1 / tile_rows(res)) + (b1 is the tile's last column).
// At 256^3 a tile is 32 rows (256 threads, four workgroups per CU): fewer rows
// without a point are transformed than with 64 (P1 39.5 -> 32.8 us, B1 29.8 ->
// 23.1, B5 33.7 -> 28.5 with 100k points of a surface) for twice the bins (binning
// +1 us). At 512^3 the bitmap of the tiles (8192 bits) is full with 32 rows.
__host__ __device__ constexpr int tile_rows(int res) {
  // where a plane pass splits a plane of res <= 128 in two, bins must not be coarser than a part
  return imin(imin(res, (res == 256 ? 256 : PSR_ROW_THREADS) / plan_TPL(res / 2)),
              (res >= PSR_PLANE_SPLIT_MIN && res <= 128) ? res / 2 : res);
}
// Plane passes: parts per plane (one workgroup each), as many chunks of rows as
// the forward direction takes a plane in, and the FP64 sums that a single
// backward's first pass leaves (one per plane and chunk) and its second adds.
__host__ __device__ constexpr int plane_parts(int res) { return res >= PSR_PLANE_SPLIT_MIN ? 2 : 1; }
__host__ __device__ constexpr int plane_sums(int res) { return res * plane_parts(res); }
__host__ __device__ constexpr int rows_block(int res) { return tile_rows(res) * plan_TPL(res / 2); }
// Workgroup size of the row passes (8 and 16, 256 and 512; the plane passes run
// between). At 8 and 16 a row tile is the whole plane and its transforms take one
// thread per row; the workgroup is widened to 256 threads for the loops over the
// plane's points and samples, the threads beyond the rows transforming scratch
// rows.
__host__ __device__ constexpr int rows_wg(int res) { return res <= 16 ? 256 : rows_block(res); }
// LDS rows of a row-pass workgroup: the tile's rows plus the scratch rows
__host__ __device__ constexpr int rows_lds(int res) {
  return rows_wg(res) / plan_TPL(res / 2) > tile_rows(res) ? rows_wg(res) / plan_TPL(res / 2) : tile_rows(res);
}
__host__ __device__ constexpr int row_tiles(int res) { return res / tile_rows(res); }
__host__ __device__ constexpr int num_bins(int res) { return 2 * res * row_tiles(res); }

}  // namespace psr
