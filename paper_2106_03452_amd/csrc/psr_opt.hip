// gfx950 kernels of the optimisation-based reconstruction loop around the
// solver (Peng et al., "Shape As Points", main Sec. 3.2): points sampled on
// the Marching Cubes mesh (the p_mesh of Eq. 5) with their backward, the
// bidirectional Chamfer loss of Eq. 5 with its gradient, and the connected
// components of the mesh for the resampling from the largest component.
//
// Sampling: FP64 face areas with their running sums per block, then per sample
// a search of u0 * total over the block sums and within the block, and the
// barycentric weights (1 - sqrt(u1), sqrt(u1) (1 - u2), sqrt(u1) u2).
// Chamfer: exact nearest neighbours over spatially sorted tiles whose boxes
// let whole tiles be skipped (the brute-force result: equal distances go to
// the lower index); FP64 sums for the loss.
// Components: label propagation over the triangles (atomic minimum) with
// pointer jumping until no label changes, FP64 areas per label, and the
// label with the greatest area (ties: the lowest label).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <cmath>

#include "psr_opt.h"

namespace psr {
namespace opt {

constexpr int kScanBlock = 1024;  // face areas per scan block
constexpr int kScanTops = 1024;   // block sums that a sampling workgroup scans itself
// samples up to which one wavefront, with the block sums scanned once for it, is
// a workgroup (see k_sample)
constexpr int64_t kSampleFew = 65536;

__device__ __forceinline__ double face_area(const float* __restrict__ v, const int32_t* __restrict__ f, int64_t i) {
  const int64_t i0 = f[3 * i], i1 = f[3 * i + 1], i2 = f[3 * i + 2];
  const double ax = (double)v[3 * i1] - v[3 * i0], ay = (double)v[3 * i1 + 1] - v[3 * i0 + 1],
               az = (double)v[3 * i1 + 2] - v[3 * i0 + 2];
  const double bx = (double)v[3 * i2] - v[3 * i0], by = (double)v[3 * i2 + 1] - v[3 * i0 + 1],
               bz = (double)v[3 * i2 + 2] - v[3 * i0 + 2];
  const double cx = ay * bz - az * by, cy = az * bx - ax * bz, cz = ax * by - ay * bx;
  return 0.5 * sqrt(cx * cx + cy * cy + cz * cz);
}

__global__ __launch_bounds__(256) void k_face_area(const float* __restrict__ v, const int32_t* __restrict__ f,
                                                   int64_t nf, double* __restrict__ a) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i < nf) a[i] = face_area(v, f, i);
}

// inclusive scan over the wavefront
__device__ __forceinline__ double wave_incl_scan(double v) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const double u = __shfl_up(v, d, 64);
    if (lane >= d) v += u;
  }
  return v;
}

// inclusive scan over the workgroup's WAVES wavefronts; sh holds WAVES values
template <int WAVES>
__device__ __forceinline__ double block_incl_scan(double v, double* sh, double& total) {
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  v = wave_incl_scan(v);
  if (lane == 63) sh[wid] = v;
  __syncthreads();
  double before = 0.0, tot = 0.0;
#pragma unroll
  for (int k = 0; k < WAVES; ++k) {
    before += k < wid ? sh[k] : 0.0;
    tot += sh[k];
  }
  total = tot;
  __syncthreads();
  return before + v;
}

// Areas of kScanBlock faces (times the face weights), their running sums
// within the block and the block's sum. One face per thread: the chain of
// loads (indices, corners) is the time, and is paid once. With k_sample, which
// scans the block sums itself, this replaces four launches (areas, block sums,
// their scan, running sums): 10.8 -> 4.5 us for 20000 faces.
__global__ __launch_bounds__(kScanBlock) void k_area_scan(const float* __restrict__ v, const int32_t* __restrict__ f,
                                                          int64_t nf, const float* __restrict__ w,
                                                          double* __restrict__ csum, double* __restrict__ bs) {
  __shared__ double sh[kScanBlock / 64];
  const int64_t i = (int64_t)blockIdx.x * kScanBlock + threadIdx.x;
  double a = 0.0;
  if (i < nf) {
    a = face_area(v, f, i);
    if (w) a *= (double)w[i];
  }
  double tot;
  const double inc = block_incl_scan<kScanBlock / 64>(a, sh, tot);
  if (i < nf) csum[i] = inc;
  if (threadIdx.x == 0) bs[blockIdx.x] = tot;
}

// exclusive scan of the block sums in place (one workgroup); the grand total
// after them. For meshes of more than kScanTops blocks only.
__global__ __launch_bounds__(256) void k_scan_tops(double* __restrict__ bs, int nb) {
  __shared__ double sh[4];
  double carry = 0.0;
  for (int c = 0; c < nb; c += 256) {
    const int i = c + threadIdx.x;
    const double v = i < nb ? bs[i] : 0.0;
    double tot;
    const double inc = block_incl_scan<4>(v, sh, tot);
    if (i < nb) bs[i] = carry + (inc - v);
    carry += tot;
  }
  if (threadIdx.x == 0) bs[nb] = carry;
}

// One sample per thread: the first face whose running area exceeds u0 times the
// total, by its scan block first (TOPS: the workgroup's first wavefront scans the
// block sums in LDS; else they are scanned already), then by binary search within
// the block.
// Cache lines of running areas fetched across the chip bound it: searches in
// rounds of 3, 7 or 31 independent loads have fewer rounds and touch more lines
// (8.0, 9.8 and 18.8 us for 20000 samples of 20000 faces; this 6.9).
// Up to kSampleFew samples a workgroup is one wavefront, so that few samples are
// spread over the chip; beyond, with TOPS, four share the scan and its 8 KB of
// LDS (3M samples of 12 faces 39.7 -> 29.0 us, 300k of 1M faces 63.5 -> 51.4;
// equal at 100k. Without TOPS there is nothing to share: 200k of 2M faces 52.1
// with one wavefront, 54.9 with four).
template <bool TOPS, int BLOCK>
__global__ __launch_bounds__(BLOCK) void k_sample(const float* __restrict__ v, const float* __restrict__ vn,
                                                const int32_t* __restrict__ f, int64_t nf,
                                                const double* __restrict__ csum, const double* __restrict__ bs, int nb,
                                                const float* __restrict__ u, int64_t m, float* __restrict__ pts,
                                                float* __restrict__ nrm, int32_t* __restrict__ face,
                                                float* __restrict__ bary) {
  __shared__ double top[TOPS ? kScanTops + 1 : 1];
  const int64_t i = (int64_t)blockIdx.x * BLOCK + threadIdx.x;
  float u0 = 0.0f, u1 = 0.0f, u2 = 0.0f;
  if (i < m) u0 = u[3 * i], u1 = u[3 * i + 1], u2 = u[3 * i + 2];
  const double* pre = bs;
  if (TOPS) {
    if (threadIdx.x < 64) {
      double carry = 0.0;
      for (int c = 0; c < nb; c += 64) {
        const int b = c + (int)threadIdx.x;
        const double s = b < nb ? bs[b] : 0.0;
        const double inc = wave_incl_scan(s);
        if (b < nb) top[b] = carry + (inc - s);
        carry += __shfl(inc, 63, 64);
      }
      if (threadIdx.x == 0) top[nb] = carry;
    }
    __syncthreads();
    pre = top;
  }
  if (i >= m) return;
  const double t = (double)u0 * pre[nb];
  int bl = 0, bh = nb - 1;
  while (bl < bh) {
    const int mid = (bl + bh) >> 1;
    if (pre[mid + 1] > t) bh = mid;
    else bl = mid + 1;
  }
  const double t0 = pre[bl];
  int64_t lo = (int64_t)bl * kScanBlock;
  int64_t hi = lo + kScanBlock < nf ? lo + kScanBlock - 1 : nf - 1;
  while (lo < hi) {
    const int64_t mid = (lo + hi) >> 1;
    if (t0 + csum[mid] > t) hi = mid;
    else lo = mid + 1;
  }
  const float s = sqrtf(u1);
  const float b0 = 1.0f - s, b1 = s * (1.0f - u2), b2 = s * u2;
  const int64_t i0 = f[3 * lo], i1 = f[3 * lo + 1], i2 = f[3 * lo + 2];
#pragma unroll
  for (int d = 0; d < 3; ++d) pts[3 * i + d] = b0 * v[3 * i0 + d] + b1 * v[3 * i1 + d] + b2 * v[3 * i2 + d];
  if (nrm) {
    float n[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) n[d] = b0 * vn[3 * i0 + d] + b1 * vn[3 * i1 + d] + b2 * vn[3 * i2 + d];
    const float il = rsqrtf(n[0] * n[0] + n[1] * n[1] + n[2] * n[2]);
#pragma unroll
    for (int d = 0; d < 3; ++d) nrm[3 * i + d] = n[d] * il;
  }
  face[i] = (int32_t)lo;
  bary[3 * i] = b0;
  bary[3 * i + 1] = b1;
  bary[3 * i + 2] = b2;
}

__global__ __launch_bounds__(256) void k_fill0(float* __restrict__ x, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) x[i] = 0.0f;
}

// One thread per sample and corner: the atomics, at the rate of the memory side
// that all XCDs share, bound it; nine by one thread took 13.2 us for 20000
// samples, three by each of three take 9.9.
__global__ __launch_bounds__(256) void k_sample_bwd(const int32_t* __restrict__ f, const int32_t* __restrict__ face,
                                                    const float* __restrict__ bary, const float* __restrict__ dp,
                                                    int64_t m, float* __restrict__ dv) {
  const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (t >= 3 * m) return;
  const int64_t i = t / 3;
  const int64_t vi = f[3 * (int64_t)face[i] + (t - 3 * i)];
  const float b = bary[t];
#pragma unroll
  for (int d = 0; d < 3; ++d) atomicAdd(&dv[3 * vi + d], b * dp[3 * i + d]);
}

// ---------------------------------------------------------------------------
// Nearest neighbours for the Chamfer loss: an exact search that skips whole
// tiles of the reference cloud. Both clouds are counting-sorted into
// the cells of a grid over [0,1)^3 (32^3 or 64^3 by cloud size) in Hilbert order
// (points outside fall into the border cells), cut into tiles of kNnTile
// sorted points, and each tile gets its bounding box. A query group
// (kNnTile sorted queries) visits the reference tiles nearest its own box
// first and stops where every remaining box is farther than each query's
// best so far; a tile is skipped when no query's point-to-box bound reaches
// its best. The bounds use the same FP32
// operations as the distances (monotone rounding), so a skipped point is
// strictly farther than a distance already found: the result is the
// brute-force one, the squared FP32 distance minimised with equal distances
// going to the lower reference index.
// ---------------------------------------------------------------------------

// squared length, evaluated the same way for distances and for bounds
__device__ __forceinline__ float nn_d2(float ax, float ay, float az) {
  return __fmaf_rn(az, az, __fmaf_rn(ay, ay, ax * ax));
}

__device__ __forceinline__ int nn_cell_coord(float v, int cb) {
  const int top = (1 << cb) - 1;
  const float c = v * (float)(1 << cb);
  if (!(c >= 0.0f)) return 0;  // also NaN
  return c >= (float)top ? top : (int)c;
}

__device__ __forceinline__ uint32_t nn_spread(uint32_t v) {  // up to 8 bits -> every third bit
  v = (v | (v << 8)) & 0x0300F00Fu;
  v = (v | (v << 4)) & 0x030C30C3u;
  v = (v | (v << 2)) & 0x09249249u;
  return v;
}

// Index of the point's cell along the Hilbert curve of the 2^cb per axis grid
// (Skilling, "Programming the Hilbert curve", 2004: the axes to transpose
// transform), so that consecutive cells are neighbours: in Morton order a tile
// that spans a jump of the curve has a box of up to the whole domain, and a
// query group of 64 surface points scanned 20 tiles on average and 50 at most
// against 15 and 42.
__device__ __forceinline__ int nn_key(float px, float py, float pz, int cb) {
  int x = nn_cell_coord(px, cb), y = nn_cell_coord(py, cb), z = nn_cell_coord(pz, cb);
  for (int q = 1 << (cb - 1); q > 1; q >>= 1) {
    const int p = q - 1;
    x ^= (x & q) ? p : 0;
    const int ty = (x ^ y) & p, fy = y & q;
    x ^= fy ? p : ty;
    y ^= fy ? 0 : ty;
    const int tz = (x ^ z) & p, fz = z & q;
    x ^= fz ? p : tz;
    z ^= fz ? 0 : tz;
  }
  y ^= x;
  z ^= y;
  int t = 0;
  for (int q = 1 << (cb - 1); q > 1; q >>= 1) t ^= (z & q) ? q - 1 : 0;
  return (int)((nn_spread(x ^ t) << 2) | (nn_spread(y ^ t) << 1) | nn_spread(z ^ t));
}

__global__ __launch_bounds__(256) void k_nn_zero(int* __restrict__ cnt, int n) {
  for (int i = blockIdx.x * 256 + threadIdx.x; i < n; i += gridDim.x * 256) cnt[i] = 0;
}

// cell counts of both clouds (x: points [0, nx), y: the next ny)
__global__ __launch_bounds__(256) void k_nn_count(const float* __restrict__ x, int64_t nx,
                                                  const float* __restrict__ y, int64_t ny, int* __restrict__ cnt,
                                                  int cb) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= nx + ny) return;
  const bool isy = i >= nx;
  const float* p = isy ? y + 3 * (i - nx) : x + 3 * i;
  atomicAdd(&cnt[(isy ? 1 << (3 * cb) : 0) + nn_key(p[0], p[1], p[2], cb)], 1);
}

// exclusive scan of one cloud's nc cell counts in place (workgroup = cloud;
// each thread owns nc / 1024 consecutive counts)
__global__ __launch_bounds__(1024) void k_nn_scan(int* __restrict__ cnt, int nc) {
  __shared__ int wsum[16];
  int4* c = reinterpret_cast<int4*>(cnt + (int64_t)blockIdx.x * nc);
  const int per4 = nc / 4096;
  const int t = threadIdx.x, lane = t & 63, wid = t >> 6;
  int s = 0;
  for (int k = 0; k < per4; ++k) {
    const int4 a = c[t * per4 + k];
    s += a.x + a.y + a.z + a.w;
  }
  int inc = s;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const int u = __shfl_up(inc, d, 64);
    if (lane >= d) inc += u;
  }
  if (lane == 63) wsum[wid] = inc;
  __syncthreads();
  int run = inc - s;
  for (int v = 0; v < wid; ++v) run += wsum[v];
  for (int k = 0; k < per4; ++k) {
    const int4 a = c[t * per4 + k];
    int4 o;
    o.x = run;
    o.y = o.x + a.x;
    o.z = o.y + a.y;
    o.w = o.z + a.z;
    run = o.w + a.w;
    c[t * per4 + k] = o;
  }
}

// points into cell order: (x, y, z, original index bits); the offsets end as
// the cells' ends
__global__ __launch_bounds__(256) void k_nn_scatter(const float* __restrict__ x, int64_t nx,
                                                    const float* __restrict__ y, int64_t ny, int* __restrict__ cnt,
                                                    float4* __restrict__ sx, float4* __restrict__ sy, int cb) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= nx + ny) return;
  const bool isy = i >= nx;
  const int64_t k = isy ? i - nx : i;
  const float* p = (isy ? y : x) + 3 * k;
  const float a = p[0], b = p[1], c = p[2];
  const int pos = atomicAdd(&cnt[(isy ? 1 << (3 * cb) : 0) + nn_key(a, b, c, cb)], 1);
  (isy ? sy : sx)[pos] = make_float4(a, b, c, __int_as_float((int)k));
}

// bounding box of each tile (one wavefront per tile; NaN coordinates ignored)
__global__ __launch_bounds__(64) void k_nn_box(const float4* __restrict__ sx, int64_t nx,
                                               const float4* __restrict__ sy, int64_t ny, int64_t tx,
                                               float4* __restrict__ bx, float4* __restrict__ by) {
  const int64_t tb = blockIdx.x;
  const bool isy = tb >= tx;
  const int64_t t = isy ? tb - tx : tb, n = isy ? ny : nx;
  const int64_t i = t * kNnTile + threadIdx.x;
  const float inf = __int_as_float(0x7f800000);
  float lo[3] = {inf, inf, inf}, hi[3] = {-inf, -inf, -inf};
  if (i < n) {
    const float4 p = (isy ? sy : sx)[i];
    lo[0] = hi[0] = p.x;
    lo[1] = hi[1] = p.y;
    lo[2] = hi[2] = p.z;
    if (p.x != p.x) lo[0] = inf, hi[0] = -inf;
    if (p.y != p.y) lo[1] = inf, hi[1] = -inf;
    if (p.z != p.z) lo[2] = inf, hi[2] = -inf;
  }
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) {
#pragma unroll
    for (int a = 0; a < 3; ++a) {
      lo[a] = fminf(lo[a], __shfl_xor(lo[a], d, 64));
      hi[a] = fmaxf(hi[a], __shfl_xor(hi[a], d, 64));
    }
  }
  if (threadIdx.x == 0) {
    float4* b = (isy ? by : bx) + 2 * t;
    b[0] = make_float4(lo[0], lo[1], lo[2], 0.0f);
    b[1] = make_float4(hi[0], hi[1], hi[2], 0.0f);
  }
}

// Small clouds (up to kNnSmall points, beyond kNnOne): two launches. The keys, in cells twice
// as fine per axis as the cell ends kept for the search, go to the nn outputs,
// which the search overwrites; one workgroup computing all of its cloud's keys
// is bound by its own arithmetic (12 of 26 us for 20000 points).
constexpr int kNnFineBits = kNnSmallBits + 1;  // 32^3 cells sorted
constexpr int kNnFineCells = 1 << (3 * kNnFineBits);
constexpr int kNnSortWgs = 32;                 // workgroups per cloud
static_assert(kNnSmall <= 0xffff && kNnFineCells <= 0xffff, "counts and positions, and keys with one to spare, in 16 bits");

__global__ __launch_bounds__(256) void k_nn_keys(const float* __restrict__ x, int nx, const float* __restrict__ y,
                                                 int ny, uint16_t* __restrict__ kx, uint16_t* __restrict__ ky) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= nx + ny) return;
  const bool isy = i >= nx;
  const int k = isy ? i - nx : i;
  const float* p = (isy ? y : x) + 3 * (int64_t)k;
  (isy ? ky : kx)[k] = (uint16_t)nn_key(p[0], p[1], p[2], kNnFineBits);
}

// three minima and three maxima over the wavefront
__device__ __forceinline__ void wave_box(float (&m)[6]) {
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) {
#pragma unroll
    for (int q = 0; q < 6; ++q) {
      const float o = __shfl_xor(m[q], d, 64);
      m[q] = q < 3 ? fminf(m[q], o) : fmaxf(m[q], o);
    }
  }
}

// The counting sort of one cloud by kNnSortWgs workgroups that do not speak to
// each other: each counts and scans all keys in LDS (the keys are 2 bytes and
// are read once), then places only the cells that start in its share of the
// tiles, in LDS, and writes the sorted points and the boxes of its tiles in
// order. A cell that starts before the share and ends within it belongs to the
// workgroup before, in an order that is only known there: its points' common
// box is added to every tile of the share that it reaches (still a bound).
// One workgroup per cloud took 26 us for 20000 points each; the keys take 3 and
// this 16.5, of which half is the key arithmetic and LDS atomics of a whole
// cloud on one compute unit.
__global__ __launch_bounds__(1024) void k_nn_sort(const float* __restrict__ x, int nx, const float* __restrict__ y,
                                                  int ny, const uint16_t* __restrict__ kx,
                                                  const uint16_t* __restrict__ ky, int* __restrict__ cnt,
                                                  float4* __restrict__ sx, float4* __restrict__ sy,
                                                  float4* __restrict__ bx, float4* __restrict__ by) {
  constexpr int PAIRS = kNnSortPairs;          // key pairs per thread
  constexpr int WORDS = kNnFineCells / 2048;   // words of two 16-bit counts per thread
  constexpr int PITCH = WORDS + 4;             // a thread's words, padded against bank conflicts
  static_assert(WORDS == 16 && PITCH % 4 == 0, "hist_at() and the 16-byte accesses");
  __shared__ __attribute__((aligned(16))) uint32_t hist[1024 * PITCH];
  __shared__ uint16_t perm[kNnSmall + 1];  // the last for the points of others
  __shared__ int wsum[16];
  __shared__ int mark[7];  // own cells [0], [1) at positions [2], [3); the cell across a [4] at [5], [6)
  __shared__ float part[16][6];
  // word of a key's count; the thread's own padding for the key of no point (0xffff)
  auto hist_at = [&](int key) -> uint32_t& {
    return hist[key < kNnFineCells ? (key >> 5) * PITCH + ((key >> 1) & 15) : threadIdx.x * PITCH + WORDS];
  };
  const bool isy = blockIdx.x >= kNnSortWgs;
  const int k = isy ? blockIdx.x - kNnSortWgs : blockIdx.x;
  const float* p = isy ? y : x;
  const int n = isy ? ny : nx;
  const uint32_t* keys = reinterpret_cast<const uint32_t*>(isy ? ky : kx);
  float4* srt = isy ? sy : sx;
  float4* box = isy ? by : bx;
  int* ends = cnt + (isy ? 1 << (3 * kNnSmallBits) : 0);
  const int t = threadIdx.x, lane = t & 63, wid = t >> 6;
  const int nt = (n + kNnTile - 1) / kNnTile;
  const int share = (nt + kNnSortWgs - 1) / kNnSortWgs * kNnTile;
  const int a = min(k * share, n), b = min(a + share, n);
  uint32_t kk[PAIRS];
#pragma unroll
  for (int j = 0; j < PAIRS; ++j) {
    const int i = 2 * (j * 1024 + t);  // an odd count reads two bytes past its keys, within the 4 n of the buffer
    kk[j] = i < n ? keys[j * 1024 + t] : ~0u;
    if (i + 1 == n) kk[j] |= 0xffff0000u;
  }
#pragma unroll
  for (int c = 0; c < WORDS; c += 4) *reinterpret_cast<uint4*>(&hist[t * PITCH + c]) = make_uint4(0, 0, 0, 0);
  if (t < 7) mark[t] = t == 4 ? -1 : 0;
  __syncthreads();
  // the count before a point is its rank in its cell (both of a pair in one word)
  uint32_t rank[PAIRS];
#pragma unroll
  for (int g = 0; g < PAIRS; g += 4) {
    if (g * 2048 >= n) continue;
    uint32_t r[8];
#pragma unroll
    for (int h = 0; h < 8; ++h) {
      const int key = (int)(kk[g + h / 2] >> (16 * (h & 1))) & 0xffff;
      r[h] = atomicAdd(&hist_at(key), 1u << (16 * (key & 1)));
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const uint32_t w = kk[g + j];
      rank[g + j] = ((r[2 * j] >> (16 * (w & 1))) & 0xffff) | (r[2 * j + 1] >> (16 * ((w >> 16) & 1))) << 16;
      asm("" : "+v"(rank[g + j]), "+v"(kk[g + j]));  // packed now; the addresses are formed again below
    }
  }
  __syncthreads();
  {
    uint32_t v[WORDS];
    int s = 0;
#pragma unroll
    for (int c = 0; c < WORDS; c += 4) {
      const uint4 h = *reinterpret_cast<const uint4*>(&hist[t * PITCH + c]);
      v[c] = h.x, v[c + 1] = h.y, v[c + 2] = h.z, v[c + 3] = h.w;
    }
#pragma unroll
    for (int c = 0; c < WORDS; ++c) s += (int)(v[c] & 0xffff) + (int)(v[c] >> 16);
    int inc = s;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const int u = __shfl_up(inc, d, 64);
      if (lane >= d) inc += u;
    }
    if (lane == 63) wsum[wid] = inc;
    __syncthreads();
    int run = inc - s;
    for (int u = 0; u < wid; ++u) run += wsum[u];
    // exactly one cell holds the point before a bound greater than 0
    if ((run < a && a <= run + s) || (run < b && b <= run + s)) {
      int at = run;
#pragma unroll
      for (int c = 0; c < 2 * WORDS; ++c) {
        const int end = at + (int)((v[c >> 1] >> (16 * (c & 1))) & 0xffff);
        if (at < a && a <= end) {
          mark[0] = 2 * WORDS * t + c + 1, mark[2] = end;
          if (end > a) mark[4] = 2 * WORDS * t + c, mark[5] = at, mark[6] = end;
        }
        if (at < b && b <= end) mark[1] = 2 * WORDS * t + c + 1, mark[3] = end;
        at = end;
      }
    }
    int e[4];
#pragma unroll
    for (int c = 0; c < WORDS; ++c) {
      const int mid = run + (int)(v[c] & 0xffff), end = mid + (int)(v[c] >> 16);
      v[c] = (uint32_t)run | ((uint32_t)mid << 16);
      run = end;
      if ((c & 3) == 3) e[c >> 2] = end;
    }
#pragma unroll
    for (int c = 0; c < WORDS; c += 4)
      *reinterpret_cast<uint4*>(&hist[t * PITCH + c]) = make_uint4(v[c], v[c + 1], v[c + 2], v[c + 3]);
    if (t / (1024 / kNnSortWgs) == k) reinterpret_cast<int4*>(ends)[t] = make_int4(e[0], e[1], e[2], e[3]);
  }
  __syncthreads();
  const bool across = mark[4] >= 0;
  const int kb = mark[1], pa = mark[2], pe = mark[3], ke = mark[6];
  const int k0 = across ? mark[4] : mark[0], p0 = across ? mark[5] : pa;  // perm: positions [p0, pe)
  const float inf = __int_as_float(0x7f800000);
#pragma unroll
  for (int g = 0; g < PAIRS; g += 4) {
    if (g * 2048 >= n) continue;
#pragma unroll
    for (int h = 0; h < 8; ++h) {
      const int key = (int)(kk[g + h / 2] >> (16 * (h & 1))) & 0xffff;
      const int pos = (int)((hist_at(key) >> (16 * (key & 1))) & 0xffff) +
                      (int)((rank[g + h / 2] >> (16 * (h & 1))) & 0xffff);
      const bool own = (uint32_t)(key - k0) < (uint32_t)(kb - k0);
      perm[own ? pos - p0 : kNnSmall] = (uint16_t)(2 * ((g + h / 2) * 1024 + t) + (h & 1));
    }
  }
  __syncthreads();
  // 0..2: minima, 3..5: maxima (fminf and fmaxf pass over NaN)
  float m[6] = {inf, inf, inf, -inf, -inf, -inf};
  for (int e = p0 + t; e < pa; e += 1024) {
    const int i = perm[e - p0];
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      m[d] = fminf(m[d], p[3 * i + d]);
      m[3 + d] = fmaxf(m[3 + d], p[3 * i + d]);
    }
  }
  if (across) {  // the same for the whole workgroup
    wave_box(m);
    if (lane == 0) {
#pragma unroll
      for (int q = 0; q < 6; ++q) part[wid][q] = m[q];
    }
    __syncthreads();
    for (int w = 0; w < 16; ++w) {
#pragma unroll
      for (int q = 0; q < 6; ++q) m[q] = q < 3 ? fminf(m[q], part[w][q]) : fmaxf(m[q], part[w][q]);
    }
  }
  const int stop = max(pe, b);
  for (int i0 = a + wid * kNnTile; i0 < stop; i0 += 1024) {  // one tile per wavefront
    const int pos = i0 + lane;
    float l[6] = {inf, inf, inf, -inf, -inf, -inf};
    if (pos >= pa && pos < pe) {
      const int i = perm[pos - p0];
      const float v[3] = {p[3 * i], p[3 * i + 1], p[3 * i + 2]};
      srt[pos] = make_float4(v[0], v[1], v[2], __int_as_float(i));
#pragma unroll
      for (int d = 0; d < 3; ++d) {
        l[d] = fminf(inf, v[d]);
        l[3 + d] = fmaxf(-inf, v[d]);
      }
    }
    if (i0 >= b) continue;  // the box is the next workgroup's
    wave_box(l);
    if (lane == 0) {
#pragma unroll
      for (int q = 0; q < 6; ++q)
        if (i0 < ke) l[q] = q < 3 ? fminf(l[q], m[q]) : fmaxf(l[q], m[q]);
      box[2 * (i0 / kNnTile)] = make_float4(l[0], l[1], l[2], 0.0f);
      box[2 * (i0 / kNnTile) + 1] = make_float4(l[3], l[4], l[5], 0.0f);
    }
  }
}

// The counting sort of one cloud of up to kNnOne points by one workgroup, in the
// 16^3 cells themselves: keys, counts, scan, the sorted points in LDS, then the
// tiles with their boxes. One launch, where the finer cells take two and a
// workgroup's pass over 32768 counts: 6.0 us against 12.8 at 1000 points each,
// 12.0 against 15.3 at 3000. The key arithmetic on two compute units bounds it.
__global__ __launch_bounds__(1024) void k_nn_sort_one(const float* __restrict__ x, int nx, const float* __restrict__ y,
                                                      int ny, int* __restrict__ cnt, float4* __restrict__ sx,
                                                      float4* __restrict__ sy, float4* __restrict__ bx,
                                                      float4* __restrict__ by) {
  constexpr int CELLS = 1 << (3 * kNnSmallBits), PER = kNnOne / 1024;
  static_assert(CELLS == 4 * 1024, "four counts per thread");
  __shared__ __attribute__((aligned(16))) int hist[CELLS];
  __shared__ float4 pts[kNnOne];
  __shared__ int wsum[16];
  const bool isy = blockIdx.x == 1;
  const float* p = isy ? y : x;
  const int n = isy ? ny : nx;
  float4* srt = isy ? sy : sx;
  float4* box = isy ? by : bx;
  int* ends = cnt + (isy ? CELLS : 0);
  const int t = threadIdx.x, lane = t & 63, wid = t >> 6;
  float v[PER][3];
#pragma unroll
  for (int u = 0; u < PER; ++u) {
    const int i = u * 1024 + t;
#pragma unroll
    for (int d = 0; d < 3; ++d) v[u][d] = i < n ? p[3 * i + d] : 0.0f;
  }
  reinterpret_cast<int4*>(hist)[t] = make_int4(0, 0, 0, 0);
  __syncthreads();
  int key[PER], rank[PER];
#pragma unroll
  for (int u = 0; u < PER; ++u) {
    if (u * 1024 + t >= n) break;
    key[u] = nn_key(v[u][0], v[u][1], v[u][2], kNnSmallBits);
    rank[u] = atomicAdd(&hist[key[u]], 1);
  }
  __syncthreads();
  const int4 c = reinterpret_cast<const int4*>(hist)[t];
  const int sum = c.x + c.y + c.z + c.w;
  int inc = sum;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const int u = __shfl_up(inc, d, 64);
    if (lane >= d) inc += u;
  }
  if (lane == 63) wsum[wid] = inc;
  __syncthreads();
  int run = inc - sum;
  for (int u = 0; u < wid; ++u) run += wsum[u];
  const int4 e = make_int4(run + c.x, run + c.x + c.y, run + c.x + c.y + c.z, run + sum);
  reinterpret_cast<int4*>(hist)[t] = make_int4(run, e.x, e.y, e.z);
  reinterpret_cast<int4*>(ends)[t] = e;
  __syncthreads();
#pragma unroll
  for (int u = 0; u < PER; ++u) {
    const int i = u * 1024 + t;
    if (i < n) pts[hist[key[u]] + rank[u]] = make_float4(v[u][0], v[u][1], v[u][2], __int_as_float(i));
  }
  __syncthreads();
  const float inf = __int_as_float(0x7f800000);
  for (int i0 = wid * kNnTile; i0 < n; i0 += 1024) {  // one tile per wavefront
    const int i = i0 + lane;
    float l[6] = {inf, inf, inf, -inf, -inf, -inf};
    if (i < n) {
      const float4 q = pts[i];
      srt[i] = q;
      l[0] = fminf(inf, q.x), l[1] = fminf(inf, q.y), l[2] = fminf(inf, q.z);
      l[3] = fmaxf(-inf, q.x), l[4] = fmaxf(-inf, q.y), l[5] = fmaxf(-inf, q.z);
    }
    wave_box(l);
    if (lane == 0) {
      box[2 * (i0 / kNnTile)] = make_float4(l[0], l[1], l[2], 0.0f);
      box[2 * (i0 / kNnTile) + 1] = make_float4(l[3], l[4], l[5], 0.0f);
    }
  }
}

// squared distance bound from point q to box [lo, hi]
__device__ __forceinline__ float nn_box_d2(float qx, float qy, float qz, const float4& lo, const float4& hi) {
  return nn_d2(fmaxf(fmaxf(lo.x - qx, qx - hi.x), 0.0f), fmaxf(fmaxf(lo.y - qy, qy - hi.y), 0.0f),
               fmaxf(fmaxf(lo.z - qz, qz - hi.z), 0.0f));
}

// squared distance bound between boxes [al, ah] and [bl, bh]
__device__ __forceinline__ float nn_boxbox_d2(const float3& al, const float3& ah, const float4& bl, const float4& bh) {
  return nn_d2(fmaxf(fmaxf(bl.x - ah.x, al.x - bh.x), 0.0f), fmaxf(fmaxf(bl.y - ah.y, al.y - bh.y), 0.0f),
               fmaxf(fmaxf(bl.z - ah.z, al.z - bh.z), 0.0f));
}

// orders this wavefront's LDS writes before its own later reads (and the
// reverse) without a workgroup barrier: the wavefronts of a query group take
// different numbers of tiles
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

struct NnSide {
  const float4* q;   // sorted queries
  const float4* qbox;  // their tiles' boxes
  int64_t nq;
  const float4* r;   // sorted references
  const float4* box; // reference tile boxes (lo, hi)
  const int* rend;   // reference cell ends
  int64_t nr;
  int32_t* nn;
  float* dist;
};

constexpr int kNnWaves = 8;                  // wavefronts per query group
constexpr int kNnBlock = 64 * kNnWaves;       // threads of a query workgroup
constexpr int kNnCand = 512;  // tiles tested per pass: the capacity of the candidate list

// One group of kNnTile sorted queries per workgroup, kNnWaves wavefronts
// holding the same queries; groups [0, gx) search y from x, the rest x from y.
// 1. Each wavefront scans one of the kNnWaves tiles around the reference cell of
//    the group's first query; the largest best distance of the group then
//    bounds every neighbour.
// 2. The tiles whose box lies within that bound of the group's box are listed
//    in LDS with their boxes and ranked by the box-to-box bound.
// 3. The wavefronts take the sorted tiles in turn (the next one's points
//    prefetched) and stop at the first whose box bound exceeds every lane's
//    best; a tile is passed over when no lane's point-to-box bound reaches
//    that lane's best. A lane's best is the lowest distance any wavefront has
//    reached for it (published in LDS after every tile).
// 4. The kNnWaves results per query are merged (lower distance, then lower
//    index).
// A tile is scanned sixteen points at a time: their least distance first (6.5
// operations a pair), the index only where some lane reaches its best (one
// batch of ten after the first tile; 13 operations a pair). The chain of one
// group (cell end, first tile, list, then its tiles by eights) bounds it: 20000
// against 20000 points of two surfaces took 54 us with the index tracked in
// every step, the tiles in Morton order of 16^3 cells and the list sorted by
// exchanges, 25 now; with four wavefronts per group 31.
__global__ __launch_bounds__(kNnBlock) __attribute__((amdgpu_waves_per_eu(1, 4))) void k_nn_query(
    const NnSide A, const NnSide Bs, int64_t gx, int cb, int fine) {
  __shared__ __attribute__((aligned(16))) float stg[kNnWaves][4][kNnTile];  // x, y, z, index bits
  __shared__ float shb[kNnWaves][kNnTile];
  __shared__ int sidx[kNnWaves][kNnTile];
  __shared__ float4 cbox[kNnCand][2];  // lo (w: box bound), hi (w: tile - c0)
  __shared__ unsigned long long ckey[kNnCand];  // (box bound, slot in cbox)
  __shared__ int order[kNnCand];  // slots, nearest box first
  __shared__ int ncand;
  const bool second = blockIdx.x >= gx;
  const NnSide S = second ? Bs : A;
  const int64_t g = second ? blockIdx.x - gx : blockIdx.x;
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const float inf = __int_as_float(0x7f800000), nan = __int_as_float(0x7fc00000);
  const int64_t gi = g * kNnTile + lane;
  const bool active = gi < S.nq;
  const float4 q = active ? S.q[gi] : make_float4(nan, nan, nan, 0.0f);
  const float4 ql4 = S.qbox[2 * g], qh4 = S.qbox[2 * g + 1];  // NaN coordinates are not in it
  const float3 ql = make_float3(ql4.x, ql4.y, ql4.z), qh = make_float3(qh4.x, qh4.y, qh4.z);
  const int64_t ntr = (S.nr + kNnTile - 1) / kNnTile;
  const int key = __builtin_amdgcn_readfirstlane(nn_key(q.x, q.y, q.z, cb + fine) >> (3 * fine));
  int64_t t0 = S.rend[key] / kNnTile;
  t0 = t0 > ntr - 1 ? ntr - 1 : t0;
  int64_t s0 = t0 - kNnWaves / 2 + 1 > ntr - kNnWaves ? ntr - kNnWaves : t0 - kNnWaves / 2 + 1;
  s0 = s0 < 0 ? 0 : s0;
  const int64_t s1 = s0 + kNnWaves - 1;  // the start tiles [s0, s1] (fewer when ntr < kNnWaves)
  float best = inf;
  int bi = 0x7fffffff;
  auto publish = [&]() { __hip_atomic_store(&shb[w][lane], best, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP); };
  // the lowest distance reached for this query by any wavefront so far
  auto reached = [&]() {
    float u = best;
#pragma unroll
    for (int v = 0; v < kNnWaves; ++v)
      u = fminf(u, __hip_atomic_load(&shb[v][lane], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP));
    return u;
  };
  auto group_bound = [&](float u) {
    float b = active ? u : 0.0f;
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) b = fmaxf(b, __shfl_xor(b, d, 64));
    return b;
  };
  // this lane's point of tile t; a short last tile is padded with points at
  // infinity and the largest index, which never win
  auto tile_point = [&](int64_t t) {
    const int64_t i = t * kNnTile + lane;
    return i < S.nr ? S.r[i] : make_float4(inf, inf, inf, __int_as_float(0x7fffffff));
  };
  auto scan_tile = [&](const float4& p) {
    wave_sync();
    stg[w][0][lane] = p.x;
    stg[w][1][lane] = p.y;
    stg[w][2][lane] = p.z;
    stg[w][3][lane] = p.w;
    wave_sync();
    auto four = [&](int c, int k) { return *reinterpret_cast<const float4*>(&stg[w][c][k]); };
#pragma unroll 1
    for (int k0 = 0; k0 < kNnTile; k0 += 16) {
      float d[16], low;
#pragma unroll
      for (int u = 0; u < 16; u += 4) {
        const float4 x = four(0, k0 + u), y = four(1, k0 + u), z = four(2, k0 + u);
        d[u] = nn_d2(x.x - q.x, y.x - q.y, z.x - q.z);
        d[u + 1] = nn_d2(x.y - q.x, y.y - q.y, z.y - q.z);
        d[u + 2] = nn_d2(x.z - q.x, y.z - q.y, z.z - q.z);
        d[u + 3] = nn_d2(x.w - q.x, y.w - q.y, z.w - q.z);
      }
      low = d[0];
#pragma unroll
      for (int u = 1; u < 16; ++u) low = fminf(low, d[u]);
      if (!__any(low <= best)) continue;  // nine of ten batches after the first tile
#pragma unroll
      for (int u = 0; u < 16; ++u) {
        const int j = __float_as_int(stg[w][3][k0 + u]);
        const bool better = (d[u] < best) | ((d[u] == best) & (j < bi));
        best = better ? d[u] : best;
        bi = better ? j : bi;
      }
    }
    publish();
  };
  // a thread tests one tile per pass, whose box travels during the pass before
  // (loaded where it is tested, a pass waited on memory: 1M against 1M points
  // 4.91 ms, 1.58 now; 300k against 300k 0.54, 0.30 now)
  static_assert(kNnCand == kNnBlock, "one tile per thread and pass");
  int64_t tb = threadIdx.x < ntr ? threadIdx.x : 0;
  float4 blo = S.box[2 * tb], bhi = S.box[2 * tb + 1];
  scan_tile(tile_point(s0 + w < ntr ? s0 + w : ntr - 1));
  __syncthreads();
  float bound = group_bound(reached());
  for (int64_t c0 = 0; c0 < ntr; c0 += kNnCand) {
    if (threadIdx.x == 0) ncand = 0;
    __syncthreads();
    const int64_t t = c0 + threadIdx.x;
    const float lb = nn_boxbox_d2(ql, qh, blo, bhi);
    if (t < ntr && (t < s0 || t > s1) && lb <= bound) {
      const int k = atomicAdd(&ncand, 1);
      cbox[k][0] = make_float4(blo.x, blo.y, blo.z, lb);
      cbox[k][1] = make_float4(bhi.x, bhi.y, bhi.z, __int_as_float((int)threadIdx.x));
      ckey[k] = ((unsigned long long)__float_as_uint(lb) << 32) | (uint32_t)k;
    }
    tb = t + kNnCand < ntr ? t + kNnCand : 0;
    blo = S.box[2 * tb];
    bhi = S.box[2 * tb + 1];
    __syncthreads();
    const int nc = ncand;
    // rank by counting the lesser keys (they differ: the slot is part of the key)
    for (int i = threadIdx.x; i < nc; i += kNnBlock) {
      const unsigned long long mine = ckey[i];
      int rank = 0;
#pragma unroll 8
      for (int j = 0; j < nc; ++j) rank += ckey[j] < mine ? 1 : 0;
      order[rank] = i;
    }
    __syncthreads();
    float4 pf = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    if (w < nc) pf = tile_point(c0 + __float_as_int(cbox[order[w]][1].w));
    for (int i = w; i < nc; i += kNnWaves) {
      const int k = order[i];
      const float4 lo = cbox[k][0], hi = cbox[k][1];
      const float4 cur = pf;
      if (i + kNnWaves < nc) pf = tile_point(c0 + __float_as_int(cbox[order[i + kNnWaves]][1].w));
      const float ub = reached();
      if (!__any(active && ub >= lo.w)) break;  // every later box is farther
      if (ub < best) {  // another wavefront's: it holds the index
        best = ub;
        bi = 0x7fffffff;
      }
      const bool need = active && nn_box_d2(q.x, q.y, q.z, lo, hi) <= ub;
      if (__any(need)) scan_tile(cur);
    }
    __syncthreads();
    bound = group_bound(reached());
  }
  sidx[w][lane] = bi;
  publish();
  __syncthreads();
  if (w == 0) {
#pragma unroll
    for (int v = 1; v < kNnWaves; ++v) {
      const float d = shb[v][lane];
      const int j = sidx[v][lane];
      const bool better = (d < best) | ((d == best) & (j < bi));
      best = better ? d : best;
      bi = better ? j : bi;
    }
    if (active) {
      const int qi = __float_as_int(q.w);
      S.nn[qi] = bi == 0x7fffffff ? -1 : bi;
      S.dist[qi] = best;
    }
  }
}

// loss = mean(d_x) + mean(d_y), FP64 sums in a fixed order by point index
// (one workgroup: strided per-thread sums, then a fixed tree), so the loss
// does not depend on the order the search sorted the points in
__global__ __launch_bounds__(1024) void k_chamfer_loss(const float* __restrict__ dx, int64_t nx,
                                                       const float* __restrict__ dy, int64_t ny,
                                                       double* __restrict__ loss, float* __restrict__ loss32) {
  __shared__ double sh[16];
  const int t = threadIdx.x;
  double a = 0.0, b = 0.0;
  for (int64_t i0 = t; i0 < nx || i0 < ny; i0 += 16 * 1024) {  // 32 loads in flight
    float vx[16], vy[16];
#pragma unroll
    for (int k = 0; k < 16; ++k) {
      const int64_t i = i0 + 1024 * k;
      vx[k] = dx[i < nx ? i : 0];  // no branch between the loads
      vy[k] = dy[i < ny ? i : 0];
    }
#pragma unroll
    for (int k = 0; k < 16; ++k) {
      const int64_t i = i0 + 1024 * k;
      a += i < nx ? vx[k] : 0.0f;
      b += i < ny ? vy[k] : 0.0f;
    }
  }
  double v = a / (double)nx + b / (double)ny;
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) v += __shfl_xor(v, d, 64);
  if ((t & 63) == 0) sh[t >> 6] = v;
  __syncthreads();
  if (t == 0) {
    double tot = 0.0;
    for (int w = 0; w < 16; ++w) tot += sh[w];
    if (loss) *loss = tot;
    if (loss32) *loss32 = (float)tot;
  }
}

__global__ __launch_bounds__(256) void k_chamfer_bwd_x(const float* __restrict__ x, int64_t nx,
                                                       const float* __restrict__ y, const int32_t* __restrict__ nnx,
                                                       const float* __restrict__ scale, float* __restrict__ g) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= nx) return;
  const int64_t j = nnx[i];
  const float s = 2.0f / (float)nx, c = scale ? *scale : 1.0f;
  if (j < 0) {  // no neighbour: the query holds NaN
#pragma unroll
    for (int d = 0; d < 3; ++d) g[3 * i + d] = __int_as_float(0x7fc00000);
    return;
  }
#pragma unroll
  for (int d = 0; d < 3; ++d) g[3 * i + d] = s * (x[3 * i + d] - y[3 * j + d]) * c;
}

__global__ __launch_bounds__(256) void k_chamfer_bwd_y(const float* __restrict__ x, const float* __restrict__ y,
                                                       int64_t ny, const int32_t* __restrict__ nny,
                                                       const float* __restrict__ scale, float* __restrict__ g) {
  const int64_t j = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (j >= ny) return;
  const int64_t i = nny[j];
  if (i < 0) return;  // no neighbour: the target point holds NaN
  const float s = 2.0f / (float)ny, c = scale ? *scale : 1.0f;
#pragma unroll
  for (int d = 0; d < 3; ++d) atomicAdd(&g[3 * i + d], s * (x[3 * i + d] - y[3 * j + d]) * c);
}

__global__ void k_set_int(int32_t* __restrict__ p, int32_t v) { *p = v; }

__global__ __launch_bounds__(256) void k_lab_init(int32_t* __restrict__ lab, int64_t nv) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i < nv) lab[i] = (int32_t)i;
}

__global__ __launch_bounds__(256) void k_lab_faces(const int32_t* __restrict__ f, int64_t nf, int32_t* __restrict__ lab,
                                                   int32_t* __restrict__ changed) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= nf) return;
  const int32_t a = f[3 * i], b = f[3 * i + 1], c = f[3 * i + 2];
  const int32_t la = lab[a], lb = lab[b], lc = lab[c];
  const int32_t m = la < lb ? (la < lc ? la : lc) : (lb < lc ? lb : lc);
  bool ch = false;
  if (la > m) ch |= atomicMin(&lab[a], m) > m;
  if (lb > m) ch |= atomicMin(&lab[b], m) > m;
  if (lc > m) ch |= atomicMin(&lab[c], m) > m;
  if (ch) atomicOr(changed, 1);
}

// pointer jumping: labels only decrease and always name a vertex of the component
__global__ __launch_bounds__(256) void k_lab_jump(int32_t* __restrict__ lab, int64_t nv) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= nv) return;
  const int32_t l = lab[i];
  const int32_t ll = lab[l];
  if (ll < l) atomicMin(&lab[i], ll);
}

__global__ __launch_bounds__(256) void k_fill0d(double* __restrict__ x, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) x[i] = 0.0;
}

// Area per label. A mesh is mostly one or a few components, so the 64
// triangles of a wavefront usually share a label: they are then summed by
// shuffles and added with one atomic instead of 64 on the same address.
__global__ __launch_bounds__(256) void k_comp_area(const int32_t* __restrict__ f, int64_t nf,
                                                   const int32_t* __restrict__ lab, const double* __restrict__ area,
                                                   double* __restrict__ carea) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const bool ok = i < nf;
  const int l = ok ? lab[f[3 * i]] : -1;
  double a = ok ? area[i] : 0.0;
  const int l0 = __builtin_amdgcn_readfirstlane(l);  // lane 0: the wavefront's first triangle
  if (__all(l == l0 || !ok)) {
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) a += __shfl_xor(a, d, 64);
    if ((threadIdx.x & 63) == 0 && l0 >= 0) atomicAdd(&carea[l0], a);
  } else if (ok) {
    atomicAdd(&carea[l], a);
  }
}

// the label of greatest area (ties: the lowest label), one workgroup
__global__ __launch_bounds__(256) void k_comp_best(const double* __restrict__ carea, int64_t nv,
                                                   int32_t* __restrict__ best) {
  __shared__ double sa[256];
  __shared__ int64_t sl[256];
  double a = -1.0;
  int64_t l = nv;
  for (int64_t i = threadIdx.x; i < nv; i += 256) {
    if (carea[i] > a) {  // increasing i: the first of equal areas stays
      a = carea[i];
      l = i;
    }
  }
  sa[threadIdx.x] = a;
  sl[threadIdx.x] = l;
  __syncthreads();
  for (int d = 128; d > 0; d >>= 1) {
    if (threadIdx.x < d) {
      const double ob = sa[threadIdx.x + d];
      const int64_t ol = sl[threadIdx.x + d];
      if (ob > sa[threadIdx.x] || (ob == sa[threadIdx.x] && ol < sl[threadIdx.x])) {
        sa[threadIdx.x] = ob;
        sl[threadIdx.x] = ol;
      }
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) *best = (int32_t)sl[0];
}

__global__ __launch_bounds__(256) void k_face_mask(const int32_t* __restrict__ f, int64_t nf,
                                                   const int32_t* __restrict__ lab, const int32_t* __restrict__ best,
                                                   float* __restrict__ w) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= nf) return;
  w[i] = lab[f[3 * i]] == *best ? 1.0f : 0.0f;
}

static inline int nb256(int64_t n) { return (int)((n + 255) / 256); }

SampleLayout sample_layout(int64_t nf) {
  SampleLayout L;
  const int64_t nb = (nf + kScanBlock - 1) / kScanBlock;
  L.csum = 0;
  L.bs = align(nf * 8);
  L.total = L.bs + align((nb + 1) * 8);
  return L;
}

int run_sample(const float* v, const float* vn, const int32_t* f, int64_t nf, const float* w, const float* u,
               int64_t m, float* pts, float* nrm, int32_t* face, float* bary, void* ws, hipStream_t s) {
  const SampleLayout L = sample_layout(nf);
  double* a = reinterpret_cast<double*>(static_cast<char*>(ws) + L.csum);
  double* bs = reinterpret_cast<double*>(static_cast<char*>(ws) + L.bs);
  const int nb = (int)((nf + kScanBlock - 1) / kScanBlock);
  hipLaunchKernelGGL(k_area_scan, dim3(nb), dim3(kScanBlock), 0, s, v, f, nf, w, a, bs);
  const bool tops = nb <= kScanTops;
  if (!tops) hipLaunchKernelGGL(k_scan_tops, dim3(1), dim3(256), 0, s, bs, nb);
  if (tops && m > kSampleFew)
    hipLaunchKernelGGL((k_sample<true, 256>), dim3((m + 255) / 256), dim3(256), 0, s, v, vn, f, nf, a, bs, nb, u, m, pts,
                       nrm, face, bary);
  else if (m > 0)
    hipLaunchKernelGGL((tops ? k_sample<true, 64> : k_sample<false, 64>), dim3((m + 63) / 64), dim3(64), 0, s, v, vn, f,
                       nf, a, bs, nb, u, m, pts, nrm, face, bary);
  return hipGetLastError() == hipSuccess ? 0 : -4;
}

int run_sample_backward(const int32_t* f, int64_t nv, const int32_t* face, const float* bary, const float* dp,
                        int64_t m, float* dv, hipStream_t s) {
  hipLaunchKernelGGL(k_fill0, dim3(256), dim3(256), 0, s, dv, 3 * nv);
  if (m > 0) hipLaunchKernelGGL(k_sample_bwd, dim3(nb256(3 * m)), dim3(256), 0, s, f, face, bary, dp, m, dv);
  return hipGetLastError() == hipSuccess ? 0 : -4;
}

NnLayout nn_layout(int64_t nx, int64_t ny) {
  NnLayout L;
  const int64_t tx = (nx + kNnTile - 1) / kNnTile, ty = (ny + kNnTile - 1) / kNnTile;
  L.cell_bits = nn_cell_bits(nx, ny);
  L.cnt = 0;
  L.srt_x = align(2 * ((int64_t)1 << (3 * L.cell_bits)) * 4);
  L.srt_y = L.srt_x + align(nx * 16);
  L.box_x = L.srt_y + align(ny * 16);
  L.box_y = L.box_x + align(tx * 32);
  L.total = L.box_y + align(ty * 32);
  return L;
}

size_t chamfer_ws(int64_t nx, int64_t ny) { return nn_layout(nx, ny).total; }

int run_chamfer(const float* x, int64_t nx, const float* y, int64_t ny, int32_t* nnx, float* dx, int32_t* nny,
                float* dy, double* loss, float* loss32, void* ws, hipStream_t s) {
  const NnLayout L = nn_layout(nx, ny);
  char* b = static_cast<char*>(ws);
  int* cnt = reinterpret_cast<int*>(b + L.cnt);
  float4* sx = reinterpret_cast<float4*>(b + L.srt_x);
  float4* sy = reinterpret_cast<float4*>(b + L.srt_y);
  float4* bx = reinterpret_cast<float4*>(b + L.box_x);
  float4* by = reinterpret_cast<float4*>(b + L.box_y);
  const int64_t tx = (nx + kNnTile - 1) / kNnTile, ty = (ny + kNnTile - 1) / kNnTile;
  const int cb = L.cell_bits, nc = 1 << (3 * cb);
  const bool one = nn_one(nx, ny), small = !one && nn_small(nx, ny);
  if (one) {
    hipLaunchKernelGGL(k_nn_sort_one, dim3(2), dim3(1024), 0, s, x, (int)nx, y, (int)ny, cnt, sx, sy, bx, by);
  } else if (small) {
    uint16_t *kx = reinterpret_cast<uint16_t*>(nnx), *ky = reinterpret_cast<uint16_t*>(nny);
    hipLaunchKernelGGL(k_nn_keys, dim3(nb256(nx + ny)), dim3(256), 0, s, x, (int)nx, y, (int)ny, kx, ky);
    hipLaunchKernelGGL(k_nn_sort, dim3(2 * kNnSortWgs), dim3(1024), 0, s, x, (int)nx, y, (int)ny, kx, ky, cnt, sx, sy, bx,
                       by);
  } else {
    hipLaunchKernelGGL(k_nn_zero, dim3(64), dim3(256), 0, s, cnt, 2 * nc);
    hipLaunchKernelGGL(k_nn_count, dim3(nb256(nx + ny)), dim3(256), 0, s, x, nx, y, ny, cnt, cb);
    hipLaunchKernelGGL(k_nn_scan, dim3(2), dim3(1024), 0, s, cnt, nc);
    hipLaunchKernelGGL(k_nn_scatter, dim3(nb256(nx + ny)), dim3(256), 0, s, x, nx, y, ny, cnt, sx, sy, cb);
    hipLaunchKernelGGL(k_nn_box, dim3(tx + ty), dim3(64), 0, s, sx, nx, sy, ny, tx, bx, by);
  }
  const NnSide A{sx, bx, nx, sy, by, cnt + nc, ny, nnx, dx};  // samples x against the target y
  const NnSide B{sy, by, ny, sx, bx, cnt, nx, nny, dy};       // and back
  hipLaunchKernelGGL(k_nn_query, dim3(tx + ty), dim3(kNnBlock), 0, s, A, B, tx, cb,
                     small ? kNnFineBits - kNnSmallBits : 0);
  if (loss || loss32)
    hipLaunchKernelGGL(k_chamfer_loss, dim3(1), dim3(1024), 0, s, dx, nx, dy, ny, loss, loss32);
  return hipGetLastError() == hipSuccess ? 0 : -4;
}

int run_chamfer_backward(const float* x, int64_t nx, const float* y, int64_t ny, const int32_t* nnx,
                         const int32_t* nny, const float* scale, float* g, hipStream_t s) {
  hipLaunchKernelGGL(k_chamfer_bwd_x, dim3(nb256(nx)), dim3(256), 0, s, x, nx, y, nnx, scale, g);
  hipLaunchKernelGGL(k_chamfer_bwd_y, dim3(nb256(ny)), dim3(256), 0, s, x, y, ny, nny, scale, g);
  return hipGetLastError() == hipSuccess ? 0 : -4;
}

// Adam (Kingma and Ba): m <- b1 m + (1 - b1) g, v <- b2 v + (1 - b2) g^2,
// p <- p - (lr / (1 - b1^t)) m / (sqrt(v) / sqrt(1 - b2^t) + eps); the bias
// corrections come from the host in double precision.
__global__ __launch_bounds__(256) void k_adam(float* __restrict__ p, float* __restrict__ m, float* __restrict__ v,
                                              const float* __restrict__ g, int64_t n, float b1, float b2,
                                              float step, float inv_sqrt_bc2, float eps, int wrap) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
  const float gi = g[i];
  const float mi = b1 * m[i] + (1.0f - b1) * gi;
  const float vi = b2 * v[i] + (1.0f - b2) * gi * gi;
  m[i] = mi;
  v[i] = vi;
  float pi = p[i] - step * mi / (sqrtf(vi) * inv_sqrt_bc2 + eps);
  if (wrap) pi -= floorf(pi);
  p[i] = pi;
}

int run_adam(float* p, float* m, float* v, const float* g, int64_t n, int64_t t, float lr, float b1, float b2,
             float eps, bool wrap, hipStream_t s) {
  const double bc1 = 1.0 - std::pow((double)b1, (double)t), bc2 = 1.0 - std::pow((double)b2, (double)t);
  if (n > 0)
    hipLaunchKernelGGL(k_adam, dim3(nb256(n)), dim3(256), 0, s, p, m, v, g, n, b1, b2, (float)(lr / bc1),
                       (float)(1.0 / std::sqrt(bc2)), eps, wrap ? 1 : 0);
  return hipGetLastError() == hipSuccess ? 0 : -4;
}

CompLayout comp_layout(int64_t nv, int64_t nf) {
  CompLayout L;
  L.flag = 0;
  L.best = 256;
  L.carea = 512;
  L.area = L.carea + align(nv * 8);
  L.total = L.area + align(nf * 8);
  return L;
}

int run_components(const float* v, int64_t nv, const int32_t* f, int64_t nf, int32_t* lab, float* w, void* ws,
                   hipStream_t s, int max_iters) {
  const CompLayout L = comp_layout(nv, nf);
  char* b = static_cast<char*>(ws);
  int32_t* flag = reinterpret_cast<int32_t*>(b + L.flag);
  int32_t* best = reinterpret_cast<int32_t*>(b + L.best);
  double* carea = reinterpret_cast<double*>(b + L.carea);
  double* area = reinterpret_cast<double*>(b + L.area);
  hipLaunchKernelGGL(k_lab_init, dim3(nb256(nv)), dim3(256), 0, s, lab, nv);
  int it = 0;
  for (; it < max_iters; ++it) {
    hipLaunchKernelGGL(k_set_int, dim3(1), dim3(1), 0, s, flag, 0);
    hipLaunchKernelGGL(k_lab_faces, dim3(nb256(nf)), dim3(256), 0, s, f, nf, lab, flag);
    hipLaunchKernelGGL(k_lab_jump, dim3(nb256(nv)), dim3(256), 0, s, lab, nv);
    int32_t h = 0;
    if (hipMemcpyAsync(&h, flag, sizeof(h), hipMemcpyDeviceToHost, s) != hipSuccess) return -4;
    if (hipStreamSynchronize(s) != hipSuccess) return -4;
    if (!h) break;
  }
  // a pass that changed nothing leaves one label per component: the smallest
  // vertex index in it, whose own label never changes
  if (it == max_iters) return -5;
  if (w) {
    hipLaunchKernelGGL(k_face_area, dim3(nb256(nf)), dim3(256), 0, s, v, f, nf, area);
    hipLaunchKernelGGL(k_fill0d, dim3(256), dim3(256), 0, s, carea, nv);
    hipLaunchKernelGGL(k_comp_area, dim3(nb256(nf)), dim3(256), 0, s, f, nf, lab, area, carea);
    hipLaunchKernelGGL(k_comp_best, dim3(1), dim3(256), 0, s, carea, nv, best);
    hipLaunchKernelGGL(k_face_mask, dim3(nb256(nf)), dim3(256), 0, s, f, nf, lab, best, w);
  }
  return hipGetLastError() == hipSuccess ? 0 : -4;
}

}  // namespace opt
}  // namespace psr
