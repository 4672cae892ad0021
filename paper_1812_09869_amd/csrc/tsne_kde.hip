// Perplexity-adaptive kernel density estimate of a 2-D map (paKDE, section
// "Perplexity-adaptive Kernel Density Estimation"): every map point gets the
// precision beta_j of the same perplexity search as the input affinities, run
// on the map's squared distances; the density is the sample smoothing
// estimator with bivariate Gaussian kernels of bandwidth h_j^2 = 1 / beta_j,
//   f(c) = (S / n) sum_j (beta_j / pi) exp(-beta_j |c - y_j|^2),
// evaluated at the centres of a regular raster with cells of area S.
#include <hip/hip_runtime.h>
#include <math.h>

#include <type_traits>

#include "../../include/tsne355.h"
#include "tsne_internal.h"

namespace {

constexpr int kKdeTile = 32;     // raster tile of a workgroup: 32 x 32 cells
constexpr int kKdeStage = 64;    // points a wave stages at a time
constexpr int kKdeChunk = 256;   // points summed in FP32 before their sum goes to FP64
constexpr double kLog2e = 1.4426950408889634074;
constexpr double kInvPi = 0.31830988618379067154;

typedef float v16f __attribute__((ext_vector_type(16)));

template <int W>
struct KdeSmem {
  union {
    float4 pts[W][kKdeStage];                // {x, y, beta log2(e), beta / pi}
    double sum[W][kKdeTile][kKdeTile];       // the shares' partial rasters
  };
};

// The Gaussian of a point is the product of one along x and one along y, so
// the raster is a contraction over the points,
//   f(v, u) = sum_j [beta_j / pi exp(-beta_j (cy_v - y_j)^2)] exp(-beta_j (cx_u - x_j)^2),
// which v_mfma_f32_32x32x2_f32 forms: two points a step, lane l supplying the
// factors of point l / 32 for row v = l % 32 (A) and column u = l % 32 (B), and
// receiving cells (8 (r / 4) + 4 (l / 32) + r % 4, l % 32), r = 0 .. 15. A step
// is two exponentials per lane for 2,048 cell terms, where a sum over the
// cells takes one exponential each. What bounds it: the two exponentials and
// seven other instructions (60 issue cycles) against the 64 cycles of the MFMA,
// on the four waves of a SIMD. 65,536 points on 512 x 512 cells: 0.395 ms
// (4.3e13 cell terms a second) against 3.74 ms for one exponential per term.
// A workgroup covers one tile; its W waves share the points in contiguous
// pieces, so that a small raster still fills its compute units. 256 points are
// summed in FP32 and the chunk sums in FP64; the shares' sums meet in LDS in
// their order.
template <int W>
__global__ __launch_bounds__(64 * W) void k_kde_raster(const float2 *__restrict__ y,
                                                       const double *__restrict__ beta, int64_t n,
                                                       tsne_raster g, float *__restrict__ out) {
  __shared__ KdeSmem<W> sm;
  const int t = threadIdx.x, w = t >> 6, l = t & 63, li = l & 31, lk = l >> 5;
  // the wave's share. Few chunks fall to shares 16 / chunks apart, and waves a
  // multiple of 4 apart sit on one SIMD, so the shares go to the SIMDs (w % 4) in
  // blocks of four: 1,000 points on 512 x 512 cells 29.9 us, with sixteen waves now
  // 14.8 (and the stages past the last point left out)
  const int share = W > 4 ? (w & 3) * (W / 4) + (w >> 2) : w;
  const unsigned across = (unsigned)(((int64_t)g.gx + kKdeTile - 1) / kKdeTile);
  const unsigned tile = blockIdx.y * gridDim.x + blockIdx.x;
  const int64_t u0 = (int64_t)(tile % across) * kKdeTile, v0 = (int64_t)(tile / across) * kKdeTile;
  if (v0 >= g.gy) return;  // past the last tile (the grid's last row)
  const float cx = g.x0 + ((float)(u0 + li) + 0.5f) * g.cx;
  const float cy = g.y0 + ((float)(v0 + li) + 0.5f) * g.cy;
  // this wave's points: whole chunks
  const int64_t chunks = (n + kKdeChunk - 1) / kKdeChunk;
  const int64_t c0 = chunks * share / W, c1 = chunks * (share + 1) / W;
  double acc[16];
#pragma unroll
  for (int r = 0; r < 16; ++r) acc[r] = 0.0;
  float4 *pts = sm.pts[w];
  // past the end: the last point with weight 0 (a point of no width anywhere else
  // would be 0 times infinity at a cell whose distance from it overflows)
  auto fetch = [&](int64_t j) {
    const int64_t i = j < n ? j : n - 1;
    const float2 p = y[i];
    const double b = beta[i];
    return make_float4(p.x, p.y, (float)(b * kLog2e), j < n ? (float)(b * kInvPi) : 0.f);
  };
  float4 next = c0 < c1 ? fetch(c0 * kKdeChunk + l) : make_float4(0.f, 0.f, 0.f, 0.f);
  for (int64_t c = c0; c < c1; ++c) {
    v16f s = {};
    const int64_t left = n - c * kKdeChunk;  // stages past the last point are left out
    const int m = left < kKdeChunk ? (int)left : kKdeChunk;
#pragma unroll 1
    for (int q = 0; q < m; q += kKdeStage) {
      // one wave writes and reads this buffer: no barrier between waves
      __builtin_amdgcn_wave_barrier();
      pts[l] = next;
      __builtin_amdgcn_wave_barrier();
      next = fetch(c * kKdeChunk + q + kKdeStage + l);  // in flight over this stage
#pragma unroll 8
      for (int k = 0; k < kKdeStage; k += 2) {
        const float4 p = pts[k + lk];
        const float dx = cx - p.x, dy = cy - p.y;
        const float ey = p.w * __builtin_amdgcn_exp2f(-p.z * (dy * dy));
        const float ex = __builtin_amdgcn_exp2f(-p.z * (dx * dx));
        s = __builtin_amdgcn_mfma_f32_32x32x2f32(ey, ex, s, 0, 0, 0);
      }
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] += (double)s[r];
  }
  __syncthreads();  // the staged points give way to the sums
#pragma unroll
  for (int r = 0; r < 16; ++r) sm.sum[share][8 * (r >> 2) + 4 * lk + (r & 3)][li] = acc[r];
  __syncthreads();
#pragma unroll
  for (int c = t; c < kKdeTile * kKdeTile; c += 64 * W) {
    const int64_t v = v0 + (c >> 5), u = u0 + (c & 31);
    if (v >= g.gy || u >= g.gx) continue;
    double f = 0.0;
#pragma unroll
    for (int q = 0; q < W; ++q) f += sm.sum[q][c >> 5][c & 31];
    out[v * g.gx + u] = (float)(f * ((double)g.cx * (double)g.cy / (double)n));
  }
}

constexpr int kKdeThreads = 256;
constexpr int kKdeCells = 4;  // cells per thread (consecutive along x)

// One exponential per cell term, for rasters whose tiles would be mostly
// padding, and for a handful of points. One thread: kKdeCells consecutive cells
// of one raster row. Points pass through LDS in chunks of 256; each cell sums a
// chunk in FP32 and the chunk sums in FP64.
__global__ __launch_bounds__(kKdeThreads) void k_kde_cells(const float2 *__restrict__ y,
                                                           const double *__restrict__ beta,
                                                           int64_t n, tsne_raster g,
                                                           float *__restrict__ out) {
  __shared__ float4 pts[kKdeThreads];
  const int64_t per_row = ((int64_t)g.gx + kKdeCells - 1) / kKdeCells;
  const int64_t slot = (int64_t)blockIdx.x * kKdeThreads + threadIdx.x;
  const int64_t v = slot / per_row, u0 = (slot - v * per_row) * kKdeCells;
  const bool live = v < g.gy;
  const float cy = g.y0 + ((float)v + 0.5f) * g.cy;
  float cx[kKdeCells];
#pragma unroll
  for (int k = 0; k < kKdeCells; ++k) cx[k] = g.x0 + ((float)(u0 + k) + 0.5f) * g.cx;
  double acc[kKdeCells] = {};
  for (int64_t j0 = 0; j0 < n; j0 += kKdeThreads) {
    __syncthreads();
    const int64_t j = j0 + threadIdx.x;
    if (j < n) {
      const float2 p = y[j];
      const double b = beta[j];
      pts[threadIdx.x] = make_float4(p.x, p.y, (float)(b * kLog2e), (float)(b * kInvPi));
    }
    __syncthreads();
    const int cnt = (int)((n - j0) < kKdeThreads ? (n - j0) : kKdeThreads);
    float s[kKdeCells] = {};
    for (int q = 0; q < cnt; ++q) {
      const float4 p = pts[q];
      const float dy = cy - p.y, dy2 = dy * dy;
#pragma unroll
      for (int k = 0; k < kKdeCells; ++k) {
        const float dx = cx[k] - p.x;
        const float r2 = fmaf(dx, dx, dy2);
        s[k] = fmaf(p.w, __builtin_amdgcn_exp2f(-p.z * r2), s[k]);
      }
    }
#pragma unroll
    for (int k = 0; k < kKdeCells; ++k) acc[k] += (double)s[k];
  }
  if (!live) return;
  const double scale = (double)g.cx * (double)g.cy / (double)n;
#pragma unroll
  for (int k = 0; k < kKdeCells; ++k)
    if (u0 + k < g.gx) out[v * g.gx + u0 + k] = (float)(acc[k] * scale);
}

}  // namespace

namespace tsne {

hipError_t launch_kde_raster(const float *y, int64_t n, const double *beta, const tsne_raster &g,
                             float *out, hipStream_t st) {
  const float2 *yy = reinterpret_cast<const float2 *>(y);
  const int64_t tiles = (((int64_t)g.gx + kKdeTile - 1) / kKdeTile) *
                        (((int64_t)g.gy + kKdeTile - 1) / kKdeTile);
  const int64_t slots = (int64_t)g.gy * (((int64_t)g.gx + kKdeCells - 1) / kKdeCells);
  // A tile costs n x 5.8 ns x tiles / 256 once the chip is full, the thread per four cells n x
  // max(56, 39 x slots / 65,536) ns: the threads are faster from about 2,560 tiles with up to 37
  // slots each, rasters of at most four rows or columns (10,000 points: 262,144 x 4 cells 1.65 ms
  // against 1.88, x 8 3.16 against 1.87; 32,768 x 1 0.57 against 0.27). And a tile's sums and
  // exchange take 4 us whatever the points: one point on 2,048 x 2,048 cells 14 us against 17,
  // 64 points 53 against 17.
  if (n <= 16 || (tiles > 2560 && slots <= 37 * tiles)) {
    hipLaunchKernelGGL(k_kde_cells, dim3((unsigned)((slots + kKdeThreads - 1) / kKdeThreads)),
                       dim3(kKdeThreads), 0, st, yy, beta, n, g, out);
    return hipGetLastError();
  }
  // tiles over both grid dimensions: a launch holds fewer than 2^32 threads along x, and a raster
  // of one row or column of 2^30 cells has 2^25 tiles
  constexpr int64_t kAlong = (int64_t)1 << 20;
  const dim3 grid((unsigned)(tiles < kAlong ? tiles : kAlong),
                  (unsigned)((tiles + kAlong - 1) / kAlong));
  auto tiled = [&](auto w) {
    constexpr int W = decltype(w)::value;
    static_assert(kAlong * 64 * W < ((int64_t)1 << 32), "threads along x");
    static_assert(sizeof(KdeSmem<W>) <= 160 * 1024, "one workgroup per compute unit");
    hipLaunchKernelGGL(k_kde_raster<W>, grid, dim3(64 * W), 0, st, yy, beta, n, g, out);
  };
  // Waves to a tile: no more than there are chunks, and sixteen only where there is no more than
  // a tile to a compute unit. 2,048 x 2,048 cells, sixteen, four and one: 256 points 160, 54 and
  // 36 us, 1,000 163, 110 and 110, 4,096 433, 389 and 403; 512 x 512 cells: 1,000 points 14.8,
  // 14.4 and 37, 65,536 440, 513 and 1,922.
  if (n <= kKdeChunk)
    tiled(std::integral_constant<int, 1>{});
  else if (n <= 4 * kKdeChunk || tiles > 256)
    tiled(std::integral_constant<int, 4>{});
  else
    tiled(std::integral_constant<int, 16>{});
  return hipGetLastError();
}

}  // namespace tsne
