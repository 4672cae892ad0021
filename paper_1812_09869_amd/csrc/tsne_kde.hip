// Perplexity-adaptive kernel density estimate of a 2-D map (paKDE, section
// "Perplexity-adaptive Kernel Density Estimation"): every map point gets the
// precision beta_j of the same perplexity search as the input affinities, run
// on the map's squared distances; the density is the sample smoothing
// estimator with bivariate Gaussian kernels of bandwidth h_j^2 = 1 / beta_j,
//   f(c) = (S / n) sum_j (beta_j / pi) exp(-beta_j |c - y_j|^2),
// evaluated at the centres of a regular raster with cells of area S.
#include <hip/hip_runtime.h>
#include <math.h>

#include "../../include/tsne355.h"
#include "tsne_internal.h"

namespace {

constexpr int kKdeTile = 32;     // raster tile of a workgroup: 32 x 32 cells
constexpr int kKdeWaves = 16;    // waves of a workgroup, each a share of the points
constexpr int kKdeStage = 64;    // points a wave stages at a time
constexpr int kKdeChunk = 256;   // points summed in FP32 before their sum goes to FP64
constexpr double kLog2e = 1.4426950408889634074;
constexpr double kInvPi = 0.31830988618379067154;

typedef float v16f __attribute__((ext_vector_type(16)));

struct KdeSmem {
  union {
    float4 pts[kKdeWaves][kKdeStage];                // {x, y, beta log2(e), beta / pi}
    double sum[kKdeWaves][kKdeTile][kKdeTile];       // the waves' partial rasters
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
// A workgroup covers one tile; its waves share the points in contiguous
// pieces, so that a small raster still fills its compute units. As before, 256
// points are summed in FP32 and the chunk sums in FP64; the waves' sums meet in
// LDS in wave order.
__global__ __launch_bounds__(64 * kKdeWaves) void k_kde_raster(const float2 *__restrict__ y,
                                                               const double *__restrict__ beta,
                                                               int64_t n, tsne_raster g,
                                                               float *__restrict__ out) {
  __shared__ KdeSmem sm;
  const int t = threadIdx.x, w = t >> 6, l = t & 63, li = l & 31, lk = l >> 5;
  const unsigned across = (unsigned)(((int64_t)g.gx + kKdeTile - 1) / kKdeTile);
  const unsigned tile = blockIdx.y * gridDim.x + blockIdx.x;
  const int64_t u0 = (int64_t)(tile % across) * kKdeTile, v0 = (int64_t)(tile / across) * kKdeTile;
  if (v0 >= g.gy) return;  // past the last tile (the grid's last row)
  const float cx = g.x0 + ((float)(u0 + li) + 0.5f) * g.cx;
  const float cy = g.y0 + ((float)(v0 + li) + 0.5f) * g.cy;
  // this wave's points: whole chunks
  const int64_t chunks = (n + kKdeChunk - 1) / kKdeChunk;
  const int64_t c0 = chunks * w / kKdeWaves, c1 = chunks * (w + 1) / kKdeWaves;
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
#pragma unroll 1
    for (int q = 0; q < kKdeChunk; q += kKdeStage) {
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
  for (int r = 0; r < 16; ++r) sm.sum[w][8 * (r >> 2) + 4 * lk + (r & 3)][li] = acc[r];
  __syncthreads();
  const int64_t v = v0 + (t >> 5), u = u0 + (t & 31);
  if (v >= g.gy || u >= g.gx) return;
  double f = 0.0;
#pragma unroll
  for (int q = 0; q < kKdeWaves; ++q) f += sm.sum[q][t >> 5][t & 31];
  out[v * g.gx + u] = (float)(f * ((double)g.cx * (double)g.cy / (double)n));
}

}  // namespace

namespace tsne {

hipError_t launch_kde_raster(const float *y, int64_t n, const double *beta, const tsne_raster &g,
                             float *out, hipStream_t st) {
  static_assert(sizeof(KdeSmem) <= 160 * 1024, "one workgroup per compute unit");
  const int64_t tiles = (((int64_t)g.gx + kKdeTile - 1) / kKdeTile) *
                        (((int64_t)g.gy + kKdeTile - 1) / kKdeTile);
  // tiles over both grid dimensions: a launch holds fewer than 2^32 threads along x, and a raster
  // of one row or column of 2^30 cells has 2^25 tiles
  constexpr int64_t kAlong = (int64_t)1 << 20;
  static_assert(kAlong * 64 * kKdeWaves < ((int64_t)1 << 32), "threads along x");
  const dim3 grid((unsigned)(tiles < kAlong ? tiles : kAlong),
                  (unsigned)((tiles + kAlong - 1) / kAlong));
  hipLaunchKernelGGL(k_kde_raster, grid, dim3(64 * kKdeWaves), 0, st,
                     reinterpret_cast<const float2 *>(y), beta, n, g, out);
  return hipGetLastError();
}

}  // namespace tsne
