// Input affinities P on the GPU (section "Similarities in the input space",
// Eqs. 1-3 of the bigMap paper):
//   1. centre X (distances are translation invariant) and form row norms;
//   2. per block of T rows: squared distances to all points on MFMA
//      (d_ij = |x_i|^2 + |x_j|^2 - 2 x_i.x_j), a per-row bracketed search on
//      the Gaussian precision beta_i so that the entropy of p_{.|i} equals
//      ln(perplexity), and a copy of the block's upper-triangle tiles into
//      the P store;
//   3. in place over the stored tiles: p_ij = (p_{j|i} + p_{i|j}) / (2n).
#include <float.h>
#include <math.h>

#include <type_traits>

#include "tsne_internal.h"
#include "tsne_tile.h"

namespace tsne {

namespace {

constexpr double kLog2e = 1.4426950408889634074;
constexpr double kLn2 = 0.69314718055994530942;
constexpr float kBig = 3.0e38f;  // stands for an excluded entry (self pair)


__device__ inline void flag_error(Hdr *h, uint32_t bit) { atomicOr(&h->err, bit); }

// Implicit P: the kernels of a pass run only on a workspace whose header
// records implicit affinities for the same n, d and distance mode (its layout,
// hence every offset these kernels use, depends on all three); key is
// implicit_key(d, mode).
__device__ inline bool implicit_ready(const Hdr *h, int64_t n, int32_t key) {
  return h->magic == kMagic && h->n == n && implicit_key(h->d, h->mode) == key && h->ready == 2;
}

// ----------------------------------------------------------------------------
// Wave / block reductions (fixed order, hence deterministic)
// ----------------------------------------------------------------------------
__device__ inline double wave_sum_d(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}
__device__ inline int wave_max_i(int v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = max(v, __shfl_xor(v, o, 64));
  return __builtin_amdgcn_readfirstlane(v);
}
__device__ inline float wave_min_f(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = fminf(v, __shfl_xor(v, o, 64));
  return v;
}

// x plus the x of another lane of its row of 16 (a DPP control).
template <int CTRL>
__device__ __forceinline__ double dpp_add(double x) {
  const int2 a = __builtin_bit_cast(int2, x);
  return x + __builtin_bit_cast(
                 double, make_int2(__builtin_amdgcn_mov_dpp(a.x, CTRL, 0xf, 0xf, true),
                                   __builtin_amdgcn_mov_dpp(a.y, CTRL, 0xf, 0xf, true)));
}

// ----------------------------------------------------------------------------
// 0. Header
// ----------------------------------------------------------------------------
__global__ void k_init_hdr(Hdr *h, int64_t n, int32_t d, int32_t mode, double perplexity) {
  if (threadIdx.x == 0) {
    h->magic = kMagic;
    h->n = n;
    h->d = d;
    h->ready = 0;
    h->err = 0;
    h->mode = mode;
    h->perplexity = perplexity;
    h->z = 0.0;
    h->c_p = 0.0;
    h->p_sum = 0.0;
    h->xmax = 0.f;
  }
}

// ----------------------------------------------------------------------------
// 1. Column means (FP64) and centred, transposed X with FP64 row norms
// ----------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_colmean(const float *__restrict__ x, int64_t n, int32_t d,
                                                 double *__restrict__ mean) {
  __shared__ double red[4];
  const int k = blockIdx.x;
  double s = 0.0;
  for (int64_t i = threadIdx.x; i < n; i += 256) s += (double)x[i * d + k];
  s = wave_sum_d(s);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0) mean[k] = (red[0] + red[1] + red[2] + red[3]) / (double)n;
}

__global__ __launch_bounds__(256) void k_centre(const float *__restrict__ x, int64_t n, int32_t d,
                                                int64_t npad, int32_t dpad,
                                                const double *__restrict__ mean,
                                                double *__restrict__ xcT,
                                                double *__restrict__ norms, Hdr *h) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= npad) return;
  double nrm = 0.0;
  bool bad = false;
  float amax = 0.f;
  for (int k = 0; k < dpad; ++k) {
    double v = 0.0;
    if (i < n && k < d) {
      float xv = x[i * d + k];
      bad |= !isfinite(xv);
      v = (double)xv - mean[k];
    }
    xcT[(int64_t)k * npad + i] = v;
    nrm += v * v;
    amax = fmaxf(amax, fabsf((float)v));
  }
  norms[i] = nrm;
  if (bad) flag_error(h, kErrNonFinite);
  // max |centred x| over the wave, then one atomic per wave (non-negative
  // floats order like their bit patterns)
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) amax = fmaxf(amax, __shfl_xor(amax, o, 64));
  if ((threadIdx.x & 63) == 0 && isfinite(amax))
    atomicMax(reinterpret_cast<unsigned int *>(&h->xmax), __float_as_uint(amax));
}

// Place of a workgroup of a distance launch: column strip x of nx, 64-row strip
// of row block z of the group. Consecutive workgroups go to the eight XCDs in
// turn, so the strips of an XCD's turn are the row strips of one column strip:
// its columns come into that XCD's L2 once (in row-major order every row strip
// read all columns anew, 4.2 MB an XCD at n = 65,536 against 4 MB of L2). The
// affinity stage there: 23.4 ms, so 22.7; the FP64 kernel, whose strips are half as
// wide and which is bound by its MFMAs, keeps the row order (29.1 against 31.0).
// False for the padding workgroups of the last turn. Grid: dist_grid.
__device__ __forceinline__ bool dist_place(int nx, int blocks, int &x, int &row0, int &z) {
  const unsigned rows = (unsigned)blocks * (T / 64), k = blockIdx.x / 8;
  x = (int)(8 * (k / rows) + blockIdx.x % 8);
  row0 = 64 * (int)(k % rows % (T / 64));
  z = (int)(k % rows / (T / 64));
  return x < nx;
}
static dim3 dist_grid(int64_t nx, int blocks) {
  return dim3((unsigned)((nx + 7) / 8 * 8 * blocks * (T / 64)));
}

// ----------------------------------------------------------------------------
// 2a. Distance block on FP64 MFMA: rows b*T .. b*T+T-1 against all columns.
//
// v_mfma_f64_16x16x4f64 computes a 16x16 block of A(16x4) B(4x16). Lane l
// supplies A[l%16][l/16] and B[l/16][l%16] and receives D[l/16 + 4r][l%16]
// in accumulator element r (rows interleaved by 4, unlike the FP32/BF16
// 16x16 variants, whose element r holds row 4(l/16) + r). X is stored transposed (k-major), so the 16
// lanes that share a k read 16 consecutive doubles. A wave computes a
// 64 x 16 kDistCT block (4 x kDistCT MFMA tiles, small enough for two waves
// per SIMD); a workgroup of 4 waves covers 64 rows x 64 kDistCT columns.
// ----------------------------------------------------------------------------
constexpr int kDistCT = 2;  // 16-column MFMA tiles per wave (a wave covers 64 x 16 kDistCT)

// With P given, the block row's tiles (J >= b) also go straight to their
// place in the packed buffer, in the layout k_stage writes, as in k_dist_x3:
// for each of its rows a lane holds columns cl + li and cl + 16 + li of the
// tile (cl = 128 h + 32 w, h the half of the tile this workgroup covers),
// the two consecutive elements 2 (w mod 2) and 2 (w mod 2) + 1 of one float4
// there. The column strips are rotated so that the diagonal tile's are
// dispatched first.
static_assert(kDistCT == 2, "the packed stores assume 32 columns per wave");
__global__ __launch_bounds__(256) void k_dist_f64(const double *__restrict__ xcT,
                                                  const double *__restrict__ norms, int64_t npad,
                                                  int32_t dpad, int32_t b,
                                                  float *__restrict__ dblock,
                                                  float4 *__restrict__ P, int32_t nb) {
  b += blockIdx.z;  // row block of the group, its distances in the group's slot
  dblock += (size_t)blockIdx.z * T * npad;
  const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
  const int xs = (int)((blockIdx.x + 2u * (unsigned)b) % gridDim.x);  // column strip
  const int row0_loc = blockIdx.y * 64;
  const int J = xs >> 1, cl = 128 * (xs & 1) + 32 * w;
  const int64_t col0 = (int64_t)xs * (64 * kDistCT) + w * (16 * kDistCT);
  const int64_t row0 = (int64_t)b * T + row0_loc;
  const int li = l & 15, lk = l >> 4;
  v4d acc[4][kDistCT];
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int c = 0; c < kDistCT; ++c) acc[a][c] = (v4d){0.0, 0.0, 0.0, 0.0};
  for (int k0 = 0; k0 < dpad; k0 += 4) {
    const double *xk = xcT + (int64_t)(k0 + lk) * npad;
    double av[4], bv[kDistCT];
#pragma unroll
    for (int a = 0; a < 4; ++a) av[a] = xk[row0 + a * 16 + li];
#pragma unroll
    for (int c = 0; c < kDistCT; ++c) bv[c] = xk[col0 + c * 16 + li];
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
      for (int c = 0; c < kDistCT; ++c)
        acc[a][c] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[a], bv[c], acc[a][c], 0, 0, 0);
  }
  // every norm is loaded before the first store, so no store waits on a load
  double ni[4][4], nj[kDistCT];
#pragma unroll
  for (int c = 0; c < kDistCT; ++c) nj[c] = norms[col0 + c * 16 + li];
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int r = 0; r < 4; ++r) ni[a][r] = norms[(int64_t)b * T + row0_loc + a * 16 + lk + 4 * r];
  float *pt = (P != nullptr && J > b)
                  ? reinterpret_cast<float *>(P + (size_t)(tile_start(b, nb) + (J - b)) * TT4)
                  : nullptr;
  float *pd = (P != nullptr && J == b) ? reinterpret_cast<float *>(P + (size_t)tile_start(b, nb) * TT4)
                                       : nullptr;
  auto packed = [](int i, int j) {  // float of (row i, column j) of a tile
    return 4 * ((4 * (i >> 4) + (j >> 6)) * 256 + 16 * (i & 15) + (j & 15)) + ((j >> 4) & 3);
  };
#pragma unroll
  for (int a = 0; a < 4; ++a) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int il = row0_loc + a * 16 + lk + 4 * r;
      float v[kDistCT];
#pragma unroll
      for (int c = 0; c < kDistCT; ++c) {
        const int64_t j = col0 + c * 16 + li;
        double dd = ni[a][r] + nj[c] - 2.0 * acc[a][c][r];
        v[c] = (float)fmax(dd, 0.0);
        dblock[(int64_t)il * npad + j] = v[c];
      }
      if (pt) {
        *reinterpret_cast<float2 *>(pt + packed(il, cl + li)) = make_float2(v[0], v[1]);
      } else if (pd) {
#pragma unroll
        for (int c = 0; c < kDistCT; ++c) {
          const int jl = cl + 16 * c + li;  // column within the tile
          if (jl >= il) {
            pd[packed(il, jl)] = v[c];
            if (jl > il) pd[packed(jl, il)] = v[c];
          }
        }
      }
    }
  }
}

// ----------------------------------------------------------------------------
// 2a'. Reduced-precision distance contraction (the precision path).
//
// FP32 mode: the FP64-centred X rounded to FP32, v_mfma_f32_16x16x4f32, norms
// of the rounded points, d = (n_i + n_j) - 2 x.y in FP32.
// BF16 / FP16 modes: operands rounded to 16 bits, v_mfma_f32_16x16x32_{bf16,f16}
// with FP32 accumulation, and the norms of the rounded operands, so that d is
// the exact squared distance of two slightly moved points (never negative, no
// cancellation blow-up of the dot-product error). FP16 operands are scaled by
// a power of two so that max |x| maps to <= 256 (exact, undone after the
// contraction).
// These three keep the cancellation of |x|^2 + |y|^2 - 2 x.y: near pairs
// have d ~ 200 against |x|^2 ~ 1,350 on the benchmark data, so an FP32
// rounding of the large terms moves d by ~1e-4. The x3 modes (2a'' below)
// remove it.
// 16x16x32 layout: lane l supplies A[l%16][8(l/16) .. 8(l/16)+7] and the
// matching B column slice, and receives D[4(l/16) + r][l%16] in element r.
// ----------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_prep_f32(const double *__restrict__ xcT, int64_t npad,
                                                  int32_t dpad, float *__restrict__ xfT,
                                                  float *__restrict__ norms32) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= npad) return;
  double nrm = 0.0;
  for (int k = 0; k < dpad; ++k) {
    const float v = (float)xcT[(int64_t)k * npad + i];
    xfT[(int64_t)k * npad + i] = v;
    nrm += (double)v * (double)v;
  }
  norms32[i] = (float)nrm;
}

template <typename H, bool SCALE>
__global__ __launch_bounds__(256) void k_prep_lp(const double *__restrict__ xcT, int64_t npad,
                                                 int32_t d, int32_t k32, H *__restrict__ xa,
                                                 float *__restrict__ norms32, const Hdr *h) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= npad) return;
  const float s = SCALE ? fp16_scale(h) : 1.f;
  H *ra = xa + i * k32;
  double nrm = 0.0;
  for (int k = 0; k < k32; ++k) {
    const float v = (k < d) ? (float)xcT[(int64_t)k * npad + i] : 0.f;
    const H hi = (H)(v * s);
    ra[k] = hi;
    const double hv = (double)(float)hi / (double)s;
    nrm += hv * hv;
  }
  norms32[i] = (float)nrm;
}

__global__ __launch_bounds__(256) void k_dist_f32(const float *__restrict__ xfT,
                                                  const float *__restrict__ norms, int64_t npad,
                                                  int32_t dpad, int32_t b,
                                                  float *__restrict__ dblock) {
  b += blockIdx.z;
  dblock += (size_t)blockIdx.z * T * npad;
  const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
  const int64_t col0 = (int64_t)blockIdx.x * 256 + w * 64;
  const int row0_loc = blockIdx.y * 64;
  const int64_t row0 = (int64_t)b * T + row0_loc;
  const int li = l & 15, lk = l >> 4;
  v4f acc[4][4];
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int c = 0; c < 4; ++c) acc[a][c] = (v4f){0.f, 0.f, 0.f, 0.f};
  for (int k0 = 0; k0 < dpad; k0 += 4) {
    const float *xk = xfT + (int64_t)(k0 + lk) * npad;
    float av[4], bv[4];
#pragma unroll
    for (int a = 0; a < 4; ++a) av[a] = xk[row0 + a * 16 + li];
#pragma unroll
    for (int c = 0; c < 4; ++c) bv[c] = xk[col0 + c * 16 + li];
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
      for (int c = 0; c < 4; ++c)
        acc[a][c] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[a], bv[c], acc[a][c], 0, 0, 0);
  }
  // every norm is loaded before the first store, so no store waits on a load
  float ni[4][4], nj[4];
#pragma unroll
  for (int c = 0; c < 4; ++c) nj[c] = norms[col0 + c * 16 + li];
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int r = 0; r < 4; ++r) ni[a][r] = norms[(int64_t)b * T + row0_loc + a * 16 + 4 * lk + r];
#pragma unroll
  for (int a = 0; a < 4; ++a) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int il = row0_loc + a * 16 + 4 * lk + r;
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const int64_t j = col0 + c * 16 + li;
        const float dd = (ni[a][r] + nj[c]) - 2.f * acc[a][c][r];
        dblock[(int64_t)il * npad + j] = fmaxf(dd, 0.f);
      }
    }
  }
}

template <typename H, typename V8, bool SCALE>
__global__ __launch_bounds__(256) void k_dist_lp(const H *__restrict__ xa,
                                                 const float *__restrict__ norms, int64_t npad,
                                                 int32_t kk, int32_t b, float *__restrict__ dblock,
                                                 const Hdr *h) {
  b += blockIdx.z;
  dblock += (size_t)blockIdx.z * T * npad;
  const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
  const int64_t col0 = (int64_t)blockIdx.x * 256 + w * 64;
  const int row0_loc = blockIdx.y * 64;
  const int64_t row0 = (int64_t)b * T + row0_loc;
  const int li = l & 15, lk = l >> 4;
  float inv_s2 = 1.f;
  if (SCALE) {
    const float s = fp16_scale(h);
    inv_s2 = 1.f / (s * s);
  }
  v4f acc[4][4];
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int c = 0; c < 4; ++c) acc[a][c] = (v4f){0.f, 0.f, 0.f, 0.f};
  for (int k0 = 0; k0 < kk; k0 += 32) {
    V8 av[4], bv[4];
#pragma unroll
    for (int a = 0; a < 4; ++a)
      av[a] = *reinterpret_cast<const V8 *>(xa + (row0 + a * 16 + li) * kk + k0 + 8 * lk);
#pragma unroll
    for (int c = 0; c < 4; ++c)
      bv[c] = *reinterpret_cast<const V8 *>(xa + (col0 + c * 16 + li) * kk + k0 + 8 * lk);
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        if constexpr (sizeof(H) == 2 && __is_same(H, __bf16))
          acc[a][c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av[a], bv[c], acc[a][c], 0, 0, 0);
        else
          acc[a][c] = __builtin_amdgcn_mfma_f32_16x16x32_f16(av[a], bv[c], acc[a][c], 0, 0, 0);
      }
  }
  // every norm is loaded before the first store, so no store waits on a load
  float ni[4][4], nj[4];
#pragma unroll
  for (int c = 0; c < 4; ++c) nj[c] = norms[col0 + c * 16 + li];
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int r = 0; r < 4; ++r) ni[a][r] = norms[(int64_t)b * T + row0_loc + a * 16 + 4 * lk + r];
#pragma unroll
  for (int a = 0; a < 4; ++a) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int il = row0_loc + a * 16 + 4 * lk + r;
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const int64_t j = col0 + c * 16 + li;
        const float dd = (ni[a][r] + nj[c]) - 2.f * (acc[a][c][r] * inv_s2);
        dblock[(int64_t)il * npad + j] = fmaxf(dd, 0.f);
      }
    }
  }
}

// ----------------------------------------------------------------------------
// 2a''. The x3 modes: exact-accumulate slices and a compensated FP32 combine.
//
// Every centred coordinate is cut on one grid for the whole data set,
//   x = sigma (h1 + 2^-b h2 + 2^-2b h3) + r,  sigma = 2^(E - b), max |x| < 2^E,
// rounding to the nearest integer at each level (|h1| <= 2^b, |h2|, |h3| <=
// 2^(b-1), |r| <= sigma 2^(-2b-1)). b is the largest value with
// 2b + log2(K) <= 24 (K = d rounded up to 32), at most 10 for FP16 and 8 for
// BF16, so each slice is exact in 16 bits and
//   A0 = sum_k h1 h1'
// is an integer below 2^24: the MFMA's FP32 accumulation adds it exactly, in
// whatever order it works. The rest of the contraction, scaled by 2^b,
//   R = sum_k (h1 h2' + h2 h1') + 2^-b (h1 h3' + h2 h2' + h3 h1')
//       + 2^-2b (h2 h3' + h3 h2'),
// is 2^-b smaller and is allowed to round. Its operands are stored as four
// slices per point, [h1 | h2 | 2^-b h2 | 2^-b h3] (all normal numbers in
// both formats), so R takes seven MFMA products and A0 one. Then
//   x.y = sigma^2 (A0 + 2^-b R);
// the product left out (h3 h3') is below sigma^2 2^-4b K 2^2b.
// The norms are FP32 pairs (hi, lo) of the FP64 norm of the represented point
// sigma (h1 + 2^-b h2 + 2^-2b h3). d = n_i + n_j - 2 x.y cancels most of its
// operands, so it is formed with error-free transformations: TwoSum of the
// two hi parts, the exact difference of that sum and 2 sigma^2 A0, then the
// small terms (the TwoSum error, the lo parts and 2 sigma^2 2^-b R) added to
// the leading difference. d then carries about one FP32 rounding of d
// itself instead of one of |x|^2.
// Operand layout: per point, per block of 32 values of k, the four slices'
// 32 values in a row ([point][k / 32][slice][32]), so that the four
// fragments a lane loads for one MFMA step sit in one 256-byte segment.
// ----------------------------------------------------------------------------
template <typename H>
__global__ __launch_bounds__(256) void k_prep_x3(const double *__restrict__ xcT, int64_t npad,
                                                 int32_t d, int32_t k32, int32_t b,
                                                 H *__restrict__ xs, float2 *__restrict__ nhl,
                                                 const Hdr *h) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= npad) return;
  const int E = x3_exp(h);
  H *row = xs + i * (4 * (int64_t)k32);
  double nrm = 0.0;
  for (int k = 0; k < k32; ++k) {
    const double v = (k < d) ? xcT[(int64_t)k * npad + i] : 0.0;
    const double q = ldexp(v, b - E);
    const double h1 = rint(q);
    double r = ldexp(q - h1, b);
    const double h2 = rint(r);
    r = ldexp(r - h2, b);
    const double h3 = rint(r);
    H *blk = row + (k >> 5) * 128 + (k & 31);
    blk[0] = (H)(float)h1;
    blk[32] = (H)(float)h2;
    blk[64] = (H)(float)ldexp(h2, -b);
    blk[96] = (H)(float)ldexp(h3, -b);
    const double xr = ldexp(h1 + ldexp(h2 + ldexp(h3, -b), -b), E - b);
    nrm += xr * xr;
  }
  const float hi = (float)nrm;
  nhl[i] = make_float2(hi, (float)(nrm - (double)hi));
}

// Distance block of the x3 modes: a workgroup covers 64 rows x 256 columns,
// as k_dist_lp. With P given, the block row's tiles (J >= b) also go
// straight to their place in the packed buffer, in the layout k_stage
// writes, so that no staging pass follows: lane (li, lk) of wave w holds,
// for each of its rows tr + 16 k of a tile, columns li + 16 (4 w + c),
// c = 0 .. 3, which is the float4 4 k + w of thread 16 tr + li there.
template <typename H, typename V8>
__global__ __launch_bounds__(256, 2) void k_dist_x3(const H *__restrict__ xs,
                                                 const float2 *__restrict__ nhl, int64_t npad,
                                                 int32_t k32, int32_t bits, int32_t b,
                                                 int32_t blocks, float *__restrict__ dblock,
                                                 const Hdr *h, float4 *__restrict__ P,
                                                 int32_t nb) {
  int strip, row0_loc, z;
  if (!dist_place(nb, blocks, strip, row0_loc, z)) return;
  b += z;
  dblock += (size_t)z * T * npad;
  const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
  // column tile, rotated so that the diagonal one (the workgroups with the
  // most stores) is dispatched first
  const int J = (int)((unsigned)(strip + b) % (unsigned)nb);
  const int64_t col0 = (int64_t)J * 256 + w * 64;
  const int64_t row0 = (int64_t)b * T + row0_loc;
  const int li = l & 15, lk = l >> 4;
  v4f A0[4][4], R[4][4];
  __shared__ X3Smem<V8> sm;
  x3_contract<H, V8>(xs, k32, row0, col0, threadIdx.x, A0, R, sm);
  const X3Scale sc = x3_scale(h, bits);
  // every norm is loaded before the first store, so no store waits on a load
  float2 nj[4], ni[4][4];
#pragma unroll
  for (int c = 0; c < 4; ++c) nj[c] = nhl[col0 + c * 16 + li];
#pragma unroll
  for (int t = 0; t < 4; ++t)
#pragma unroll
    for (int r = 0; r < 4; ++r) ni[t][r] = nhl[(int64_t)b * T + row0_loc + t * 16 + 4 * lk + r];
  float4 *pt = (P != nullptr && J > b) ? P + (size_t)(tile_start(b, nb) + (J - b)) * TT4 : nullptr;
  // the diagonal tile is symmetrised as k_stage does it: each value of the
  // upper triangle (diagonal included) goes to its own place and to the
  // mirrored one, one float at a time
  float *pd = (P != nullptr && J == b) ? reinterpret_cast<float *>(P + (size_t)tile_start(b, nb) * TT4)
                                       : nullptr;
  // float of (row i, column j) of a tile in that layout
  auto packed = [](int i, int j) {
    return 4 * ((4 * (i >> 4) + (j >> 6)) * 256 + 16 * (i & 15) + (j & 15)) + ((j >> 4) & 3);
  };
#pragma unroll
  for (int t = 0; t < 4; ++t) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int il = row0_loc + t * 16 + 4 * lk + r;
      float v[4];
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const int64_t j = col0 + c * 16 + li;
        v[c] = x3_combine(ni[t][r], nj[c], A0[t][c][r], R[t][c][r], sc);
        dblock[(int64_t)il * npad + j] = v[c];
      }
      if (pt) {
        pt[((il >> 4) * 4 + w) * 256 + 16 * (il & 15) + li] = make_float4(v[0], v[1], v[2], v[3]);
      } else if (pd) {
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          const int jl = 64 * w + 16 * c + li;  // column within the tile
          if (jl >= il) {
            pd[packed(il, jl)] = v[c];
            if (jl > il) pd[packed(jl, il)] = v[c];
          }
        }
      }
    }
  }
}

// ----------------------------------------------------------------------------
// 2b. Per-row search for beta (Eqs. 1-2).
//
// One workgroup of 1024 threads per row, one launch for the rows of a group
// of consecutive row blocks (their distances side by side in the scratch;
// b is the group's first block), so that rows needing more passes than
// others are spread over the compute units instead of setting the length of
// every block's launch. The row's distances, shifted by the row minimum m,
// are held in registers (VPT per thread) when they fit, else re-read from
// the scratch on every pass. Each pass forms, with FP32
// exponentials and FP32 per-thread partial sums combined in FP64,
//   S = sum_j exp(-beta (d_j - m)),  T = sum_j (d_j - m) exp(-beta (d_j - m)),
//   Q = sum_j (d_j - m)^2 exp(-beta (d_j - m)),
//   H = ln S + beta T / S,  dH/dbeta = -beta (Q / S - (T / S)^2),
// where beta is the FP32-rounded precision actually applied. The paper
// leaves the search to a supplement it does not include; H decreases in
// beta, so any bracketed search that reaches the tolerance finds the same
// root. Bracket logic: start with [0, inf) at the beta of the same position
// in the row block before the group (a nearby point in the locality order;
// 1 for the first group); each pass moves one end of the bracket to beta, then takes
// the Newton step if it lands inside the bracket, else doubles beta (no
// upper end yet) or bisects. Stops at |H - ln u| <= tol_h, at a bracket
// narrower than FP32 resolution, or after max_bisect passes (then the row is
// flagged as not converged).
// The per-wave FP64 partial sums meet in LDS; the first wave adds them in a
// fixed order and takes the step (all sixteen doing so cost 1.7 us of FP64
// issue a pass, four waves to a SIMD, against 0.8 and a barrier).
//
// What bounds it: one workgroup's registers hold the row, so nothing hides the
// load of the next (256 KB a compute unit at n = 65,536), then the chain of a pass
// (sums, barrier, FP64 step, barrier).
// Rows in the locality order: most waves' 64 consecutive points are too far to
// add anything (n = 65,536, perplexity 50: 95% of them) and are passed over, bit
// for bit; the test costs unordered rows more than the 4% it finds there.
// 1,024 rows of 65,536: 163 us, now 117 (20,000 points, 32 a thread: 93 and 68).
// Rows of a map (bandwidths): the distances are formed here, in FP64 from the
// coordinates, instead of written by one kernel (62 us) and read by this one
// (173 us): 180 us for both.
// ----------------------------------------------------------------------------
constexpr int kCalThreads = 1024;

struct CalOut {
  double *beta, *S, *H;
  float *m, *a, *r;
  int32_t *evals;
};

// Sums over the wave of R rows' values. R = 1: every lane ends with the total.
// R = 4: lane l ends with the total of row l / 16; the first two levels
// (distances 32 and 16) exchange whole rows between the halves with the
// lane-swap instructions, each halving the rows a lane carries, and the last
// four rotate inside the 16 lanes. The additions are those of an xor
// butterfly from distance 32 down, in its order (operands swapped at most).
__device__ __forceinline__ double swap32_add(double x, double y) {
  const int2 a = __builtin_bit_cast(int2, x), b = __builtin_bit_cast(int2, y);
  const auto lo = __builtin_amdgcn_permlane32_swap(a.x, b.x, false, false);
  const auto hi = __builtin_amdgcn_permlane32_swap(a.y, b.y, false, false);
  return __builtin_bit_cast(double, make_int2(lo[0], hi[0])) +
         __builtin_bit_cast(double, make_int2(lo[1], hi[1]));
}
__device__ __forceinline__ double swap16_add(double x, double y) {
  const int2 a = __builtin_bit_cast(int2, x), b = __builtin_bit_cast(int2, y);
  const auto lo = __builtin_amdgcn_permlane16_swap(a.x, b.x, false, false);
  const auto hi = __builtin_amdgcn_permlane16_swap(a.y, b.y, false, false);
  return __builtin_bit_cast(double, make_int2(lo[0], hi[0])) +
         __builtin_bit_cast(double, make_int2(lo[1], hi[1]));
}
template <int R>
__device__ __forceinline__ double rows_sum_d(const double (&x)[R]) {
  static_assert(R == 1 || R == 4, "a row to 16 lanes, or one row");
  double v;
  if constexpr (R == 1) {
    v = swap32_add(x[0], x[0]);
    v = swap16_add(v, v);
  } else {
    // lower half rows 0, 1, upper half rows 2, 3; then one row to 16 lanes
    v = swap16_add(swap32_add(x[0], x[2]), swap32_add(x[1], x[3]));
  }
  v = dpp_add<0x128>(v);
  v = dpp_add<0x124>(v);
  v = dpp_add<0x122>(v);
  return dpp_add<0x121>(v);
}

// Where the row's distances come from: the scratch (natural or locality order),
// or a map of two coordinates, FP64 as k_centre and k_dist_f64 form them.
enum CalRow { kCalPlain, kCalOrdered, kCalMap };

template <int VPT, CalRow ROW>
__global__ __launch_bounds__(kCalThreads) void k_calibrate(const float *__restrict__ dblock,
                                                           int64_t n, int64_t npad, int32_t b,
                                                           double logu, int max_bisect,
                                                           double tol_h, CalOut out, Hdr *h,
                                                           const float *__restrict__ y,
                                                           const double *__restrict__ ymean,
                                                           uint8_t *__restrict__ cand,
                                                           int32_t nb) {
  constexpr bool SKIP = ROW == kCalOrdered, MAP = ROW == kCalMap;
  static_assert(VPT > 0 || ROW == kCalPlain, "rows in registers");
  constexpr int NW = kCalThreads / 64;
  static_assert(NW == 16, "one partial per lane of a 16-lane group");
  __shared__ double sred[3][NW];
  __shared__ double snext, slo;
  __shared__ int sdone;
  __shared__ float smin[NW];
  const int tid = threadIdx.x, wv = tid >> 6, ln = tid & 63;
  const int64_t i = (int64_t)b * T + blockIdx.x;
  if (i >= n) return;
  const float *row = dblock + (MAP ? 0 : (int64_t)blockIdx.x * npad);

  // row minimum over j != i, j < n
  float mn = INFINITY;
  float v[VPT > 0 ? VPT : 1];
  if constexpr (VPT > 0) {
    const int nn = (int)n, ii = (int)i, j0 = __builtin_amdgcn_readfirstlane(wv) * 64;
    if constexpr (MAP) {
      const double m0 = ymean[0], m1 = ymean[1];
      const double c0 = (double)y[2 * i] - m0, c1 = (double)y[2 * i + 1] - m1;
      const double ni = fma(c1, c1, c0 * c0);
#pragma unroll
      for (int q = 0; q < VPT; ++q) {
        const float *p = y + 2 * min(q * kCalThreads + tid, nn - 1);
        const double x0 = (double)p[0] - m0, x1 = (double)p[1] - m1;
        const double nj = fma(x1, x1, x0 * x0);
        v[q] = (float)fmax(fma(-2.0, fma(c1, x1, c0 * x0), ni + nj), 0.0);
      }
    } else {
#pragma unroll
      for (int q = 0; q < VPT; ++q) {
        const int jq = q * kCalThreads;
        v[q] = row[jq + j0 < nn ? jq + tid : ln];  // (past n: any column there is)
      }
    }
#pragma unroll
    for (int q = 0; q < VPT; ++q) {
      // a wave's 64 columns: all valid unless they hold row i or pass n
      const int jq = q * kCalThreads + j0;
      if (jq + 64 > nn || (unsigned)(ii - jq) < 64u)
        v[q] = (jq + ln < nn && jq + ln != ii) ? v[q] : INFINITY;
      mn = fminf(mn, v[q]);
    }
  } else {
    for (int64_t j = tid; j < n; j += kCalThreads)
      if (j != i) mn = fminf(mn, row[j]);
  }
  mn = wave_min_f(mn);
  if (ln == 0) smin[wv] = mn;
  __syncthreads();
  float m = smin[0];
#pragma unroll
  for (int q = 1; q < NW; ++q) m = fminf(m, smin[q]);
  if constexpr (VPT > 0) {
#pragma unroll
    for (int q = 0; q < VPT; ++q) {
      // (only given dissimilarities can hold a NaN, which stays one)
      if (ROW == kCalPlain)
        v[q] = (v[q] == INFINITY) ? kBig : v[q] - m;
      else
        v[q] = fminf(v[q] - m, kBig);
    }
  }

  double beta = 1.0;
  if (b > 0) {
    const double bp = out.beta[(int64_t)(b - 1) * T + (blockIdx.x & (T - 1))];
    if (bp > 0.0 && isfinite(bp)) beta = bp;
  }
  double lo = 0.0, hi = INFINITY, S = 0.0, H = 0.0;
  float a = 0.f;
  int it = 0, done = 0;
  // MAP: once the bracket has a lower end, the points whose exponentials vanish
  // there (94% at n = 65,536, perplexity 100) do so in every later pass: each lane
  // copies its others to LDS, those of even q from the front of its column, those
  // of odd q from the back, and later passes read only them, in the same
  // order. A wave with a lane of more than kCap of them goes on with all.
  constexpr bool COMPACT = MAP && VPT >= 16;
  constexpr int kCap = COMPACT ? VPT / 2 + 4 : 1;
  __shared__ float kept[COMPACT ? NW : 1][kCap][64];
  int ne = 0, no = 0, me = -1, mo = 0, tries = 0;  // me, mo: longest of the wave; -1: not kept
  double lo_kept = 0.0;
  for (;;) {
    ++it;
    a = fmaxf((float)(beta * kLog2e), 1e-30f);
    float s0 = 0.f, s1 = 0.f, t0 = 0.f, t1 = 0.f, q0 = 0.f, q1 = 0.f;
    if (COMPACT && me >= 0) {
      auto add = [&](float d, float &s, float &t, float &qq) {
        const float e = __builtin_amdgcn_exp2f(-a * d);
        const float ve = d * e;
        s += e;
        t += ve;
        qq = fmaf(d, ve, qq);
      };
#pragma unroll 4
      for (int k = 0; k < me; ++k) add(k < ne ? kept[wv][k][ln] : kBig, s0, t0, q0);
#pragma unroll 4
      for (int k = 0; k < mo; ++k) add(k < no ? kept[wv][kCap - 1 - k][ln] : kBig, s1, t1, q1);
    } else if constexpr (VPT > 0) {
      // exp2(-a v) is exactly 0 from a v = 152 on, and adds exactly 0 to all
      // three sums: nothing to do where it is so for the wave's 64 points
      const float far = 153.f / a;
#pragma unroll
      for (int q = 0; q < VPT; ++q) {
        if (SKIP && !__builtin_amdgcn_ballot_w64(v[q] < far)) continue;
        const float e = __builtin_amdgcn_exp2f(-a * v[q]);
        const float ve = v[q] * e;  // 0 for an excluded entry (e = 0)
        float &s = q & 1 ? s1 : s0, &t = q & 1 ? t1 : t0, &qq = q & 1 ? q1 : q0;
        s += e;
        t += ve;
        qq = fmaf(v[q], ve, qq);
      }
    } else {
      for (int64_t j = tid; j < n; j += kCalThreads) {
        const float dm = (j == i) ? kBig : row[j] - m;
        const float e = __builtin_amdgcn_exp2f(-a * dm);
        const float ve = dm * e;
        s0 += e;
        t0 += ve;
        q0 = fmaf(dm, ve, q0);
      }
    }
    const double xs[3][1] = {{(double)(s0 + s1)}, {(double)(t0 + t1)}, {(double)(q0 + q1)}};
    const double ds = rows_sum_d(xs[0]), dt = rows_sum_d(xs[1]), dq = rows_sum_d(xs[2]);
    if (ln == 0) {
      sred[0][wv] = ds;
      sred[1][wv] = dt;
      sred[2][wv] = dq;
    }
    __syncthreads();
    if (wv == 0) {
      // the 16 wave partials, summed in one fixed order, and the step
      auto sum16 = [&](const double *part) {
        return dpp_add<0x121>(dpp_add<0x122>(dpp_add<0x124>(dpp_add<0x128>(part[ln & 15]))));
      };
      const double SS = sum16(sred[0]), TT = sum16(sred[1]), QQ = sum16(sred[2]);
      const double beff = (double)a * kLn2;
      S = SS;
      const double mean = TT / SS;
      H = log(SS) + beff * mean;
      if (fabs(H - logu) <= tol_h) {
        done = 1;
      } else if (isfinite(hi) && (hi - lo) <= hi * 0x1p-24) {
        done = 1;
      } else if (it >= max_bisect) {
        done = 2;
      } else {
        // H falls with beta (dH/dbeta = -beta Var(d)): shrink the bracket of
        // FP64 iterates, then take the Newton step if it lands inside it,
        // else bisect (H was taken at beff, within 2^-24 of beta)
        if (H > logu)
          lo = beta;
        else
          hi = beta;
        const double var = QQ / SS - mean * mean;
        const double nb = beta + (H - logu) / (beff * var);
        if (var > 0.0 && nb > lo && nb < hi && isfinite(nb))
          beta = nb;
        else
          beta = isinf(hi) ? 2.0 * beta : 0.5 * (lo + hi);
      }
      if (ln == 0) {
        snext = done ? 1.0 / (2.0 * (double)n * S) : beta;
        slo = lo;
        sdone = done;
      }
    }
    __syncthreads();
    if (sdone) break;
    beta = snext;
    if (COMPACT && me < 0 && tries < 2 && slo > lo_kept) {
      ++tries;
      lo_kept = slo;
      // every later a is at least this one
      const float far = 153.f / fmaxf((float)(lo_kept * kLog2e), 1e-30f);
      ne = no = 0;
#pragma unroll
      for (int q = 0; q < VPT; ++q) {
        if (v[q] < far) {
          if (ne + no < kCap) kept[wv][q & 1 ? kCap - 1 - no : ne][ln] = v[q];
          if (q & 1)
            ++no;
          else
            ++ne;
        }
      }
      if (!__builtin_amdgcn_ballot_w64(ne + no > kCap)) {
        me = wave_max_i(ne);
        mo = wave_max_i(no);
      }
    }
  }
  // Tiles this row may give a nonzero p to; all others are zero and need no pass
  // over their distances. A stored p below FLT_MIN = 2^-126 is zero, and from
  // here on a side's term exp2(-a v) r is below 2^-128, so that both sides'
  // sum is too (each order of a pair marks the same tile).
  const float rs = (float)snext;
  if constexpr (SKIP) {
    const float far = (128.5f + __builtin_amdgcn_logf(rs)) / a;
    const int I = (int)(i / T);
#pragma unroll
    for (int q = 0; q < VPT; ++q) {
      if (!__builtin_amdgcn_ballot_w64(!(v[q] >= far))) continue;
      // groups past the last tile have none, whatever far came to (a row whose search ends
      // without a finite sum has no limit: all of its tiles are marked)
      const int J = (q * kCalThreads + wv * 64) / T;
      if (ln == 0 && J < nb) cand[tile_start(min(I, J), nb) + (I < J ? J - I : I - J)] = 1;
    }
  }
  if (tid == 0) {
    const double beff = (double)a * kLn2;
    const bool ok = (done == 1);
    out.beta[i] = beff;
    out.S[i] = S;
    out.H[i] = H;
    out.m[i] = m;
    out.a[i] = a;
    out.r[i] = rs;
    out.evals[i] = ok ? it : -it;
    if (!ok) flag_error(h, kErrNoConv);
    if (!isfinite(H) || !isfinite(S)) flag_error(h, kErrNonFinite);
  }
}

// The search of a row kept in the registers of one wave. Lane l holds the state
// of row l / 16 (R = 4) or of the one row (R = 1): the FP64 arithmetic of a step,
// several times the exponentials of 16 points a lane, is done once for all rows
// of the wave.
struct RowSearch {
  double S, H;
  float a, m;
  int it, done;
  // Results of row i, by one lane. bad: a non-finite distance.
  __device__ void store(const CalOut &out, int64_t i, int64_t n, bool bad, Hdr *h) const {
    out.beta[i] = (double)a * kLn2;
    out.S[i] = S;
    out.H[i] = H;
    out.m[i] = m;
    out.a[i] = a;
    out.r[i] = (float)(1.0 / (2.0 * (double)n * S));
    out.evals[i] = done == 1 ? it : -it;
    if (done != 1) flag_error(h, kErrNoConv);
    if (bad || !isfinite(H) || !isfinite(S)) flag_error(h, kErrNonFinite);
  }
};

// v: the distances of the wave's rows, VPT per lane, INFINITY where excluded
// (shifted by the row minimum in place). ok: the lane's row exists. G: points of a
// lane that are summed in FP32 before their sum goes to FP64 (fewer than VPT: in two
// alternating sums, as in k_calibrate).
template <int VPT, int R, int G>
__device__ __forceinline__ RowSearch search_rows(float (&v)[R][VPT], int64_t n, bool ok,
                                                 double logu, int max_bisect, double tol_h) {
  const int g = R == 4 ? (threadIdx.x & 63) >> 4 : 0;
  RowSearch f{0.0, 0.0, 0.f, 0.f, 0, ok ? 0 : 1};
#pragma unroll
  for (int r = 0; r < R; ++r) {
    float mn = INFINITY;
#pragma unroll
    for (int q = 0; q < VPT; ++q) mn = fminf(mn, v[r][q]);
    mn = wave_min_f(mn);
#pragma unroll
    for (int q = 0; q < VPT; ++q) v[r][q] = (v[r][q] == INFINITY) ? kBig : v[r][q] - mn;
    if (r == g) f.m = mn;
  }
  // Start of the search: at beta = 0 the entropy is ln(n - 1), its slope is
  // zero and its curvature -Var(d), so it falls to ln u near
  // beta = sqrt(2 ln((n - 1) / u) / Var(d)); one pass without exponentials. (From
  // beta = 1, partial problems of 1,000 points at perplexity 400 took 13 passes,
  // most of them halvings; from here 4.) Where far points make up the variance
  // (clusters a thousand widths apart, one stray point), the start is far too
  // small and the first Newton step, over the near points' variance, far too
  // large; a bracket so wide is halved in the exponent (1,000 points, two clusters:
  // 19 passes by halves, 9 so).
  double beta, lo = 0.0, hi = INFINITY;
  bool spread;  // the row's distances differ
  {
    double T1[R], T2[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
      float t1 = 0.f, t2 = 0.f;
#pragma unroll
      for (int q = 0; q < VPT; ++q) {
        const float x = v[r][q] < kBig ? v[r][q] : 0.f;  // 0 for an excluded entry
        t1 += x;
        t2 = fmaf(x, x, t2);
      }
      T1[r] = (double)t1;
      T2[r] = (double)t2;
    }
    const double cnt = (double)(n - 1), mean = rows_sum_d<R>(T1) / cnt;
    spread = mean > 0.0;
    const double var = rows_sum_d<R>(T2) / cnt - mean * mean;
    beta = sqrt(2.0 * (log(cnt) - logu) / var);
    if (!(beta > 0.0) || !isfinite(beta)) beta = 1.0;
  }
  // The result is that of the last pass with finite sums (of the last one if none
  // has them): where ties at the minimum keep the entropy above its target at any
  // beta, the search ends at the largest FP32 precision, half of the time one
  // pass beyond it. Where all of a row's distances are equal (identical points, a
  // row whose input is not a number) it is that of the last pass, always beyond
  // it: not finite, and reported.
  float a = 0.f;
  bool finite = false;
  while (!__all(f.done)) {
    // a row that has stopped goes along with its last beta, unused
    if (!f.done) {
      ++f.it;
      a = fmaxf((float)(beta * kLog2e), 1e-30f);
    }
    double SS[R], TT[R], QQ[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const float ar = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(a), 16 * r));
      SS[r] = TT[r] = QQ[r] = 0.0;
#pragma unroll
      for (int q0 = 0; q0 < VPT; q0 += G) {
        float s[2] = {}, tt[2] = {}, qq[2] = {};
#pragma unroll
        for (int q = q0; q < q0 + G; ++q) {
          const int o = G < VPT ? q & 1 : 0;
          const float ex = __builtin_amdgcn_exp2f(-ar * v[r][q]);
          const float ve = v[r][q] * ex;  // 0 for an excluded entry (ex = 0)
          s[o] += ex;
          tt[o] += ve;
          qq[o] = fmaf(v[r][q], ve, qq[o]);
        }
        SS[r] += (double)(s[0] + s[1]);
        TT[r] += (double)(tt[0] + tt[1]);
        QQ[r] += (double)(qq[0] + qq[1]);
      }
    }
    const double ss = rows_sum_d<R>(SS), ts = rows_sum_d<R>(TT), qs = rows_sum_d<R>(QQ);
    if (f.done) continue;
    const double beff = (double)a * kLn2;
    const double mean = ts / ss;
    const double H = log(ss) + beff * mean;
    if (isfinite(H) || !finite) {
      finite = spread && isfinite(H);
      f.S = ss;
      f.H = H;
      f.a = a;
    }
    if (fabs(H - logu) <= tol_h) {
      f.done = 1;
    } else if (isfinite(hi) && (hi - lo) <= hi * 0x1p-24) {
      f.done = 1;
    } else if (f.it >= max_bisect) {
      f.done = 2;
    } else {
      // H falls with beta (dH/dbeta = -beta Var(d)): shrink the bracket,
      // then take the Newton step if it lands inside it, else bisect
      // (the bracket holds the FP64 iterates; H was taken at their FP32
      // rounding beff, within 2^-24 of beta)
      if (H > logu)
        lo = beta;
      else
        hi = beta;
      const double var = qs / ss - mean * mean;
      const double nb = beta + (H - logu) / (beff * var);
      if (var > 0.0 && nb > lo && nb < hi && isfinite(nb))
        beta = nb;
      else if (isinf(hi))
        beta = 2.0 * beta;
      else
        beta = lo > 0.0 && hi > 16.0 * lo ? sqrt(lo) * sqrt(hi) : 0.5 * (lo + hi);
    }
  }
  return f;
}

// Search for problems of at most kCalWaveN points: R rows to a wave, as in the
// many-problem path, instead of a workgroup of 1,024 threads to a row, most of
// whose time at two points a thread went into its barriers and wave sums. All
// rows of the problem in one launch where the workspace has room for their
// distances (else a group of four row blocks at a time), each
// from its own start. n = 2,000: 22 us against 149 (two launches). G: a workgroup to
// a row had 1, 2 or 4 points a thread, summed in FP32, and all else in FP64; so here
// (a lane's 32 or 64 points summed in FP32: 19 us, but rows that miss tol_h).
constexpr int64_t kCalWaveN = 4096;
constexpr int kCalWaves = 4;  // waves per workgroup
template <int VPT, int R, int G>
__global__ __launch_bounds__(kCalWaves * 64) void k_calibrate_wave(
    const float *__restrict__ dblock, int64_t n, int64_t npad, int32_t b, double logu,
    int max_bisect, double tol_h, CalOut out, Hdr *h) {
  const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
  const int64_t r0 = ((int64_t)blockIdx.x * kCalWaves + w) * R;  // row within the group
  const int64_t i0 = (int64_t)b * T + r0;
  if (i0 >= n) return;
  float v[R][VPT];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int64_t i = i0 + r;
    const float *row = dblock + (r0 + r) * npad;
#pragma unroll
    for (int q = 0; q < VPT; ++q) {
      const int64_t j = (int64_t)q * 64 + l;
      v[r][q] = (i < n && j < n && j != i) ? row[j] : INFINITY;
    }
  }
  const int g = R == 4 ? l >> 4 : 0;
  const RowSearch f = search_rows<VPT, R, G>(v, n, i0 + g < n, logu, max_bisect, tol_h);
  if ((R == 4 ? (l & 15) : l) == 0 && i0 + g < n) f.store(out, i0 + g, n, false, h);
}

// ----------------------------------------------------------------------------
// 2c. Copy the block's tiles (b, J >= b) into the P store in consumer order.
// The diagonal tile holds both orders of each pair; both take the distance
// of the upper element so that the stored P is exactly symmetric.
// ----------------------------------------------------------------------------
// Grid (nb - b, kStageSplit, blocks), blocks b .. of one group.
constexpr int kStageSplit = 4;
__global__ __launch_bounds__(256) void k_stage(const float *__restrict__ dblock, int64_t npad,
                                               int32_t nb, int32_t b, float4 *__restrict__ P) {
  b += blockIdx.z;
  dblock += (size_t)blockIdx.z * T * npad;
  const int J = b + blockIdx.x;
  if (J >= nb) return;
  const int t = threadIdx.x, w = t >> 6, l = t & 63;
  const int tc = l & 15, tr = (l >> 4) + 4 * w;
  float4 *dst = P + (size_t)tile_start(b, nb) * TT4 + (size_t)blockIdx.x * TT4;
  const float *src = dblock + (int64_t)J * T;
  // workgroup y of the tile copies float4 rows s0 .. s1 - 1 of its 64
  const int s0 = blockIdx.y * (64 / kStageSplit), s1 = s0 + 64 / kStageSplit;
  if (J != b) {
#pragma unroll 4
    for (int s = s0; s < s1; ++s) {
      const int k = s >> 2, mq = s & 3;
      const float *rp = src + (int64_t)(tr + 16 * k) * npad + tc + 64 * mq;
      dst[s * 256 + t] = make_float4(rp[0], rp[16], rp[32], rp[48]);
    }
  } else {
    for (int s = s0; s < s1; ++s) {
      const int k = s >> 2, mq = s & 3;
      const int il = tr + 16 * k;
      float v[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int jl = tc + 16 * (4 * mq + e);
        const int lo = il < jl ? il : jl, hi = il < jl ? jl : il;
        v[e] = src[(int64_t)lo * npad + hi];
      }
      dst[s * 256 + t] = make_float4(v[0], v[1], v[2], v[3]);
    }
  }
}

// ----------------------------------------------------------------------------
// 2d. Implicit P: the distances (or with PACK the P) of the tiles tile0 .. tile0 +
// gridDim.x - 1 (whole block rows) straight into the tile buffer, strips over
// blockIdx.y. skip: the zero tiles are known and are left alone.
// ----------------------------------------------------------------------------
template <int MODE, bool PACK>
__global__ __launch_bounds__(256, 2) void k_tdist(TileSrc src, int32_t nb, int64_t tile0,
                                                  int64_t tile_base, float *__restrict__ Pb,
                                                  int32_t gkey, const uint8_t *__restrict__ nz,
                                                  bool skip) {
  __shared__ RowStats<MODE> rows;
  // a workspace prepared for another n, d or mode is flagged and left alone
  if (!implicit_ready(src.h, src.n, gkey)) {
    if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0)
      flag_error(const_cast<Hdr *>(src.h), kErrState);
    return;
  }
  const int64_t tile = tile0 + blockIdx.x;
  if (skip && !nz[tile]) return;
  int I, J;
  tile_coords(tile, nb, I, J);
  tile_strip<MODE, PACK>(src, I, J, blockIdx.y, Pb + (size_t)(tile - tile_base) * T * T, rows);
}

// ----------------------------------------------------------------------------
// 3. Symmetrise and normalise in place (Eq. 3):
//    p_ij = exp2(-a_i (d - m_i)) r_i + exp2(-a_j (d - m_j)) r_j,  r = 1/(2 n S).
// Also per tile: sum p and sum p ln p over ordered pairs (off-diagonal tiles
// stand for both (i, j) and (j, i)).
// ----------------------------------------------------------------------------
__device__ __forceinline__ void pack_tile(float4 *__restrict__ P, const float *__restrict__ a,
                                          const float *__restrict__ m,
                                          const float *__restrict__ r, int64_t n, int32_t nb,
                                          double2 *__restrict__ ppart,
                                          uint8_t *__restrict__ nzflag, int2 *__restrict__ tmap,
                                          int64_t tile, int64_t pslot) {
  __shared__ double red[2][4];
  __shared__ float srow[3][T];  // a, m, r of the tile's rows (0 past n)
  int I, J;
  tile_coords(tile, nb, I, J);
  if (threadIdx.x == 0) tmap[tile] = make_int2(I, J);
  const int t = threadIdx.x, w = t >> 6, l = t & 63;
  const int tc = l & 15, tr = (l >> 4) + 4 * w;
  const bool diag = (I == J);
  {
    const int64_t i = (int64_t)I * T + t;
    const bool ok = i < n;
    srow[0][t] = ok ? a[i] : 0.f;
    srow[1][t] = ok ? m[i] : 0.f;
    srow[2][t] = ok ? r[i] : 0.f;
  }
  float ac[16], mc[16], rc[16];
  uint32_t rvalid = 0, cvalid = 0;  // bit k: row tr+16k (column tc+16k) is a real point
#pragma unroll
  for (int k = 0; k < 16; ++k) {
    rvalid |= ((int64_t)I * T + tr + 16 * k < n) ? (1u << k) : 0u;
    const int64_t j = (int64_t)J * T + tc + 16 * k;
    const bool ok = j < n;
    cvalid |= ok ? (1u << k) : 0u;
    ac[k] = ok ? a[j] : 0.f;
    mc[k] = ok ? m[j] : 0.f;
    rc[k] = ok ? r[j] : 0.f;
  }
  __syncthreads();
  float4 *tp = P + (size_t)pslot * TT4;
  float psum = 0.f, plp = 0.f;
  bool any = false;
  // row k of the thread's block is four float4 (one per column quarter mq);
  // rows alternate between two register buffers, so the next row's four
  // loads are in flight while a row is converted
  auto convert_row = [&](int k, const float4 (&dv)[4]) {
    const int row = tr + 16 * k;
    const float ark = srow[0][row], mrk = srow[1][row], rrk = srow[2][row];
#pragma unroll
    for (int mq = 0; mq < 4; ++mq) {
      const float dd[4] = {dv[mq].x, dv[mq].y, dv[mq].z, dv[mq].w};
      float pv[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int mm = 4 * mq + e;
        float p = pair_p(dd[e], ark, mrk, rrk, ac[mm], mc[mm], rc[mm]);
        if (diag && tr == tc && k == mm) p = 0.f;
        if (!((rvalid >> k) & (cvalid >> mm) & 1u)) p = 0.f;
        // values below the normal FP32 range are stored as 0 (they change no
        // sum by more than 1e-38); a tile whose entries are all 0 is skipped
        // by the attractive part of the force pass
        if (p < FLT_MIN) p = 0.f;
        any |= p > 0.f;
        pv[e] = p;
        psum += p;
        // denormal p (< FLT_MIN) contribute below 1e-36 and are skipped: the
        // hardware log flushes them to zero
        plp += (p >= FLT_MIN) ? p * __builtin_amdgcn_logf(p) : 0.f;
      }
      tp[(k * 4 + mq) * 256 + t] = make_float4(pv[0], pv[1], pv[2], pv[3]);
    }
  };
  float4 ba[4], bb[4];
#pragma unroll
  for (int mq = 0; mq < 4; ++mq) ba[mq] = tp[mq * 256 + t];
#pragma unroll 1
  for (int k = 0; k < 16; k += 2) {
#pragma unroll
    for (int mq = 0; mq < 4; ++mq) bb[mq] = tp[((k + 1) * 4 + mq) * 256 + t];
    convert_row(k, ba);
    if (k + 2 < 16) {
#pragma unroll
      for (int mq = 0; mq < 4; ++mq) ba[mq] = tp[((k + 2) * 4 + mq) * 256 + t];
    }
    convert_row(k + 1, bb);
  }
  double ds = wave_sum_d((double)psum), dl = wave_sum_d((double)plp);
  if (l == 0) {
    red[0][w] = ds;
    red[1][w] = dl;
  }
  const int tile_any = __syncthreads_or(any ? 1 : 0);
  if (t == 0) {
    nzflag[tile] = tile_any ? 1 : 0;
    double mult = diag ? 1.0 : 2.0;
    double S = red[0][0] + red[0][1] + red[0][2] + red[0][3];
    double Lg = red[1][0] + red[1][1] + red[1][2] + red[1][3];
    ppart[tile] = make_double2(mult * S, mult * Lg * kLn2);
  }
}

// known: the search marked the tiles that may hold a nonzero p in nzflag; the
// others are all zero (sums, flag and coordinates are written, their distances
// stay where they are, and nothing reads them). n = 65,536: 4,620 of 32,896 tiles,
// 3.3 ms, now 0.52.
__global__ __launch_bounds__(256) void k_pack(float4 *__restrict__ P, const float *__restrict__ a,
                                              const float *__restrict__ m,
                                              const float *__restrict__ r, int64_t n, int32_t nb,
                                              double2 *__restrict__ ppart,
                                              uint8_t *__restrict__ nzflag,
                                              int2 *__restrict__ tmap, bool known) {
  const int64_t tile = blockIdx.x;
  if (known && !nzflag[tile]) {
    int I, J;
    tile_coords(tile, nb, I, J);
    if (threadIdx.x == 0) {
      tmap[tile] = make_int2(I, J);
      ppart[tile] = make_double2(0.0, 0.0);
    }
    return;
  }
  pack_tile(P, a, m, r, n, nb, ppart, nzflag, tmap, tile, tile);
}

__global__ __launch_bounds__(256) void k_clear_flags(uint8_t *__restrict__ f, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i < n) f[i] = 0;
}

__device__ __forceinline__ void pack_reduce_wg(const double2 *__restrict__ ppart, int64_t nt,
                                               Hdr *h, int32_t ready = 1) {
  __shared__ double red[2][16];
  double s = 0.0, lg = 0.0;
  for (int64_t q = threadIdx.x; q < nt; q += 1024) {
    s += ppart[q].x;
    lg += ppart[q].y;
  }
  s = wave_sum_d(s);
  lg = wave_sum_d(lg);
  if ((threadIdx.x & 63) == 0) {
    red[0][threadIdx.x >> 6] = s;
    red[1][threadIdx.x >> 6] = lg;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    double S = 0.0, Lg = 0.0;
    for (int q = 0; q < 16; ++q) {
      S += red[0][q];
      Lg += red[1][q];
    }
    h->p_sum = S;
    h->c_p = Lg;
    if (!isfinite(S) || !isfinite(Lg)) atomicOr(&h->err, kErrNonFinite);
    h->ready = ready;
  }
}

__global__ __launch_bounds__(1024) void k_pack_reduce(const double2 *__restrict__ ppart,
                                                      int64_t nt, Hdr *h) {
  pack_reduce_wg(ppart, nt, h);
}

// ----------------------------------------------------------------------------
// 4. Locality reordering (not part of the method: it only changes the order
// in which P is stored and summed).
//
// Points whose affinities are nonzero lie close in the input space, so an
// order in which nearby points are contiguous concentrates the nonzero p_ij in
// few tiles and leaves the rest all-zero (skipped by the attractive part of
// every force pass). The order is a principal-direction bisection tree with
// tile-aligned leaves: at level l the internal positions split into 2^l
// segments [floor(s nb / 2^l) T, floor((s + 1) nb / 2^l) T); each segment is
// sorted by the projection of its centred points on their leading principal
// direction (a few power iterations from a fixed start), so that its two
// halves at the next level are the two sides of that direction. Every step is
// deterministic (fixed reduction orders, a fixed sorting network).
// ----------------------------------------------------------------------------
constexpr int kTreeThreads = 256;
constexpr int kTreeMaxD = 2048;
constexpr int kTreePowerIters = 4;
constexpr int kTreeTargetGroups = 1024;  // workgroups per level at the shallow levels
constexpr int kSortBlock = 4096;         // keys per workgroup in the LDS sorting stages

// Given dissimilarities (any measure may enter, section "ptSNE: parallelized
// t-SNE"): the squares of rows b*T .. b*T + T - 1 of the n x n matrix into the
// distance block, in place of the contraction. Grid (npad / 256, T / 16, blocks):
// workgroup (c, g) covers columns 256 c .. 256 c + 255 of rows 16 g .. 16 g + 15.
__global__ __launch_bounds__(256) void k_dissim_block(const float *__restrict__ dis, int64_t n,
                                                      int64_t npad, int32_t b,
                                                      float *__restrict__ dblock, Hdr *h) {
  b += blockIdx.z;  // row block of the group, its squares in the group's slot
  dblock += (size_t)blockIdx.z * T * npad;
  const int64_t j = (int64_t)blockIdx.x * 256 + threadIdx.x;
  bool bad = false;
  for (int r = 16 * blockIdx.y; r < 16 * (blockIdx.y + 1); ++r) {
    const int64_t i = (int64_t)b * T + r;
    float v = 0.f;
    if (i < n && j < n) {
      const float dv = dis[i * n + j];
      bad |= !(dv >= 0.f && dv < INFINITY) && j != i;
      v = dv * dv;
    }
    dblock[(int64_t)r * npad + j] = v;
  }
  if (bad) flag_error(h, kErrNonFinite);
}

__global__ void k_reorder_init(int64_t n, int64_t npad, int32_t *__restrict__ perm,
                               int32_t *__restrict__ inv) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= npad) return;
  perm[i] = (int32_t)i;
  inv[i] = (int32_t)i;
}

// Segment s of level `level`: internal positions [lo, hi).
struct TreeSeg {
  int64_t lo, hi;
};

__device__ inline TreeSeg tree_segment(int64_t s, int level, int32_t nb, int64_t n) {
  TreeSeg g;
  g.lo = ((s * nb) >> level) * T;
  g.hi = (((s + 1) * nb) >> level) * T;
  if (g.lo > n) g.lo = n;
  if (g.hi > n) g.hi = n;
  return g;
}

// Sum of acc[0..7] over the workgroup into out[0..7] (LDS), in a fixed order.
__device__ inline void tree_block_sum8(double (&acc)[8], double (*red)[8], double *out) {
  const int t = threadIdx.x, w = t >> 6, l = t & 63;
#pragma unroll
  for (int q = 0; q < 8; ++q) acc[q] = wave_sum_d(acc[q]);
  if (l == 0) {
#pragma unroll
    for (int q = 0; q < 8; ++q) red[w][q] = acc[q];
  }
  __syncthreads();
  if (t < 8) {
    double s = 0.0;
    for (int g = 0; g < kTreeThreads / 64; ++g) s += red[g][t];
    out[t] = s;
  }
  __syncthreads();
}

__device__ inline uint32_t orderable_f32(float f) {
  const uint32_t u = __float_as_uint(f);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// Partial sums of one chunk (workgroup blockIdx.x = s * C + c) of a segment:
//   MODE 0: sum_r x_r                       (for the mean)
//   MODE 1: sum_r (x_r - mean) w_r, w_r = (x_r - mean) . v   (power iteration)
// into part[blockIdx.x][0 .. d). Each thread keeps w_r of its own rows in
// wbuf and reads back only what it wrote.
template <int MODE>
__global__ __launch_bounds__(kTreeThreads) void k_tree_partial(
    const double *__restrict__ xcT, int64_t npad, int32_t d, int64_t n, int32_t nb, int level,
    int32_t C, const int32_t *__restrict__ perm, const double *__restrict__ segmean,
    const double *__restrict__ segv, double *__restrict__ wbuf, double *__restrict__ part) {
  __shared__ double mean[MODE ? kTreeMaxD : 1], v[MODE ? kTreeMaxD : 1];
  __shared__ double red[kTreeThreads / 64][8];
  __shared__ double out8[8];
  const int t = threadIdx.x;
  const int64_t s = blockIdx.x / C, c = blockIdx.x % C;
  const TreeSeg g = tree_segment(s, level, nb, n);
  if (g.hi - g.lo <= T) return;  // leaves are not split
  const int64_t len = g.hi - g.lo;
  const int64_t r0 = g.lo + len * c / C, r1 = g.lo + len * (c + 1) / C;
  double *out = part + (int64_t)blockIdx.x * d;
  if (MODE == 1) {
    for (int k = t; k < d; k += kTreeThreads) {
      mean[k] = segmean[s * d + k];
      v[k] = segv[s * d + k];
    }
    __syncthreads();
    for (int64_t r = r0 + t; r < r1; r += kTreeThreads) {
      const int64_t i = perm[r];
      double wsum = 0.0;
      for (int k = 0; k < d; ++k) wsum += (xcT[(int64_t)k * npad + i] - mean[k]) * v[k];
      wbuf[r] = wsum;
    }
  }
  for (int k0 = 0; k0 < d; k0 += 8) {
    double acc[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) acc[q] = 0.0;
    for (int64_t r = r0 + t; r < r1; r += kTreeThreads) {
      const int64_t i = perm[r];
      const double wr = MODE ? wbuf[r] : 1.0;
#pragma unroll
      for (int q = 0; q < 8; ++q)
        if (k0 + q < d) {
          const double xv = xcT[(int64_t)(k0 + q) * npad + i];
          acc[q] += MODE ? (xv - mean[MODE ? k0 + q : 0]) * wr : xv;
        }
    }
    tree_block_sum8(acc, red, out8);
    if (t < 8 && k0 + t < d) out[k0 + t] = out8[t];
  }
}

// Per segment: MODE 0 turns the chunk sums into the mean and sets the fixed
// start vector; MODE 1 turns them into the next (normalised) direction.
template <int MODE>
__global__ __launch_bounds__(kTreeThreads) void k_tree_reduce(const double *__restrict__ part,
                                                              int32_t d, int64_t n, int32_t nb,
                                                              int level, int32_t C,
                                                              double *__restrict__ segmean,
                                                              double *__restrict__ segv) {
  __shared__ double red[kTreeThreads / 64];
  __shared__ double scale;
  const int t = threadIdx.x;
  const int64_t s = blockIdx.x;
  const TreeSeg g = tree_segment(s, level, nb, n);
  if (g.hi - g.lo <= T) return;
  double ss = 0.0;
  for (int k = t; k < d; k += kTreeThreads) {
    double sum = 0.0;
    for (int c = 0; c < C; ++c) sum += part[(s * C + c) * d + k];
    if (MODE == 0) {
      segmean[s * d + k] = sum / (double)(g.hi - g.lo);
      const uint32_t hsh = (uint32_t)(k + 1) * 2654435761u;
      segv[s * d + k] = 0.5 + (double)(hsh >> 8) * (1.0 / 16777216.0);
    } else {
      segv[s * d + k] = sum;
      ss += sum * sum;
    }
  }
  if (MODE == 0) return;
  ss = wave_sum_d(ss);
  if ((t & 63) == 0) red[t >> 6] = ss;
  __syncthreads();
  if (t == 0) {
    double tot = 0.0;
    for (int q = 0; q < kTreeThreads / 64; ++q) tot += red[q];
    scale = tot > 0.0 ? 1.0 / sqrt(tot) : 0.0;  // coincident points: projections all 0
  }
  __syncthreads();
  for (int k = t; k < d; k += kTreeThreads) segv[s * d + k] *= scale;
}

// Sort keys (segment << 32 | projection on the segment's direction) and the
// caller indices of the positions; leaves keep their order.
__global__ __launch_bounds__(kTreeThreads) void k_tree_keys(
    const double *__restrict__ xcT, int64_t npad, int32_t d, int64_t n, int32_t nb, int level,
    int32_t C, const int32_t *__restrict__ perm, const double *__restrict__ segmean,
    const double *__restrict__ segv, uint64_t *__restrict__ keys, int32_t *__restrict__ vals) {
  __shared__ double mean[kTreeMaxD], v[kTreeMaxD];
  const int t = threadIdx.x;
  const int64_t s = blockIdx.x / C, c = blockIdx.x % C;
  const TreeSeg g = tree_segment(s, level, nb, n);
  const int64_t len = g.hi - g.lo;
  const int64_t r0 = g.lo + len * c / C, r1 = g.lo + len * (c + 1) / C;
  const uint64_t seg = (uint64_t)s << 32;
  if (len <= T) {
    for (int64_t r = r0 + t; r < r1; r += kTreeThreads) {
      keys[r] = seg | (uint64_t)(r - g.lo);
      vals[r] = perm[r];
    }
    return;
  }
  for (int k = t; k < d; k += kTreeThreads) {
    mean[k] = segmean[s * d + k];
    v[k] = segv[s * d + k];
  }
  __syncthreads();
  for (int64_t r = r0 + t; r < r1; r += kTreeThreads) {
    const int64_t i = perm[r];
    double p = 0.0;
    for (int k = 0; k < d; ++k) p += (xcT[(int64_t)k * npad + i] - mean[k]) * v[k];
    keys[r] = seg | (uint64_t)orderable_f32((float)p);
    vals[r] = perm[r];
  }
}

// ----------------------------------------------------------------------------
// The same tree for d <= kTreeRowD, from the input rows themselves. The kernels
// above read the centred X by column through the order, 8 bytes from each
// cache line and each row twice per power iteration, and a level of a small
// problem is eleven launches and a sort. Here 16 lanes share a row (Q of its
// coordinates each, in registers from one contiguous read), so a power
// iteration is one sweep: the row's product with the direction is a sum over
// the 16 lanes, and the row times it goes into the lanes' accumulators. The
// arithmetic is FP64 as above, in another order of summation, so the
// projections round to the same FP32 keys but for one in about 10^8.
// A segment of at most kSegRows rows is one workgroup for its whole level: mean,
// power iterations, projections, an LDS sort of (projection, position) in one
// 64-bit word, the new order. n = 2,000, d = 10: 44 us a level (5 of them each
// power iteration, 13 the sort) against 110 for its launches; 65,536 x 50: 1.9
// ms for all eight levels against 4.7.
// ----------------------------------------------------------------------------
constexpr int kTreeRowD = 128;
constexpr int kSegRows = 4096;
constexpr int kSegThreads = 1024;

// Q coordinates (tc + 16 q) of one row, zero past d.
template <int Q>
__device__ __forceinline__ void row_coords(const float *__restrict__ x, int64_t i, int32_t d,
                                           int tc, float (&c)[Q]) {
  const float *xr = x + i * d;
#pragma unroll
  for (int q = 0; q < Q; ++q) c[q] = tc + 16 * q < d ? xr[tc + 16 * q] : 0.f;
}

// Sum over the 16 lanes of a row group, the same in every lane.
__device__ __forceinline__ double rot16_sum_d(double v) {
  v = dpp_add<0x128>(v);
  v = dpp_add<0x124>(v);
  v = dpp_add<0x122>(v);
  return dpp_add<0x121>(v);
}

// fn(r, coordinates) for rows first, first + step, ... < r1 (a row to 16 lanes,
// at(r) its point), with the reads of four rows in flight (16 made no difference).
template <int Q, class At, class Fn>
__device__ __forceinline__ void tree_rows(const float *__restrict__ x, int32_t d, int64_t first,
                                          int64_t r1, int step, int tc, At at, Fn fn) {
  constexpr int U = Q > 4 ? 2 : 4;
  for (int64_t r = first; r < r1; r += U * step) {
    int64_t i[U];
    float c[U][Q];
#pragma unroll
    for (int u = 0; u < U; ++u) i[u] = at(r + u * step < r1 ? r + u * step : r);
#pragma unroll
    for (int u = 0; u < U; ++u) row_coords<Q>(x, i[u], d, tc, c[u]);
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (r + u * step < r1) fn(r + u * step, i[u], c[u]);
  }
}

// One sweep, x being centred by the column means gm first. POWER: acc += (x -
// mean) ((x - mean) . v), else acc += x.
template <int Q, bool POWER, class At>
__device__ __forceinline__ void tree_sweep(const float *__restrict__ x, int32_t d, int64_t first,
                                           int64_t r1, int step, int tc, At at,
                                           const double (&gm)[Q], const double (&mean)[Q],
                                           const double (&v)[Q], double (&acc)[Q]) {
#pragma unroll
  for (int q = 0; q < Q; ++q) acc[q] = 0.0;
  tree_rows<Q>(x, d, first, r1, step, tc, at, [&](int64_t, int64_t, float (&c)[Q]) {
    if (POWER) {
      double e[Q], w = 0.0;
#pragma unroll
      for (int q = 0; q < Q; ++q) {
        e[q] = ((double)c[q] - gm[q]) - mean[q];
        w = fma(e[q], v[q], w);  // v is zero past d
      }
      w = rot16_sum_d(w);
#pragma unroll
      for (int q = 0; q < Q; ++q) acc[q] = fma(e[q], w, acc[q]);
    } else {
#pragma unroll
      for (int q = 0; q < Q; ++q) acc[q] += (double)c[q] - gm[q];
    }
  });
}

// Sums of acc over the workgroup's row groups into out[0 .. d) (LDS, FP64, a
// fixed order). W waves.
template <int Q, int W>
__device__ __forceinline__ void tree_gather(const double (&acc)[Q], int32_t d, int tc,
                                            double (*red)[kTreeRowD], double *out) {
  const int t = threadIdx.x, w = t >> 6, l = t & 63;
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    double s = acc[q];
    s += __shfl_xor(s, 16, 64);
    s += __shfl_xor(s, 32, 64);
    if (l < 16) red[w][tc + 16 * q] = s;
  }
  __syncthreads();
  if (t < d) {
    double s = 0.0;
    for (int g = 0; g < W; ++g) s += red[g][t];
    out[t] = s;
  }
  __syncthreads();
}

// Start direction: fixed and the same for every segment.
__device__ __forceinline__ double tree_start(int k) {
  const uint32_t hsh = (uint32_t)(k + 1) * 2654435761u;
  return 0.5 + (double)(hsh >> 8) * (1.0 / 16777216.0);
}

// 1 / |v| (0 for a zero vector: coincident points keep their order), by one wave.
__device__ __forceinline__ double tree_scale(const double *v, int32_t d) {
  double ss = 0.0;
  for (int k = threadIdx.x & 63; k < d; k += 64) ss += v[k] * v[k];
  ss = wave_sum_d(ss);
  return ss > 0.0 ? 1.0 / sqrt(ss) : 0.0;
}

template <int Q>
__global__ __launch_bounds__(kSegThreads) void k_tree_seg(const float *__restrict__ x,
                                                          const double *__restrict__ gmean,
                                                          int32_t d, int64_t n, int32_t nb,
                                                          int level, int32_t *__restrict__ perm) {
  constexpr int W = kSegThreads / 64;
  __shared__ double red[W][kTreeRowD];
  __shared__ double mean_s[kTreeRowD], v_s[kTreeRowD];
  __shared__ uint64_t key[kSegRows];
  __shared__ int32_t point[kSegRows];  // the segment's order
  __shared__ double scale_s;
  const int t = threadIdx.x, tc = t & 15;
  const int64_t s = blockIdx.x;
  const TreeSeg g = tree_segment(s, level, nb, n);
  const int len = (int)(g.hi - g.lo);
  if (len <= T || len > kSegRows) return;  // leaves are not split; the host sends no longer ones
  for (int e = t; e < len; e += kSegThreads) point[e] = perm[g.lo + e];
  __syncthreads();
  constexpr int kStep = kSegThreads / 16;
  auto at = [&](int64_t r) -> int64_t { return point[r]; };
  double gm[Q], mean[Q] = {}, v[Q] = {}, acc[Q];
#pragma unroll
  for (int q = 0; q < Q; ++q) gm[q] = tc + 16 * q < d ? gmean[tc + 16 * q] : 0.0;
  tree_sweep<Q, false>(x, d, t >> 4, len, kStep, tc, at, gm, mean, v, acc);
  tree_gather<Q, W>(acc, d, tc, red, mean_s);
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    const int k = tc + 16 * q;
    mean[q] = k < d ? mean_s[k] / (double)len : 0.0;
    v[q] = k < d ? tree_start(k) : 0.0;
  }
  for (int it = 0; it < kTreePowerIters; ++it) {
    tree_sweep<Q, true>(x, d, t >> 4, len, kStep, tc, at, gm, mean, v, acc);
    tree_gather<Q, W>(acc, d, tc, red, v_s);
    if (t < 64) {
      const double sc = tree_scale(v_s, d);
      if (t == 0) scale_s = sc;
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const int k = tc + 16 * q;
      v[q] = k < d ? v_s[k] * scale_s : 0.0;
    }
    __syncthreads();
  }
  // projections; padding sorts last
  int np2 = 2 * T;
  while (np2 < len) np2 <<= 1;
  tree_rows<Q>(x, d, t >> 4, len, kStep, tc, at, [&](int64_t e, int64_t, float (&c)[Q]) {
    double w = 0.0;
#pragma unroll
    for (int q = 0; q < Q; ++q) w = fma(((double)c[q] - gm[q]) - mean[q], v[q], w);
    w = rot16_sum_d(w);
    if (tc == 0) key[e] = ((uint64_t)orderable_f32((float)w) << 32) | (uint32_t)e;
  });
  for (int e = len + t; e < np2; e += kSegThreads) key[e] = ~0ull;
  __syncthreads();
  // bitonic sort, one compare-exchange per thread and pair
  for (int k = 2; k <= np2; k <<= 1) {
    for (int j = k >> 1; j > 0; j >>= 1) {
      for (int c = t; c < np2 / 2; c += kSegThreads) {
        const int lo = 2 * c - (c & (j - 1)), hi = lo + j;
        const uint64_t a = key[lo], b = key[hi];
        if ((a > b) == ((lo & k) == 0)) {
          key[lo] = b;
          key[hi] = a;
        }
      }
      __syncthreads();
    }
  }
  for (int e = t; e < len; e += kSegThreads) perm[g.lo + e] = point[(uint32_t)key[e]];
}

// Levels whose segments are longer: chunk c of segment s (workgroup s C + c).
// POWER: the chunk's part of the next direction, else of the mean.
template <int Q, bool POWER>
__global__ __launch_bounds__(kTreeThreads) void k_tree_chunk(
    const float *__restrict__ x, const double *__restrict__ gmean, int32_t d, int64_t n,
    int32_t nb, int level, int32_t C, const int32_t *__restrict__ perm,
    const double *__restrict__ segmean,
    const double *__restrict__ segv, double *__restrict__ part) {
  __shared__ double red[kTreeThreads / 64][kTreeRowD];
  __shared__ double out[kTreeRowD];
  const int t = threadIdx.x, tc = t & 15;
  const int64_t s = blockIdx.x / C, c = blockIdx.x % C;
  const TreeSeg g = tree_segment(s, level, nb, n);
  const int64_t len = g.hi - g.lo;
  if (len <= T) return;
  const int64_t r0 = g.lo + len * c / C, r1 = g.lo + len * (c + 1) / C;
  double gm[Q], mean[Q], v[Q], acc[Q];
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    const int k = tc + 16 * q;
    gm[q] = k < d ? gmean[k] : 0.0;
    mean[q] = POWER && k < d ? segmean[s * d + k] : 0.0;
    v[q] = POWER && k < d ? segv[s * d + k] : 0.0;
  }
  auto at = [&](int64_t r) -> int64_t { return perm[r]; };
  tree_sweep<Q, POWER>(x, d, r0 + (t >> 4), r1, kTreeThreads / 16, tc, at, gm, mean, v, acc);
  tree_gather<Q, kTreeThreads / 64>(acc, d, tc, red, out);
  if (t < d) part[(int64_t)blockIdx.x * d + t] = out[t];
}

// Per segment: the chunk sums to the mean (and the start direction), or to the
// next direction, normalised. A wave sums one coordinate's chunks.
template <bool POWER>
__global__ __launch_bounds__(kTreeThreads) void k_tree_join(const double *__restrict__ part,
                                                            int32_t d, int64_t n, int32_t nb,
                                                            int level, int32_t C,
                                                            double *__restrict__ segmean,
                                                            double *__restrict__ segv) {
  __shared__ double out[kTreeRowD];
  __shared__ double scale_s;
  const int t = threadIdx.x, w = t >> 6, l = t & 63;
  const int64_t s = blockIdx.x;
  const TreeSeg g = tree_segment(s, level, nb, n);
  if (g.hi - g.lo <= T) return;
  for (int k = w; k < d; k += kTreeThreads / 64) {
    double sum = 0.0;
    for (int c = l; c < C; c += 64) sum += part[(s * C + c) * d + k];
    sum = wave_sum_d(sum);
    if (l == 0) out[k] = sum;
  }
  __syncthreads();
  if (POWER && t < 64) {
    const double sc = tree_scale(out, d);
    if (t == 0) scale_s = sc;
  }
  __syncthreads();
  if (t >= d) return;
  if (POWER) {
    segv[s * d + t] = out[t] * scale_s;
  } else {
    segmean[s * d + t] = out[t] / (double)(g.hi - g.lo);
    segv[s * d + t] = tree_start(t);
  }
}

// Sort keys of a chunk's rows, as k_tree_keys.
template <int Q>
__global__ __launch_bounds__(kTreeThreads) void k_tree_rowkeys(
    const float *__restrict__ x, const double *__restrict__ gmean, int32_t d, int64_t n,
    int32_t nb, int level, int32_t C, const int32_t *__restrict__ perm,
    const double *__restrict__ segmean,
    const double *__restrict__ segv, uint64_t *__restrict__ keys, int32_t *__restrict__ vals) {
  const int t = threadIdx.x, tc = t & 15;
  const int64_t s = blockIdx.x / C, c = blockIdx.x % C;
  const TreeSeg g = tree_segment(s, level, nb, n);
  const int64_t len = g.hi - g.lo;
  const int64_t r0 = g.lo + len * c / C, r1 = g.lo + len * (c + 1) / C;
  const uint64_t seg = (uint64_t)s << 32;
  double gm[Q], mean[Q], v[Q];
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    const int k = tc + 16 * q;
    gm[q] = k < d ? gmean[k] : 0.0;
    mean[q] = len > T && k < d ? segmean[s * d + k] : 0.0;
    v[q] = len > T && k < d ? segv[s * d + k] : 0.0;
  }
  auto at = [&](int64_t r) -> int64_t { return perm[r]; };
  tree_rows<Q>(x, d, r0 + (t >> 4), r1, kTreeThreads / 16, tc, at,
               [&](int64_t r, int64_t i, float (&cc)[Q]) {
                 double w = 0.0;
#pragma unroll
                 for (int q = 0; q < Q; ++q) w = fma(((double)cc[q] - gm[q]) - mean[q], v[q], w);
                 w = rot16_sum_d(w);
                 if (tc == 0) {
                   keys[r] = seg | (len > T ? (uint64_t)orderable_f32((float)w)
                                            : (uint64_t)(r - g.lo));
                   vals[r] = (int32_t)i;
                 }
               });
}

// Keys of positions beyond n sort last.
__global__ void k_tree_pad(int64_t n, int64_t npow2, uint64_t *__restrict__ keys,
                           int32_t *__restrict__ vals) {
  const int64_t r = n + (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (r >= npow2) return;
  keys[r] = ~0ull;
  vals[r] = (int32_t)(r < INT32_MAX ? r : INT32_MAX);
}

// Bitonic sort (ascending) of (key, value) pairs over npow2 entries.
// Global stage: one compare-exchange distance j >= kSortBlock / 2 ... of
// merge size k.
__global__ void k_bitonic(uint64_t *__restrict__ keys, int32_t *__restrict__ vals, int64_t npow2,
                          int64_t j, int64_t k) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= npow2) return;
  const int64_t l = i ^ j;
  if (l <= i) return;
  const uint64_t a = keys[i], b = keys[l];
  const bool up = (i & k) == 0;
  if ((a > b) == up) {
    keys[i] = b;
    keys[l] = a;
    const int32_t va = vals[i];
    vals[i] = vals[l];
    vals[l] = va;
  }
}

// LDS stages on blocks of `blk` consecutive entries (blk a power of two, at
// most kSortBlock): with k0 = 0, every merge size k = 2 .. blk and all its
// distances (a full sort of each block in the global direction pattern);
// otherwise the distances blk / 2 .. 1 of merge size k0.
__global__ __launch_bounds__(1024) void k_bitonic_local(uint64_t *__restrict__ keys,
                                                        int32_t *__restrict__ vals, int64_t blk,
                                                        int64_t k0) {
  __shared__ uint64_t sk[kSortBlock];
  __shared__ int32_t sv[kSortBlock];
  const int64_t base = (int64_t)blockIdx.x * blk;
  for (int64_t e = threadIdx.x; e < blk; e += 1024) {
    sk[e] = keys[base + e];
    sv[e] = vals[base + e];
  }
  __syncthreads();
  const int64_t kfirst = k0 ? k0 : 2, klast = k0 ? k0 : blk;
  for (int64_t k = kfirst; k <= klast; k <<= 1) {
    for (int64_t j = (k0 ? blk : k) >> 1; j > 0; j >>= 1) {
      for (int64_t e = threadIdx.x; e < blk; e += 1024) {
        const int64_t l = e ^ j;
        if (l > e) {
          const uint64_t a = sk[e], b = sk[l];
          const bool up = ((base + e) & k) == 0;
          if ((a > b) == up) {
            sk[e] = b;
            sk[l] = a;
            const int32_t va = sv[e];
            sv[e] = sv[l];
            sv[l] = va;
          }
        }
      }
      __syncthreads();
    }
  }
  for (int64_t e = threadIdx.x; e < blk; e += 1024) {
    keys[base + e] = sk[e];
    vals[base + e] = sv[e];
  }
}

__global__ void k_tree_apply(const int32_t *__restrict__ vals, int64_t n,
                             int32_t *__restrict__ perm) {
  const int64_t r = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (r < n) perm[r] = vals[r];
}

__global__ void k_inverse(const int32_t *__restrict__ perm, int64_t npad,
                          int32_t *__restrict__ inv) {
  const int64_t r = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (r < npad) inv[perm[r]] = (int32_t)r;
}

// Centred X and its norms in the internal order (padding rows stay zero).
__global__ __launch_bounds__(256) void k_permute_x(const double *__restrict__ xcT,
                                                   const double *__restrict__ norms,
                                                   const int32_t *__restrict__ perm, int64_t n,
                                                   int64_t npad, int32_t dpad,
                                                   double *__restrict__ xcT2,
                                                   double *__restrict__ norms2) {
  const int64_t r = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (r >= npad) return;
  const int64_t i = r < n ? perm[r] : -1;
  for (int k = 0; k < dpad; ++k) xcT2[(int64_t)k * npad + r] = i >= 0 ? xcT[(int64_t)k * npad + i] : 0.0;
  norms2[r] = i >= 0 ? norms[i] : 0.0;
}

// ----------------------------------------------------------------------------
// Exports (test hooks)
// ----------------------------------------------------------------------------
__device__ inline bool state_ok(const Hdr *h, int64_t n) {
  return h->magic == kMagic && h->n == n && h->ready == 1;
}

__global__ __launch_bounds__(256) void k_export_rows(const float4 *__restrict__ P, int64_t n,
                                                     int32_t nb, int64_t row0, int64_t nrows,
                                                     const int32_t *__restrict__ inv,
                                                     const uint8_t *__restrict__ nz,
                                                     float *__restrict__ out, Hdr *h) {
  if (!state_ok(h, n)) {
    if (blockIdx.x == 0 && threadIdx.x == 0) flag_error(h, kErrState);
    return;
  }
  // one thread per output element (row rr, column j)
  const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (idx >= nrows * n) return;
  const int64_t rr = idx / n, j = idx % n;
  int64_t i = inv[row0 + rr], jj = inv[j];  // internal positions of the caller's (row, column)
  if (i / T > jj / T) {  // lower triangle: read the mirrored entry
    int64_t tmp = i;
    i = jj;
    jj = tmp;
  }
  const int I = (int)(i / T), J = (int)(jj / T);
  const int il = (int)(i % T), jl = (int)(jj % T);
  const int tr = il & 15, k = il >> 4, tc = jl & 15, mmi = jl >> 4;
  const int mq = mmi >> 2, e = mmi & 3;
  const int th = (tr >> 2) * 64 + (tr & 3) * 16 + tc;
  const int s = k * 4 + mq;
  const int64_t t = tile_start(I, nb) + (J - I);
  const float *tile = reinterpret_cast<const float *>(P + (size_t)t * TT4);
  out[idx] = nz[t] ? tile[((size_t)s * 256 + th) * 4 + e] : 0.f;  // (zero tiles are not stored)
}

__global__ void k_export_stats(int64_t n, const double *__restrict__ beta,
                               const float *__restrict__ m, const double *__restrict__ S,
                               const double *__restrict__ H, const int32_t *__restrict__ ev,
                               const int32_t *__restrict__ inv, double *ob, float *om, double *oS,
                               double *oH, int32_t *oe, Hdr *h) {
  // affinities for this n complete (stored or implicit P): the order exists
  if (!(h->magic == kMagic && h->n == n && (h->ready == 1 || h->ready == 2))) {
    if (blockIdx.x == 0 && threadIdx.x == 0) flag_error(h, kErrState);
    return;
  }
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
  const int64_t r = inv[i];
  if (ob) ob[i] = beta[r];
  if (om) om[i] = m[r];
  if (oS) oS[i] = S[r];
  if (oH) oH[i] = H[r];
  if (oe) oe[i] = ev[r];
}

// The internal order and the zero-tile flags, after checking that the
// workspace holds affinities for this n.
__global__ __launch_bounds__(256) void k_export_order(const Hdr *h, int64_t n, int64_t nt,
                                                      const int32_t *__restrict__ perm,
                                                      const uint8_t *__restrict__ nz,
                                                      int32_t *__restrict__ operm,
                                                      uint8_t *__restrict__ oflags) {
  if (!(h->magic == kMagic && h->n == n && (h->ready == 1 || h->ready == 2))) {
    if (blockIdx.x == 0 && threadIdx.x == 0) flag_error(const_cast<Hdr *>(h), kErrState);
    return;
  }
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (operm && i < n) operm[i] = perm[i];
  // the flags exist only where P is stored
  if (oflags && h->ready == 1 && i < nt) oflags[i] = nz[i];
}

__global__ void k_export_scalars(int64_t n, const Hdr *h, double *out) {
  if (threadIdx.x != 0) return;
  const bool ok = h->magic == kMagic && h->n == n;
  out[0] = ok ? h->p_sum : NAN;
  out[1] = ok ? h->c_p : NAN;
  out[2] = ok ? h->z : NAN;
  out[3] = ok ? h->perplexity : NAN;
}

// Tile lists for the force pass: all-zero tiles in ascending order, then the
// others in ascending order (one workgroup; ballot prefix counts in a fixed
// order).
__device__ __forceinline__ void tile_lists_wg(const uint8_t *__restrict__ nz, int64_t nt,
                                              int32_t *__restrict__ tlist,
                                              int32_t *__restrict__ tcount) {
  __shared__ int32_t wz[16], wn[16];
  __shared__ int32_t zbase, nbase, zeros;
  const int t = threadIdx.x, l = t & 63, w = t >> 6;
  // pass 1: number of all-zero tiles
  int32_t cnt = 0;
  for (int64_t q = t; q < nt; q += 1024) cnt += nz[q] == 0;
  for (int o = 32; o > 0; o >>= 1) cnt += __shfl_xor(cnt, o, 64);
  if (l == 0) wz[w] = cnt;
  __syncthreads();
  if (t == 0) {
    int32_t z = 0;
    for (int q = 0; q < 16; ++q) z += wz[q];
    zeros = z;
    zbase = 0;
    nbase = z;
  }
  __syncthreads();
  // pass 2: positions
  for (int64_t q0 = 0; q0 < nt; q0 += 1024) {
    const int64_t q = q0 + t;
    const bool valid = q < nt;
    const bool isz = valid && nz[q] == 0, isn = valid && nz[q] != 0;
    const uint64_t mz = __ballot(isz), mn = __ballot(isn);
    const uint64_t below = (l == 0) ? 0ull : (~0ull >> (64 - l));
    if (l == 0) {
      wz[w] = __popcll(mz);
      wn[w] = __popcll(mn);
    }
    __syncthreads();
    int32_t oz = zbase, on = nbase;
    for (int k = 0; k < w; ++k) {
      oz += wz[k];
      on += wn[k];
    }
    if (isz) tlist[oz + __popcll(mz & below)] = (int32_t)q;
    if (isn) tlist[on + __popcll(mn & below)] = (int32_t)q;
    __syncthreads();
    if (t == 0) {
      for (int k = 0; k < 16; ++k) {
        zbase += wz[k];
        nbase += wn[k];
      }
    }
    __syncthreads();
  }
  if (t == 0) {
    tcount[0] = zeros;
    tcount[1] = (int32_t)(nt - zeros);
  }
}

__global__ __launch_bounds__(1024) void k_tile_lists(const uint8_t *__restrict__ nz, int64_t nt,
                                                     int32_t *__restrict__ tlist,
                                                     int32_t *__restrict__ tcount) {
  tile_lists_wg(nz, nt, tlist, tcount);
}

// Per row block b, the slots s (tiles (b, s) or (s, b)) whose P is not all
// zero, in increasing s: the update reads the attractive partial sums of
// these slots only. One workgroup per block; a fixed-order prefix count.
__device__ __forceinline__ void slot_list_wg(const uint8_t *__restrict__ nz, int32_t nb,
                                             int32_t *__restrict__ slots,
                                             int32_t *__restrict__ nslots, int b) {
  __shared__ int32_t wsum[4];
  __shared__ int32_t base;
  const int t = threadIdx.x, l = t & 63, w = t >> 6;
  if (t == 0) base = 0;
  __syncthreads();
  for (int s0 = 0; s0 < nb; s0 += 256) {
    const int s = s0 + t;
    int f = 0;
    if (s < nb) {
      const int64_t tile = s >= b ? tile_start(b, nb) + (s - b) : tile_start(s, nb) + (b - s);
      f = nz[tile] != 0;
    }
    const uint64_t mask = __ballot(f);
    const int before = __popcll(mask & ((l == 0) ? 0ull : (~0ull >> (64 - l))));
    if (l == 0) wsum[w] = __popcll(mask);
    __syncthreads();
    int off = base;
    for (int q = 0; q < w; ++q) off += wsum[q];
    if (f) slots[(int64_t)b * nb + off + before] = s;
    __syncthreads();
    if (t == 0) base += wsum[0] + wsum[1] + wsum[2] + wsum[3];
    __syncthreads();
  }
  if (t == 0) nslots[b] = base;
}

__global__ __launch_bounds__(256) void k_slot_lists(const uint8_t *__restrict__ nz, int32_t nb,
                                                    int32_t *__restrict__ slots,
                                                    int32_t *__restrict__ nslots) {
  slot_list_wg(nz, nb, slots, nslots, blockIdx.x);
}

// ----------------------------------------------------------------------------
// 5. Many small problems at once (the partial problems of the parallel
// scheme). Same method as above with one wave per row: the row's squared
// distances (FP64 direct differences, rounded to FP32 like the distance
// block of the large path) stay in registers for the bisection, whose sums
// are wave reductions, so no workgroup barrier sits inside the search (several
// rows to a wave where they fit, see k_small_calibrate). The rows of a
// workgroup belong to one problem and share the staging of
// the other points' coordinates in LDS. The distances of tiles (I, J >= I)
// go straight into the P store in consumer order; the pack, reduction and
// list steps are the same device code as the single-problem path.
// ----------------------------------------------------------------------------

__device__ inline int small_find(const SmallEntry *tab, int count, int64_t key, int which) {
  int lo = 0, hi = count - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    const int64_t start = which == 0 ? tab[mid].wg0 : which == 1 ? tab[mid].tile0 : tab[mid].blk0;
    if (start <= key)
      lo = mid;
    else
      hi = mid - 1;
  }
  return lo;
}

// Position of element (il, jl) of a tile in the consumer order of the P store
// (the order the stage and pack kernels use), as a float index in the tile.
__device__ inline int small_pos(int il, int jl) {
  const int tr = il & 15, k = il >> 4, tc = jl & 15, mm = jl >> 4;
  const int s = k * 4 + (mm >> 2), t = 64 * (tr >> 2) + tc + 16 * (tr & 3);
  return (s * 256 + t) * 4 + (mm & 3);
}

// Header and identity order of every problem: one workgroup per row block.
__global__ __launch_bounds__(256) void k_small_init(const SmallEntry *__restrict__ tab, int count) {
  const int p = small_find(tab, count, blockIdx.x, 2);
  const SmallEntry &e = tab[p];
  const int64_t b = (int64_t)blockIdx.x - e.blk0;
  if (b < 0 || b >= e.nb) return;
  if (b == 0 && threadIdx.x == 0) {
    Hdr *h = e.h;
    h->magic = kMagic;
    h->n = e.n;
    h->d = e.d;
    h->ready = 0;
    h->err = 0;
    h->mode = TSNE_DIST_FP64;
    h->perplexity = e.perplexity;
    h->z = 0.0;
    h->c_p = 0.0;
    h->p_sum = 0.0;
    h->xmax = 0.f;
  }
  const int64_t i = b * T + threadIdx.x;
  e.perm[i] = (int32_t)i;
  e.inv[i] = (int32_t)i;
}

// R rows to a wave. What bounds a pass over 1,000 points is not its 16
// exponentials a lane but the three wave sums, the logarithm and the divisions
// in FP64, which every lane repeats for the one row; and in the distances one
// read of a double per lane feeds two FP64 instructions, which is the LDS rate.
// With four rows the wave reduces all their sums together and takes their four
// steps in the four groups of 16 lanes at once, and a read of a pair of
// coordinates (ds_read_b128; the row stride is twice an odd number of doubles,
// which spreads 16 lanes over all banks) feeds sixteen instructions. Every
// row's sums and steps are those of R = 1, so its results are too. 120,000 rows
// of 1,000 points in 30 dimensions, perplexity 400: 2.25 ms with one row to a
// wave, 2.32 with four rows and four separate steps, 1.62 this way, 1.12 with
// the start in search_rows. Four rows up to 1,024 points, one above, where two rows'
// distances no longer stay in registers.
template <int VPT, int R>
__global__ __launch_bounds__(kSmallWaves * 64) void k_small_calibrate(
    const SmallEntry *__restrict__ tab, int count, int32_t dstride, int max_bisect,
    double tol_h) {
  // LDS (FP64, converted once): two buffers of 64 points ([64][dstride]
  // each), then the own rows; the columns past d are zero
  extern __shared__ __align__(16) double sx[];
  constexpr int kThr = kSmallWaves * 64;
  constexpr int kRows = kSmallWaves * R;
  constexpr int kPre = 64 * kSmallMaxD / kThr;  // prefetch registers per thread
  const int p = small_find(tab, count, blockIdx.x, 0);
  const SmallEntry &e = tab[p];
  const int64_t n = e.n;
  const int32_t d = e.d;
  const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
  const int64_t r0 = ((int64_t)blockIdx.x - e.wg0) * kRows;
  const int64_t i0 = r0 + R * w;  // the wave's rows i0 .. i0 + R - 1
  double *own = sx + 2 * 64 * dstride;
  for (int q = threadIdx.x; q < (2 * 64 + kRows) * dstride; q += kThr) {
    const int rr = q / dstride - 2 * 64, k = q % dstride;
    sx[q] = rr >= 0 && k < d && r0 + rr < n ? (double)e.x[(r0 + rr) * d + k] : 0.0;
  }
  __syncthreads();
  const int nchunk = (int)((n + 63) / 64);
  // chunk c holds points 64c .. 64c + 63 as rows of d floats (contiguous in x)
  auto fetch = [&](int c, float (&pre)[kPre]) {
    const int64_t base = (int64_t)c * 64 * d, lim = (n - (int64_t)c * 64) * d;
#pragma unroll
    for (int u = 0; u < kPre; ++u) {
      const int idx = threadIdx.x + u * kThr;
      pre[u] = (idx < 64 * d && idx < lim) ? e.x[base + idx] : 0.f;
    }
  };
  // (row, coordinate) of this thread's first value and of the step between two
  const int rr0 = threadIdx.x / d, k0 = threadIdx.x - rr0 * d, rs = kThr / d, ks = kThr - rs * d;
  auto put = [&](int c, const float (&pre)[kPre]) {
    double *buf = sx + (c & 1) * 64 * dstride;
    int rr = rr0, k = k0;
#pragma unroll
    for (int u = 0; u < kPre; ++u) {
      if (rr < 64) buf[rr * dstride + k] = (double)pre[u];
      rr += rs;
      k += ks;
      if (k >= d) {
        k -= d;
        ++rr;
      }
    }
  };
  float pre[kPre];
  fetch(0, pre);
  put(0, pre);
  __syncthreads();
  float v[R][VPT];
  bool bad[R] = {};
#pragma unroll
  for (int q = 0; q < VPT; ++q) {
#pragma unroll
    for (int r = 0; r < R; ++r) v[r][q] = INFINITY;
    if (q < nchunk) {  // uniform over the workgroup
      if (q + 1 < nchunk) fetch(q + 1, pre);  // in flight while this chunk is used
      const int64_t j = (int64_t)q * 64 + l;
      if (i0 < n) {
        double acc[R];
#pragma unroll
        for (int r = 0; r < R; ++r) acc[r] = 0.0;
        const double2 *xj = reinterpret_cast<const double2 *>(sx + (q & 1) * 64 * dstride +
                                                              l * dstride);
        const double2 *xi = reinterpret_cast<const double2 *>(own + R * w * dstride);
        const int half = dstride / 2;
        // pairs of coordinates; past d both sides are zero
        for (int k = 0; k < (d + 1) / 2; ++k) {
          const double2 a = xj[k];
#pragma unroll
          for (int r = 0; r < R; ++r) {
            const double2 c = xi[r * half + k];
            const double d0 = a.x - c.x, d1 = a.y - c.y;
            acc[r] = fma(d0, d0, acc[r]);
            acc[r] = fma(d1, d1, acc[r]);
          }
        }
#pragma unroll
        for (int r = 0; r < R; ++r) {
          const int64_t i = i0 + r;
          if (i < n && j < n) {
            const float dv = (float)acc[r];
            bad[r] |= !isfinite(dv);
            const int I = (int)(i / T), J = (int)(j / T);
            if (J >= I) {
              float *tp =
                  reinterpret_cast<float *>(e.P + (size_t)(tile_start(I, e.nb) + (J - I)) * TT4);
              tp[small_pos((int)(i - (int64_t)I * T), (int)(j - (int64_t)J * T))] = dv;
            }
            if (j != i) v[r][q] = dv;
          }
        }
      }
      if (q + 1 < nchunk) put(q + 1, pre);  // the other buffer: last read two chunks ago
      __syncthreads();
    }
  }
  if (i0 >= n) return;  // no barrier below this point
  const int g = R == 4 ? l >> 4 : 0;
  const RowSearch f =
      search_rows<VPT, R, VPT>(v, n, i0 + g < n, log(e.perplexity), max_bisect, tol_h);
  bool any_bad = false;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const bool ab = __any(bad[r]);
    if (r == g) any_bad = ab;
  }
  if ((R == 4 ? (l & 15) : l) == 0 && i0 + g < n)
    f.store(CalOut{e.beta, e.S, e.H, e.m, e.a, e.r, e.evals}, i0 + g, n, any_bad, e.h);
}

__global__ __launch_bounds__(256) void k_small_pack(const SmallEntry *__restrict__ tab,
                                                    int count) {
  const int p = small_find(tab, count, blockIdx.x, 1);
  const SmallEntry &e = tab[p];
  const int64_t tile = (int64_t)blockIdx.x - e.tile0;
  if (tile < 0 || tile >= e.nt) return;
  pack_tile(e.P, e.a, e.m, e.r, e.n, e.nb, e.ppart, e.nz, e.tmap, tile, tile);
}

__global__ __launch_bounds__(256) void k_small_slots(const SmallEntry *__restrict__ tab,
                                                     int count) {
  const int p = small_find(tab, count, blockIdx.x, 2);
  const SmallEntry &e = tab[p];
  const int64_t b = (int64_t)blockIdx.x - e.blk0;
  if (b < 0 || b >= e.nb) return;
  slot_list_wg(e.nz, e.nb, e.slots, e.nslots, (int)b);
}

// One workgroup per problem: the sums of P (marks the problem ready), then
// the tile lists.
__global__ __launch_bounds__(1024) void k_small_lists(const SmallEntry *__restrict__ tab) {
  const SmallEntry &e = tab[blockIdx.x];
  pack_reduce_wg(e.ppart, e.nt, e.h);
  __syncthreads();
  tile_lists_wg(e.nz, e.nt, e.tlist, e.tcount);
}

// ----------------------------------------------------------------------------
// 6. Implicit P: the workspace keeps a buffer of implicit_capacity(L) tiles. The
// affinity stage ends with one pass over every tile (launch_implicit_discover):
// by buffers of whole block rows, k_tdist forms the distances, slot x holding tile
// base + x, and k_pack_range packs them, which gives the zero tiles, the sums of P
// and the lists. Later passes leave the zero tiles out and form the P of the others
// with their distances (k_tdist with PACK; above kImplicitTiles tiles a force pass
// takes a tile at a time, in a slot of the buffer for each workgroup:
// k_force_implicit). The arithmetic is that of the stored P, so the values are
// bitwise the same.
// ----------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_pack_range(float4 *__restrict__ Pb,
                                                    const float *__restrict__ a,
                                                    const float *__restrict__ m,
                                                    const float *__restrict__ r, int64_t n,
                                                    int32_t nb, double2 *__restrict__ ppart,
                                                    uint8_t *__restrict__ nzflag,
                                                    int2 *__restrict__ tmap, int64_t tile0,
                                                    int64_t tile_base, const Hdr *guard,
                                                    int32_t gkey) {
  if (!implicit_ready(guard, n, gkey)) {
    if (blockIdx.x == 0 && threadIdx.x == 0) flag_error(const_cast<Hdr *>(guard), kErrState);
    return;
  }
  const int64_t tile = tile0 + blockIdx.x;
  pack_tile(Pb, a, m, r, n, nb, ppart, nzflag, tmap, tile, tile - tile_base);
}

// After all blocks of a pass: sums of P (the header keeps ready = 2).
__global__ __launch_bounds__(1024) void k_implicit_sums(const double2 *__restrict__ ppart,
                                                        int64_t nt, int64_t n, int32_t key,
                                                        Hdr *h) {
  if (!implicit_ready(h, n, key)) return;
  pack_reduce_wg(ppart, nt, h, 2);
}

// Before the pass that discovers an implicit P's zero tiles: no tile flagged and
// empty slot lists (the pass writes both).
__global__ __launch_bounds__(256) void k_implicit_init(uint8_t *__restrict__ nz, int64_t nt,
                                                       int32_t *__restrict__ nslots, int32_t nb,
                                                       Hdr *h) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i < nt) nz[i] = 0;
  if (i < nb) nslots[i] = 0;
}

__global__ void k_set_ready(Hdr *h, int32_t ready) {
  if (threadIdx.x == 0) h->ready = ready;
}

}  // namespace

// ----------------------------------------------------------------------------
// Host-side sequencing
// ----------------------------------------------------------------------------

// Distances of row blocks b .. b + blocks - 1 against all columns into dblock
// (the group scratch), in the workspace's distance mode, one launch. xc, nrm: the centred X and its norms for the
// FP64 mode (the reduced modes read their prepared operands).
// P: the packed buffer, for the modes whose distance kernel stages the block
// row's tiles itself (FP64 and the x3 modes), else nullptr. Returns whether
// it did.
static bool launch_dist(const Layout &L, void *ws, int b, int blocks, const double *xc,
                        const double *nrm, float *dblock, float4 *P, hipStream_t st) {
  const Hdr *h = at<const Hdr>(ws, L.hdr);
  const float *norms32 = at<const float>(ws, L.norms32);
  const dim3 dgrid((unsigned)(L.npad / 256), T / 64, (unsigned)blocks);
  switch (L.mode) {
    case TSNE_DIST_FP32:
      hipLaunchKernelGGL(k_dist_f32, dgrid, dim3(256), 0, st, at<const float>(ws, L.xfT), norms32,
                         L.npad, L.dpad, b, dblock);
      break;
    case TSNE_DIST_BF16:
      hipLaunchKernelGGL((k_dist_lp<__bf16, v8bf, false>), dgrid, dim3(256), 0, st,
                         at<const __bf16>(ws, L.xa), norms32, L.npad,
                         L.kk, b, dblock, h);
      break;
    case TSNE_DIST_FP16:
      hipLaunchKernelGGL((k_dist_lp<_Float16, v8h, true>), dgrid, dim3(256), 0, st,
                         at<const _Float16>(ws, L.xa), norms32,
                         L.npad, L.kk, b, dblock, h);
      break;
    case TSNE_DIST_BF16X3:
      hipLaunchKernelGGL((k_dist_x3<__bf16, v8bf>), dist_grid(L.nb, blocks), dim3(256), 0, st,
                         at<const __bf16>(ws, L.xa), at<const float2>(ws, L.norms32), L.npad,
                         L.kk / 4, x3_bits(L.kk / 4, true), b, blocks, dblock, h, P, L.nb);
      return P != nullptr;
    case TSNE_DIST_FP16X3:
      hipLaunchKernelGGL((k_dist_x3<_Float16, v8h>), dist_grid(L.nb, blocks), dim3(256), 0, st,
                         at<const _Float16>(ws, L.xa), at<const float2>(ws, L.norms32), L.npad,
                         L.kk / 4, x3_bits(L.kk / 4, false), b, blocks, dblock, h, P, L.nb);
      return P != nullptr;
    default:
      hipLaunchKernelGGL(k_dist_f64,
                         dim3((unsigned)(L.npad / (64 * kDistCT)), T / 64, (unsigned)blocks),
                         dim3(256), 0, st, xc, nrm, L.npad, L.dpad, b, dblock, P, L.nb);
      return P != nullptr;
  }
  return false;
}

hipError_t launch_affinities(const Layout &L, const float *x, const float *dis, double perplexity,
                             int max_bisect, double tol_h, int reorder, void *ws, hipStream_t st,
                             bool stats_only, bool implicit) {
  Hdr *h = at<Hdr>(ws, L.hdr);
  hipLaunchKernelGGL(k_init_hdr, dim3(1), dim3(64), 0, st, h, L.n, L.d, L.mode, perplexity);
  double *mean = at<double>(ws, L.xmean);
  double *xcT = at<double>(ws, L.xcT);
  double *norms = at<double>(ws, L.norms);
  float *dblock = at<float>(ws, L.dblock);
  float4 *P = at<float4>(ws, L.P);
  int32_t *perm = at<int32_t>(ws, L.perm), *inv = at<int32_t>(ws, L.inv);
  const unsigned pgrid = (unsigned)((L.npad + 255) / 256);
  if (!dis) {
    hipLaunchKernelGGL(k_colmean, dim3(L.d), dim3(256), 0, st, x, L.n, L.d, mean);
    hipLaunchKernelGGL(k_centre, dim3(pgrid), dim3(256), 0, st, x, L.n, L.d, L.npad, L.dpad,
                       mean, xcT, norms, h);
  }
  hipLaunchKernelGGL(k_reorder_init, dim3(pgrid), dim3(256), 0, st, L.n, L.npad, perm, inv);
  CalOut co{at<double>(ws, L.beta), at<double>(ws, L.S), at<double>(ws, L.H),
            at<float>(ws, L.m),     at<float>(ws, L.a),  at<float>(ws, L.r),
            at<int32_t>(ws, L.evals)};
  const double logu = log(perplexity);
  const int64_t vpt_need = (L.n + kCalThreads - 1) / kCalThreads;
  const int32_t k32 = (L.d + 31) / 32 * 32;
  float *norms32 = at<float>(ws, L.norms32);
  float *xfT = at<float>(ws, L.xfT);
  __bf16 *xa_b = at<__bf16>(ws, L.xa);
  _Float16 *xa_h = at<_Float16>(ws, L.xa);
  float2 *nhl = at<float2>(ws, L.norms32);
  double2 *ppart = at<double2>(ws, L.ppart);
  uint8_t *nz = at<uint8_t>(ws, L.nz);

  // Reduced-precision operands of the contraction, from centred X in the
  // current order.
  auto prep = [&](const double *xc) {
    switch (L.mode) {
      case TSNE_DIST_FP32:
        hipLaunchKernelGGL(k_prep_f32, dim3(pgrid), dim3(256), 0, st, xc, L.npad, L.dpad, xfT,
                           norms32);
        break;
      case TSNE_DIST_BF16:
        hipLaunchKernelGGL((k_prep_lp<__bf16, false>), dim3(pgrid), dim3(256), 0, st, xc, L.npad,
                           L.d, k32, xa_b, norms32, h);
        break;
      case TSNE_DIST_BF16X3:
        hipLaunchKernelGGL(k_prep_x3<__bf16>, dim3(pgrid), dim3(256), 0, st, xc, L.npad, L.d, k32,
                           x3_bits(k32, true), xa_b, nhl, h);
        break;
      case TSNE_DIST_FP16:
        hipLaunchKernelGGL((k_prep_lp<_Float16, true>), dim3(pgrid), dim3(256), 0, st, xc,
                           L.npad, L.d, k32, xa_h, norms32, h);
        break;
      case TSNE_DIST_FP16X3:
        hipLaunchKernelGGL(k_prep_x3<_Float16>, dim3(pgrid), dim3(256), 0, st, xc, L.npad, L.d,
                           k32, x3_bits(k32, false), xa_h, nhl, h);
        break;
      default:
        break;
    }
  };
  // Row blocks are handled in groups of L.cal_group: block b's distances go
  // to slot b - b0 of the scratch (b0 the group's first block). One launch of
  // each kernel per group.
  auto group_end = [&](int b0) { return b0 + L.cal_group < L.nb ? b0 + L.cal_group : L.nb; };
  // Distances of a group's row blocks (into their slots), all columns.
  // Whether the distance kernel staged the block rows' tiles itself.
  bool staged = false;
  auto dist = [&](int b0, const double *xc, const double *nrm) {
    staged = launch_dist(L, ws, b0, group_end(b0) - b0, xc, nrm, dblock,
                         (stats_only || implicit) ? nullptr : P, st);
  };
  // The search over every row of the group starting at block b. ordered: in the
  // locality order.
  const bool ordered = !dis && reorder && !stats_only && L.nb >= 2 && L.d <= kTreeMaxD;
  // whether the search marks the tiles that can be nonzero
  const bool marked = ordered && !implicit && L.n > kCalWaveN && vpt_need <= 64;
  // bandwidths of a map: the search forms the distances itself
  const bool map = stats_only && !dis && L.d == 2 && L.mode == TSNE_DIST_FP64 && vpt_need <= 64;
  auto calibrate = [&](int b) {
    const int64_t left = L.n - (int64_t)b * T, span = (int64_t)L.cal_group * T;
    const int rows = (int)(left < span ? left : span);
    dim3 g(rows), blk(kCalThreads);
    if (L.n <= kCalWaveN && !stats_only) {
#define TSNE_CAL(V, R, G)                                                                       \
  hipLaunchKernelGGL((k_calibrate_wave<V, R, G>),                                               \
                     dim3((unsigned)((rows + kCalWaves * R - 1) / (kCalWaves * R))),            \
                     dim3(kCalWaves * 64), 0, st, dblock, L.n, L.npad, b, logu, max_bisect,     \
                     tol_h, co, h)
      // (rows to a wave as in small_rows: distances of four rows stay in
      // registers up to 16 a lane)
      if (L.n <= 256)
        TSNE_CAL(4, 4, 1);
      else if (L.n <= 512)
        TSNE_CAL(8, 4, 1);
      else if (L.n <= 1024)
        TSNE_CAL(16, 4, 1);
      else if (L.n <= 2048)
        TSNE_CAL(32, 1, 2);
      else
        TSNE_CAL(64, 1, 4);
#undef TSNE_CAL
      return;
    }
    // (below 8 points a thread only maps come here: kCalWaveN)
    auto run = [&](auto vpt) {
      constexpr int V = decltype(vpt)::value;
      static_assert(4 * kCalThreads <= kCalWaveN, "rows of points are searched by waves");
      auto *k = &k_calibrate<V, (V == 0 || V > 4) ? kCalPlain : kCalMap>;
      if constexpr (V > 4) {
        if (ordered) k = &k_calibrate<V, kCalOrdered>;
        if (map) k = &k_calibrate<V, kCalMap>;
      }
      hipLaunchKernelGGL(k, g, blk, 0, st, dblock, L.n, L.npad, b, logu, max_bisect, tol_h, co, h, x,
                         mean, nz, L.nb);
    };
    if (vpt_need <= 1)
      run(std::integral_constant<int, 1>{});
    else if (vpt_need <= 2)
      run(std::integral_constant<int, 2>{});
    else if (vpt_need <= 4)
      run(std::integral_constant<int, 4>{});
    else if (vpt_need <= 8)
      run(std::integral_constant<int, 8>{});
    else if (vpt_need <= 16)
      run(std::integral_constant<int, 16>{});
    else if (vpt_need <= 32)
      run(std::integral_constant<int, 32>{});
    else if (vpt_need <= 64)
      run(std::integral_constant<int, 64>{});
    else
      run(std::integral_constant<int, 0>{});
  };
  auto stage = [&](int b0) {
    hipLaunchKernelGGL(k_stage, dim3(L.nb - b0, kStageSplit, (unsigned)(group_end(b0) - b0)),
                       dim3(256), 0, st, dblock, L.npad, L.nb, b0, P);
  };
  auto pack = [&]() {
    hipLaunchKernelGGL(k_pack, dim3((unsigned)L.nt), dim3(256), 0, st, P, co.a, co.m, co.r, L.n,
                       L.nb, ppart, nz, at<int2>(ws, L.tmap), marked);
    hipLaunchKernelGGL(k_pack_reduce, dim3(1), dim3(1024), 0, st, ppart, L.nt, h);
    hipLaunchKernelGGL(k_slot_lists, dim3(L.nb), dim3(256), 0, st, nz, L.nb,
                       at<int32_t>(ws, L.slots), at<int32_t>(ws, L.nslots));
    hipLaunchKernelGGL(k_tile_lists, dim3(1), dim3(1024), 0, st, nz, L.nt,
                       at<int32_t>(ws, L.tlist), at<int32_t>(ws, L.tcount));
  };

  if (dis) {
    // given dissimilarities: no coordinates, so no ordering tree; the squared
    // rows take the place of the contraction
    for (int b0 = 0; b0 < L.nb; b0 += L.cal_group) {
      hipLaunchKernelGGL(k_dissim_block,
                         dim3((unsigned)(L.npad / 256), T / 16, (unsigned)(group_end(b0) - b0)),
                         dim3(256), 0, st, dis, L.n, L.npad, b0, dblock, h);
      calibrate(b0);
      stage(b0);
    }
    pack();
    return hipGetLastError();
  }
  const double *xc = xcT, *nrm = norms;
  if (ordered) {
    // Internal order: bisection tree over the centred X, then X in that order.
    uint64_t *keys = at<uint64_t>(ws, L.keys);
    int32_t *vals = at<int32_t>(ws, L.vals);
    // tree scratch in the (still idle) distance block: w per row, chunk
    // partial sums, segment means and directions (each at most nb x d)
    double *wbuf = reinterpret_cast<double *>(dblock);
    double *part = wbuf + L.npad;
    double *segmean = part + (size_t)L.nb * L.d;
    double *segv = segmean + (size_t)L.nb * L.d;
    const unsigned ngrid = (unsigned)((L.n + 255) / 256);
    const int64_t blk = L.npow2 < kSortBlock ? L.npow2 : kSortBlock;
    int levels = 0;
    while ((1 << levels) < L.nb) ++levels;
    // coordinates per lane of the row kernels (0: d too large for them)
    const int Q = L.d <= 16 ? 1 : L.d <= 32 ? 2 : L.d <= 64 ? 4 : L.d <= kTreeRowD ? 8 : 0;
    auto rows = [&](auto run) {
      if (Q == 1)
        run(std::integral_constant<int, 1>{});
      else if (Q == 2)
        run(std::integral_constant<int, 2>{});
      else if (Q == 4)
        run(std::integral_constant<int, 4>{});
      else
        run(std::integral_constant<int, 8>{});
    };
    for (int lev = 0; lev < levels; ++lev) {
      const int32_t S = 1 << lev;
      int32_t C = kTreeTargetGroups / S;
      if (C > L.nb / S) C = L.nb / S;  // at least a tile of rows per chunk on average
      if (C < 1) C = 1;
      const dim3 chunks((unsigned)(S * C)), segs((unsigned)S), tb(kTreeThreads);
      // segments of at most kSegRows rows (the longest has ceil(nb / S) tiles)
      if (Q && (L.nb + S - 1) / S <= kSegRows / T) {
        rows([&](auto q) {
          hipLaunchKernelGGL(k_tree_seg<decltype(q)::value>, segs, dim3(kSegThreads), 0, st, x,
                             mean, L.d, L.n, L.nb, lev, perm);
        });
        continue;
      }
      if (Q) {
        rows([&](auto q) {
          constexpr int kq = decltype(q)::value;
          hipLaunchKernelGGL((k_tree_chunk<kq, false>), chunks, tb, 0, st, x, mean, L.d, L.n, L.nb,
                             lev, C, perm, segmean, segv, part);
          hipLaunchKernelGGL(k_tree_join<false>, segs, tb, 0, st, part, L.d, L.n, L.nb, lev, C,
                             segmean, segv);
          for (int it = 0; it < kTreePowerIters; ++it) {
            hipLaunchKernelGGL((k_tree_chunk<kq, true>), chunks, tb, 0, st, x, mean, L.d, L.n, L.nb,
                               lev, C, perm, segmean, segv, part);
            hipLaunchKernelGGL(k_tree_join<true>, segs, tb, 0, st, part, L.d, L.n, L.nb, lev, C,
                               segmean, segv);
          }
          hipLaunchKernelGGL(k_tree_rowkeys<kq>, chunks, tb, 0, st, x, mean, L.d, L.n, L.nb, lev, C,
                             perm, segmean, segv, keys, vals);
        });
      } else {
        hipLaunchKernelGGL(k_tree_partial<0>, chunks, tb, 0, st, xcT, L.npad, L.d, L.n, L.nb, lev,
                           C, perm, segmean, segv, wbuf, part);
        hipLaunchKernelGGL(k_tree_reduce<0>, segs, tb, 0, st, part, L.d, L.n, L.nb, lev, C, segmean,
                           segv);
        for (int it = 0; it < kTreePowerIters; ++it) {
          hipLaunchKernelGGL(k_tree_partial<1>, chunks, tb, 0, st, xcT, L.npad, L.d, L.n, L.nb, lev,
                             C, perm, segmean, segv, wbuf, part);
          hipLaunchKernelGGL(k_tree_reduce<1>, segs, tb, 0, st, part, L.d, L.n, L.nb, lev, C,
                             segmean, segv);
        }
        hipLaunchKernelGGL(k_tree_keys, chunks, tb, 0, st, xcT, L.npad, L.d, L.n, L.nb, lev, C,
                           perm, segmean, segv, keys, vals);
      }
      if (L.npow2 > L.n)
        hipLaunchKernelGGL(k_tree_pad, dim3((unsigned)((L.npow2 - L.n + 255) / 256)), dim3(256),
                           0, st, L.n, L.npow2, keys, vals);
      const unsigned nblk = (unsigned)(L.npow2 / blk);
      hipLaunchKernelGGL(k_bitonic_local, dim3(nblk), dim3(1024), 0, st, keys, vals, blk,
                         (int64_t)0);
      for (int64_t k = 2 * blk; k <= L.npow2; k <<= 1) {
        for (int64_t j = k >> 1; j >= blk; j >>= 1)
          hipLaunchKernelGGL(k_bitonic, dim3((unsigned)(L.npow2 / 256)), dim3(256), 0, st, keys,
                             vals, L.npow2, j, k);
        hipLaunchKernelGGL(k_bitonic_local, dim3(nblk), dim3(1024), 0, st, keys, vals, blk, k);
      }
      hipLaunchKernelGGL(k_tree_apply, dim3(ngrid), dim3(256), 0, st, vals, L.n, perm);
    }
    hipLaunchKernelGGL(k_inverse, dim3(pgrid), dim3(256), 0, st, perm, L.npad, inv);
    double *xcT2 = at<double>(ws, L.xcT2), *norms2 = at<double>(ws, L.norms2);
    hipLaunchKernelGGL(k_permute_x, dim3(pgrid), dim3(256), 0, st, xcT, norms, perm, L.n, L.npad,
                       L.dpad, xcT2, norms2);
    xc = xcT2;
    nrm = norms2;
  }
  // Distances, calibration and staging block by block, then P.
  prep(xc);
  if (marked)
    hipLaunchKernelGGL(k_clear_flags, dim3((unsigned)((L.nt + 255) / 256)), dim3(256), 0, st, nz,
                       L.nt);
  for (int b0 = 0; b0 < L.nb; b0 += L.cal_group) {
    if (!map) dist(b0, xc, nrm);
    calibrate(b0);
    if (!stats_only && !implicit && !staged) stage(b0);
  }
  if (implicit) {
    // every pass rebuilds P from the contraction operands in the internal
    // order: the prepared ones of a reduced mode stay where prep() wrote
    // them; the FP64 mode reads the centred X from the second buffer (the
    // identity order copies it there)
    if (L.mode == TSNE_DIST_FP64 && xc != at<double>(ws, L.xcT2))
      hipLaunchKernelGGL(k_permute_x, dim3(pgrid), dim3(256), 0, st, xcT, norms, perm, L.n,
                         L.npad, L.dpad, at<double>(ws, L.xcT2), at<double>(ws, L.norms2));
    const int64_t m = L.nt > L.nb ? L.nt : L.nb;
    hipLaunchKernelGGL(k_implicit_init, dim3((unsigned)((m + 255) / 256)), dim3(256), 0, st,
                       at<uint8_t>(ws, L.nz), L.nt, at<int32_t>(ws, L.nslots), L.nb, h);
    hipLaunchKernelGGL(k_set_ready, dim3(1), dim3(64), 0, st, h, 2);
    hipError_t e = launch_implicit_discover(L, ws, st);
    if (e != hipSuccess) return e;
  } else if (!stats_only) {
    pack();
  }
  return hipGetLastError();
}

TileSrc tile_src(const Layout &L, void *ws) {
  TileSrc s{};
  s.h = at<const Hdr>(ws, L.hdr);
  s.n = L.n;
  s.npad = L.npad;
  s.dpad = L.dpad;
  s.kk = L.kk;
  switch (L.mode) {
    case TSNE_DIST_FP32:
      s.x = at<const float>(ws, L.xfT);
      s.norms = at<const float>(ws, L.norms32);
      break;
    case TSNE_DIST_BF16:
    case TSNE_DIST_FP16:
      s.x = at<const void>(ws, L.xa);
      s.norms = at<const float>(ws, L.norms32);
      break;
    case TSNE_DIST_BF16X3:
    case TSNE_DIST_FP16X3:
      s.x = at<const void>(ws, L.xa);
      s.norms = at<const float2>(ws, L.norms32);
      s.kk = L.kk / 4;
      s.bits = x3_bits(s.kk, L.mode == TSNE_DIST_BF16X3);
      break;
    default:
      s.x = at<const double>(ws, L.xcT2);
      s.norms = at<const double>(ws, L.norms2);
  }
  s.a = at<const float>(ws, L.a);
  s.m = at<const float>(ws, L.m);
  s.r = at<const float>(ws, L.r);
  return s;
}

template <bool PACK>
static void launch_tdist(const Layout &L, void *ws, int64_t tile0, int64_t count,
                         int64_t tile_base, bool skip_zero, hipStream_t st) {
  const TileSrc src = tile_src(L, ws);
  with_mode(L.mode, [&](auto mode) {
    constexpr int M = decltype(mode)::value;
    hipLaunchKernelGGL((k_tdist<M, PACK>), dim3((unsigned)count, tile_strips(M)), dim3(256), 0, st,
                       src, L.nb, tile0, tile_base, at<float>(ws, L.P),
                       implicit_key(L.d, L.mode), at<const uint8_t>(ws, L.nz), skip_zero);
  });
}

hipError_t launch_implicit_tiles(const Layout &L, void *ws, int64_t tile0, int64_t count,
                                 int64_t tile_base, bool skip_zero, bool pack, hipStream_t st) {
  if (pack)
    launch_tdist<true>(L, ws, tile0, count, tile_base, skip_zero, st);
  else
    launch_tdist<false>(L, ws, tile0, count, tile_base, skip_zero, st);
  return hipGetLastError();
}

// Pack (Eq. 3) the tiles tile0 .. tile0 + count - 1 of the buffer, with their
// sums, flags and coordinates.
static hipError_t launch_implicit_pack(const Layout &L, void *ws, int64_t tile0, int64_t count,
                                       int64_t tile_base, hipStream_t st) {
  hipLaunchKernelGGL(k_pack_range, dim3((unsigned)count), dim3(256), 0, st, at<float4>(ws, L.P),
                     at<const float>(ws, L.a), at<const float>(ws, L.m), at<const float>(ws, L.r),
                     L.n, L.nb, at<double2>(ws, L.ppart), at<uint8_t>(ws, L.nz),
                     at<int2>(ws, L.tmap), tile0, tile_base, at<const Hdr>(ws, L.hdr),
                     implicit_key(L.d, L.mode));
  return hipGetLastError();
}

// The end of the affinity stage of implicit P: one pass over every tile
// (distances, stage, pack) finds the zero tiles, the sums of P and the tile
// coordinates; P is the same in every later pass, so those passes recompute
// only the nonzero tiles and take the all-zero ones with the repulsion-only
// body, as the stored path does.
hipError_t launch_implicit_discover(const Layout &L, void *ws, hipStream_t st) {
  const int64_t cap = implicit_capacity(L);
  for (int b0 = 0; b0 < L.nb;) {
    int b1 = b0 + 1;
    while (b1 < L.nb && tile_start(b1 + 1, L.nb) - tile_start(b0, L.nb) <= cap) ++b1;
    const int64_t base = tile_start(b0, L.nb), count = tile_start(b1, L.nb) - base;
    hipError_t e = launch_implicit_tiles(L, ws, base, count, base, false, false, st);
    if (e != hipSuccess) return e;
    e = launch_implicit_pack(L, ws, base, count, base, st);
    if (e != hipSuccess) return e;
    b0 = b1;
  }
  uint8_t *nz = at<uint8_t>(ws, L.nz);
  hipLaunchKernelGGL(k_implicit_sums, dim3(1), dim3(1024), 0, st, at<const double2>(ws, L.ppart),
                     L.nt, L.n, implicit_key(L.d, L.mode), at<Hdr>(ws, L.hdr));
  hipLaunchKernelGGL(k_slot_lists, dim3(L.nb), dim3(256), 0, st, nz, L.nb,
                     at<int32_t>(ws, L.slots), at<int32_t>(ws, L.nslots));
  hipLaunchKernelGGL(k_tile_lists, dim3(1), dim3(1024), 0, st, nz, L.nt,
                     at<int32_t>(ws, L.tlist), at<int32_t>(ws, L.tcount));
  return hipGetLastError();
}

void small_entry(const Layout &L, void *ws, const float *x, double perplexity, SmallEntry &e) {
  e.x = x;
  e.n = L.n;
  e.nt = L.nt;
  e.d = L.d;
  e.nb = L.nb;
  e.perplexity = perplexity;
  e.h = at<Hdr>(ws, L.hdr);
  e.a = at<float>(ws, L.a);
  e.m = at<float>(ws, L.m);
  e.r = at<float>(ws, L.r);
  e.beta = at<double>(ws, L.beta);
  e.S = at<double>(ws, L.S);
  e.H = at<double>(ws, L.H);
  e.evals = at<int32_t>(ws, L.evals);
  e.P = at<float4>(ws, L.P);
  e.ppart = at<double2>(ws, L.ppart);
  e.nz = at<uint8_t>(ws, L.nz);
  e.tmap = at<int2>(ws, L.tmap);
  e.tlist = at<int32_t>(ws, L.tlist);
  e.tcount = at<int32_t>(ws, L.tcount);
  e.slots = at<int32_t>(ws, L.slots);
  e.nslots = at<int32_t>(ws, L.nslots);
  e.perm = at<int32_t>(ws, L.perm);
  e.inv = at<int32_t>(ws, L.inv);
}

hipError_t launch_affinities_small(const SmallEntry *tab, int count, int64_t wgs, int64_t tiles,
                                   int64_t blocks, int64_t nmax, int32_t dmax, int max_bisect,
                                   double tol_h, hipStream_t st) {
  if (nmax > kSmallMaxN || dmax > kSmallMaxD || count < 1) return hipErrorInvalidValue;
  // row stride in doubles: twice an odd number (16-byte aligned pairs, 16
  // lanes' pairs in different banks)
  const int32_t dstride = 2 * (((dmax + 1) / 2) | 1);
  const int rows = small_rows(nmax);
  const size_t lds = (size_t)(2 * 64 + rows) * dstride * sizeof(double);
  hipLaunchKernelGGL(k_small_init, dim3((unsigned)blocks), dim3(256), 0, st, tab, count);
  const dim3 g((unsigned)wgs), b(kSmallWaves * 64);
  const int vpt = (int)((nmax + 63) / 64);
#define TSNE_SMALL(V, R)                                                                        \
  hipLaunchKernelGGL((k_small_calibrate<V, R>), g, b, lds, st, tab, count, dstride, max_bisect, \
                     tol_h)
  // (rows to a wave as in small_rows)
  if (vpt <= 4)
    TSNE_SMALL(4, 4);
  else if (vpt <= 8)
    TSNE_SMALL(8, 4);
  else if (vpt <= 16)
    TSNE_SMALL(16, 4);
  else if (vpt <= 32)
    TSNE_SMALL(32, 1);
  else
    TSNE_SMALL(64, 1);
#undef TSNE_SMALL
  hipLaunchKernelGGL(k_small_pack, dim3((unsigned)tiles), dim3(256), 0, st, tab, count);
  hipLaunchKernelGGL(k_small_slots, dim3((unsigned)blocks), dim3(256), 0, st, tab, count);
  hipLaunchKernelGGL(k_small_lists, dim3((unsigned)count), dim3(1024), 0, st, tab);
  return hipGetLastError();
}

hipError_t launch_export_p_rows(const Layout &L, void *ws, int64_t row0, int64_t nrows,
                                float *out, hipStream_t st) {
  const int64_t total = nrows * L.n;
  if (total == 0) return hipSuccess;
  hipLaunchKernelGGL(k_export_rows, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st,
                     at<const float4>(ws, L.P), L.n, L.nb, row0, nrows,
                     at<const int32_t>(ws, L.inv), at<const uint8_t>(ws, L.nz), out, at<Hdr>(ws, L.hdr));
  return hipGetLastError();
}

hipError_t launch_export_rowstats(const Layout &L, void *ws, double *beta, float *m, double *S,
                                  double *H, int32_t *evals, hipStream_t st) {
  hipLaunchKernelGGL(k_export_stats, dim3((unsigned)((L.n + 255) / 256)), dim3(256), 0, st, L.n,
                     at<const double>(ws, L.beta), at<const float>(ws, L.m),
                     at<const double>(ws, L.S), at<const double>(ws, L.H),
                     at<const int32_t>(ws, L.evals), at<const int32_t>(ws, L.inv), beta, m, S, H,
                     evals, at<Hdr>(ws, L.hdr));
  return hipGetLastError();
}

hipError_t launch_export_order(const Layout &L, void *ws, int32_t *perm, uint8_t *flags,
                               hipStream_t st) {
  const int64_t m = L.n > L.nt ? L.n : L.nt;
  hipLaunchKernelGGL(k_export_order, dim3((unsigned)((m + 255) / 256)), dim3(256), 0, st,
                     at<const Hdr>(ws, L.hdr), L.n, L.nt, at<const int32_t>(ws, L.perm),
                     at<const uint8_t>(ws, L.nz), perm, flags);
  return hipGetLastError();
}

hipError_t launch_export_scalars(const Layout &L, void *ws, double *out, hipStream_t st) {
  hipLaunchKernelGGL(k_export_scalars, dim3(1), dim3(64), 0, st, L.n, at<const Hdr>(ws, L.hdr),
                     out);
  return hipGetLastError();
}

}  // namespace tsne
