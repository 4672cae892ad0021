// Distances and P of one tile, recomputed from the contraction operands: shared by
// the kernels that fill a buffer of tiles (tsne_affinity.hip) and by the force
// pass that recomputes a tile and uses it at once (tsne_iterate.hip).
#pragma once

#include <float.h>

#include <type_traits>

#include "tsne_internal.h"

namespace tsne {

// Operands of a workspace's contraction in its distance mode, and the row
// statistics.
struct TileSrc {
  const Hdr *h;
  int64_t n, npad;
  const void *x;      // xcT (double) or xfT (float), [k][point]; 16-bit modes [point][k]
  const void *norms;  // double, float, or (hi, lo) pairs
  int32_t dpad, kk, bits;
  const float *a, *m, *r;
};
TileSrc tile_src(const Layout &L, void *ws);

// run(std::integral_constant<int, mode>) for a layout's distance mode
template <class F>
void with_mode(int32_t mode, F &&run) {
  switch (mode) {
    case TSNE_DIST_FP32:
      return run(std::integral_constant<int, TSNE_DIST_FP32>{});
    case TSNE_DIST_BF16:
      return run(std::integral_constant<int, TSNE_DIST_BF16>{});
    case TSNE_DIST_BF16X3:
      return run(std::integral_constant<int, TSNE_DIST_BF16X3>{});
    case TSNE_DIST_FP16:
      return run(std::integral_constant<int, TSNE_DIST_FP16>{});
    case TSNE_DIST_FP16X3:
      return run(std::integral_constant<int, TSNE_DIST_FP16X3>{});
    default:
      return run(std::integral_constant<int, TSNE_DIST_FP64>{});
  }
}

namespace {

typedef double v4d __attribute__((ext_vector_type(4)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef _Float16 v8h __attribute__((ext_vector_type(8)));

__device__ inline float fp16_scale(const Hdr *h) {
  // 2^(8 - ceil(log2 xmax)); 1 if xmax is 0
  const float xm = h->xmax;
  if (!(xm > 0.f)) return 1.f;
  int e;
  frexpf(xm, &e);  // xm = f 2^e, f in [0.5, 1)
  return ldexpf(1.f, 8 - e);
}

// The x3 modes (their derivation stands with k_prep_x3).
__host__ __device__ inline int x3_bits(int32_t k32, bool bf16) {
  int lk = 0;
  while ((1 << lk) < k32) ++lk;
  const int b = (24 - lk) / 2;
  const int bmax = bf16 ? 8 : 10;
  return b < bmax ? b : bmax;
}

// E with max |x| < 2^E (0 for an all-zero input)
__device__ inline int x3_exp(const Hdr *h) {
  const float xm = h->xmax;
  if (!(xm > 0.f)) return 0;
  int e;
  frexpf(xm, &e);
  return e;
}

template <typename H, typename V8>
__device__ __forceinline__ v4f mfma16x32(V8 a, V8 b, v4f c) {
  if constexpr (__is_same(H, __bf16))
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
  else
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0);
}

// The two sums A0 and R of a 64 x 64 block (4 x 4 MFMA tiles): rows ra .. ra+63
// against columns cb .. cb+63. Stored and recomputed P call this same routine,
// so their sums agree bit for bit.
// The workgroup's 64 rows are the same for its waves and pass through LDS (one
// coalesced load of 16 KB per 32 values of k, the next while this one is used; a
// row's pitch of 17 pieces spreads 16 rows over all banks); a wave's columns of
// one K step are in flight at once. With the fragments loaded where they were
// used, ten waits for memory a strip were what bounded it at two waves per SIMD:
// 1,024 rows of 65,536, 64 values of k: 166 us,
// now 146.
template <typename V8>
struct X3Smem {
  V8 a[2][64][17];
};
template <typename H, typename V8>
__device__ __forceinline__ void x3_contract(const H *__restrict__ xs, int32_t k32, int64_t ra,
                                            int64_t cb, int t, v4f (&A0)[4][4], v4f (&R)[4][4],
                                            X3Smem<V8> &sm) {
  const int64_t kk = 4 * (int64_t)k32;
  const int li = t & 15, lk = (t >> 4) & 3;  // also: piece li of row t / 16 (+ 16, 32, 48)
  const H *pa = xs + (ra + (t >> 4)) * kk + 8 * li, *pb = xs + (cb + li) * kk + 8 * lk;
  V8 st[4], b[4][4];  // staged rows; [slice][column tile]: h1, h2, 2^-b h2, 2^-b h3
  auto load_rows = [&](int64_t off) {
#pragma unroll
    for (int u = 0; u < 4; ++u) st[u] = *reinterpret_cast<const V8 *>(pa + 16 * u * kk + off);
  };
  auto load_cols = [&](int64_t off) {
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
      for (int q = 0; q < 4; ++q)
        b[q][c] = *reinterpret_cast<const V8 *>(pb + 16 * c * kk + off + 32 * q);
  };
  auto step = [&](auto first, int k0, int buf) {
    const int64_t next = (int64_t)((k0 >> 5) + 1) * 128;
    const v4f zero = (v4f){0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int u = 0; u < 4; ++u) sm.a[buf][(t >> 4) + 16 * u][li] = st[u];
    __syncthreads();
    if (k0 + 32 < k32) load_rows(next);
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      V8 a[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) a[q] = sm.a[buf][16 * u + li][4 * q + lk];
      constexpr int kRows[7] = {0, 1, 0, 1, 3, 2, 3}, kCols[7] = {1, 0, 3, 2, 0, 3, 2};
#pragma unroll
      for (int c = 0; c < 4; ++c)
        A0[u][c] = mfma16x32<H, V8>(a[0], b[0][c], decltype(first)::value ? zero : A0[u][c]);
#pragma unroll
      for (int p = 0; p < 7; ++p)
#pragma unroll
        for (int c = 0; c < 4; ++c)
          R[u][c] = mfma16x32<H, V8>(a[kRows[p]], b[kCols[p]][c],
                                     decltype(first)::value && p == 0 ? zero : R[u][c]);
    }
    if (k0 + 32 < k32) load_cols(next);
  };
  load_rows(0);
  load_cols(0);
  step(std::true_type{}, 0, 0);
  for (int k0 = 32, buf = 1; k0 < k32; k0 += 32, buf ^= 1) step(std::false_type{}, k0, buf);
}

// 2 sigma^2 and 2 sigma^2 2^-b
struct X3Scale {
  float s0, s1;
};
__device__ inline X3Scale x3_scale(const Hdr *h, int b) {
  const int e = 2 * (x3_exp(h) - b) + 1;
  return X3Scale{ldexpf(1.f, e), ldexpf(1.f, e - b)};
}

// d = n_i + n_j - 2 x.y from (hi, lo) norms and the two sums. The sum of the
// hi parts is taken with TwoSum (its rounding error e is kept); the leading
// difference t = s - 2 sigma^2 A0 needs no correction: the product is exact,
// and where the operands cancel (2 sigma^2 A0 >= s / 2, i.e. d below about
// s / 2) the subtraction is exact by Sterbenz's lemma, while elsewhere its
// rounding is below one FP32 ulp of d itself.
__device__ __forceinline__ float x3_combine(float2 ni, float2 nj, float a0, float r,
                                            const X3Scale &sc) {
  const float s = __fadd_rn(ni.x, nj.x);
  const float bs = __fsub_rn(s, ni.x);
  const float e = __fadd_rn(__fsub_rn(ni.x, __fsub_rn(s, bs)), __fsub_rn(nj.x, bs));
  const float t = __fsub_rn(s, __fmul_rn(sc.s0, a0));  // a0: an integer below 2^24
  const float low = __fsub_rn(__fadd_rn(e, __fadd_rn(ni.y, nj.y)), __fmul_rn(sc.s1, r));
  return fmaxf(__fadd_rn(t, low), 0.f);
}

// p_ij of Eq. 3 from the distance and both rows' statistics (a = beta
// log2(e), m = row minimum, r = 1 / (2 n S)). No contraction into an FMA, so
// that the two orders of a pair give bitwise equal sums.
__device__ __forceinline__ float pair_p(float d, float ai, float mi, float ri, float aj, float mj,
                                        float rj) {
#pragma clang fp contract(off)
  const float pi = __builtin_amdgcn_exp2f(-ai * (d - mi)) * ri;
  const float pj = __builtin_amdgcn_exp2f(-aj * (d - mj)) * rj;
  return pi + pj;
}

__device__ __forceinline__ int64_t tile_pos(int il, int jl) {
  const int tr = il & 15, k = il >> 4, tc = jl & 15, mq = jl >> 6, e = (jl >> 4) & 3;
  const int t = 64 * (tr >> 2) + 16 * (tr & 3) + tc;
  return ((int64_t)(4 * k + mq) * 256 + t) * 4 + e;
}

__device__ __forceinline__ void put_d(float *__restrict__ tp, bool diag, int il, int jl,
                                      float v) {
  if (!diag) {
    tp[tile_pos(il, jl)] = v;
  } else if (il < jl) {
    tp[tile_pos(il, jl)] = v;
    tp[tile_pos(jl, il)] = v;
  } else if (il == jl) {
    tp[tile_pos(il, il)] = v;
  }
}

// Statistics (a, m, r) of one point for the PACK epilogue; ok = false for a
// padding point (its pairs are stored as 0).
struct PtStat {
  float a, m, r;
  bool ok;
};

template <bool PACK>
__device__ __forceinline__ PtStat pt_stat(int64_t g, int64_t n, const float *__restrict__ a,
                                          const float *__restrict__ m,
                                          const float *__restrict__ r) {
  PtStat p{0.f, 0.f, 0.f, false};
  if (PACK && g < n) p = PtStat{a[g], m[g], r[g], true};
  return p;
}

// Norms and statistics of a strip's 64 rows (and the x3 modes' staged operands),
// in LDS for its epilogue: loads and
// stores of a wave complete in order, so statistics loaded between the stores
// of the rows before them would wait for those stores.
template <int MODE>
struct RowStats {
  using N = std::conditional_t<MODE == TSNE_DIST_FP64, double,
                               std::conditional_t<MODE == TSNE_DIST_BF16X3 ||
                                                      MODE == TSNE_DIST_FP16X3,
                                                  float2, float>>;
  N norm[64];
  float4 st[64];  // a, m, r; w is 1 for a point, 0 for padding
  struct None {};
  std::conditional_t<MODE == TSNE_DIST_BF16X3, X3Smem<v8bf>,
                     std::conditional_t<MODE == TSNE_DIST_FP16X3, X3Smem<v8h>, None>>
      x3;
};

// The stored value of one element: the distance, or with PACK its p_ij (the
// packed value k_pack would write: zero on the diagonal, for padding points
// and below FP32's normal range).
template <bool PACK>
__device__ __forceinline__ float tile_value(float d, bool diag, int il, int jl, const PtStat &si,
                                            const PtStat &sj) {
  if (!PACK) return d;
  // selected, not branched around: a lane's columns then run side by side
  // through the exponentials' latency
  const float v = pair_p(d, si.a, si.m, si.r, sj.a, sj.m, sj.r);
  return (diag && il == jl) || !si.ok || !sj.ok || v < FLT_MIN ? 0.f : v;
}

// Strips of a tile: 64 rows by all columns, in the FP64 mode (whose accumulators
// are twice as wide) by half of them, the second half's strips after the first's.
constexpr int kTileCT = 2;  // 16-column MFMA tiles per wave of a strip in the FP64 mode
__host__ __device__ constexpr int tile_strips(int mode) {
  return mode == TSNE_DIST_FP64 ? (T / 64) * (T / (64 * kTileCT)) : T / 64;
}

// One strip of tile (I, J) into the tile tp, in the layout k_stage produces
// (float4 s * 256 + t of a tile holds rows tr + 16 (s / 4), columns tc + 64 (s % 4)
// + 16 e), by a workgroup of four waves. The contraction of an element is the
// one the per-block-row kernels form for it (same operands, same MFMA
// sequence); a diagonal tile takes the upper element for both orders of a
// pair, as k_stage does, so P stays bitwise symmetric and bitwise that of the
// stored path. Has one barrier, after which `rows` is only read.
template <int MODE, bool PACK>
__device__ __forceinline__ void tile_strip(const TileSrc &src, int I, int J, int strip,
                                           float *__restrict__ tp, RowStats<MODE> &rows) {
  constexpr bool F64 = MODE == TSNE_DIST_FP64, F32 = MODE == TSNE_DIST_FP32;
  constexpr bool X3 = MODE == TSNE_DIST_BF16X3 || MODE == TSNE_DIST_FP16X3;
  constexpr bool BF = MODE == TSNE_DIST_BF16 || MODE == TSNE_DIST_BF16X3;
  using H = std::conditional_t<BF, __bf16, _Float16>;
  using V8 = std::conditional_t<BF, v8bf, v8h>;
  using N = typename RowStats<MODE>::N;
  constexpr int CT = F64 ? kTileCT : 4;  // a wave covers 64 rows x 16 CT columns
  const int ry = strip & 3, cx = strip >> 2;
  const bool diag = (I == J);
  if (diag && 64 * ry >= 64 * CT * (cx + 1)) return;  // wholly below the diagonal
  int t = threadIdx.x;
  // opaque, so that a caller's loop over strips or tiles computes a lane's
  // addresses anew and does not keep them (80 registers spilled there)
  asm volatile("" : "+v"(t));
  const int w = t >> 6, l = t & 63;
  const int li = l & 15, lk = l >> 4;
  const int cl0 = 64 * CT * cx + w * (16 * CT);  // first column of the wave in the tile
  const int64_t col0 = (int64_t)J * T + cl0;
  const int row0_loc = 64 * ry;
  const int64_t row0 = (int64_t)I * T + row0_loc;
  const N *norms = static_cast<const N *>(src.norms);
  if (t < 64) {
    rows.norm[t] = norms[row0 + t];
    if (PACK) {
      const PtStat p = pt_stat<PACK>(row0 + t, src.n, src.a, src.m, src.r);
      rows.st[t] = make_float4(p.a, p.m, p.r, p.ok ? 1.f : 0.f);
    }
  }
  using V4 = std::conditional_t<F64, v4d, v4f>;
  V4 acc[4][CT];
  v4f R[X3 ? 4 : 1][4];
  if constexpr (X3) {
    x3_contract<H, V8>(static_cast<const H *>(src.x), src.kk, row0, col0, t, acc, R, rows.x3);
  } else {
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
      for (int c = 0; c < CT; ++c) acc[a][c] = (V4){0, 0, 0, 0};
    if constexpr (F64 || F32) {
      using X = std::conditional_t<F64, double, float>;
      for (int k0 = 0; k0 < src.dpad; k0 += 4) {
        const X *xk = static_cast<const X *>(src.x) + (int64_t)(k0 + lk) * src.npad;
        X av[4], bv[CT];
#pragma unroll
        for (int a = 0; a < 4; ++a) av[a] = xk[row0 + a * 16 + li];
#pragma unroll
        for (int c = 0; c < CT; ++c) bv[c] = xk[col0 + c * 16 + li];
#pragma unroll
        for (int a = 0; a < 4; ++a)
#pragma unroll
          for (int c = 0; c < CT; ++c) {
            if constexpr (F64)
              acc[a][c] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[a], bv[c], acc[a][c], 0, 0, 0);
            else
              acc[a][c] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[a], bv[c], acc[a][c], 0, 0, 0);
          }
      }
    } else {
      const H *xa = static_cast<const H *>(src.x);
      for (int k0 = 0; k0 < src.kk; k0 += 32) {
        V8 av[4], bv[4];
#pragma unroll
        for (int a = 0; a < 4; ++a)
          av[a] = *reinterpret_cast<const V8 *>(xa + (row0 + a * 16 + li) * src.kk + k0 + 8 * lk);
#pragma unroll
        for (int c = 0; c < 4; ++c)
          bv[c] = *reinterpret_cast<const V8 *>(xa + (col0 + c * 16 + li) * src.kk + k0 + 8 * lk);
#pragma unroll
        for (int a = 0; a < 4; ++a)
#pragma unroll
          for (int c = 0; c < 4; ++c) acc[a][c] = mfma16x32<H, V8>(av[a], bv[c], acc[a][c]);
      }
    }
  }
  float inv_s2 = 1.f;
  if constexpr (MODE == TSNE_DIST_FP16) {
    const float s = fp16_scale(src.h);
    inv_s2 = 1.f / (s * s);
  }
  X3Scale sc{0.f, 0.f};
  if constexpr (X3) sc = x3_scale(src.h, src.bits);
  PtStat scs[CT];
  N nj[CT];
#pragma unroll
  for (int c = 0; c < CT; ++c) {
    scs[c] = pt_stat<PACK>(col0 + c * 16 + li, src.n, src.a, src.m, src.r);
    nj[c] = norms[col0 + c * 16 + li];
  }
  __syncthreads();
#pragma unroll
  for (int a = 0; a < 4; ++a) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int is = a * 16 + (F64 ? lk + 4 * r : 4 * lk + r), il = row0_loc + is;
      const N ni = rows.norm[is];
      PtStat si{0.f, 0.f, 0.f, false};
      if (PACK) {
        const float4 v = rows.st[is];
        si = PtStat{v.x, v.y, v.z, v.w != 0.f};
      }
      float v[CT];
#pragma unroll
      for (int c = 0; c < CT; ++c) {
        float dd;
        if constexpr (X3)
          dd = x3_combine(ni, nj[c], acc[a][c][r], R[a][c][r], sc);
        else if constexpr (F64)
          dd = (float)fmax(ni + nj[c] - 2.0 * acc[a][c][r], 0.0);
        else
          dd = fmaxf((ni + nj[c]) - 2.f * (acc[a][c][r] * inv_s2), 0.f);
        v[c] = tile_value<PACK>(dd, diag, il, cl0 + c * 16 + li, si, scs[c]);
      }
      // the lane's columns are consecutive elements of one float4 slot of the
      // tile layout: one store off the diagonal
      float *to = tp + tile_pos(il, cl0 + li);
      if (diag) {
#pragma unroll
        for (int c = 0; c < CT; ++c) put_d(tp, true, il, cl0 + c * 16 + li, v[c]);
      } else if constexpr (F64) {
        *reinterpret_cast<float2 *>(to) = make_float2(v[0], v[1]);
      } else {
        *reinterpret_cast<float4 *>(to) = make_float4(v[0], v[1], v[2], v[3]);
      }
    }
  }
}

}  // namespace

}  // namespace tsne
