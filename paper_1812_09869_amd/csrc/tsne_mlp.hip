// Surrogate network on the GPU: 50 -> 256 -> 256 -> 2 (d_in -> H -> H -> 2),
// ReLU, trained by mean squared error to map input points to their t-SNE
// embedding, with BF16 MFMA contractions (FP32 accumulation) for the two wide
// layers and FP32 VALU for the 2-wide output layer.
//
// Packed FP32 parameters: W1 [H][d_in], b1 [H], W2 [H][H], b2 [H], W3 [2][H],
// b3 [2]. Inputs are standardised ((x - mean) * invstd) and rounded to BF16;
// W1 and W2 are rounded to BF16 copies before each pass; hidden activations
// are kept in FP32 and rounded to BF16 where they feed a contraction.
#include <math.h>

#include <mutex>

#include "tsne_internal.h"
#include "tsne_mlp.h"

namespace tsne {

namespace {

typedef float v4f __attribute__((ext_vector_type(4)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));

constexpr int kK1 = 64;  // d_in rounded up to the MFMA K step (d_in <= 64)

// ----------------------------------------------------------------------------
// Fused inference. A persistent workgroup of W waves keeps the weights in
// registers and runs tiles of kInferRows rows through the whole network:
//
//   wave w owns hidden units [H/W w, H/W (w + 1)) of both wide layers: its
//   row slices of W1 and W2 (the A operands of the two transposed layers)
//   stay in registers for the life of the workgroup;
//   the standardised BF16 input tile and the BF16 first-layer output tile
//   live in LDS, shared by the W waves;
//   the output layer's partial sums of the W waves meet in LDS.
//
// Both wide layers are computed transposed, H1^T = W1 X^T and H2^T = W2 H1^T
// (M = hidden, N = rows). The B operand of either is one 16-byte LDS read of
// eight consecutive inputs of one row, and lane l = 16g + c receives
// H^T[h0 + 16i + 4g + r][16a + c]: four consecutive hidden units of row
// 16a + c. The first layer's four go to LDS as one 8-byte write; the second
// layer's are summed into the output layer in place, so the sum over a wave's
// hidden units needs only the four lanes of a column (two cross-lane steps).
//
// The next tile's inputs are loaded into registers at the start of a tile and
// written to LDS after its second layer, so the loads have most of a tile's
// time to arrive; the second layer's LDS reads run one K step ahead of its
// MFMAs (explicit double buffer plus scheduling groups of one read per TW
// MFMAs).
// ----------------------------------------------------------------------------
constexpr int kInferRows = 64;   // rows per tile
constexpr int kXPitch = kK1 + 8;  // BF16 elements per LDS row of the input tile

typedef __bf16 v4bf __attribute__((ext_vector_type(4)));

__device__ inline float row16_sum_f(float v) {
  v += __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x128, 0xf, 0xf, true));
  v += __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x124, 0xf, 0xf, true));
  v += __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x122, 0xf, 0xf, true));
  v += __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x121, 0xf, 0xf, true));
  return v;
}

// v + (v of lane l ^ 32) and v + (v of lane l ^ 16) in every lane, with the
// gfx950 lane-swap instructions (VALU, no LDS crossbar): permlane32_swap(v, v)
// leaves the two halves of the wave in its two results, permlane16_swap(v, v)
// the even and odd rows of 16.
__device__ inline float add_xor32(float v) {
  const auto p = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false,
                                                  false);
  return __uint_as_float(p[0]) + __uint_as_float(p[1]);
}
__device__ inline float add_xor16(float v) {
  const auto p = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false,
                                                  false);
  return __uint_as_float(p[0]) + __uint_as_float(p[1]);
}

template <int H, int W>
__global__ __launch_bounds__(64 * W, 1) void k_mlp_infer(
    const float *__restrict__ x, int64_t n, int d_in, const float *__restrict__ mean,
    const float *__restrict__ invstd, const __bf16 *__restrict__ w1b,
    const float *__restrict__ b1, const __bf16 *__restrict__ w2b, const float *__restrict__ b2,
    const float *__restrict__ w3, const float *__restrict__ b3, float *__restrict__ out) {
  constexpr int NT = 64 * W;         // threads
  constexpr int HW = H / W;          // hidden units per wave
  constexpr int TW = HW / 16;        // hidden tiles per wave
  constexpr int KS = H / 32;         // K steps of layer 2
  constexpr int RA = kInferRows / 16;  // row tiles
  constexpr int HPitch = H + 8;      // BF16 elements per LDS row of the hidden tile
  __shared__ __bf16 xs[kInferRows][kXPitch];
  __shared__ __bf16 hs[kInferRows][HPitch];
  __shared__ float po[W][kInferRows][2];
  const int t = threadIdx.x, l = t & 63, w = t >> 6;
  const int c = l & 15, g = l >> 4;
  const int h0 = w * HW;  // first hidden unit of this wave
  v8bf wa[TW][2];  // W1 rows h0 + 16i + c, inputs 32s + 8g .. + 7
#pragma unroll
  for (int i = 0; i < TW; ++i)
#pragma unroll
    for (int st = 0; st < 2; ++st)
      wa[i][st] = *reinterpret_cast<const v8bf *>(w1b + (h0 + 16 * i + c) * kK1 + 32 * st + 8 * g);
  v8bf wb[TW][KS];  // W2 rows h0 + 16e + c, inputs 32s + 8g .. + 7
#pragma unroll
  for (int e = 0; e < TW; ++e)
#pragma unroll
    for (int st = 0; st < KS; ++st)
      wb[e][st] = *reinterpret_cast<const v8bf *>(w2b + (int64_t)(h0 + 16 * e + c) * H + 32 * st + 8 * g);
  float bias1[TW][4], bias2[TW][4], u0[TW][4], u1[TW][4];
#pragma unroll
  for (int i = 0; i < TW; ++i)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int j = h0 + 16 * i + 4 * g + r;
      bias1[i][r] = b1[j];
      bias2[i][r] = b2[j];
      u0[i][r] = w3[j];
      u1[i][r] = w3[H + j];
    }
  const float c0 = b3[0], c1 = b3[1];
  const int64_t ntiles = (n + kInferRows - 1) / kInferRows;
  // the input tile: each thread loads two adjacent columns (xk, xk + 1) of
  // XM rows and stores them as one 32-bit LDS write
  constexpr int XM = kInferRows * kK1 / NT / 2;
  constexpr int RS = NT / (kK1 / 2);  // rows covered per step
  const int xk = 2 * (t & (kK1 / 2 - 1)), xr = t / (kK1 / 2);
  const bool kin0 = xk < d_in, kin1 = xk + 1 < d_in;
  const int xkc0 = kin0 ? xk : d_in - 1, xkc1 = kin1 ? xk + 1 : d_in - 1;  // padding lanes load a real element and store 0
  const float xmean0 = kin0 ? mean[xk] : 0.f, xinv0 = kin0 ? invstd[xk] : 0.f;
  const float xmean1 = kin1 ? mean[xk + 1] : 0.f, xinv1 = kin1 ? invstd[xk + 1] : 0.f;
  float xv[XM][2];
  auto load_x = [&](int64_t tl) {
    if (tl >= ntiles) return;
    const float *xt = x + tl * kInferRows * d_in;  // uniform tile base
    const int64_t lim = n - tl * kInferRows;       // rows of this tile that exist
    if (lim >= kInferRows) {
#pragma unroll
      for (int m = 0; m < XM; ++m) {
        xv[m][0] = xt[(xr + RS * m) * d_in + xkc0];
        xv[m][1] = xt[(xr + RS * m) * d_in + xkc1];
      }
    } else {
#pragma unroll
      for (int m = 0; m < XM; ++m) {
        const int rl = xr + RS * m;
        xv[m][0] = rl < lim ? xt[rl * d_in + xkc0] : 0.f;
        xv[m][1] = rl < lim ? xt[rl * d_in + xkc1] : 0.f;
      }
    }
  };
  auto store_x = [&]() {
#pragma unroll
    for (int m = 0; m < XM; ++m) {
      typedef __bf16 v2bf __attribute__((ext_vector_type(2)));
      v2bf pr;
      pr[0] = (__bf16)((xv[m][0] - xmean0) * xinv0);  // 0 in padding lanes
      pr[1] = (__bf16)((xv[m][1] - xmean1) * xinv1);
      *reinterpret_cast<v2bf *>(&xs[xr + RS * m][xk]) = pr;
    }
  };
  load_x(blockIdx.x);
  store_x();
  __syncthreads();
  for (int64_t tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
    const int64_t row0 = tile * kInferRows;
    load_x(tile + gridDim.x);
    v4f acc1[TW][RA];
#pragma unroll
    for (int i = 0; i < TW; ++i)
#pragma unroll
      for (int a = 0; a < RA; ++a) acc1[i][a] = (v4f){0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int st = 0; st < 2; ++st)
#pragma unroll
      for (int a = 0; a < RA; ++a) {
        const v8bf xb = *reinterpret_cast<const v8bf *>(&xs[16 * a + c][32 * st + 8 * g]);
#pragma unroll
        for (int i = 0; i < TW; ++i)
          acc1[i][a] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wa[i][st], xb, acc1[i][a], 0, 0, 0);
      }
#pragma unroll
    for (int i = 0; i < TW; ++i)
#pragma unroll
      for (int a = 0; a < RA; ++a) {
        v4bf hv;
#pragma unroll
        for (int r = 0; r < 4; ++r) hv[r] = (__bf16)fmaxf(acc1[i][a][r] + bias1[i][r], 0.f);
        *reinterpret_cast<v4bf *>(&hs[16 * a + c][h0 + 16 * i + 4 * g]) = hv;
      }
    __syncthreads();
    // layer 2, transposed: acc2[e][a] = H2^T[h0 + 16e + 4g + r][16a + c]
    v4f acc2[TW][RA];
#pragma unroll
    for (int e = 0; e < TW; ++e)
#pragma unroll
      for (int a = 0; a < RA; ++a) acc2[e][a] = (v4f){0.f, 0.f, 0.f, 0.f};
    v8bf hb[2][RA];
#pragma unroll
    for (int a = 0; a < RA; ++a) hb[0][a] = *reinterpret_cast<const v8bf *>(&hs[16 * a + c][8 * g]);
#pragma unroll
    for (int st = 0; st < KS; ++st) {
      if (st + 1 < KS) {
#pragma unroll
        for (int a = 0; a < RA; ++a)
          hb[(st + 1) & 1][a] = *reinterpret_cast<const v8bf *>(&hs[16 * a + c][32 * (st + 1) + 8 * g]);
      }
#pragma unroll
      for (int a = 0; a < RA; ++a)
#pragma unroll
        for (int e = 0; e < TW; ++e)
          acc2[e][a] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wb[e][st], hb[st & 1][a], acc2[e][a], 0, 0, 0);
    }
    __builtin_amdgcn_sched_group_barrier(0x100, RA, 0);
#pragma unroll
    for (int q = 0; q < (KS - 1) * RA; ++q) {
      __builtin_amdgcn_sched_group_barrier(0x008, TW, 0);
      __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
    }
    __builtin_amdgcn_sched_group_barrier(0x008, TW * RA, 0);
    // output layer: lane (c, g) holds 4 TW hidden units of row 16a + c
#pragma unroll
    for (int a = 0; a < RA; ++a) {
      float s0 = 0.f, s1 = 0.f;
#pragma unroll
      for (int e = 0; e < TW; ++e)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const float hh = fmaxf(acc2[e][a][r] + bias2[e][r], 0.f);
          s0 = fmaf(u0[e][r], hh, s0);
          s1 = fmaf(u1[e][r], hh, s1);
        }
      s0 = add_xor32(s0);
      s1 = add_xor32(s1);
      s0 = add_xor16(s0);
      s1 = add_xor16(s1);
      po[w][16 * a + c][0] = s0;  // the four lanes of a column hold the same sums
      po[w][16 * a + c][1] = s1;
    }
    __builtin_amdgcn_sched_barrier(0);
    store_x();
    __syncthreads();
    if (t < kInferRows * 2) {
      const int rr = t >> 1, o = t & 1;
      const int64_t row = row0 + rr;
      float sum = 0.f;
#pragma unroll
      for (int q = 0; q < W; ++q) sum += po[q][rr][o];
      if (row < n) out[2 * row + o] = sum + (o ? c1 : c0);
    }
  }
}


// BF16 copies of W1 (zero-padded to [H][kK1]), W2 and W2 transposed.
__global__ void k_mlp_cast(const float *__restrict__ p, int d_in, int H, __bf16 *__restrict__ w1b,
                           __bf16 *__restrict__ w2b, __bf16 *__restrict__ w2tb) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const float *w1 = p, *w2 = p + (int64_t)H * d_in + H;
  if (i < (int64_t)H * kK1) {
    const int j = (int)(i / kK1), k = (int)(i % kK1);
    w1b[i] = (__bf16)(k < d_in ? w1[(int64_t)j * d_in + k] : 0.f);
  }
  if (i < (int64_t)H * H) {
    const int j = (int)(i / H), k = (int)(i % H);
    const __bf16 v = (__bf16)w2[i];
    w2b[i] = v;
    w2tb[(int64_t)k * H + j] = v;
  }
}

// ----------------------------------------------------------------------------
// Training: one kernel takes a tile of 16 rows of the batch forward and back,
// one more forms every parameter gradient. As single layers a step was 13
// launches of 3 to 22 us, each the latency of a few dependent loads on 64
// workgroups or fewer, with the activations written and read between them and
// their transposes stored two bytes at a time.
//
// k_mlp_rows: wave w owns hidden units [H/W w, H/W (w + 1)) of both layers in
// both directions and loads its rows of W1 and W2 while the inputs arrive and those
// of W2^T beside the first layer. All three products are formed transposed, so a lane holds four
// consecutive hidden units of one row, and the layers' operands pass through LDS:
//   H1^T = W1 X^T, H2^T = W2 H1^T, out = W3 H2 + b3 (FP32, partial sums of the
//   waves in LDS), dout = (out - y) / B, dH2 = W3^T dout where H2 > 0,
//   dH1^T = W2^T dH2^T where H1 > 0.
// The contractions' K steps are summed in KP parts whose sums are added in
// order. Out of a tile go the BF16 operands of the weight gradients as
// [tile][unit][16 rows], whose 16-byte pieces are the next kernel's operands,
// and the tile's FP32 sums over its 16 rows for db1, db2, dW3, db3 and the loss.
//
// k_mlp_wgrad: workgroups of eight waves, 32 x 32 blocks of dW2 = dH2^T H1 and
// dW1 = dH1^T X with the batch split over the waves (their partial results meet
// in LDS, added in wave order); the last ones add the tiles' sums, in FP64.
//
// What bounds them at B = 1,024, H = 256 is the chain of one tile (index, row,
// two layers, output, two layers back: five barriers), 14.2 us with cold caches,
// and 4.2 us for the weight gradients; a gradient took 136 us and takes 21
// (B = 4,096: 223 and 28; 65,536: 2,369 and 271).
// ----------------------------------------------------------------------------
constexpr int kTrainRows = 16;

template <int KS, int KP, int TW>
__device__ __forceinline__ void train_layer(const v8bf (&wt)[TW][KS], const __bf16 *row, int g,
                                            v4f (&acc)[TW]) {
  v8bf b[KS];
#pragma unroll
  for (int st = 0; st < KS; ++st)
    b[st] = *reinterpret_cast<const v8bf *>(row + 32 * st + 8 * g);
#pragma unroll
  for (int i = 0; i < TW; ++i) {
#pragma unroll
    for (int p = 0; p < KP; ++p) {
      v4f s = (v4f){0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int st = KS / KP * p; st < KS / KP * (p + 1); ++st)
        s = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wt[i][st], b[st], s, 0, 0, 0);
      acc[i] = p ? acc[i] + s : s;
    }
  }
}

// Partial sums of a tile: db1[H], db2[H], dW3[2][H], db3[2].
__host__ __device__ inline int train_sums(int H) { return 4 * H + 2; }

template <int H, int W>
__global__ __launch_bounds__(64 * W, 1) void k_mlp_rows(
    const float *__restrict__ x, const float *__restrict__ y, int d_in,
    const float *__restrict__ mean, const float *__restrict__ invstd,
    const int32_t *__restrict__ idx, int64_t B, int64_t Bpad, const __bf16 *__restrict__ w1b,
    const float *__restrict__ b1, const __bf16 *__restrict__ w2b,
    const __bf16 *__restrict__ w2tb, const float *__restrict__ b2, const float *__restrict__ w3,
    const float *__restrict__ b3, double inv_batch, __bf16 *__restrict__ xbt,
    __bf16 *__restrict__ h1t, __bf16 *__restrict__ dh2t, __bf16 *__restrict__ dh1t,
    float *__restrict__ sums, double *__restrict__ loss_part) {
  constexpr int HW = H / W, TW = HW / 16, KS = H / 32;
  constexpr int KP = KS % 4 == 0 ? 4 : 2;
  constexpr int HPitch = H + 8;
  __shared__ __bf16 xs[kTrainRows][kXPitch];
  __shared__ __bf16 hs[kTrainRows][HPitch];  // H1, then dH2
  __shared__ float po[W][kTrainRows][2];
  __shared__ v4f vec[4][H / 4];  // b1, b2 and the two rows of W3
  const int t = threadIdx.x, l = t & 63, w = t >> 6;
  const int c = l & 15, g = l >> 4;
  const int h0 = w * HW;
  for (int e = t; e < 4 * H; e += 64 * W) {
    const int j = e % H;
    const float *src = e < H ? b1 + j : e < 2 * H ? b2 + j : w3 + (e - 2 * H);
    reinterpret_cast<float *>(vec)[e] = *src;
  }
  v8bf wa[TW][2], wb[TW][KS], wt[TW][KS];
#pragma unroll
  for (int i = 0; i < TW; ++i) {
#pragma unroll
    for (int st = 0; st < 2; ++st)
      wa[i][st] =
          *reinterpret_cast<const v8bf *>(w1b + (h0 + 16 * i + c) * kK1 + 32 * st + 8 * g);
#pragma unroll
    for (int st = 0; st < KS; ++st)
      wb[i][st] =
          *reinterpret_cast<const v8bf *>(w2b + (h0 + 16 * i + c) * H + 32 * st + 8 * g);
  }
  const float c0 = b3[0], c1 = b3[1];
  const int64_t tile = blockIdx.x;
  const int64_t row0 = tile * kTrainRows;
  // standardised inputs, zero past the batch and past d_in
  for (int e = t; e < kTrainRows * kK1; e += 64 * W) {
    const int r = e / kK1, k = e % kK1;
    const int64_t b = row0 + r;
    float v = 0.f;
    if (b < B && k < d_in) {
      const int64_t i = idx ? (int64_t)idx[b] : b;
      v = (x[i * d_in + k] - mean[k]) * invstd[k];
    }
    xs[r][k] = (__bf16)v;
  }
  const int64_t br = row0 + c;  // this lane's row
  __bf16 *h1o = h1t + row0 * H, *dh2o = dh2t + row0 * H, *dh1o = dh1t + row0 * H;
  const bool live = br < B;
  float y0 = 0.f, y1 = 0.f;
  if (live) {
    const int64_t i = idx ? (int64_t)idx[br] : br;
    y0 = y[2 * i];
    y1 = y[2 * i + 1];
  }
  __syncthreads();
  __bf16 *xt = xbt + row0 * kK1;
  for (int e = t; e < kTrainRows * kK1; e += 64 * W) {
    const int k = e / kTrainRows, r = e % kTrainRows;
    xt[e] = xs[r][k];
  }
#pragma unroll
  for (int i = 0; i < TW; ++i)
#pragma unroll
    for (int st = 0; st < KS; ++st)
      wt[i][st] =
          *reinterpret_cast<const v8bf *>(w2tb + (h0 + 16 * i + c) * H + 32 * st + 8 * g);
  // first layer
  v4f acc[TW];
  train_layer<2, 2, TW>(wa, xs[c], g, acc);
  uint32_t on1 = 0;  // units of this lane with H1 > 0
#pragma unroll
  for (int i = 0; i < TW; ++i) {
    v4bf hv;
    const v4f bias = vec[0][(h0 + 16 * i) / 4 + g];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int j = h0 + 16 * i + 4 * g + r;
      const float h = fmaxf(acc[i][r] + bias[r], 0.f);
      on1 |= h > 0.f ? 1u << (4 * i + r) : 0u;
      hv[r] = (__bf16)h;
      h1o[kTrainRows * j + c] = hv[r];
    }
    *reinterpret_cast<v4bf *>(&hs[c][h0 + 16 * i + 4 * g]) = hv;
  }
  __syncthreads();
  // second layer and the output layer's share of this wave
  train_layer<KS, KP, TW>(wb, hs[c], g, acc);
  float h2[TW][4], s0 = 0.f, s1 = 0.f;
#pragma unroll
  for (int i = 0; i < TW; ++i) {
    const int v = (h0 + 16 * i) / 4 + g;
    const v4f bias = vec[1][v], u0 = vec[2][v], u1 = vec[3][v];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      h2[i][r] = live ? fmaxf(acc[i][r] + bias[r], 0.f) : 0.f;
      s0 = fmaf(u0[r], h2[i][r], s0);
      s1 = fmaf(u1[r], h2[i][r], s1);
    }
  }
  s0 = add_xor16(add_xor32(s0));
  s1 = add_xor16(add_xor32(s1));
  if (g == 0) {
    po[w][c][0] = s0;
    po[w][c][1] = s1;
  }
  __syncthreads();  // also: every wave is done with H1 in hs
  float o0 = 0.f, o1 = 0.f;
#pragma unroll
  for (int q = 0; q < W; ++q) {
    o0 += po[q][c][0];
    o1 += po[q][c][1];
  }
  const float e0 = live ? o0 + c0 - y0 : 0.f, e1 = live ? o1 + c1 - y1 : 0.f;
  const float d0 = (float)(e0 * inv_batch), d1 = (float)(e1 * inv_batch);
  float *sp = sums + tile * train_sums(H);
  if (w == 0) {
    double ls = l < 16 ? 0.5 * ((double)e0 * e0 + (double)e1 * e1) : 0.0;
#pragma unroll
    for (int o = 8; o > 0; o >>= 1) ls += __shfl_xor(ls, o, 64);
    const float t0 = row16_sum_f(d0), t1 = row16_sum_f(d1);
    if (l == 0) {
      loss_part[tile] = ls;
      sp[4 * H] = t0;
      sp[4 * H + 1] = t1;
    }
  }
  // dH2, and the sums over the 16 rows
#pragma unroll
  for (int i = 0; i < TW; ++i) {
    v4bf dv;
    const int v = (h0 + 16 * i) / 4 + g;
    const v4f u0 = vec[2][v], u1 = vec[3][v];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int j = h0 + 16 * i + 4 * g + r;
      float dh = fmaf(d0, u0[r], d1 * u1[r]);
      if (!(h2[i][r] > 0.f)) dh = 0.f;
      dv[r] = (__bf16)dh;
      dh2o[kTrainRows * j + c] = dv[r];
      const float sb = row16_sum_f(dh), sw0 = row16_sum_f(d0 * h2[i][r]),
                  sw1 = row16_sum_f(d1 * h2[i][r]);
      if (c == 0) {
        sp[H + j] = sb;
        sp[2 * H + j] = sw0;
        sp[3 * H + j] = sw1;
      }
    }
    *reinterpret_cast<v4bf *>(&hs[c][h0 + 16 * i + 4 * g]) = dv;
  }
  __syncthreads();
  train_layer<KS, KP, TW>(wt, hs[c], g, acc);
#pragma unroll
  for (int i = 0; i < TW; ++i)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int j = h0 + 16 * i + 4 * g + r;
      const float dh = (on1 >> (4 * i + r)) & 1u ? acc[i][r] : 0.f;
      dh1o[kTrainRows * j + c] = (__bf16)dh;
      const float sb = row16_sum_f(dh);
      if (c == 0) sp[j] = sb;
    }
}

constexpr int kWgWaves = 8;

// C block (bm, bn) of 32 x 32: C[m][n] = sum_b A[m][b] D[n][b], columns n < nvalid;
// A and D hold ma and na units to a tile of 16 rows.
__device__ __forceinline__ void wgrad_block(const __bf16 *__restrict__ A, int ma,
                                            const __bf16 *__restrict__ D, int na, int64_t Bpad,
                                            int bm, int bn, float *__restrict__ C, int ldc,
                                            int nvalid, v4f (*red)[4][64]) {
  const int t = threadIdx.x, l = t & 63, w = t >> 6, li = l & 15, lk = l >> 4;
  const int steps = (int)(Bpad / 32), s0 = steps * w / kWgWaves, s1 = steps * (w + 1) / kWgWaves;
  v4f acc[2][2];
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int c = 0; c < 2; ++c) acc[a][c] = (v4f){0.f, 0.f, 0.f, 0.f};
  // batch rows 32 st + 8 lk .. + 7: tile 2 st + lk / 2, half lk % 2
  const __bf16 *ap = A + ((int64_t)(lk >> 1) * ma + 32 * bm + li) * kTrainRows + 8 * (lk & 1);
  const __bf16 *dp = D + ((int64_t)(lk >> 1) * na + 32 * bn + li) * kTrainRows + 8 * (lk & 1);
  const int64_t as = 2 * kTrainRows * (int64_t)ma, ds = 2 * kTrainRows * (int64_t)na;
  int st = s0;
  for (; st + 4 <= s1; st += 4) {  // four steps' loads in flight
    v8bf av[4][2], dv[4][2];
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
      for (int a = 0; a < 2; ++a) {
        av[u][a] = *reinterpret_cast<const v8bf *>(ap + as * (st + u) + 16 * kTrainRows * a);
        dv[u][a] = *reinterpret_cast<const v8bf *>(dp + ds * (st + u) + 16 * kTrainRows * a);
      }
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
      for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int c = 0; c < 2; ++c)
          acc[a][c] =
              __builtin_amdgcn_mfma_f32_16x16x32_bf16(av[u][a], dv[u][c], acc[a][c], 0, 0, 0);
  }
  for (; st < s1; ++st) {
    v8bf av[2], dv[2];
#pragma unroll
    for (int a = 0; a < 2; ++a) {
      av[a] = *reinterpret_cast<const v8bf *>(ap + as * st + 16 * kTrainRows * a);
      dv[a] = *reinterpret_cast<const v8bf *>(dp + ds * st + 16 * kTrainRows * a);
    }
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
      for (int c = 0; c < 2; ++c)
        acc[a][c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av[a], dv[c], acc[a][c], 0, 0, 0);
  }
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int c = 0; c < 2; ++c) red[w][2 * a + c][l] = acc[a][c];
  __syncthreads();
  // thread (q, lane): the waves' results of one MFMA tile in wave order
  if (t >= 256) return;
  const int q = t >> 6;
  v4f s = red[0][q][l];
#pragma unroll
  for (int v = 1; v < kWgWaves; ++v) s += red[v][q][l];
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int m = 32 * bm + 16 * (q >> 1) + 4 * lk + r, n = 32 * bn + 16 * (q & 1) + li;
    if (n < nvalid) C[(int64_t)m * ldc + n] = s[r];
  }
}

__global__ __launch_bounds__(64 * kWgWaves) void k_mlp_wgrad(
    const __bf16 *__restrict__ xbt, const __bf16 *__restrict__ h1t,
    const __bf16 *__restrict__ dh2t, const __bf16 *__restrict__ dh1t, int64_t Bpad, int H,
    int d_in, const float *__restrict__ sums, const double *__restrict__ loss_part,
    double inv_batch, float *__restrict__ g_w1, float *__restrict__ g_b1,
    float *__restrict__ g_w2, float *__restrict__ g_b2, float *__restrict__ g_w3,
    float *__restrict__ g_b3, double *__restrict__ loss) {
  __shared__ v4f red[kWgWaves][4][64];
  const int hb = H / 32, n2 = hb * hb, n1 = hb * (kK1 / 32);
  const int wg = blockIdx.x;
  if (wg < n2) {
    wgrad_block(dh2t, H, h1t, H, Bpad, wg / hb, wg % hb, g_w2, H, H, red);
    return;
  }
  if (wg < n2 + n1) {
    const int q = wg - n2;
    wgrad_block(dh1t, H, xbt, kK1, Bpad, q / (kK1 / 32), q % (kK1 / 32), g_w1, d_in, d_in, red);
    return;
  }
  // sums over the tiles: 64 values to a workgroup, one to a lane, the tiles split over the
  // waves, whose sums are added in order; the value past the sums is the loss
  const int64_t tiles = Bpad / kTrainRows;
  const int l = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int ns = train_sums(H), e = (wg - n2 - n1) * 64 + l;
  const int64_t q0 = tiles * w / kWgWaves, q1 = tiles * (w + 1) / kWgWaves;
  double s = 0.0;
  if (e < ns) {
    int64_t q = q0;
    for (; q + 8 <= q1; q += 8) {
      float v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = sums[(q + u) * ns + e];
#pragma unroll
      for (int u = 0; u < 8; ++u) s += (double)v[u];
    }
    for (; q < q1; ++q) s += (double)sums[q * ns + e];
  } else if (e == ns) {
    for (int64_t q = q0; q < q1; ++q) s += loss_part[q];
  }
  double(*part)[64] = reinterpret_cast<double(*)[64]>(red);
  part[w][l] = s;
  __syncthreads();
  if (w > 0 || e > ns) return;
#pragma unroll
  for (int v = 1; v < kWgWaves; ++v) s += part[v][l];
  if (e == ns) {
    *loss = s * inv_batch;
    return;
  }
  float *dst = e < H ? g_b1 + e : e < 2 * H ? g_b2 + (e - H)
                                 : e < 4 * H ? g_w3 + (e - 2 * H) : g_b3 + (e - 4 * H);
  *dst = (float)s;
}

__global__ void k_adam(float *__restrict__ p, const float *__restrict__ g, float *__restrict__ m,
                       float *__restrict__ v, int64_t count, float lr, float beta1, float beta2,
                       float eps, float inv_c1, float inv_c2) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= count) return;
  const float gi = g[i];
  const float mi = beta1 * m[i] + (1.f - beta1) * gi;
  const float vi = beta2 * v[i] + (1.f - beta2) * gi * gi;
  m[i] = mi;
  v[i] = vi;
  p[i] -= lr * (mi * inv_c1) / (sqrtf(vi * inv_c2) + eps);
}

}  // namespace

// ----------------------------------------------------------------------------
// Workspace layout for a batch of up to Bpad rows (Bpad multiple of 64)
// ----------------------------------------------------------------------------
MlpLayout make_mlp_layout(int d_in, int H, int64_t Bpad, bool train) {
  MlpLayout L;
  L.d_in = d_in;
  L.H = H;
  L.Bpad = Bpad;
  size_t o = 0;
  auto take = [&](size_t bytes) {
    size_t at = o;
    o = (o + bytes + 255) / 256 * 256;
    return at;
  };
  const size_t B = (size_t)Bpad, Hs = (size_t)H;
  L.w1b = take(Hs * kK1 * 2);
  L.w2b = take(Hs * Hs * 2);
  L.w2tb = take(Hs * Hs * 2);
  // (a forward pass keeps its activations in the kernel, whatever the batch)
  if (train) {
    L.xbt = take(B * kK1 * 2);
    L.h1t = take(B * Hs * 2);
    L.dh2t = take(B * Hs * 2);
    L.dh1t = take(B * Hs * 2);
    L.sums = take(B / kTrainRows * train_sums(H) * 4);
    L.loss_part = take(B / kTrainRows * 8);
  }
  L.total = o;
  return L;
}

// Forward pass of rows [row0, row0 + B) (or idx[0..B)) of x into out.
hipError_t launch_mlp_cast(const MlpLayout &L, const float *params, void *ws, hipStream_t st) {
  const int64_t cnt = (int64_t)L.H * (L.H > kK1 ? L.H : kK1);
  hipLaunchKernelGGL(k_mlp_cast, dim3((unsigned)((cnt + 255) / 256)), dim3(256), 0, st, params,
                     L.d_in, L.H, at<__bf16>(ws, L.w1b), at<__bf16>(ws, L.w2b),
                     at<__bf16>(ws, L.w2tb));
  return hipGetLastError();
}

hipError_t launch_mlp_forward(const MlpLayout &L, const float *params, const float *mean,
                              const float *invstd, const float *x, int64_t n, float *out, void *ws,
                              hipStream_t st) {
  hipError_t e = launch_mlp_cast(L, params, ws, st);
  if (e != hipSuccess) return e;
  const int H = L.H;
  const float *b1 = params + (int64_t)H * L.d_in, *b2 = b1 + H + (int64_t)H * H;
  const float *w3 = b2 + H, *b3 = w3 + 2 * H;
  const __bf16 *w1b = at<const __bf16>(ws, L.w1b), *w2b = at<const __bf16>(ws, L.w2b);
  // persistent: at most one workgroup per compute unit (the weights fill the
  // registers of a wave per SIMD), fewer when there are fewer tiles
  const int64_t ntiles = (n + kInferRows - 1) / kInferRows;
  const dim3 grid((unsigned)(ntiles < 256 ? ntiles : 256));
  switch (H) {
    case 64:
      hipLaunchKernelGGL((k_mlp_infer<64, 4>), grid, dim3(256), 0, st, x, n, L.d_in, mean, invstd,
                         w1b, b1, w2b, b2, w3, b3, out);
      break;
    case 128:
      hipLaunchKernelGGL((k_mlp_infer<128, 8>), grid, dim3(512), 0, st, x, n, L.d_in, mean,
                         invstd, w1b, b1, w2b, b2, w3, b3, out);
      break;
    case 192:
      hipLaunchKernelGGL((k_mlp_infer<192, 4>), grid, dim3(256), 0, st, x, n, L.d_in, mean,
                         invstd, w1b, b1, w2b, b2, w3, b3, out);
      break;
    default:
      hipLaunchKernelGGL((k_mlp_infer<256, 8>), grid, dim3(512), 0, st, x, n, L.d_in, mean,
                         invstd, w1b, b1, w2b, b2, w3, b3, out);
  }
  return hipGetLastError();
}

// ----------------------------------------------------------------------------
// Scratch of the allocation-free forward entry point: the BF16 weight copies
// of a forward pass (the whole 64-row forward layout, under 0.4 MiB for every
// supported d_in and H). One copy per device, held until the process ends and
// shared by every call on that device. Host code never passes the array's
// name to a kernel (on the host it is only a stand-in for the symbol): the
// device address is looked up once per device, with that device current, and
// kept here.
// ----------------------------------------------------------------------------
static __device__ __align__(256) unsigned char scratch[kNoAllocScratchBytes];

namespace {
std::mutex g_scratch_mu;
void *g_scratch_ptr[64] = {};
}  // namespace

hipError_t noalloc_scratch(void **out) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= 64) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void *p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (!p) return hipErrorInvalidSymbol;
    g_scratch_ptr[dev] = p;
  }
  *out = g_scratch_ptr[dev];
  return hipSuccess;
}

hipError_t launch_mlp_gradient(const MlpLayout &L, const float *params, const float *mean,
                               const float *invstd, const float *x, const float *y,
                               const int32_t *idx, int64_t B, float *grad, double *loss,
                               void *ws, hipStream_t st) {
  const int H = L.H, d_in = L.d_in;
  const int64_t Bpad = (B + 63) / 64 * 64;
  const float *b1 = params + (int64_t)H * d_in, *b2 = b1 + H + (int64_t)H * H;
  const float *w3 = b2 + H, *b3 = w3 + 2 * H;
  float *g_w1 = grad, *g_b1 = g_w1 + (int64_t)H * d_in, *g_w2 = g_b1 + H,
        *g_b2 = g_w2 + (int64_t)H * H, *g_w3 = g_b2 + H, *g_b3 = g_w3 + 2 * H;
  __bf16 *xbt = at<__bf16>(ws, L.xbt), *h1t = at<__bf16>(ws, L.h1t),
         *dh2t = at<__bf16>(ws, L.dh2t), *dh1t = at<__bf16>(ws, L.dh1t);
  float *sums = at<float>(ws, L.sums);
  double *lp = at<double>(ws, L.loss_part);
  const double inv = 1.0 / (double)B;
  hipError_t err = launch_mlp_cast(L, params, ws, st);
  if (err != hipSuccess) return err;
  const int64_t tiles = Bpad / kTrainRows;
  const dim3 grid((unsigned)tiles);
#define TSNE_ROWS(HH, W)                                                                        \
  hipLaunchKernelGGL((k_mlp_rows<HH, W>), grid, dim3(64 * W), 0, st, x, y, d_in, mean, invstd,  \
                     idx, B, Bpad, at<const __bf16>(ws, L.w1b), b1, at<const __bf16>(ws, L.w2b), \
                     at<const __bf16>(ws, L.w2tb), b2, w3, b3, inv, xbt, h1t, dh2t, dh1t, sums, \
                     lp)
  switch (H) {
    case 64:
      TSNE_ROWS(64, 4);
      break;
    case 128:
      TSNE_ROWS(128, 8);
      break;
    case 192:
      TSNE_ROWS(192, 12);
      break;
    default:
      TSNE_ROWS(256, 16);
  }
#undef TSNE_ROWS
  const int hb = H / 32;
  const unsigned wgs = (unsigned)(hb * hb + hb * (kK1 / 32) + train_sums(H) / 64 + 1);
  hipLaunchKernelGGL(k_mlp_wgrad, dim3(wgs), dim3(64 * kWgWaves), 0, st, xbt, h1t, dh2t, dh1t, Bpad,
                     H, d_in, sums, lp, inv, g_w1, g_b1, g_w2, g_b2, g_w3, g_b3, loss);
  return hipGetLastError();
}

hipError_t launch_adam(float *p, const float *g, float *m, float *v, int64_t count, float lr,
                       float beta1, float beta2, float eps, int32_t t, hipStream_t st) {
  const double c1 = 1.0 - pow((double)beta1, t), c2 = 1.0 - pow((double)beta2, t);
  hipLaunchKernelGGL(k_adam, dim3((unsigned)((count + 255) / 256)), dim3(256), 0, st, p, g, m, v,
                     count, lr, beta1, beta2, eps, (float)(1.0 / c1), (float)(1.0 / c2));
  return hipGetLastError();
}

}  // namespace tsne
