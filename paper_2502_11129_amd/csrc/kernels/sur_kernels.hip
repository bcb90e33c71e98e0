// Kernels of the learned fitness surrogate: genotype features, BF16 MFMA
// products with fused bias/GELU/GELU' epilogues, the prediction head and its
// deterministic reductions, Adam with BF16 weight copies, and top-k selection.
//
// Matrix products use v_mfma_f32_16x16x32_bf16 (gfx950): a wave multiplies a
// 16x32 BF16 tile of A by a 32x16 tile of B into a 16x16 FP32 tile.  Lane l
// supplies row (l mod 16) of A and column (l mod 16) of B, eight consecutive
// k each (k = 8 floor(l/16) ...); it receives rows 4 floor(l/16) + i,
// i = 0..3, of column (l mod 16) of the result.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <mutex>

#include "../sur_launch.h"

namespace surk {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// ----------------------------------------------------------------------------- scalar helpers
__device__ inline uint16_t f2bf(float f) {
  // round to nearest even; NaN stays NaN (quiet bit set)
  uint32_t u = __float_as_uint(f);
  if ((u & 0x7fffffffu) > 0x7f800000u) return (uint16_t)((u >> 16) | 0x40u);
  u += 0x7fffu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}
__device__ inline float bf2f(uint32_t b) { return __uint_as_float((b & 0xffffu) << 16); }

// erff takes one of two ways at |x| = 1, a branch per value.  Where all of a
// wave's values keep clear of it (near_zero), the argument's range is told to the
// compiler, which leaves the one polynomial: the same results, 8 instructions.
template <bool SMALL>
__device__ inline float erf_half(float z) {
  const float x = z * 0.70710678118654752f;
  if (SMALL) __builtin_assume(__builtin_fabsf(x) < 1.0f);
  return erff(x);
}
// |z| < 1.4 for all values of all lanes (false with a NaN among them)
__device__ inline bool near_zero(const float (&z)[4]) {
  const float m = __builtin_elementwise_maximum(
      __builtin_elementwise_maximum(__builtin_fabsf(z[0]), __builtin_fabsf(z[1])),
      __builtin_elementwise_maximum(__builtin_fabsf(z[2]), __builtin_fabsf(z[3])));
  return __builtin_amdgcn_ballot_w64(!(m < 1.4f)) == 0;
}
template <bool SMALL>
__device__ inline float gelu(float z) {
  return 0.5f * z * (1.0f + erf_half<SMALL>(z));
}

// Place of element (row, k) of a BF16 matrix that is an operand of products over
// k, in the order of a wave's registers for them: 16 rows and 32 k after each
// other, lane (row % 16, k / 8 % 4) with its eight k.  A wave's load then takes
// 1 KB of whole lines; by rows of k it touched a line per lane, 64 where 8 do:
// 10 007 predictions took 15.9 us instead of 10.2, a training batch 40 instead of 33.
__device__ inline int64_t operand(int row, int64_t k, int rows) {
  return (((k >> 5) * (rows / 16) + (row >> 4)) * 64 + ((k >> 3) & 3) * 16 + (row & 15)) * 8 + (k & 7);
}

constexpr uint16_t kOne = 0x3F80;
constexpr uint16_t kNaN = 0x7FC0;

// ----------------------------------------------------------------------------- whole-network prediction
// The four layers of one tile of 16 NT rows without leaving the CU.  A
// workgroup's eight waves (two per SIMD) hold the three weight matrices in
// their registers, 32 output columns each (160 registers), and walk over tiles;
// activations go from layer to layer through LDS in BF16.  The products run
// with the weights as the row operand, so a lane's four results are four
// consecutive columns of one row and go to LDS as eight bytes.
// 1 M rows: 472 us, 700 TFLOP/s; layer at a time, with the activations (1.5 KB a
// row) through HBM, 1816 us.  10 007 rows: 10 us, 39 in four launches.  What bounds
// it is the matrix cores (274 us at the 1200 TFLOP/s of a large product), the exact erf
// of 768 GELUs a row (8 vector instructions each, up to 46 where values are large:
// then 790 us) and the LDS reads, which the barriers of a layer keep apart.
constexpr int kPredWaves = 8;
constexpr int kXS = kFeat + 8, kHS = kHid + 8;  // LDS row strides in BF16 (16-byte aligned, banks spread)

// Sum over the 64 lanes by lane distances 32, 16, 8, 4, 2, 1, without LDS; every
// lane gets the result.
template <int CTRL>
__device__ inline float dpp_move(float x) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xF, 0xF, false));
}
__device__ inline float wave_sum(float v) {
  auto a = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = __uint_as_float(a[0]) + __uint_as_float(a[1]);
  a = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = __uint_as_float(a[0]) + __uint_as_float(a[1]);
  v += dpp_move<0x128>(v);  // row_ror:8
  v += dpp_move<0x124>(v);  // row_ror:4 (lanes 8 apart agree by now)
  v += dpp_move<0x4E>(v);   // quad_perm [2,3,0,1]
  v += dpp_move<0xB1>(v);   // quad_perm [1,0,3,2]
  return v;
}

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
// two floats to BF16, round to nearest even
__device__ inline uint32_t pack_bf16(float a, float b) {
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{a, b}, bf16x2));
}

// acc[m][t] = W[32 columns of the wave] . act[tile rows] over K = 32 KS; W in
// registers, act in LDS (row stride ST).
template <int KS, int ST, int NT>
__device__ inline void tile_product(const bf16x8 (&w)[2][KS], const uint16_t* act, int r16, int g, f32x4 (&acc)[2][NT]) {
#pragma unroll
  for (int m = 0; m < 2; ++m)
#pragma unroll
    for (int t = 0; t < NT; ++t) acc[m][t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) {
    bf16x8 b[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t)
      b[t] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4*>(&act[(t * 16 + r16) * ST + ks * 32 + 8 * g]));
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
      for (int t = 0; t < NT; ++t) acc[m][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[m][ks], b[t], acc[m][t], 0, 0, 0);
  }
}

// h = bf16(GELU(acc + bias)) into LDS, 16 rows.
__device__ inline void tile_gelu(const f32x4 (&acc)[2][1], const float* bias, uint16_t* h, int c0, int r16, int g) {
#pragma unroll
  for (int m = 0; m < 2; ++m) {
    const float4 bv = *reinterpret_cast<const float4*>(&bias[c0 + m * 16 + 4 * g]);
    const float z[4] = {acc[m][0][0] + bv.x, acc[m][0][1] + bv.y, acc[m][0][2] + bv.z, acc[m][0][3] + bv.w};
    uint2 o;
    if (near_zero(z)) {
      o.x = pack_bf16(gelu<true>(z[0]), gelu<true>(z[1]));
      o.y = pack_bf16(gelu<true>(z[2]), gelu<true>(z[3]));
    } else {
      o.x = pack_bf16(gelu<false>(z[0]), gelu<false>(z[1]));
      o.y = pack_bf16(gelu<false>(z[2]), gelu<false>(z[3]));
    }
    *reinterpret_cast<uint2*>(&h[r16 * kHS + c0 + m * 16 + 4 * g]) = o;
  }
}

// One layer of a tile, 16 rows at a time: while one of a SIMD's two waves has the
// matrix cores the other forms its GELUs.
template <int KS, int ST, int NT>
__device__ inline void tile_layer(const bf16x8 (&w)[2][KS], const uint16_t* act, const float* bias, uint16_t* h, int c0,
                                  int r16, int g) {
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    f32x4 acc[2][1];
    tile_product<KS, ST, 1>(w, act + t * 16 * ST, r16, g, acc);
    tile_gelu(acc, bias, h + t * 16 * kHS, c0, r16, g);
  }
}

template <int KS>
__device__ inline void load_weights(bf16x8 (&w)[KS], const uint16_t* wt, int c0, int r16, int g) {
#pragma unroll
  for (int ks = 0; ks < KS; ++ks)
    w[ks] = __builtin_bit_cast(bf16x8,
                               *reinterpret_cast<const uint4*>(&wt[operand(c0 + r16, ks * 32 + 8 * g, kHid)]));
}
template <int KS>
__device__ inline void load_weights(bf16x8 (&w)[2][KS], const uint16_t* wt, int c0, int r16, int g) {
#pragma unroll
  for (int m = 0; m < 2; ++m) load_weights(w[m], wt, c0 + m * 16, r16, g);
}

template <int NT>
__global__ __launch_bounds__(64 * kPredWaves) __attribute__((amdgpu_waves_per_eu(2, 2)))
void predict_kernel(int64_t n, const uint16_t* __restrict__ X, int64_t x_rows, const int32_t* __restrict__ idx,
                    const uint16_t* __restrict__ wt1, const uint16_t* __restrict__ wt2,
                    const uint16_t* __restrict__ wt3, const float* __restrict__ b1, const float* __restrict__ b2,
                    const float* __restrict__ b3, const float* __restrict__ w4, const float* __restrict__ b4,
                    float* __restrict__ y) {
  constexpr int R = 16 * NT;                       // rows of a tile
  constexpr int T = 64 * kPredWaves;
  constexpr int CH = (R * (kFeat / 8) + T - 1) / T;  // 16-byte chunks of a tile per thread
  __shared__ __attribute__((aligned(16))) uint16_t xs[R * kXS];
  __shared__ __attribute__((aligned(16))) uint16_t hs[2][R * kHS];
  __shared__ __attribute__((aligned(16))) float bias[3][kHid];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, r16 = lane & 15, g = lane >> 4;
  const int c0 = 32 * wave;
  const int64_t tiles = (n + R - 1) / R;

  uint4 xv[CH];
  // rows past n read as zero, a gathered row outside the stored ones as NaN
  auto fetch = [&](int64_t tile) {
#pragma unroll
    for (int q = 0; q < CH; ++q) {
      const int e = tid + q * T, r = e >> 4, c = e & 15;
      const int64_t row = tile * R + r;
      uint4 v = make_uint4(0, 0, 0, 0);
      if (r < R && row < n) {
        const int64_t src = idx ? (int64_t)idx[row] : row;
        if (src >= 0 && src < x_rows) v = *reinterpret_cast<const uint4*>(X + src * kFeat + c * 8);
        else v = make_uint4(kNaN * 0x10001u, kNaN * 0x10001u, kNaN * 0x10001u, kNaN * 0x10001u);
      }
      xv[q] = v;
    }
  };
  auto stage = [&]() {
#pragma unroll
    for (int q = 0; q < CH; ++q) {
      const int e = tid + q * T, r = e >> 4, c = e & 15;
      if (r < R) *reinterpret_cast<uint4*>(&xs[r * kXS + c * 8]) = xv[q];
    }
  };

  fetch(blockIdx.x);
  bf16x8 w1[2][kFeat / 32], w2[2][kHid / 32], w3[2][kHid / 32];
  load_weights(w1, wt1, c0, r16, g);
  load_weights(w2, wt2, c0, r16, g);
  load_weights(w3, wt3, c0, r16, g);
  for (int e = tid; e < kHid; e += T) {
    bias[0][e] = b1[e];
    bias[1][e] = b2[e];
    bias[2][e] = b3[e];
  }
  const float4 wv = *reinterpret_cast<const float4*>(w4 + 4 * lane);
  const float b4v = b4[0];
  stage();
  __syncthreads();

  int cur = 0;  // buffer of the odd layers; swapped per tile, so that a tile's
                // first layer does not write what a slower wave's head still reads
  for (int64_t tile = blockIdx.x; tile < tiles; tile += gridDim.x, cur ^= 1) {
    uint16_t* ha = hs[cur];
    uint16_t* hb = hs[cur ^ 1];
    if (tile + gridDim.x < tiles) fetch(tile + gridDim.x);
    tile_layer<kFeat / 32, kXS, NT>(w1, xs, bias[0], ha, c0, r16, g);
    __syncthreads();
    if (tile + gridDim.x < tiles) stage();
    tile_layer<kHid / 32, kHS, NT>(w2, ha, bias[1], hb, c0, r16, g);
    __syncthreads();
    tile_layer<kHid / 32, kHS, NT>(w3, hb, bias[2], ha, c0, r16, g);
    __syncthreads();
    // head: one wave per row, lane l owns hidden units 4l .. 4l+3
#pragma unroll
    for (int q = 0; q < R / kPredWaves; ++q) {
      const int r = wave + q * kPredWaves;
      const uint2 hv = *reinterpret_cast<const uint2*>(&ha[r * kHS + 4 * lane]);
      const float v = wave_sum(bf2f(hv.x) * wv.x + bf2f(hv.x >> 16) * wv.y + bf2f(hv.y) * wv.z +
                                   bf2f(hv.y >> 16) * wv.w);
      const int64_t row = tile * R + r;
      if (lane == 0 && row < n) y[row] = v + b4v;
    }
  }
}

// Rows per tile: as few as still give every CU (256) at most one tile, since a
// tile's latency is what a small call waits for.  Beyond that a tile of R rows
// costs a CU about 0.11 us x (R + 6), so the size whose rounds cost least: at
// 1 M rows 48, 64 and 96 rows take 500, 487 and 472 us, at 16 000 rows 22.3,
// 18.5 and 21.7 us, at 50 000 rows 40.5, 41.6 and 44.8 us (with 5 us more for
// the weights than they now take).
hipError_t predict(int64_t n, const uint16_t* X, int64_t x_rows, const int32_t* idx, const uint16_t* wt1,
                   const uint16_t* wt2, const uint16_t* wt3, const float* b1, const float* b2, const float* b3,
                   const float* w4, const float* b4, float* y, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  constexpr int64_t kCus = 256;
  int nt = n <= 16 * kCus ? 1 : 2;
  if (n > 32 * kCus) {
    auto cost = [&](int64_t c) { return (n + 16 * c * kCus - 1) / (16 * c * kCus) * (16 * c + 6); };
    nt = 3;
    for (int c : {4, 6})
      if (cost(c) < cost(nt)) nt = c;
  }
  const int64_t tiles = (n + 16 * nt - 1) / (16 * nt);
  const dim3 grid((unsigned)(tiles < kCus ? tiles : kCus)), block(64 * kPredWaves);
#define SUR_PREDICT(NT)                                                                                              \
  case NT:                                                                                                           \
    hipLaunchKernelGGL((predict_kernel<NT>), grid, block, 0, s, n, X, x_rows, idx, wt1, wt2, wt3, b1, b2, b3, w4, b4, y); \
    break;
  switch (nt) { SUR_PREDICT(1) SUR_PREDICT(2) SUR_PREDICT(3) SUR_PREDICT(4) SUR_PREDICT(6) }
#undef SUR_PREDICT
  return hipGetLastError();
}

// ----------------------------------------------------------------------------- features
// 64 candidates per workgroup.  Every value is formed in double and rounded to
// float, then to BF16 (the same two roundings for every feature).  Bound by
// memory (304 bytes in and 256 out per candidate): controllers and rows go by
// whole lines through an LDS tile, and a thread walks five hinges of a candidate
// up to the core at once.  One thread per candidate, with its row in 128
// registers, read 240-byte rows lane by lane: 200 000 candidates 72 us, now 33 us.
constexpr int kFC = 64, kFThreads = 256;
constexpr int kFS = kFeat + 4;  // row of the tile in LDS: 8-byte aligned, two banks on from the last

// Byte-wise for four hinges: parent | face << 5 | axis << 7, and parent 31 (no
// earlier body) where parent is not 0..19, face not 0..3 or axis not 0 or 1.
__device__ inline uint32_t pack_genes(uint32_t p, uint32_t f, uint32_t a) {
  const uint32_t p_bad = ((p & 0x7f7f7f7fu) + 0x6c6c6c6cu) | p;
  const uint32_t f_bad = ((f & 0x7f7f7f7fu) + 0x7c7c7c7cu) | f;
  const uint32_t a_bad = ((a & 0x7f7f7f7fu) + 0x7e7e7e7eu) | a;
  const uint32_t bad = ((p_bad | f_bad | a_bad) >> 7) & 0x01010101u;
  return (p & 0x1f1f1f1fu) | (bad * 31u) | ((f & 0x03030303u) << 5) | ((a & 0x01010101u) << 7);
}

// Word e of a byte array, also where the array does not start at a word.
__device__ inline uint32_t gene_word(const int8_t* g, int e) {
  if (((uintptr_t)g & 3) == 0) return reinterpret_cast<const uint32_t*>(g)[e];
  uint32_t v = 0;
#pragma unroll
  for (int q = 0; q < 4; ++q) v |= (uint32_t)(uint8_t)g[4 * e + q] << (8 * q);
  return v;
}

__global__ __launch_bounds__(kFThreads) void features_kernel(int64_t n, const int32_t* __restrict__ nh,
                                                             const int8_t* __restrict__ parent,
                                                             const int8_t* __restrict__ face,
                                                             const int8_t* __restrict__ axis,
                                                             const float* __restrict__ cpg,
                                                             uint16_t* __restrict__ X) {
  constexpr int W = kMaxH / 4;  // words of a candidate's parents, faces or axes
  __shared__ __attribute__((aligned(16))) uint16_t tile[kFC * kFS];
  __shared__ uint32_t genes[kFC * W];
  // per candidate: bodies at depth 1..5 and z axes (5 bits each); faces of the
  // core, depths (from bit 5) and invalid (bit 31); bodies of the limb from each body
  __shared__ uint32_t sums[kFC], bits[kFC], limb[W + 1][kFC];
  __shared__ uint16_t by20[kMaxH + 1];
  const int tid = threadIdx.x;
  const int64_t i0 = (int64_t)blockIdx.x * kFC;
  const int rows = (int)(n - i0 < kFC ? n - i0 : kFC);
  const float* C = cpg + i0 * kMaxH * 3;
  const bool wide = ((uintptr_t)C & 15) == 0;
  if (tid < kFC) {
    sums[tid] = bits[tid] = 0;
#pragma unroll
    for (int q = 0; q <= W; ++q) limb[q][tid] = 0;
  } else if (tid <= kFC + kMaxH) {
    by20[tid - kFC] = f2bf((float)((double)(tid - kFC) / 20.0));
  }
  for (int e = tid; e < rows * W; e += kFThreads)
    genes[e] = pack_genes(gene_word(parent + i0 * kMaxH, e), gene_word(face + i0 * kMaxH, e),
                          gene_word(axis + i0 * kMaxH, e));
#pragma unroll
  for (int u = 0; u < kFC * 15 / kFThreads + 1; ++u) {
    const int e = tid + u * kFThreads;
    if (e < rows * 15) {
      const int r = e / 15, c = 4 * (e - 15 * r);
      float4 v;
      if (wide) v = reinterpret_cast<const float4*>(C)[e];
      else v = make_float4(C[4 * e], C[4 * e + 1], C[4 * e + 2], C[4 * e + 3]);
      const int h = nh[i0 + r];
      const float x[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int j = (c + q) / 3, part = c + q - 3 * j;
        const double by = part == 0 ? 1.0 : part == 1 ? 6.0 : 6.283185307179586;
        const uint16_t f = f2bf((float)((double)x[q] / by));
        tile[r * kFS + part * kMaxH + j] = j < h ? f : (uint16_t)0;
      }
    }
  }
  __syncthreads();

  const int r = tid & (kFC - 1), w = tid / kFC;
  const int h = r < rows ? nh[i0 + r] : 0;
  uint16_t* row = tile + r * kFS;
  if (r < rows) {
    const uint8_t* gene = reinterpret_cast<const uint8_t*>(genes) + r * kMaxH;
    uint32_t sum = 0, bit = h >= 1 && h <= kMaxH ? 0u : 1u << 31;
    int cur[W], d[W];
#pragma unroll
    for (int k = 0; k < W; ++k) {
      cur[k] = w + 4 * k + 1;
      d[k] = 1;
    }
    // a parent that is not an earlier body ends the walk (and the row is NaN)
    for (bool more = true; more;) {
      more = false;
#pragma unroll
      for (int k = 0; k < W; ++k) {
        const int p = gene[cur[k] - 1] & 31;
        if (p > 0 && p < cur[k]) {
          cur[k] = p;
          ++d[k];
          more = true;
        }
      }
    }
#pragma unroll
    for (int k = 0; k < W; ++k) {
      const int j = w + 4 * k;
      uint16_t ax_f = 0, d_f = 0;
      if (j < h) {
        const int gn = gene[j], p = gn & 31, fc = (gn >> 5) & 3, ax = gn >> 7;
        if (p > j) bit |= 1u << 31;
        ax_f = ax == 0 ? 0x3f80 : 0xbf80;
        d_f = f2bf(0.25f * (float)d[k]);
        sum += (d[k] <= 5 ? 1u << (5 * (d[k] - 1)) : 0u) + (ax == 0 ? 1u << 25 : 0u);
        bit |= (16u << d[k]) | (p == 0 ? 1u << fc : 0u);
        atomicAdd(&limb[cur[k] >> 2][r], 1u << (8 * (cur[k] & 3)));
      }
      row[60 + j] = ax_f;
      row[80 + j] = d_f;
    }
    atomicAdd(&sums[r], sum);
    atomicOr(&bits[r], bit);
  }
  __syncthreads();

  if (r < rows && !(bits[r] >> 31)) {
    if (w == 0) {
      const uint32_t s = sums[r], b = bits[r] >> 4;  // bit d: some body at depth d
      const int nz = s >> 25;
      row[100] = by20[h];
      row[101] = by20[nz];
      row[102] = by20[h - nz];
      row[103] = f2bf(0.25f * (float)(31 - __builtin_clz(b)));
#pragma unroll
      for (int q = 0; q < 5; ++q) row[104 + q] = by20[(s >> (5 * q)) & 31];
    } else if (w == 1) {
      uint32_t bins = 0;  // limbs of 1, 2, 3-4, 5-8 and more bodies, 5 bits each
#pragma unroll
      for (int b = 1; b <= kMaxH; ++b) {
        const int s = (limb[b >> 2][r] >> (8 * (b & 3))) & 255;
        bins += s == 0 ? 0u : 1u << (s == 1 ? 0 : s == 2 ? 5 : s <= 4 ? 10 : s <= 8 ? 15 : 20);
      }
#pragma unroll
      for (int q = 0; q < 5; ++q) row[109 + q] = f2bf(0.25f * (float)((bins >> (5 * q)) & 31));
    } else if (w == 2) {
#pragma unroll
      for (int q = 0; q < 4; ++q) row[114 + q] = (bits[r] >> q) & 1 ? 0x3f80 : 0;
#pragma unroll
      for (int q = 118; q < kFeat; ++q) row[q] = 0;
    }
  }
  __syncthreads();

  uint4* out = reinterpret_cast<uint4*>(X + i0 * kFeat);
  const uint32_t nan2 = (uint32_t)f2bf(__builtin_nanf("")) * 0x10001u;
#pragma unroll
  for (int u = 0; u < kFC * (kFeat / 8) / kFThreads; ++u) {
    const int e = tid + u * kFThreads, q = e / (kFeat / 8);
    if (q < rows) {
      const uint2* v = reinterpret_cast<const uint2*>(&tile[q * kFS + (e % (kFeat / 8)) * 8]);
      const uint2 lo = v[0], hi = v[1];
      out[e] = bits[q] >> 31 ? make_uint4(nan2, nan2, nan2, nan2) : make_uint4(lo.x, lo.y, hi.x, hi.y);
    }
  }
}

hipError_t features(int64_t n, const int32_t* nh, const int8_t* parent, const int8_t* face, const int8_t* axis,
                    const float* cpg, uint16_t* X, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  const int64_t blocks = (n + kFC - 1) / kFC;
  hipLaunchKernelGGL(features_kernel, dim3((unsigned)blocks), dim3(kFThreads), 0, s, n, nh, parent, face, axis, cpg, X);
  return hipGetLastError();
}

// ----------------------------------------------------------------------------- Adam + BF16 copies
struct Copies {
  uint16_t *wt1, *wt2, *wt3, *wb2, *wb3;
  float* w4f;
};

// wt_l(o, i) (forward operand) and wb_l(i, o) (backward operand) hold bf16(W_l[i][o]).
__device__ inline void write_copy(int i, float val, const Copies& c) {
  const uint16_t b = f2bf(val);
  if (i < kOffB1) {
    const int in = i / kHid, o = i % kHid;
    c.wt1[operand(o, in, kHid)] = b;
  } else if (i >= kOffW2 && i < kOffB2) {
    const int j = i - kOffW2, in = j / kHid, o = j % kHid;
    c.wt2[operand(o, in, kHid)] = b;
    c.wb2[operand(in, o, kHid)] = b;
  } else if (i >= kOffW3 && i < kOffB3) {
    const int j = i - kOffW3, in = j / kHid, o = j % kHid;
    c.wt3[operand(o, in, kHid)] = b;
    c.wb3[operand(in, o, kHid)] = b;
  } else if (i >= kOffW4 && i < kOffB4) {
    c.w4f[i - kOffW4] = bf2f(b);
  }
}

struct AdamArgs {
  float *p, *m, *v;
  float c1, c2, lr, b1, omb1, b2, omb2, eps;
};
// 1 - beta and the bias corrections 1 - beta^t are formed in double, then rounded once
static AdamArgs adam_args(float* p, float* m, float* v, int64_t t, double lr, double b1, double b2, double eps) {
  return AdamArgs{p, m, v, (float)(1.0 - pow(b1, (double)t)), (float)(1.0 - pow(b2, (double)t)), (float)lr,
                  (float)b1, (float)(1.0 - b1), (float)b2, (float)(1.0 - b2), (float)eps};
}
__device__ inline void adam_update(int i, float gi, const AdamArgs& a, const Copies& cp) {
  const float mi = a.b1 * a.m[i] + a.omb1 * gi;
  const float vi = a.b2 * a.v[i] + a.omb2 * gi * gi;
  const float mh = mi / a.c1, vh = vi / a.c2;
  const float pi = a.p[i] - a.lr * mh / (sqrtf(vh) + a.eps);
  a.m[i] = mi;
  a.v[i] = vi;
  a.p[i] = pi;
  write_copy(i, pi, cp);
}

__global__ __launch_bounds__(256) void adam_kernel(const float* __restrict__ g, AdamArgs a, Copies cp) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= kNParams) return;
  adam_update(i, g[i], a, cp);
}

__global__ __launch_bounds__(256) void refresh_kernel(const float* __restrict__ p, Copies cp) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= kNParams) return;
  write_copy(i, p[i], cp);
}

hipError_t adam(float* p, float* m, float* v, const float* g, int64_t t, double lr, double b1, double b2, double eps,
                uint16_t* wt1, uint16_t* wt2, uint16_t* wt3, uint16_t* wb2, uint16_t* wb3, float* w4f,
                hipStream_t s) {
  hipLaunchKernelGGL(adam_kernel, dim3((kNParams + 255) / 256), dim3(256), 0, s, g,
                     adam_args(p, m, v, t, lr, b1, b2, eps), Copies{wt1, wt2, wt3, wb2, wb3, w4f});
  return hipGetLastError();
}

hipError_t refresh_copies(const float* p, uint16_t* wt1, uint16_t* wt2, uint16_t* wt3, uint16_t* wb2,
                          uint16_t* wb3, float* w4f, hipStream_t s) {
  Copies cp{wt1, wt2, wt3, wb2, wb3, w4f};
  hipLaunchKernelGGL(refresh_kernel, dim3((kNParams + 255) / 256), dim3(256), 0, s, p, cp);
  return hipGetLastError();
}

// ----------------------------------------------------------------------------- training step
// A step is three launches: activations and their gradients of all rows, the
// weight-gradient products, the parameter update.  (Layer at a time it was
// thirteen, 175 us a batch of 4096, most of it launches and single-block sums.)
//
// Activations, features and gradients that the weight products (sums over batch
// rows) read are kept in BF16 as their operands: a column is a row, a batch row a k.

// GELU and its derivative from one erf.
template <bool SMALL>
__device__ inline void gelu_pair(float z, float* h, float* d) {
  const float e1 = 1.0f + erf_half<SMALL>(z);
  *h = 0.5f * z * e1;
  *d = 0.5f * e1 + z * expf(-0.5f * z * z) * 0.39894228040143268f;
}

// An LDS tile of 16 batch rows (stride ST) to its place in an operand of W rows.
template <int ST, int W>
__device__ inline void store_operand(const uint16_t* tile, uint16_t* __restrict__ out, int64_t row0, int tid) {
  for (int e = tid; e < 2 * W; e += 64 * kPredWaves) {
    const int c = (e >> 5) * 16 + (e & 15), r = ((e >> 4) & 1) * 8;
    uint32_t v[4];
#pragma unroll
    for (int j = 0; j < 4; ++j)
      v[j] = (uint32_t)tile[(r + 2 * j) * ST + c] | ((uint32_t)tile[(r + 2 * j + 1) * ST + c] << 16);
    *reinterpret_cast<uint4*>(out + operand(c, row0 + r, W)) = make_uint4(v[0], v[1], v[2], v[3]);
  }
}

// Forward and backward over the layers for one tile of 16 batch rows per
// workgroup, as in predict_kernel, the weights of two layers in registers at a
// time; z never leaves the registers (GELU' is formed with GELU), the gradients
// take the way back through the same LDS buffers.  Rows past the batch have zero
// features and zero gradient.  Bound by the weights' way from L2 (590 KB a
// workgroup) and the erf and exp of 768 units a row.  Six batches of 4096 (a
// launch per layer and direction before, activations through HBM): 1053 -> 180 us
// in the three launches, a batch 15 us here, 9 us in the weight gradients and
// 5 us in the update.
__global__ __launch_bounds__(64 * kPredWaves) __attribute__((amdgpu_waves_per_eu(2, 2)))
void train_rows_kernel(TrainArgs a) {
  constexpr int NT = 1, R = 16 * NT;
  constexpr int T = 64 * kPredWaves;
  __shared__ __attribute__((aligned(16))) uint16_t xs[R * kXS];
  __shared__ __attribute__((aligned(16))) uint16_t hs[2][R * kHS];
  __shared__ __attribute__((aligned(16))) float bias[3][kHid];
  __shared__ __attribute__((aligned(16))) float w4s[kHid];
  __shared__ float dys[R], ts[R];  // dL/dy and target of each row
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, r16 = lane & 15, g = lane >> 4;
  const int c0 = 32 * wave;
  const int64_t row0 = (int64_t)blockIdx.x * R;

  // Half the threads take a 16-byte piece of a row each, sixteen others the
  // targets (in the head their two dependent loads would stop every wave): first
  // the indices, then what does not wait for them, then the rows.
  static_assert(R * (kFeat / 8) <= T - R, "one piece per thread");
  const int pr = tid < R * (kFeat / 8) ? tid >> 4 : tid >= T - R ? tid - (T - R) : -1;
  const bool in = pr >= 0 && row0 + pr < a.B;
  const int64_t src = in ? a.idx[row0 + pr] : -1;
  bf16x8 wa[2][kHid / 32], wb[2][kHid / 32], w1[2][kFeat / 32];
  load_weights(w1, a.wt1, c0, r16, g);
  float bv[4] = {0.f, 0.f, 0.f, 0.f};
  if (tid < kHid) {
    bv[0] = a.p[kOffB1 + tid];
    bv[1] = a.p[kOffB2 + tid];
    bv[2] = a.p[kOffB3 + tid];
    bv[3] = a.w4[tid];
  }
  const float b4 = a.p[kOffB4];
  const bool stored = src >= 0 && src < a.x_rows;
  if (tid < R * (kFeat / 8)) {
    uint4 v = make_uint4(0, 0, 0, 0);
    if (stored) v = *reinterpret_cast<const uint4*>(a.X + src * kFeat + (tid & 15) * 8);
    else if (in) v = make_uint4(kNaN * 0x10001u, kNaN * 0x10001u, kNaN * 0x10001u, kNaN * 0x10001u);
    *reinterpret_cast<uint4*>(&xs[pr * kXS + (tid & 15) * 8]) = v;
  } else if (tid >= T - R) {
    ts[pr] = stored ? a.target[src] : __builtin_nanf("");
  }
  if (tid < kHid) {
    bias[0][tid] = bv[0];
    bias[1][tid] = bv[1];
    bias[2][tid] = bv[2];
    w4s[tid] = bv[3];
  }
  load_weights(wa, a.wt2, c0, r16, g);
  __syncthreads();

  f32x4 acc[2][NT], d1[2][NT], d2[2][NT], d3[2][NT];
  // h = bf16(GELU(acc + b)) to LDS, GELU' to d, and the next weights for w on
  // their way between: a layer's 128 KB keep the address unit busy for 2048 cycles,
  // and a wave that asked for all of its part at once would wait for that first
  auto activate = [&](const float* b, uint16_t* h, f32x4 (&d)[2][NT], bf16x8 (&w)[2][kHid / 32], const uint16_t* wt) {
#pragma unroll
    for (int m = 0; m < 2; ++m) {
      const float4 bv = *reinterpret_cast<const float4*>(&b[c0 + m * 16 + 4 * g]);
      const float bb[4] = {bv.x, bv.y, bv.z, bv.w};
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        float z[4], hv[4], dv[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) z[i] = acc[m][t][i] + bb[i];
        if (near_zero(z)) {
#pragma unroll
          for (int i = 0; i < 4; ++i) gelu_pair<true>(z[i], &hv[i], &dv[i]);
        } else {
#pragma unroll
          for (int i = 0; i < 4; ++i) gelu_pair<false>(z[i], &hv[i], &dv[i]);
        }
        d[m][t] = f32x4{dv[0], dv[1], dv[2], dv[3]};
        *reinterpret_cast<uint2*>(&h[(t * 16 + r16) * kHS + c0 + m * 16 + 4 * g]) =
            make_uint2(pack_bf16(hv[0], hv[1]), pack_bf16(hv[2], hv[3]));
      }
      __builtin_amdgcn_sched_barrier(0);
      load_weights(w[m], wt, c0 + m * 16, r16, g);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  // dz = bf16(v * GELU') to LDS
  auto put_grad = [&](const f32x4 (&v)[2][NT], const f32x4 (&d)[2][NT], uint16_t* h) {
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
      for (int t = 0; t < NT; ++t)
        *reinterpret_cast<uint2*>(&h[(t * 16 + r16) * kHS + c0 + m * 16 + 4 * g]) =
            make_uint2(pack_bf16(v[m][t][0] * d[m][t][0], v[m][t][1] * d[m][t][1]),
                       pack_bf16(v[m][t][2] * d[m][t][2], v[m][t][3] * d[m][t][3]));
  };

  store_operand<kXS, kFeat>(xs, a.XT, row0, tid);
  tile_product<kFeat / 32, kXS, NT>(w1, xs, r16, g, acc);
  activate(bias[0], hs[0], d1, wb, a.wt3);
  __syncthreads();
  store_operand<kHS, kHid>(hs[0], a.h1T, row0, tid);
  tile_product<kHid / 32, kHS, NT>(wa, hs[0], r16, g, acc);
  activate(bias[1], hs[1], d2, wa, a.wb3);
  __syncthreads();
  store_operand<kHS, kHid>(hs[1], a.h2T, row0, tid);
  tile_product<kHid / 32, kHS, NT>(wb, hs[1], r16, g, acc);
  activate(bias[2], hs[0], d3, wb, a.wb2);
  __syncthreads();
  // head: one wave per row, lane l owns hidden units 4l .. 4l+3
  {
    const float4 wv = *reinterpret_cast<const float4*>(&w4s[4 * lane]);
#pragma unroll
    for (int q = 0; q < R / kPredWaves; ++q) {
      const int r = wave + q * kPredWaves;
      const int64_t row = row0 + r;
      const uint2 hv = *reinterpret_cast<const uint2*>(&hs[0][r * kHS + 4 * lane]);
      const float s = wave_sum(bf2f(hv.x) * wv.x + bf2f(hv.x >> 16) * wv.y + bf2f(hv.y) * wv.z +
                               bf2f(hv.y >> 16) * wv.w);
      if (lane == 0) {
        float rr = 0.f, d = 0.f;
        if (row < a.B) {
          rr = (s + b4) - ts[r];
          d = 2.0f * rr / (float)a.B;
          a.r[row] = rr;
          a.dy[row] = d;
        }
        dys[r] = d;
      }
    }
  }
  store_operand<kHS, kHid>(hs[0], a.h3T, row0, tid);
  __syncthreads();
  {
    f32x4 v[2][NT];
#pragma unroll
    for (int m = 0; m < 2; ++m) {
      const float4 wv = *reinterpret_cast<const float4*>(&w4s[c0 + m * 16 + 4 * g]);
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        const float d = dys[t * 16 + r16];
        v[m][t] = f32x4{d * wv.x, d * wv.y, d * wv.z, d * wv.w};
      }
    }
    put_grad(v, d3, hs[1]);
  }
  __syncthreads();
  store_operand<kHS, kHid>(hs[1], a.d3T, row0, tid);
  tile_product<kHid / 32, kHS, NT>(wa, hs[1], r16, g, acc);
  put_grad(acc, d2, hs[0]);
  __syncthreads();
  store_operand<kHS, kHid>(hs[0], a.d2T, row0, tid);
  tile_product<kHid / 32, kHS, NT>(wb, hs[0], r16, g, acc);
  put_grad(acc, d1, hs[1]);
  __syncthreads();
  store_operand<kHS, kHid>(hs[1], a.d1T, row0, tid);
}

// Weight gradients [W_l; b_l] = [h | 1]^T dz_l over layer z of the batch rows (a
// ones row of the activation operand gives the bias gradient), 128 x 128 outputs
// per workgroup, 64 x 64 per wave straight from the operands, the
// partial sums of each layer of rows in the flat parameter layout (activations as
// the row operand: a lane's results then lie in the columns beside its neighbours',
// 16 lines a store and not 64, 1.7 us a batch of 4096 less); in the last
// workgroups the head's sums (W4, b4 and the squared residuals) over chunks of
// kHeadChunk rows, each in row order.
constexpr int kHeadCols = kHid + 2;
constexpr int kGradTiles = 4 + 4 + 2;  // workgroups per layer of rows: W3, W2 (256 x 256), W1 (128 x 256)

__global__ __launch_bounds__(256) void train_grad_kernel(TrainArgs a) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, r16 = lane & 15, g = lane >> 4;
  if ((int)blockIdx.x >= kGradTiles * a.layers) {
    // column c < 256: sum_m h3[m][c] dy[m]; c = 256: sum dy; c = 257: sum r^2
    __shared__ float dys[kHeadChunk], rs[kHeadChunk];
    const int q = blockIdx.x - kGradTiles * a.layers;
    const int m0 = q * kHeadChunk, rows = min(a.B - m0, kHeadChunk);
    if (tid < kHeadChunk) {
      dys[tid] = tid < rows ? a.dy[m0 + tid] : 0.f;
      rs[tid] = tid < rows ? a.r[m0 + tid] : 0.f;
    }
    __syncthreads();
    // 64 rows in flight: one block at a time waits on memory once per 16 rows
    float s = 0.f;
    const int last = (rows - 1) / 16 * 16;
    for (int m = 0; m < rows; m += 64) {
      uint4 hb[8];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int64_t row = m0 + min(m + 16 * u, last);
        hb[2 * u] = *reinterpret_cast<const uint4*>(a.h3T + operand(tid, row, kHid));
        hb[2 * u + 1] = *reinterpret_cast<const uint4*>(a.h3T + operand(tid, row + 8, kHid));
      }
#pragma unroll
      for (int j = 0; j < 64; ++j) {
        const uint4 hv = hb[j >> 3];
        const uint32_t hw = (j & 7) < 2 ? hv.x : (j & 7) < 4 ? hv.y : (j & 7) < 6 ? hv.z : hv.w;
        const float next = s + bf2f(hw >> (16 * (j & 1))) * dys[m + j];
        s = m + j < rows ? next : s;
      }
    }
    a.head_partial[q * kHeadCols + tid] = s;
    if (tid == 0) {  // the zeros past the last row change nothing
      float t = 0.f;
#pragma unroll 32
      for (int m = 0; m < kHeadChunk; ++m) t += dys[m];
      a.head_partial[q * kHeadCols + kHid] = t;
    } else if (tid == 64) {
      float t = 0.f;
#pragma unroll 32
      for (int m = 0; m < kHeadChunk; ++m) t += rs[m] * rs[m];
      a.head_partial[q * kHeadCols + kHid + 1] = t;
    }
    return;
  }
  const int z = blockIdx.x / kGradTiles, tile = blockIdx.x % kGradTiles;
  const int prod = tile < 4 ? 2 : tile < 8 ? 1 : 0;  // layer index: W3, W2, W1
  const int tt = tile - (prod == 2 ? 0 : prod == 1 ? 4 : 8);
  const int width = prod == 0 ? kFeat : kHid;        // columns of the activation operand
  const uint16_t* h = prod == 2 ? a.h2T : prod == 1 ? a.h1T : a.XT;
  const uint16_t* d = prod == 2 ? a.d3T : prod == 1 ? a.d2T : a.d1T;
  const int mb = tt >> 1;
  const int m0 = mb * 128 + (wave >> 1) * 64, n0 = (tt & 1) * 128 + (wave & 1) * 64;
  const bool bias_row = mb == 0 && wave < 2;
  f32x4 acc[4][4], accb[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    accb[i] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  const uint32_t one2 = r16 == 0 ? kOne * 0x10001u : 0u;
  const bf16x8 ones = __builtin_bit_cast(bf16x8, make_uint4(one2, one2, one2, one2));
  const int kbeg = z * a.kchunk, kend = min(a.B, kbeg + a.kchunk);
#pragma unroll 2
  for (int k0 = kbeg; k0 < kend; k0 += 32) {
    // rows past the batch up to the next multiple of 32 hold zero gradients
    const int64_t row = k0 + 8 * g;
    bf16x8 df[4], hf[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      df[i] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4*>(d + operand(n0 + i * 16 + r16, row, kHid)));
      hf[i] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4*>(h + operand(m0 + i * 16 + r16, row, width)));
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
#pragma unroll
      for (int j = 0; j < 4; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(hf[j], df[i], acc[i][j], 0, 0, 0);
      if (bias_row) accb[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ones, df[i], accb[i], 0, 0, 0);
    }
  }
  float* out = a.partial + (size_t)z * kOffW4 + (prod == 2 ? kOffW3 : prod == 1 ? kOffW2 : kOffW1);
#pragma unroll
  for (int i = 0; i < 4; ++i) {
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) out[(m0 + j * 16 + 4 * g + r) * kHid + n0 + i * 16 + r16] = acc[i][j][r];
    if (bias_row && g == 0) out[width * kHid + n0 + i * 16 + r16] = accb[i][0];
  }
}

// Gradient of every parameter (the layers' partial sums in layer order, the
// head's in chunk order), Adam, and the BF16 copies of the new weights.
__global__ __launch_bounds__(256) void train_update_kernel(TrainArgs a, AdamArgs ad, Copies cp) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i > kNParams) return;
  float gi = 0.f;
  if (i < kOffW4) {
    float v[kMaxSplitK];
#pragma unroll
    for (int z = 0; z < kMaxSplitK; ++z) v[z] = z < a.layers ? a.partial[(size_t)z * kOffW4 + i] : 0.f;
#pragma unroll
    for (int z = 0; z < kMaxSplitK; ++z)
      if (z < a.layers) gi += v[z];
  } else {
    const float* hp = a.head_partial + (i - kOffW4);
#pragma unroll 8
    for (int q = 0; q < a.chunks; ++q) gi += hp[q * kHeadCols];
    if (i == kNParams) {
      a.loss[0] = gi / (float)a.B;
      return;
    }
  }
  a.g[i] = gi;
  adam_update(i, gi, ad, cp);
}

hipError_t train(const TrainArgs& args, float* p, float* m, float* v, int64_t t, double lr, double b1, double b2,
                 double eps, uint16_t* wt1, uint16_t* wt2, uint16_t* wt3, uint16_t* wb2, uint16_t* wb3, float* w4f,
                 hipStream_t s) {
  TrainArgs a = args;
  // the batch (the reduction) is long and a product's output small: split it over
  // layers of at least kSplitKRows rows
  a.layers = a.B / kSplitKRows < 1 ? 1 : a.B / kSplitKRows > kMaxSplitK ? kMaxSplitK : a.B / kSplitKRows;
  a.kchunk = ((a.B + a.layers - 1) / a.layers + 31) / 32 * 32;
  a.chunks = (a.B + kHeadChunk - 1) / kHeadChunk;
  // whole 32-row steps of the products are written
  const int rows = (a.B + 31) / 32 * 32;
  hipLaunchKernelGGL(train_rows_kernel, dim3(rows / 16), dim3(64 * kPredWaves), 0, s, a);
  hipLaunchKernelGGL(train_grad_kernel, dim3(kGradTiles * a.layers + a.chunks), dim3(256), 0, s, a);
  hipLaunchKernelGGL(train_update_kernel, dim3(kNParams / 256 + 1), dim3(256), 0, s, a,
                     adam_args(p, m, v, t, lr, b1, b2, eps), Copies{wt1, wt2, wt3, wb2, wb3, w4f});
  return hipGetLastError();
}

// ----------------------------------------------------------------------------- top-k
// Order-preserving key: larger score -> larger key; NaN -> 0 (below -inf), -0 -> +0.
__device__ inline uint32_t score_key(float f) {
  uint32_t u = __float_as_uint(f);
  if ((u & 0x7fffffffu) > 0x7f800000u) return 0u;
  if (u == 0x80000000u) u = 0u;
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// A radix select over digits of 11, 11 and 10 bits finds the k-th largest key T
// (a wide first digit spreads scores of like size over many counters), then the
// scores above T and the first of those equal to it go out in index order.
// Bound by launches and, per pass, by the way to memory and back: 1 000 003
// scores 29 us; 115 us with 8-bit digits, 2048 workgroups adding to one histogram,
// a serial choice of the digit and a scan of the counts in launches of their own.
// 8 keys a thread and round: when 1 000 003 scores took 37 us, 4 and 16 keys took
// 39 and 41.
constexpr int kTkThreads = 1024, kTkWaves = kTkThreads / 64;
constexpr int kTkKeys = 8;                        // keys of a thread in one round
constexpr int kTkRound = kTkThreads * kTkKeys;
constexpr int kTkBins = kTopkHistWords / 3, kTkLast = 1024;  // bins of a pass, of the last one

// Sum of v over the threads up to and with this one; *total over all threads.
__device__ inline uint32_t thread_scan(uint32_t v, uint32_t* wave_sums, uint32_t* total) {
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const uint32_t a = __shfl_up(v, off);
    v += lane >= off ? a : 0u;
  }
  __syncthreads();
  if (lane == 63) wave_sums[wave] = v;
  __syncthreads();
  uint32_t before = 0, all = 0;
#pragma unroll
  for (int w = 0; w < kTkWaves; ++w) {
    const uint32_t c = wave_sums[w];
    before += w < wave ? c : 0u;
    all += c;
  }
  *total = all;
  return before + v;
}

// The digit of the left-th largest of the keys counted in c (this thread's bins
// from the top: 2 of kTkBins, or 1 of kTkLast) and how many remain below it.
template <int BINS>
__device__ inline void choose_digit(const uint32_t (&c)[BINS / kTkThreads], uint32_t left, uint32_t* wave_sums,
                                    uint32_t* chosen) {
  constexpr int PER = BINS / kTkThreads;
  uint32_t sum = 0, all;
#pragma unroll
  for (int q = 0; q < PER; ++q) sum += c[q];
  uint32_t above = thread_scan(sum, wave_sums, &all) - sum;
#pragma unroll
  for (int q = 0; q < PER; ++q) {
    if (above < left && left <= above + c[q]) {
      chosen[0] = BINS - 1 - (int)threadIdx.x * PER - q;
      chosen[1] = left - above;
    }
    above += c[q];
  }
  __syncthreads();
}

// Writes the indices of one round's keys (thread t: base + 1024 j + t) that are
// above T or among the first keq equal to it; rg and re count those before.
template <int K>
__device__ inline void emit(const uint32_t (&key)[K], int64_t base, int64_t n, uint32_t T, uint32_t keq, uint32_t* rg,
                            uint32_t* re, uint32_t* counts, int32_t* __restrict__ out) {
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  constexpr int PER = K * kTkWaves / 64;
  uint64_t gt[K], eq[K];
#pragma unroll
  for (int j = 0; j < K; ++j) {
    const bool in = base + j * kTkThreads + t < n;
    gt[j] = __ballot(in && key[j] > T);
    eq[j] = __ballot(in && key[j] == T);
    if (lane == 0) counts[j * kTkWaves + wave] = (uint32_t)__popcll(gt[j]) | ((uint32_t)__popcll(eq[j]) << 16);
  }
  __syncthreads();
  // exclusive sums over the waves in index order, at most 16384 of each kind
  if (wave == 0) {
    uint32_t c[PER], sum = 0;
#pragma unroll
    for (int q = 0; q < PER; ++q) {
      c[q] = counts[lane * PER + q];
      sum += c[q];
    }
    uint32_t inc = sum;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const uint32_t a = __shfl_up(inc, off);
      inc += lane >= off ? a : 0u;
    }
    if (lane == 63) counts[K * kTkWaves] = inc;
    uint32_t before = inc - sum;
#pragma unroll
    for (int q = 0; q < PER; ++q) {
      counts[lane * PER + q] = before;
      before += c[q];
    }
  }
  __syncthreads();
  const uint64_t below = ((uint64_t)1 << lane) - 1;
#pragma unroll
  for (int j = 0; j < K; ++j) {
    const uint32_t c = counts[j * kTkWaves + wave];
    const uint32_t g = *rg + (c & 0xffffu) + (uint32_t)__popcll(gt[j] & below);
    const uint32_t e = *re + (c >> 16) + (uint32_t)__popcll(eq[j] & below);
    const int32_t i = (int32_t)(base + j * kTkThreads + t);
    if ((gt[j] >> lane) & 1) out[g + (e < keq ? e : keq)] = i;
    else if (((eq[j] >> lane) & 1) && e < keq) out[g + e] = i;
  }
  const uint32_t all = counts[K * kTkWaves];
  *rg += all & 0xffffu;
  *re += all >> 16;
  __syncthreads();
}

// Up to kTkThreads * K scores: keys in registers, counters in LDS.
template <int K>
__global__ __launch_bounds__(kTkThreads) void topk_single_kernel(int64_t n, const float* __restrict__ s, uint32_t k,
                                                                 int32_t* __restrict__ out) {
  __shared__ uint32_t hist[kTkBins], counts[K * kTkWaves + 1], wave_sums[kTkWaves], chosen[2];
  const int t = threadIdx.x;
  uint32_t key[K];
#pragma unroll
  for (int j = 0; j < K; ++j) key[j] = j * kTkThreads + t < n ? score_key(s[j * kTkThreads + t]) : 0u;
  uint32_t T = 0, left = k;
#pragma unroll
  for (int pass = 0; pass < 3; ++pass) {
    const int shift = pass == 0 ? 21 : pass == 1 ? 10 : 0;
    for (int q = t; q < kTkBins; q += kTkThreads) hist[q] = 0;
    __syncthreads();
#pragma unroll
    for (int j = 0; j < K; ++j)
      if (j * kTkThreads + t < n && (pass == 0 || key[j] >> (pass == 1 ? 21 : 10) == T))
        atomicAdd(&hist[(key[j] >> shift) & (pass == 2 ? kTkLast - 1 : kTkBins - 1)], 1u);
    __syncthreads();
    if (pass < 2) {
      const uint32_t c[2] = {hist[kTkBins - 1 - 2 * t], hist[kTkBins - 2 - 2 * t]};
      choose_digit<kTkBins>(c, left, wave_sums, chosen);
      T = T << 11 | chosen[0];
    } else {
      const uint32_t c[1] = {hist[kTkLast - 1 - t]};
      choose_digit<kTkLast>(c, left, wave_sums, chosen);
      T = T << 10 | chosen[0];
    }
    left = chosen[1];
  }
  uint32_t rg = 0, re = 0;
  emit<K>(key, 0, n, T, left, &rg, &re, counts, out);
}

__global__ __launch_bounds__(kTkThreads) void topk_init_kernel(uint32_t* hist) {
  hist[blockIdx.x * kTkThreads + threadIdx.x] = 0;
}

// This thread's scores of the round at b, zero past the end.
__device__ inline void load_round(float (&x)[kTkKeys], const float* __restrict__ s, int64_t b, int64_t end) {
#pragma unroll
  for (int j = 0; j < kTkKeys; ++j) {
    const int64_t i = b + j * kTkThreads + threadIdx.x;
    x[j] = i < end ? s[i] : 0.f;
  }
}

// The key's leading bits after the first PASSES digits, and how many of the keys
// that share them are taken: every workgroup picks the last of those digits from
// the finished histogram while its scores are on their way (a pick by the workgroup
// that finishes last would wait for its counts, a ticket and the histogram in turn,
// 7 us a pass for 5); workgroup 0 leaves it for the pass after.
template <int PASSES>
__device__ inline void chosen_bits(const uint32_t* hist, uint32_t* state, uint32_t k, uint32_t* wave_sums,
                                   uint32_t* chosen, uint32_t* bits, uint32_t* left) {
  constexpr int BINS = PASSES == 3 ? kTkLast : kTkBins, PER = BINS / kTkThreads;
  const uint32_t* h = hist + (PASSES - 1) * kTkBins + BINS - 1 - threadIdx.x * PER;
  uint32_t c[PER];
#pragma unroll
  for (int q = 0; q < PER; ++q) c[q] = h[-q];
  const uint32_t before = PASSES == 1 ? 0u : state[2 * PASSES - 4], from = PASSES == 1 ? k : state[2 * PASSES - 3];
  choose_digit<BINS>(c, from, wave_sums, chosen);
  *bits = before << (PASSES == 3 ? 10 : 11) | chosen[0];
  *left = chosen[1];
  if (PASSES < 3 && blockIdx.x == 0 && threadIdx.x == 0) {
    state[2 * PASSES - 2] = *bits;
    state[2 * PASSES - 1] = *left;
  }
}

// Pass PASS over this workgroup's tile of scores: its counts join the histogram.
// The last pass also leaves, per tile and digit d, how many of its keys are
// above (bits, d); the entry before digit 0's counts those at or above (bits, 0).
template <int PASS>
__global__ __launch_bounds__(kTkThreads) void topk_pass_kernel(int64_t n, const float* __restrict__ s, uint32_t k,
                                                               int64_t tile, uint32_t* hist, uint32_t* state,
                                                               uint32_t* above) {
  constexpr int BINS = PASS == 2 ? kTkLast : kTkBins, PER = BINS / kTkThreads;
  constexpr int SHIFT = PASS == 0 ? 21 : PASS == 1 ? 10 : 0, TOP = PASS == 1 ? 21 : 10;
  __shared__ uint32_t lh[BINS], wave_sums[kTkWaves], chosen[2];
  const int t = threadIdx.x;
  const int64_t beg = blockIdx.x * tile, end = beg + tile < n ? beg + tile : n;
  float x[kTkKeys];
  load_round(x, s, beg, end);
#pragma unroll
  for (int q = 0; q < PER; ++q) lh[q * kTkThreads + t] = 0;
  uint32_t bits = 0, left = k, higher = 0;
  if constexpr (PASS > 0) chosen_bits<PASS>(hist, state, k, wave_sums, chosen, &bits, &left);
  else __syncthreads();
  for (int64_t b = beg; b < end; b += kTkRound) {
    uint32_t key[kTkKeys];
#pragma unroll
    for (int j = 0; j < kTkKeys; ++j) key[j] = score_key(x[j]);
    load_round(x, s, b + kTkRound, end);
#pragma unroll
    for (int j = 0; j < kTkKeys; ++j) {
      const bool in = b + j * kTkThreads + t < end;
      if (in && (PASS == 0 || key[j] >> TOP == bits)) atomicAdd(&lh[(key[j] >> SHIFT) & (BINS - 1)], 1u);
      if (PASS == 2) higher += in && key[j] >> TOP > bits;
    }
  }
  __syncthreads();
  uint32_t c[PER];
#pragma unroll
  for (int q = 0; q < PER; ++q) {
    const int d = BINS - 1 - t * PER - q;
    c[q] = lh[d];
    if (c[q]) atomicAdd(&hist[PASS * kTkBins + d], c[q]);
  }
  if (PASS == 2) {
    uint32_t all_higher, all;
    thread_scan(higher, wave_sums, &all_higher);
    const uint32_t upto = thread_scan(c[0], wave_sums, &all);
    uint32_t* out = above + (size_t)blockIdx.x * (kTkLast + 1);
    out[BINS - t] = all_higher + upto - c[0];  // digit BINS - 1 - t
    if (t == 0) out[0] = all_higher + all;
  }
}

__global__ __launch_bounds__(kTkThreads) void topk_write_kernel(int64_t n, const float* __restrict__ s, uint32_t k,
                                                                int64_t tile, const uint32_t* hist, uint32_t* state,
                                                                const uint32_t* __restrict__ above,
                                                                int32_t* __restrict__ out) {
  __shared__ uint32_t counts[kTkKeys * kTkWaves + 1], wave_sums[kTkWaves], chosen[2];
  const int t = threadIdx.x;
  const int64_t beg = blockIdx.x * tile, end = beg + tile < n ? beg + tile : n;
  float x[kTkKeys];
  load_round(x, s, beg, end);
  uint32_t T, keq;
  chosen_bits<3>(hist, state, k, wave_sums, chosen, &T, &keq);
  // those of the tiles before: above T, and equal to it
  uint32_t g = 0, e = 0, rg, re;
  if (t < (int)blockIdx.x) {
    const uint32_t* a = above + (size_t)t * (kTkLast + 1) + (T & (kTkLast - 1));
    g = a[1];
    e = a[0] - g;
  }
  thread_scan(g, wave_sums, &rg);
  thread_scan(e, wave_sums, &re);
  for (int64_t b = beg; b < end; b += kTkRound) {
    uint32_t key[kTkKeys];
#pragma unroll
    for (int j = 0; j < kTkKeys; ++j) key[j] = score_key(x[j]);
    load_round(x, s, b + kTkRound, end);
    emit<kTkKeys>(key, b, end, T, keq, &rg, &re, counts, out);
  }
}

hipError_t topk(int64_t n, const float* scores, int64_t k, int32_t* out, const TopkScratch& ws, hipStream_t s) {
  if (k <= 0 || n <= 0) return hipSuccess;
  // One launch for five up to 16 384 scores: there one workgroup takes 14 us and
  // the tiles 22.  With 32 keys a thread it would take 24 us for 32 768 (tiles
  // 22), and 16 instead of 10 us for 1000; the short form takes 9 us for those.
  if (n <= 16 * kTkThreads) {
    if (n <= 4 * kTkThreads)
      hipLaunchKernelGGL(topk_single_kernel<4>, dim3(1), dim3(kTkThreads), 0, s, n, scores, (uint32_t)k, out);
    else
      hipLaunchKernelGGL(topk_single_kernel<16>, dim3(1), dim3(kTkThreads), 0, s, n, scores, (uint32_t)k, out);
    return hipGetLastError();
  }
  // whole rounds, as few as at most kTopkTiles tiles allow
  const int64_t rounds = (n + kTkRound - 1) / kTkRound;
  const int64_t tile = (rounds + kTopkTiles - 1) / kTopkTiles * kTkRound;
  const dim3 grid((unsigned)((n + tile - 1) / tile)), block(kTkThreads);
  hipLaunchKernelGGL(topk_init_kernel, dim3(kTopkHistWords / kTkThreads), block, 0, s, ws.hist);
  const uint32_t kk = (uint32_t)k;
  hipLaunchKernelGGL(topk_pass_kernel<0>, grid, block, 0, s, n, scores, kk, tile, ws.hist, ws.state, ws.above);
  hipLaunchKernelGGL(topk_pass_kernel<1>, grid, block, 0, s, n, scores, kk, tile, ws.hist, ws.state, ws.above);
  hipLaunchKernelGGL(topk_pass_kernel<2>, grid, block, 0, s, n, scores, kk, tile, ws.hist, ws.state, ws.above);
  hipLaunchKernelGGL(topk_write_kernel, grid, block, 0, s, n, scores, kk, tile, ws.hist, ws.state, ws.above, out);
  return hipGetLastError();
}

// ----------------------------------------------------------------------------- top-k without allocation
// Scratch of topk_noalloc: the histogram, the state (padded to 64 words) and the
// tiles' counts of one selection.  A file-scope device array: each GPU the
// library runs on holds its own copy until the process ends; every call on a GPU
// uses that GPU's copy, so calls that overlap on one GPU race.  topk_init_kernel
// clears what must start at zero.
constexpr int64_t kTopkStaticWords = kTopkHistWords + 64 + kTopkAboveWords;
static __device__ __align__(256) uint32_t scratch[kTopkStaticWords];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
uint32_t* g_scratch_ptr[kMaxDevices] = {};
}  // namespace

// Device address of the current GPU's scratch copy, taken once per device (the
// array's name in host code is only a stand-in for the symbol).
static hipError_t static_scratch(uint32_t** out) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* ptr = nullptr;
    e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    g_scratch_ptr[dev] = static_cast<uint32_t*>(ptr);
  }
  *out = g_scratch_ptr[dev];
  return hipSuccess;
}

hipError_t topk_noalloc(int64_t n, const float* scores, int64_t k, int32_t* out, hipStream_t s) {
  if (n > kTopkStaticMax) return hipErrorInvalidValue;
  uint32_t* base = nullptr;
  const hipError_t e = static_scratch(&base);
  if (e != hipSuccess) return e;
  const TopkScratch ws{base, base + kTopkHistWords, base + kTopkHistWords + 64};
  return topk(n, scores, k, out, ws, s);
}

// ----------------------------------------------------------------------------- target standardisation
// One block: mean and (population) standard deviation accumulated in double
// in a fixed order, then z = (y - mean) / std.  stats = (mean, std).
__global__ __launch_bounds__(1024) void standardize_kernel(int64_t n, const float* __restrict__ y,
                                                           float* __restrict__ z, double* __restrict__ stats) {
  __shared__ double sh[1024];
  const int t = threadIdx.x;
  double s = 0.0;
  for (int64_t i = t; i < n; i += 1024) s += (double)y[i];
  sh[t] = s;
  __syncthreads();
  for (int off = 512; off > 0; off >>= 1) {
    if (t < off) sh[t] += sh[t + off];
    __syncthreads();
  }
  const double mean = sh[0] / (double)n;
  __syncthreads();
  double q = 0.0;
  for (int64_t i = t; i < n; i += 1024) {
    const double d = (double)y[i] - mean;
    q += d * d;
  }
  sh[t] = q;
  __syncthreads();
  for (int off = 512; off > 0; off >>= 1) {
    if (t < off) sh[t] += sh[t + off];
    __syncthreads();
  }
  const double sd = sqrt(sh[0] / (double)n);
  const double inv = sd > 0.0 ? 1.0 / sd : 1.0;
  for (int64_t i = t; i < n; i += 1024) z[i] = (float)(((double)y[i] - mean) * inv);
  if (t == 0) {
    stats[0] = mean;
    stats[1] = sd;
  }
}

hipError_t standardize(int64_t n, const float* y, float* z, double* stats, hipStream_t s) {
  hipLaunchKernelGGL(standardize_kernel, dim3(1), dim3(1024), 0, s, n, y, z, stats);
  return hipGetLastError();
}

}  // namespace surk
