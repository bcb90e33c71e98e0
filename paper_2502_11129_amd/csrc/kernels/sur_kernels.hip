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

__device__ inline float gelu(float z) { return 0.5f * z * (1.0f + erff(z * 0.70710678118654752f)); }

constexpr uint16_t kOne = 0x3F80;
constexpr uint16_t kNaN = 0x7FC0;

// ----------------------------------------------------------------------------- whole-network prediction
// The four layers of one tile of 16 NT rows without leaving the CU.  A
// workgroup's eight waves (two per SIMD) hold the three weight matrices in
// their registers, 32 output columns each (160 registers), and walk over tiles;
// activations go from layer to layer through LDS in BF16.  The products run
// with the weights as the row operand, so a lane's four results are four
// consecutive columns of one row and go to LDS as eight bytes.
// 1 M rows: 600 us, 550 TFLOP/s; layer at a time, with the activations (1.5 KB a
// row) through HBM, 1816 us.  10 007 rows: 17 us, 39 in four launches.  What bounds
// it is the exact erf of 768 GELUs a row (20 to 46 VALU instructions each, by the
// size of the argument), then the matrix cores.
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

// h = bf16(GELU(acc + bias)) into LDS.
template <int NT>
__device__ inline void tile_gelu(const f32x4 (&acc)[2][NT], const float* bias, uint16_t* h, int c0, int r16, int g) {
#pragma unroll
  for (int m = 0; m < 2; ++m) {
    const float4 bv = *reinterpret_cast<const float4*>(&bias[c0 + m * 16 + 4 * g]);
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      uint2 o;
      o.x = pack_bf16(gelu(acc[m][t][0] + bv.x), gelu(acc[m][t][1] + bv.y));
      o.y = pack_bf16(gelu(acc[m][t][2] + bv.z), gelu(acc[m][t][3] + bv.w));
      *reinterpret_cast<uint2*>(&h[(t * 16 + r16) * kHS + c0 + m * 16 + 4 * g]) = o;
    }
  }
}

template <int KS>
__device__ inline void load_weights(bf16x8 (&w)[2][KS], const uint16_t* wt, int c0, int r16, int g) {
#pragma unroll
  for (int m = 0; m < 2; ++m)
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
      w[m][ks] = __builtin_bit_cast(
          bf16x8, *reinterpret_cast<const uint4*>(&wt[(c0 + m * 16 + r16) * (32 * KS) + ks * 32 + 8 * g]));
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
    f32x4 acc[2][NT];
    tile_product<kFeat / 32, kXS, NT>(w1, xs, r16, g, acc);
    tile_gelu<NT>(acc, bias[0], ha, c0, r16, g);
    __syncthreads();
    if (tile + gridDim.x < tiles) stage();
    tile_product<kHid / 32, kHS, NT>(w2, ha, r16, g, acc);
    tile_gelu<NT>(acc, bias[1], hb, c0, r16, g);
    __syncthreads();
    tile_product<kHid / 32, kHS, NT>(w3, hb, r16, g, acc);
    tile_gelu<NT>(acc, bias[2], ha, c0, r16, g);
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
// tile's latency is what a small call waits for; 48 beyond that (64 rows would
// spill 15 of the 256 registers).
hipError_t predict(int64_t n, const uint16_t* X, int64_t x_rows, const int32_t* idx, const uint16_t* wt1,
                   const uint16_t* wt2, const uint16_t* wt3, const float* b1, const float* b2, const float* b3,
                   const float* w4, const float* b4, float* y, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  constexpr int64_t kCus = 256;
  const int nt = n <= 16 * kCus ? 1 : n <= 32 * kCus ? 2 : 3;
  const int64_t tiles = (n + 16 * nt - 1) / (16 * nt);
  const dim3 grid((unsigned)(tiles < kCus ? tiles : kCus)), block(64 * kPredWaves);
#define SUR_PREDICT(NT)                                                                                              \
  case NT:                                                                                                           \
    hipLaunchKernelGGL((predict_kernel<NT>), grid, block, 0, s, n, X, x_rows, idx, wt1, wt2, wt3, b1, b2, b3, w4, b4, y); \
    break;
  switch (nt) { SUR_PREDICT(1) SUR_PREDICT(2) SUR_PREDICT(3) }
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

// wt_l[o][i] (forward operand) and wb_l[i][o] (backward operand) hold bf16(W_l[i][o]).
__device__ inline void write_copy(int i, float val, const Copies& c) {
  const uint16_t b = f2bf(val);
  if (i < kOffB1) {
    const int in = i / kHid, o = i % kHid;
    c.wt1[o * kFeat + in] = b;
  } else if (i >= kOffW2 && i < kOffB2) {
    const int j = i - kOffW2, in = j / kHid, o = j % kHid;
    c.wt2[o * kHid + in] = b;
    c.wb2[j] = b;
  } else if (i >= kOffW3 && i < kOffB3) {
    const int j = i - kOffW3, in = j / kHid, o = j % kHid;
    c.wt3[o * kHid + in] = b;
    c.wb3[j] = b;
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
// Activations, features and gradients that the weight products read are kept
// in BF16 blocks of 16 rows, transposed: element (row, col) of a matrix of W
// columns at ((row / 16) W + col) 16 + row % 16.  The products sum over rows, so
// this is the order in which a lane wants its eight operands, and both sides
// move whole lines.
__device__ inline int64_t blk16(int64_t row, int col, int width) {
  return ((row >> 4) * width + col) * 16 + (row & 15);
}

// GELU and its derivative from one erf.
__device__ inline void gelu_pair(float z, float* h, float* d) {
  const float e1 = 1.0f + erff(z * 0.70710678118654752f);
  *h = 0.5f * z * e1;
  *d = 0.5f * e1 + z * expf(-0.5f * z * z) * 0.39894228040143268f;
}

// An LDS tile of R rows (stride ST) to its transposed blocks at row0.
template <int R, int ST, int W>
__device__ inline void store_blocks(const uint16_t* tile, uint16_t* __restrict__ out, int64_t row0, int tid) {
  for (int e = tid; e < W * (R / 8); e += 64 * kPredWaves) {
    const int c = e % W, r = (e / W) * 8;
    uint32_t v[4];
#pragma unroll
    for (int j = 0; j < 4; ++j)
      v[j] = (uint32_t)tile[(r + 2 * j) * ST + c] | ((uint32_t)tile[(r + 2 * j + 1) * ST + c] << 16);
    *reinterpret_cast<uint4*>(out + blk16(row0 + r, c, W)) = make_uint4(v[0], v[1], v[2], v[3]);
  }
}

// Forward and backward over the layers for one tile of 16 batch rows per
// workgroup, as in predict_kernel, the weights of two layers in registers at a
// time; z never leaves the registers (GELU' is formed with GELU), the gradients
// take the way back through the same LDS buffers.  Rows past the batch have zero
// features and zero gradient.  Bound by the weights' way from L2 (590 KB a
// workgroup) and the erf and exp of 768 units a row.  Six batches of 4096 (a
// launch per layer and direction before, activations through HBM): 1053 -> 243 us
// in the three launches, a batch 25 us here, 10 us in the weight gradients and
// 6 us in the update.
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

  for (int e = tid; e < R * (kFeat / 8); e += T) {
    const int r = e >> 4, c = e & 15;
    const int64_t row = row0 + r;
    uint4 v = make_uint4(0, 0, 0, 0);
    if (row < a.B) {
      const int64_t src = a.idx[row];
      if (src >= 0 && src < a.x_rows) v = *reinterpret_cast<const uint4*>(a.X + src * kFeat + c * 8);
      else v = make_uint4(kNaN * 0x10001u, kNaN * 0x10001u, kNaN * 0x10001u, kNaN * 0x10001u);
    }
    *reinterpret_cast<uint4*>(&xs[r * kXS + c * 8]) = v;
  }
  // the targets now: in the head their two dependent loads would stop every wave
  if (tid >= T - R && row0 + tid - (T - R) < a.B) {
    const int64_t ti = a.idx[row0 + tid - (T - R)];
    ts[tid - (T - R)] = (ti >= 0 && ti < a.x_rows) ? a.target[ti] : __builtin_nanf("");
  }
  for (int e = tid; e < kHid; e += T) {
    bias[0][e] = a.p[kOffB1 + e];
    bias[1][e] = a.p[kOffB2 + e];
    bias[2][e] = a.p[kOffB3 + e];
    w4s[e] = a.w4[e];
  }
  bf16x8 wa[2][kHid / 32], wb[2][kHid / 32], w1[2][kFeat / 32];
  load_weights(w1, a.wt1, c0, r16, g);
  load_weights(wa, a.wt2, c0, r16, g);
  const float b4 = a.p[kOffB4];
  __syncthreads();

  f32x4 acc[2][NT], d1[2][NT], d2[2][NT], d3[2][NT];
  // h = bf16(GELU(acc + b)) to LDS, GELU' to d
  auto activate = [&](const float* b, uint16_t* h, f32x4 (&d)[2][NT]) {
#pragma unroll
    for (int m = 0; m < 2; ++m) {
      const float4 bv = *reinterpret_cast<const float4*>(&b[c0 + m * 16 + 4 * g]);
      const float bb[4] = {bv.x, bv.y, bv.z, bv.w};
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        float hv[4], dv[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          gelu_pair(acc[m][t][i] + bb[i], &hv[i], &dv[i]);
          d[m][t][i] = dv[i];
        }
        *reinterpret_cast<uint2*>(&h[(t * 16 + r16) * kHS + c0 + m * 16 + 4 * g]) =
            make_uint2(pack_bf16(hv[0], hv[1]), pack_bf16(hv[2], hv[3]));
      }
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

  store_blocks<R, kXS, kFeat>(xs, a.XT, row0, tid);
  tile_product<kFeat / 32, kXS, NT>(w1, xs, r16, g, acc);
  load_weights(wb, a.wt3, c0, r16, g);
  activate(bias[0], hs[0], d1);
  __syncthreads();
  store_blocks<R, kHS, kHid>(hs[0], a.h1T, row0, tid);
  tile_product<kHid / 32, kHS, NT>(wa, hs[0], r16, g, acc);
  load_weights(wa, a.wb3, c0, r16, g);
  activate(bias[1], hs[1], d2);
  __syncthreads();
  store_blocks<R, kHS, kHid>(hs[1], a.h2T, row0, tid);
  tile_product<kHid / 32, kHS, NT>(wb, hs[1], r16, g, acc);
  load_weights(wb, a.wb2, c0, r16, g);
  activate(bias[2], hs[0], d3);
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
  store_blocks<R, kHS, kHid>(hs[0], a.h3T, row0, tid);
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
  store_blocks<R, kHS, kHid>(hs[1], a.d3T, row0, tid);
  tile_product<kHid / 32, kHS, NT>(wa, hs[1], r16, g, acc);
  put_grad(acc, d2, hs[0]);
  __syncthreads();
  store_blocks<R, kHS, kHid>(hs[0], a.d2T, row0, tid);
  tile_product<kHid / 32, kHS, NT>(wb, hs[0], r16, g, acc);
  put_grad(acc, d1, hs[1]);
  __syncthreads();
  store_blocks<R, kHS, kHid>(hs[1], a.d1T, row0, tid);
}

// Weight gradients [W_l; b_l] = [h | 1]^T dz_l over layer z of the batch rows (a
// ones row of the activation operand gives the bias gradient), 128 x 128 outputs
// per workgroup, 64 x 64 per wave straight from the transposed blocks, the
// partial sums of each layer of rows in the flat parameter layout; in the last
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
        const uint4* hp = reinterpret_cast<const uint4*>(a.h3T + blk16(m0 + min(m + 16 * u, last), tid, kHid));
        hb[2 * u] = hp[0];
        hb[2 * u + 1] = hp[1];
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
      df[i] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4*>(d + blk16(row, n0 + i * 16 + r16, kHid)));
      hf[i] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4*>(h + blk16(row, m0 + i * 16 + r16, width)));
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
#pragma unroll
      for (int j = 0; j < 4; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(df[i], hf[j], acc[i][j], 0, 0, 0);
      if (bias_row) accb[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(df[i], ones, accb[i], 0, 0, 0);
    }
  }
  float* out = a.partial + (size_t)z * kOffW4 + (prod == 2 ? kOffW3 : prod == 1 ? kOffW2 : kOffW1);
#pragma unroll
  for (int i = 0; i < 4; ++i) {
#pragma unroll
    for (int j = 0; j < 4; ++j)
      *reinterpret_cast<f32x4*>(&out[(m0 + j * 16 + r16) * kHid + n0 + i * 16 + 4 * g]) = acc[i][j];
    if (bias_row && r16 == 0) *reinterpret_cast<f32x4*>(&out[width * kHid + n0 + i * 16 + 4 * g]) = accb[i];
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

__global__ __launch_bounds__(256) void topk_init_kernel(uint32_t* hist, uint32_t* state, uint32_t k) {
  hist[threadIdx.x] = 0;
  if (threadIdx.x < 4) state[threadIdx.x] = threadIdx.x == 2 ? k : 0u;
}

__global__ __launch_bounds__(256) void topk_hist_kernel(int64_t n, const float* __restrict__ s,
                                                        const uint32_t* __restrict__ state, uint32_t* hist,
                                                        int shift) {
  __shared__ uint32_t lh[256];
  const int t = threadIdx.x;
  lh[t] = 0;
  __syncthreads();
  const uint32_t prefix = state[0], mask = state[1];
  for (int64_t i = (int64_t)blockIdx.x * 256 + t; i < n; i += (int64_t)gridDim.x * 256) {
    const uint32_t k = score_key(s[i]);
    if ((k & mask) == prefix) atomicAdd(&lh[(k >> shift) & 255u], 1u);
  }
  __syncthreads();
  if (lh[t]) atomicAdd(&hist[t], lh[t]);
}

// Pick the digit of the k-th largest key among those matching the prefix.
__global__ __launch_bounds__(256) void topk_select_kernel(uint32_t* hist, uint32_t* state, int shift) {
  __shared__ uint32_t c[256];
  const int t = threadIdx.x;
  c[t] = hist[t];
  hist[t] = 0;
  __syncthreads();
  if (t == 0) {
    const uint32_t kleft = state[2];
    uint32_t above = 0;
    int d = 255;
    for (; d > 0; --d) {
      if (above + c[d] >= kleft) break;
      above += c[d];
    }
    state[0] = state[0] | ((uint32_t)d << shift);
    state[1] = state[1] | (255u << shift);
    state[2] = kleft - above;
  }
}

// Inclusive scan of one value per thread over a 256-thread block.
__device__ inline uint32_t block_scan(uint32_t v, uint32_t* sh) {
  const int t = threadIdx.x;
  sh[t] = v;
  __syncthreads();
  for (int off = 1; off < 256; off <<= 1) {
    const uint32_t a = t >= off ? sh[t - off] : 0u;
    __syncthreads();
    sh[t] += a;
    __syncthreads();
  }
  const uint32_t r = sh[t];
  __syncthreads();
  return r;
}

// Per block of kTopkBlock scores: (#key > T, #key == T), packed as gt << 16 | eq.
__global__ __launch_bounds__(256) void topk_count_kernel(int64_t n, const float* __restrict__ s,
                                                         const uint32_t* __restrict__ state, uint32_t* blocks) {
  __shared__ uint32_t sh[256];
  const uint32_t T = state[0];
  const int64_t base = (int64_t)blockIdx.x * kTopkBlock + 4 * threadIdx.x;
  uint32_t gt = 0, eq = 0;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    if (base + j < n) {
      const uint32_t k = score_key(s[base + j]);
      gt += k > T;
      eq += k == T;
    }
  }
  const uint32_t tot = block_scan((gt << 16) | eq, sh);
  if (threadIdx.x == 255) blocks[blockIdx.x] = tot;
}

// Exclusive prefix over blocks of the greater and equal counts (one block).
__global__ __launch_bounds__(256) void topk_scan_kernel(int64_t nb, uint32_t* blocks, uint32_t* pre) {
  __shared__ uint32_t sh[256];
  __shared__ uint32_t carry_gt, carry_eq;
  const int t = threadIdx.x;
  if (t == 0) carry_gt = carry_eq = 0;
  __syncthreads();
  for (int64_t b0 = 0; b0 < nb; b0 += 256) {
    const int64_t b = b0 + t;
    const uint32_t v = b < nb ? blocks[b] : 0u;
    const uint32_t gt_in = block_scan(v >> 16, sh);
    const uint32_t eq_in = block_scan(v & 0xffffu, sh);
    const uint32_t cg = carry_gt, ce = carry_eq;
    if (b < nb) {
      pre[2 * b] = cg + gt_in - (v >> 16);
      pre[2 * b + 1] = ce + eq_in - (v & 0xffffu);
    }
    __syncthreads();
    if (t == 255) {
      carry_gt = cg + gt_in;
      carry_eq = ce + eq_in;
    }
    __syncthreads();
  }
}

__global__ __launch_bounds__(256) void topk_write_kernel(int64_t n, const float* __restrict__ s,
                                                         const uint32_t* __restrict__ state,
                                                         const uint32_t* __restrict__ pre, int32_t* __restrict__ out) {
  __shared__ uint32_t sh[256];
  const uint32_t T = state[0], keq = state[2];
  const int64_t base = (int64_t)blockIdx.x * kTopkBlock + 4 * threadIdx.x;
  uint32_t key[4];
  uint32_t gt = 0, eq = 0;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    key[j] = base + j < n ? score_key(s[base + j]) : 0u;
    const bool in = base + j < n;
    gt += in && key[j] > T;
    eq += in && key[j] == T;
  }
  const uint32_t inc = block_scan((gt << 16) | eq, sh);
  uint32_t rg = pre[2 * blockIdx.x] + (inc >> 16) - gt;
  uint32_t re = pre[2 * blockIdx.x + 1] + (inc & 0xffffu) - eq;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    if (base + j >= n) break;
    if (key[j] > T) {
      out[rg + (re < keq ? re : keq)] = (int32_t)(base + j);
      ++rg;
    } else if (key[j] == T) {
      if (re < keq) out[rg + re] = (int32_t)(base + j);
      ++re;
    }
  }
}

hipError_t topk(int64_t n, const float* scores, int64_t k, int32_t* out, const TopkScratch& ws, hipStream_t s) {
  if (k <= 0 || n <= 0) return hipSuccess;
  hipLaunchKernelGGL(topk_init_kernel, dim3(1), dim3(256), 0, s, ws.hist, ws.state, (uint32_t)k);
  const int64_t hb = (n + 255) / 256;
  const unsigned hist_blocks = (unsigned)(hb < 2048 ? hb : 2048);
  for (int pass = 0; pass < 4; ++pass) {
    const int shift = 24 - 8 * pass;
    hipLaunchKernelGGL(topk_hist_kernel, dim3(hist_blocks), dim3(256), 0, s, n, scores, ws.state, ws.hist, shift);
    hipLaunchKernelGGL(topk_select_kernel, dim3(1), dim3(256), 0, s, ws.hist, ws.state, shift);
  }
  const int64_t nb = (n + kTopkBlock - 1) / kTopkBlock;
  uint32_t* counts = ws.blocks;
  uint32_t* pre = ws.blocks + nb;
  hipLaunchKernelGGL(topk_count_kernel, dim3((unsigned)nb), dim3(256), 0, s, n, scores, ws.state, counts);
  hipLaunchKernelGGL(topk_scan_kernel, dim3(1), dim3(256), 0, s, nb, counts, pre);
  hipLaunchKernelGGL(topk_write_kernel, dim3((unsigned)nb), dim3(256), 0, s, n, scores, ws.state, pre, out);
  return hipGetLastError();
}

// ----------------------------------------------------------------------------- top-k without allocation
// Scratch of topk_noalloc: the histogram (256 words), the state (4 words, padded
// to 64) and the per-block counts and prefixes (3 words per kTopkBlock scores)
// of one selection over at most kTopkStaticMax scores.  A file-scope device
// array: each GPU the library runs on holds its own copy until the process
// ends; every call on a GPU uses that GPU's copy, so calls that overlap on one
// GPU race.  topk_init_kernel clears what must start at zero.
constexpr int64_t kTopkStaticWords = 256 + 64 + 3 * (kTopkStaticMax / kTopkBlock);
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
  const TopkScratch ws{base, base + 256, base + 256 + 64};
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
