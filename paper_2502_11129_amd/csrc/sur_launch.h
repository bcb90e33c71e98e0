// Launchers of the surrogate kernels (defined in kernels/sur_kernels.hip).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace surk {

constexpr int kFeat = 128;
constexpr int kHid = 256;
constexpr int kMaxH = 20;
constexpr int kNParams = 164865;
// offsets of the flat parameter vector
constexpr int kOffW1 = 0;
constexpr int kOffB1 = kOffW1 + kFeat * kHid;
constexpr int kOffW2 = kOffB1 + kHid;
constexpr int kOffB2 = kOffW2 + kHid * kHid;
constexpr int kOffW3 = kOffB2 + kHid;
constexpr int kOffB3 = kOffW3 + kHid * kHid;
constexpr int kOffW4 = kOffB3 + kHid;
constexpr int kOffB4 = kOffW4 + kHid;
static_assert(kOffB4 + 1 == kNParams, "parameter layout");

// Rows of the head reduction handled per block.
constexpr int kHeadChunk = 128;
// Tiles of scores in a top-k selection, at most.
constexpr int kTopkTiles = 256;
constexpr int kTopkHistWords = 3 * 2048;  // a histogram per pass
constexpr int kTopkAboveWords = kTopkTiles * 1025;

// Layers of batch rows a weight-gradient product is split over, and rows per layer at least.
constexpr int kMaxSplitK = 16;
constexpr int kSplitKRows = 256;

// One training step: B batch rows, row i at X[idx[i]] (x_rows stored rows, other
// indices read as NaN) with target[idx[i]].
struct TrainArgs {
  int B;
  int64_t x_rows;
  const uint16_t* X;
  const int32_t* idx;
  const float* target;
  // parameters and BF16 weights, in the order their products load them
  const float *p, *w4;
  const uint16_t *wt1, *wt2, *wt3, *wb2, *wb3;
  // workspace: residual and dL/dy per row; features, activations and their
  // gradients as operands of the weight products (train_block_words); partial sums
  float *r, *dy;
  uint16_t *XT, *h1T, *h2T, *h3T, *d1T, *d2T, *d3T;
  float *partial, *head_partial;
  // results: gradient of every parameter, mean squared residual
  float *g, *loss;
  // set by train(): layers of rows of the weight products, rows per layer, head chunks
  int layers, kchunk, chunks;
};
// 16-bit words of a width-column matrix of R batch rows as an operand.
constexpr int64_t train_block_words(int64_t R, int width) { return (R + 31) / 32 * 32 * width; }

hipError_t train(const TrainArgs& a, float* p, float* m, float* v, int64_t t, double lr, double b1, double b2,
                 double eps, uint16_t* wt1, uint16_t* wt2, uint16_t* wt3, uint16_t* wb2, uint16_t* wb3, float* w4f,
                 hipStream_t s);

// Predictions of n rows of X (x_rows stored rows; idx: optional gather, an index
// outside gives NaN) in one launch: y = head(GELU layers), weights wt_l[out][in].
hipError_t predict(int64_t n, const uint16_t* X, int64_t x_rows, const int32_t* idx, const uint16_t* wt1,
                   const uint16_t* wt2, const uint16_t* wt3, const float* b1, const float* b2, const float* b3,
                   const float* w4, const float* b4, float* y, hipStream_t s);

hipError_t features(int64_t n, const int32_t* nh, const int8_t* parent, const int8_t* face, const int8_t* axis,
                    const float* cpg, uint16_t* X, hipStream_t s);

hipError_t adam(float* p, float* m, float* v, const float* g, int64_t t, double lr, double b1, double b2, double eps,
                uint16_t* wt1, uint16_t* wt2, uint16_t* wt3, uint16_t* wb2, uint16_t* wb3, float* w4f,
                hipStream_t s);
// Refresh the BF16 weight copies from the masters (after an upload).
hipError_t refresh_copies(const float* p, uint16_t* wt1, uint16_t* wt2, uint16_t* wt3, uint16_t* wb2,
                          uint16_t* wb3, float* w4f, hipStream_t s);

// Top-k: radix select of the threshold key, then an index-ordered compaction.
struct TopkScratch {
  uint32_t* hist;   // [kTopkHistWords]
  uint32_t* state;  // [4]: after the first and the second digit, key bits and how many keys with them are taken
  uint32_t* above;  // [kTopkAboveWords]: per tile and last digit, keys above
};
hipError_t topk(int64_t n, const float* scores, int64_t k, int32_t* out, const TopkScratch& ws, hipStream_t s);
// The same selection with its scratch in a static device array of the library
// (no allocation, no workspace argument); n <= kTopkStaticMax, the limit of the
// C call (the scratch is enough for any n).
constexpr int64_t kTopkStaticMax = int64_t(1) << 24;
hipError_t topk_noalloc(int64_t n, const float* scores, int64_t k, int32_t* out, hipStream_t s);

// z = (y - mean) / std over n values (std of the population; 1 when zero); stats = (mean, std).
hipError_t standardize(int64_t n, const float* y, float* z, double* stats, hipStream_t s);

}  // namespace surk
