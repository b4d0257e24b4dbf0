// Pieces of TIP scoring (paper Sec. 4.1) shared by the scoring kernel and the one-launch decode step.
#pragma once

#include "fasa_device.h"

namespace fasa {

template <typename ET> struct ScoreTraits;
template <> struct ScoreTraits<uint16_t> { static constexpr int TPT = 4; };  // tokens per 16-byte load
template <> struct ScoreTraits<float> { static constexpr int TPT = 2; };

template <typename ET>
__device__ __forceinline__ void fma_pairs(const uint4& w, float qlo, float qhi, float* acc);

template <>
__device__ __forceinline__ void fma_pairs<uint16_t>(const uint4& w, float qlo, float qhi, float* acc) {
  acc[0] = fmaf(qhi, bf16_hi(w.x), fmaf(qlo, bf16_lo(w.x), acc[0]));
  acc[1] = fmaf(qhi, bf16_hi(w.y), fmaf(qlo, bf16_lo(w.y), acc[1]));
  acc[2] = fmaf(qhi, bf16_hi(w.z), fmaf(qlo, bf16_lo(w.z), acc[2]));
  acc[3] = fmaf(qhi, bf16_hi(w.w), fmaf(qlo, bf16_lo(w.w), acc[3]));
}

template <>
__device__ __forceinline__ void fma_pairs<float>(const uint4& w, float qlo, float qhi, float* acc) {
  acc[0] = fmaf(qhi, __uint_as_float(w.y), fmaf(qlo, __uint_as_float(w.x), acc[0]));
  acc[1] = fmaf(qhi, __uint_as_float(w.w), fmaf(qlo, __uint_as_float(w.z), acc[1]));
}

// Sample of a row's scores from which a cut is taken that few scores besides the B best reach: of m (kSample)
// evenly spaced scores the sample_rank-th best, 3.5 standard deviations (and three) above the B m / N of them
// that are expected among the B best.  In one row of a few thousand the cut still comes out too high;
// whoever uses it checks that B scores reach it and otherwise looks at all of them.
constexpr int kSample = 128;
__host__ __device__ __forceinline__ int sample_rank(int bsel, int n, int m = kSample) {
  const float ps = (float)bsel * ((float)m / (float)n);
  return (int)(ps + 3.5f * sqrtf(ps) + 3.0f);
}

}  // namespace fasa
