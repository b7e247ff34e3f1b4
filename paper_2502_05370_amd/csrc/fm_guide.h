// Guiding probabilities of a query's matched map(s), shared by the
// selection (Section 4.3, Eq. 6-8) and the priority ordering (Section 4.5):
// the best match's stored row, or the similarity-weighted mean of the rows of
// the k matches (weights max(score, 0), the plain mean if all are 0), summed
// in match order with explicit float64 roundings.
#pragma once

#include "fm_device.h"
#include "fm_internal.h"

namespace fm {

struct GuideView {
  const void* planes;
  int64_t plane_elems;
  int32_t n, row;
  fm_dtype dtype;
};

// (a float32, or a bf16 widened: exact in float32)
__device__ __forceinline__ float stored_prob(const GuideView& v, int y, int l, int j) {
  const int64_t off = static_cast<int64_t>(l) * v.plane_elems + tile_offset(y, j, v.row);
  if (v.dtype == FM_F32) return static_cast<const float*>(v.planes)[off];
  return bf16_to_f32(static_cast<const uint16_t*>(v.planes)[off]);
}

// The k matches of one query in ranking order (-1: none, or past the store).
struct Matches {
  int32_t y[kMaxK];
  float score[kMaxK];
};
__device__ __forceinline__ Matches load_matches(int32_t n, const int32_t* idx_b, const float* score_b, int k) {
  Matches m;
#pragma unroll
  for (int i = 0; i < kMaxK; ++i) {
    m.y[i] = i < k ? idx_b[i] : -1;
    m.score[i] = i < k ? score_b[i] : 0.0f;
    if (m.y[i] >= n) m.y[i] = -1;
  }
  return m;
}

// Blended p of expert j at layer l for one query from its matches (-1 entries
// are skipped, y[0] is none of them).  The rows of all matches load together:
// one after the other in the sum's order, each waited for the one before (top-8
// rows of 100 queries, merge and selection 13.7 -> 10.0 us; the blended
// selection of 512 x 24 rows of 60 experts 24.6 -> 21.9 us).
__device__ __forceinline__ double blended_prob(const GuideView& v, const Matches& m, int l, int j) {
  float p[kMaxK];
#pragma unroll
  for (int i = 0; i < kMaxK; ++i) p[i] = m.y[i] >= 0 ? stored_prob(v, m.y[i], l, j) : 0.0f;
  bool any_pos = false;
#pragma unroll
  for (int i = 0; i < kMaxK; ++i) any_pos = any_pos || (m.y[i] >= 0 && m.score[i] > 0.0f);
  double num = 0.0, den = 0.0;
#pragma unroll
  for (int i = 0; i < kMaxK; ++i) {
    if (m.y[i] < 0) continue;
    const double s = static_cast<double>(m.score[i]);
    const double wgt = any_pos ? (s > 0.0 ? s : 0.0) : 1.0;
    num = __dadd_rn(num, __dmul_rn(wgt, static_cast<double>(p[i])));
    den = __dadd_rn(den, wgt);
  }
  return __ddiv_rn(num, den);
}

}  // namespace fm
