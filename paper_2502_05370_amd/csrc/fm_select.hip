// Similarity-aware prefetch-set selection (Section 4.3, Eq. 6-8).
//
// One lane per expert; a wavefront holds 64 / SW rows of (query, layer), SW
// the power of two from 8 to 64 that holds the E experts (8 rows for E = 8,
// one for E = 60: a row of its own per wavefront left 56 of 64 lanes idle at
// E = 8).
//   1. Guiding probabilities: the matched map's row (float64 widening of the
//      stored value), or the similarity-weighted mean of the kept matches'
//      rows, summed in match order with explicit float64 roundings.
//   2. Threshold: fixed tau, or delta = Clip(1 - score, 0, 1).
//   3. Rank of an expert = experts ahead of it in (probability descending,
//      index ascending) order; NaN probabilities rank last.  The rank is
//      counted against the row's keys read from LDS, two instructions per
//      key (rank_row below): the kernel is bound by vector instructions.
//   4. The running sum over that order is taken sequentially in float64; k*
//      is the first prefix reaching the threshold (E if none), clamped to
//      [k_min, k_max]; the mask is the ballot of lanes with rank < k.  Past
//      k_max entries the sum cannot change the clamped size, so it stops
//      there.
#include <cstddef>

#include "fm_device.h"
#include "fm_guide.h"
#include "fm_internal.h"

namespace fm {

namespace {

struct SelArgs {
  const void* planes;
  int64_t plane_elems;
  int32_t n, L, E, row;
  fm_dtype dtype;
  const int32_t* idx;
  const float* score;
  int32_t B, k;
  const int32_t* lb;
  const int32_t* le;
  int32_t mode;
  float tau;
  int32_t k_min, k_max, blend;
  uint64_t* mask_out;
  uint8_t* count_out;
  uint32_t* flags;
};

}  // namespace

// Ordered keys of a probability: larger value -> larger key, -0 and +0
// equal, NaN lowest.  Ranking by (key desc, index asc) is the (p desc, j asc,
// NaN last) order.  Real keys are at least 1; 0 marks a lane without an
// expert.
__device__ __forceinline__ uint64_t ord_f64(double p) {
  if (p != p) return 1ull;
  const uint64_t u = static_cast<uint64_t>(__double_as_longlong(p + 0.0));
  return (u >> 63) ? ~u : (u | 0x8000000000000000ull);
}
__device__ __forceinline__ uint32_t ord_f32(float p) {
  if (p != p) return 1u;
  const uint32_t u = __float_as_uint(p + 0.0f);
  return (u >> 31) ? ~u : (u | 0x80000000u);
}

// Rank of this lane's key among the E keys of its row (SW consecutive lanes):
// the keys ahead of it, that is greater, or equal with a lower index.  The
// borrow of mine - key_i - c, with c = 1 in the lanes after i, is exactly
// "key_i is ahead of mine": one subtraction chain and one add-with-carry per
// key, no separate test for equal keys.  `row` is the row's keys in LDS.
// (gfx950: the carry mask of the subtraction is any scalar pair.)
template <int SW>
__device__ __forceinline__ int rank_row(const uint32_t* row, uint32_t mine, int E) {
  // lanes whose index in the row is above i
  uint64_t after = ~0ull;
  if constexpr (SW == 8) after = 0xFEFEFEFEFEFEFEFEull;
  else if constexpr (SW == 16) after = 0xFFFEFFFEFFFEFFFEull;
  else if constexpr (SW == 32) after = 0xFFFFFFFEFFFFFFFEull;
  else after = 0xFFFFFFFFFFFFFFFEull;
  uint32_t rank = 0;
  for (int i = 0; i < E; i += 4) {
    const uint32x4 k = *reinterpret_cast<const uint32x4*>(row + i);
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      uint32_t t;
      asm("v_subb_co_u32_e64 %0, vcc, %2, %3, %4\n\tv_addc_co_u32_e32 %1, vcc, 0, %1, vcc"
          : "=&v"(t), "+v"(rank)
          : "v"(mine), "v"(k[u]), "s"(after)
          : "vcc");
      after &= after << 1;
    }
  }
  return static_cast<int>(rank);
}
template <int SW>
__device__ __forceinline__ int rank_row(const uint64_t* row, uint64_t mine, int E) {
  uint64_t after = ~0ull;
  if constexpr (SW == 8) after = 0xFEFEFEFEFEFEFEFEull;
  else if constexpr (SW == 16) after = 0xFFFEFFFEFFFEFFFEull;
  else if constexpr (SW == 32) after = 0xFFFFFFFEFFFFFFFEull;
  else after = 0xFFFFFFFFFFFFFFFEull;
  const uint32_t mlo = static_cast<uint32_t>(mine), mhi = static_cast<uint32_t>(mine >> 32);
  uint32_t rank = 0;
  for (int i = 0; i < E; i += 2) {
    const uint32x4 k = *reinterpret_cast<const uint32x4*>(row + i);
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      uint32_t t;
      asm("v_subb_co_u32_e64 %0, vcc, %2, %4, %6\n\t"
          "v_subb_co_u32_e32 %0, vcc, %3, %5, vcc\n\t"
          "v_addc_co_u32_e32 %1, vcc, 0, %1, vcc"
          : "=&v"(t), "+v"(rank)
          : "v"(mlo), "v"(mhi), "v"(k[2 * u]), "v"(k[2 * u + 1]), "s"(after)
          : "vcc");
      after &= after << 1;
    }
  }
  return static_cast<int>(rank);
}

// LDS of one wavefront's rows: the keys (64-bit for blended rows, 32-bit
// otherwise; rank_row reads them 16 bytes at a time) and the probabilities in
// rank order.
struct SelLds {
  __align__(16) uint64_t keys[kMaxE];
  double sorted[kMaxE];
};
static_assert(alignof(SelLds) == 16 && offsetof(SelLds, keys) % 16 == 0, "16-byte reads of the keys");

// The selection of row (b, l) of the batch by the SW lanes that hold it
// (`in`: whether they hold one), from the query's matches idx_b / score_b (k
// of them, best first) and its layer bounds [lo, hi) (as given; clamped
// here).
template <int SW>
__device__ __forceinline__ void select_row(const SelArgs& a, bool in, int b, int l, int lo, int hi,
                                           const int32_t* idx_b, const float* score_b, SelLds& sm) {
  const int lane = threadIdx.x % kWave;
  const int j = lane % SW;
  const int base = lane - j;
  const int64_t row = static_cast<int64_t>(b) * a.L + l;
  lo = lo < 0 ? 0 : (lo > a.L ? a.L : lo);
  hi = hi < 0 ? 0 : (hi > a.L ? a.L : hi);
  const int y0 = in ? idx_b[0] : -1;

  // 1. guiding probability of expert j: its loads need only the matches, so
  // they are issued before the row's bounds are looked at (a row outside
  // them discards the value)
  const GuideView gv{a.planes, a.plane_elems, a.n, a.row, a.dtype};
  const bool has = j < a.E && y0 >= 0 && y0 < a.n;
  double p = 0.0;
  if (has) {
    p = a.blend == FM_BLEND_SCORE ? blended_prob(gv, load_matches(a.n, idx_b, score_b, a.k), l, j)
                                  : static_cast<double>(stored_prob(gv, y0, l, j));
  }

  bool live = in && l >= lo && l < hi && y0 >= 0;
  if (live && y0 >= a.n) {
    if (j == 0) atomicOr(a.flags, static_cast<uint32_t>(FM_FLAG_INDEX_RANGE));
    live = false;
  }
  if (in && !live && j == 0) {
    a.mask_out[row] = 0ull;
    a.count_out[row] = 0;
  }
  if (__ballot(live) == 0) return;   // every row of the wavefront is empty

  // 2. threshold
  double tau = static_cast<double>(a.tau);
  if (a.mode == FM_TAU_DYNAMIC) {
    const double s = in ? static_cast<double>(score_b[0]) : 0.0;
    if (s != s) tau = 1.0;
    else {
      const double t = 1.0 - s;
      tau = t < 0.0 ? 0.0 : (t > 1.0 ? 1.0 : t);
    }
  }

  // 3. rank (a stored value is a float32 or bf16, so its 32-bit key orders it
  // exactly; a blend is a float64)
  int rank;
  if (a.blend == FM_BLEND_SCORE) {
    const uint64_t key = j < a.E ? ord_f64(p) : 0ull;
    sm.keys[lane] = key;
    wait_lgkm0();
    __builtin_amdgcn_wave_barrier();
    rank = rank_row<SW>(sm.keys + base, key, a.E);
  } else {
    uint32_t* k32 = reinterpret_cast<uint32_t*>(sm.keys);
    const uint32_t key = j < a.E ? ord_f32(static_cast<float>(p)) : 0u;
    k32[lane] = key;
    wait_lgkm0();
    __builtin_amdgcn_wave_barrier();
    rank = rank_row<SW>(k32 + base, key, a.E);
  }
  if (j < a.E) sm.sorted[base + rank] = p;
  wait_lgkm0();
  __builtin_amdgcn_wave_barrier();

  // 4. sequential float64 prefix sum in rank order: k* is the first count
  // whose running sum reaches tau; values are read 8 at a time ahead of the
  // sequential adds
  int kstar = a.E;
  double run = 0.0;
  bool found = false;
  const int kend = a.k_max < a.E ? a.k_max : a.E;
  for (int k0 = 0; k0 < kend; k0 += 8) {
    double v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = k0 + u < kend ? sm.sorted[base + k0 + u] : 0.0;
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      if (k0 + u >= kend) break;
      if (!found && run >= tau) {
        kstar = k0 + u;
        found = true;
      }
      run = __dadd_rn(run, v[u]);
    }
    if (__ballot(live && !found) == 0) break;
  }
  int kk = kstar < a.k_min ? a.k_min : kstar;
  kk = kk > a.k_max ? a.k_max : kk;
  const uint64_t all = __ballot(j < a.E && rank < kk);
  if (live && j == 0) {
    a.mask_out[row] = SW == 64 ? all : (all >> base) & ((1ull << (SW % 64)) - 1ull);
    a.count_out[row] = static_cast<uint8_t>(kk);
  }
}

constexpr int kMergeGroups = 1536;   // workgroups of a merge-and-select launch beyond which positions stop splitting

// Lanes per row for E experts.
inline int select_width(int E) { return E <= 8 ? 8 : (E <= 16 ? 16 : (E <= 32 ? 32 : 64)); }

template <int SW>
__global__ void __launch_bounds__(256) k_select(SelArgs a) {
  constexpr int RPW = kWave / SW;
  __shared__ SelLds sm[4];
  const int wv = threadIdx.x / kWave;
  const int lane = threadIdx.x % kWave;
  const int64_t row = (static_cast<int64_t>(blockIdx.x) * 4 + wv) * RPW + lane / SW;
  const bool in = row < static_cast<int64_t>(a.B) * a.L;
  if (__ballot(in) == 0) return;
  const int b = in ? static_cast<int>(row / a.L) : 0;
  const int l = in ? static_cast<int>(row - static_cast<int64_t>(b) * a.L) : 0;
  select_row<SW>(a, in, b, l, a.lb[b], a.le[b], a.idx + static_cast<int64_t>(b) * a.k,
                 a.score + static_cast<int64_t>(b) * a.k, sm[wv]);
}

// The cross-workgroup merge of a match call with the selection after it.
// Workgroup (pos, y): its four wavefronts merge the position's partial top-k
// lists together, a list per thread (each wavefront of a row merging all of
// them by itself cost most of this kernel for top-4 and top-8 lists), the
// workgroups y = 0 write the query's matches, and the workgroup selects the
// layers of its share: row sets y * 4 + wave, + 4 * gridDim.y, ...  of 64 / SW
// layers each.  The same merge as k_finalize and the same selection as
// k_select.  Measured (kernel time): 512 positions of 256 top-4 lists, 32
// layers of 16 experts 26.6 -> 13.0 us; 100 positions of top-8 lists, 32 x 8
// 18.1 -> 10.0 us; 512 of top-1 lists, 24 x 60 18.1 -> 14.4-17.4 us, where the
// matched rows' reads bound it (a row's 15 quads lie in 15 cache lines, 94 MB
// of lines for 12,288 rows of four float32 matches).
struct MergeArgs {
  const uint64_t* partial;   // [positions][R][KTOP]
  const int32_t* perm;       // query at each position (NULL: the position itself)
  int32_t R;                 // lists per position
  const int32_t* rgrp;       // lists per query group (NULL: R)
  int32_t qg;                // positions per query group
  int32_t* idx_out;          // [B][k]
  float* score_out;          // [B][k]
  const float* rq;           // top-1 lists that rank by dot / |x|: 1/|q| per position (NULL: the keys hold the scores)
};

template <int KTOP, int SW>
__global__ void __launch_bounds__(256) k_merge_select(SelArgs a, MergeArgs m) {
  constexpr int RPW = kWave / SW;
  __shared__ SelLds sm[4];
  __shared__ uint64_t wlist[4][KTOP];
  __shared__ int32_t midx[4][kMaxK];
  __shared__ float mscore[4][kMaxK];
  const int lane = threadIdx.x % kWave;
  const int wv = threadIdx.x / kWave;
  const int pos = blockIdx.x;
  // The loads that do not depend on the merge go first, side by side: the
  // group's list count, the query index (then its layer bounds) and this
  // thread's first list of the stride (past the group's count it is read but
  // not merged).
  const int nr = m.rgrp != nullptr ? m.rgrp[pos / m.qg] : m.R;
  const int b = m.perm != nullptr ? m.perm[pos] : pos;
  const uint64_t* plist = m.partial + static_cast<int64_t>(pos) * m.R * KTOP;
  TopK<KTOP> t;
  {
    uint64_t first[KTOP];
    const bool held = static_cast<int>(threadIdx.x) < m.R;
#pragma unroll
    for (int jj = 0; jj < KTOP; ++jj) first[jj] = held ? plist[threadIdx.x * KTOP + jj] : 0ull;
#pragma unroll
    for (int jj = 0; jj < KTOP; ++jj) t.v[jj] = static_cast<int>(threadIdx.x) < nr ? first[jj] : 0ull;
  }
  const int lo = a.lb[b], hi = a.le[b];
  const float rq = KTOP == 1 && m.rq != nullptr ? m.rq[pos] : 1.0f;
  for (int r = threadIdx.x + 256; r < nr; r += 256) t.merge(plist + static_cast<int64_t>(r) * KTOP);
  // (A wavefront past the lists has nothing to merge.  The merges of longer lists
  // stay loops: two lists of 8 take over a hundred instructions, and nine copies
  // of them cost more to fetch than they save, with one query of 8,861 x 256,
  // top-8 the call 27.4 us unrolled, 25.0 as loops; those of one match are 0.4 us
  // quicker unrolled.)
  constexpr int kRounds = KTOP == 1 ? 6 : 1, kMerges = KTOP == 1 ? 3 : 1;
  if (wv * kWave < nr) {
#pragma unroll kRounds
    for (int off = 1; off < kWave; off <<= 1) {
      uint64_t o[KTOP];
#pragma unroll
      for (int jj = 0; jj < KTOP; ++jj) o[jj] = shfl_xor_u64(t.v[jj], off);
      t.merge(o);
    }
  }
  if (lane == 0) {
#pragma unroll
    for (int jj = 0; jj < KTOP; ++jj) wlist[wv][jj] = t.v[jj];
  }
  __syncthreads();
  // every wavefront merges the four lists for itself (the same result)
#pragma unroll
  for (int jj = 0; jj < KTOP; ++jj) t.v[jj] = wlist[0][jj];
#pragma unroll kMerges
  for (int ww = 1; ww < 4; ++ww)
    if (ww * kWave < nr) t.merge(wlist[ww]);
  if (lane == 0) {
#pragma unroll
    for (int jj = 0; jj < kMaxK; ++jj) {
      if (jj >= a.k) break;
      const uint64_t key = jj < KTOP ? t.v[jj < KTOP ? jj : 0] : 0ull;
      int32_t y = key_index(key);
      float sc = key_score(key);
      if constexpr (KTOP == 1)
        if (m.rq != nullptr) scale_match(key, rq, y, sc);
      midx[wv][jj] = y;
      mscore[wv][jj] = sc;
      if (blockIdx.y == 0 && wv == 0) {
        m.idx_out[static_cast<int64_t>(b) * a.k + jj] = y;
        m.score_out[static_cast<int64_t>(b) * a.k + jj] = sc;
      }
    }
  }
  // (LDS only: the bounds' loads stay in flight)
  wait_lgkm0();
  __builtin_amdgcn_wave_barrier();
  const int sets = (a.L + RPW - 1) / RPW;
  for (int rs = static_cast<int>(blockIdx.y) * 4 + wv; rs < sets; rs += 4 * static_cast<int>(gridDim.y)) {
    const int l = rs * RPW + lane / SW;
    select_row<SW>(a, l < a.L, b, l < a.L ? l : 0, lo, hi, midx[wv], mscore[wv], sm[wv]);
    __builtin_amdgcn_wave_barrier();
  }
}

// Misses of the prefetch sets (Section 3): SW lanes per (query, layer) row, as
// in the selection; lane j ranks expert j of the query's own gate
// probabilities among the row (the same order), the K best are the activated
// experts, and the count of those outside the set is written.
struct MissArgs {
  const void* q;           // [B][L][E] of the map dtype
  fm_dtype dtype;
  int32_t B, L, E, K;
  const uint64_t* masks;   // [B][L]
  const int32_t* lb;
  const int32_t* le;
  uint8_t* miss_out;       // [B][L]
};

template <int SW>
__global__ void __launch_bounds__(256) k_miss(MissArgs a) {
  constexpr int RPW = kWave / SW;
  __shared__ __align__(16) uint32_t keys[4][kMaxE];
  const int lane = threadIdx.x % kWave;
  const int wv = threadIdx.x / kWave;
  const int j = lane % SW;
  const int base = lane - j;
  const int64_t row = (static_cast<int64_t>(blockIdx.x) * 4 + wv) * RPW + lane / SW;
  const bool in = row < static_cast<int64_t>(a.B) * a.L;
  if (__ballot(in) == 0) return;
  const int b = in ? static_cast<int>(row / a.L) : 0;
  const int l = in ? static_cast<int>(row - static_cast<int64_t>(b) * a.L) : 0;
  // the row's values, set and bounds load side by side
  float p = 0.0f;
  if (in && j < a.E) {
    const int64_t i = row * a.E + j;
    p = a.dtype == FM_F32 ? static_cast<const float*>(a.q)[i] : bf16_to_f32(static_cast<const uint16_t*>(a.q)[i]);
  }
  const uint64_t set = in ? a.masks[row] : 0ull;
  int lo = a.lb[b], hi = a.le[b];
  lo = lo < 0 ? 0 : (lo > a.L ? a.L : lo);
  hi = hi < 0 ? 0 : (hi > a.L ? a.L : hi);
  const bool live = in && l >= lo && l < hi;
  if (in && !live && j == 0) a.miss_out[row] = 0;
  if (__ballot(live) == 0) return;
  const uint32_t key = j < a.E ? ord_f32(p) : 0u;
  keys[wv][lane] = key;
  wait_lgkm0();
  __builtin_amdgcn_wave_barrier();
  const int rank = rank_row<SW>(keys[wv] + base, key, a.E);
  const uint64_t all = __ballot(j < a.E && rank < a.K);
  const uint64_t act = SW == 64 ? all : (all >> base) & ((1ull << (SW % 64)) - 1ull);
  if (live && j == 0) a.miss_out[row] = static_cast<uint8_t>(__popcll(act & ~set));
}

hipError_t launch_miss(const StoreView& s, const void* q, int32_t B, int32_t K, const uint64_t* masks,
                       const int32_t* lb, const int32_t* le, uint8_t* miss_out, hipStream_t st) {
  MissArgs a;
  a.q = q;
  a.dtype = s.map_dtype;
  a.B = B;
  a.L = s.L;
  a.E = s.E;
  a.K = K;
  a.masks = masks;
  a.lb = lb;
  a.le = le;
  a.miss_out = miss_out;
  const int SW = select_width(s.E);
  const int64_t rows = static_cast<int64_t>(B) * s.L;
  const int64_t per = 4 * (kWave / SW);   // rows per workgroup
  const dim3 grid(static_cast<unsigned>((rows + per - 1) / per));
  if (SW == 8) hipLaunchKernelGGL(k_miss<8>, grid, dim3(256), 0, st, a);
  else if (SW == 16) hipLaunchKernelGGL(k_miss<16>, grid, dim3(256), 0, st, a);
  else if (SW == 32) hipLaunchKernelGGL(k_miss<32>, grid, dim3(256), 0, st, a);
  else hipLaunchKernelGGL(k_miss<64>, grid, dim3(256), 0, st, a);
  return hipGetLastError();
}

namespace {

SelArgs select_args(const StoreView& s, const int32_t* idx, const float* score, int32_t B, int32_t k,
                    const int32_t* lb, const int32_t* le, const fm_select_params& p, uint64_t* mask_out,
                    uint8_t* count_out) {
  SelArgs a;
  a.planes = s.planes;
  a.plane_elems = s.plane_elems;
  a.n = s.n;
  a.L = s.L;
  a.E = s.E;
  a.row = s.row;
  a.dtype = s.map_dtype;
  a.idx = idx;
  a.score = score;
  a.B = B;
  a.k = k;
  a.lb = lb;
  a.le = le;
  a.mode = p.mode;
  a.tau = p.tau;
  a.k_min = p.k_min;
  a.k_max = p.k_max;
  a.blend = p.blend;
  a.mask_out = mask_out;
  a.count_out = count_out;
  a.flags = s.flags;
  return a;
}

}  // namespace

hipError_t launch_select(const StoreView& s, const int32_t* idx, const float* score, int32_t B, int32_t k,
                         const int32_t* lb, const int32_t* le, const fm_select_params& p, uint64_t* mask_out,
                         uint8_t* count_out, hipStream_t st) {
  const SelArgs a = select_args(s, idx, score, B, k, lb, le, p, mask_out, count_out);
  const int SW = select_width(s.E);
  const int64_t rows = static_cast<int64_t>(B) * s.L;
  const int64_t per = 4 * (kWave / SW);   // rows per workgroup
  const dim3 grid(static_cast<unsigned>((rows + per - 1) / per));
  if (SW == 8) hipLaunchKernelGGL(k_select<8>, grid, dim3(256), 0, st, a);
  else if (SW == 16) hipLaunchKernelGGL(k_select<16>, grid, dim3(256), 0, st, a);
  else if (SW == 32) hipLaunchKernelGGL(k_select<32>, grid, dim3(256), 0, st, a);
  else hipLaunchKernelGGL(k_select<64>, grid, dim3(256), 0, st, a);
  return hipGetLastError();
}

namespace {

template <int KTOP>
void merge_select_launch(int SW, dim3 grid, const SelArgs& a, const MergeArgs& m, hipStream_t st) {
  if (SW == 8) hipLaunchKernelGGL((k_merge_select<KTOP, 8>), grid, dim3(256), 0, st, a, m);
  else if (SW == 16) hipLaunchKernelGGL((k_merge_select<KTOP, 16>), grid, dim3(256), 0, st, a, m);
  else if (SW == 32) hipLaunchKernelGGL((k_merge_select<KTOP, 32>), grid, dim3(256), 0, st, a, m);
  else hipLaunchKernelGGL((k_merge_select<KTOP, 64>), grid, dim3(256), 0, st, a, m);
}

}  // namespace

hipError_t launch_merge_select(const StoreView& s, const uint64_t* partial, const int32_t* perm, int32_t B, int32_t R,
                               int32_t k, int KTOP, const int32_t* rgrp, int32_t qg, int32_t* idx_out,
                               float* score_out, const SelectFuse& f, hipStream_t st, const float* rq) {
  const SelArgs a = select_args(s, nullptr, nullptr, B, k, f.lb, f.le, f.p, f.mask_out, f.count_out);
  MergeArgs m;
  m.partial = partial;
  m.perm = perm;
  m.R = R;
  m.rgrp = rgrp;
  m.qg = qg > 0 ? qg : 1;
  m.idx_out = idx_out;
  m.score_out = score_out;
  m.rq = rq;
  // Workgroups per position: enough that every wavefront selects one set of
  // rows, fewer (each then selects several in turn) once the batch alone
  // fills the chip, since every workgroup of a position repeats its merge.
  const int SW = select_width(s.E);
  const int sets = (s.L + kWave / SW - 1) / (kWave / SW);
  int S = (sets + 3) / 4;
  const int most = (kMergeGroups + B - 1) / B;
  if (S > most) S = most;
  const dim3 grid(static_cast<unsigned>(B), static_cast<unsigned>(S));
  if (KTOP == 1) merge_select_launch<1>(SW, grid, a, m, st);
  else if (KTOP == 4) merge_select_launch<4>(SW, grid, a, m, st);
  else merge_select_launch<8>(SW, grid, a, m, st);
  return hipGetLastError();
}

}  // namespace fm
