// Prefetch and eviction priorities (Section 4.5).
//
//   PRI^prefetch_{l,j} = p_{l,j} / (l - l_now)   experts of the query's
//                                                 prefetch set, layers l > l_now
//   PRI^evict_{l,j}    = 1 / (p_{l,j} freq_{l,j}) cached experts
//
// with p the query's guiding probabilities (as for the selection).  One
// workgroup per query: the candidates' priorities are computed in float64,
// rounded to float32 and packed with their expert index into 64-bit keys
// (priority order, then the lower l * E + j; NaN last), collected in LDS and
// placed by counting the keys above each one (up to 1024 candidates) or by a
// bitonic sort, then written out in that order.
#include "fm_device.h"
#include "fm_guide.h"
#include "fm_internal.h"

namespace fm {

namespace {

constexpr int kPriThreads = 256;
constexpr int kPriMax = kMaxL * kMaxE;   // candidates per query at most
constexpr int kCountMax = 1024;          // up to this many candidates are ranked by counting

struct PriArgs {
  GuideView gv;
  int32_t L, E;
  const int32_t* idx;
  const float* score;
  int32_t B, k, blend, kind;
  const uint64_t* masks;   // PREFETCH: [B][L]; EVICT: [L]
  const int32_t* l_now;    // [B] (PREFETCH)
  const float* freq;       // [L][E] (EVICT)
  int32_t cap;
  int32_t* order_out;      // [B][cap]
  float* pri_out;          // [B][cap]
  int32_t* count_out;      // [B]
  uint32_t* flags;
};

// Order-preserving map of a float32 to uint32 (NaN -> 0, below every number;
// -0 and +0 equal).
__device__ __forceinline__ uint32_t ord_value(float s) {
  if (s != s) return 0u;
  s = s + 0.0f;
  const uint32_t u = __float_as_uint(s);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

}  // namespace

// Place the candidates by counting: a candidate's place is the number of keys
// above its own (keys are distinct), read from LDS as broadcasts, eight in
// flight (64 queries of about 700 candidates of 24 x 60: the call 22.6 us, with
// four 27.5); OWN candidates per thread.
template <int OWN>
__device__ __forceinline__ void place_by_count(const PriArgs& a, const uint64_t* keys, int N, int b) {
  const int tid = threadIdx.x;
  uint64_t mine[OWN];
  int rank[OWN];
#pragma unroll
  for (int u = 0; u < OWN; ++u) {
    mine[u] = tid + u * kPriThreads < N ? keys[tid + u * kPriThreads] : 0ull;
    rank[u] = 0;
  }
#pragma unroll 8
  for (int i = 0; i < N; ++i) {
    const uint64_t x = keys[i];
#pragma unroll
    for (int u = 0; u < OWN; ++u) rank[u] += x > mine[u] ? 1 : 0;
  }
#pragma unroll
  for (int u = 0; u < OWN; ++u) {
    if (tid + u * kPriThreads >= N || rank[u] >= a.cap) continue;
    const int64_t o = static_cast<int64_t>(b) * a.cap + rank[u];
    a.order_out[o] = static_cast<int32_t>(~static_cast<uint32_t>(mine[u]));
    a.pri_out[o] = unord_score(static_cast<uint32_t>(mine[u] >> 32));
  }
}

// One workgroup per query.  The candidates are listed before any
// probability is read (a set bit's place is the set bits before it), so that
// a thread reads and ranks only candidates: with a slot of the thread's own
// for every (layer, expert) pair, most slots were empty and each cost its
// guarded loads and four 64-bit comparisons per key (512 queries of 24 x 60
// with sets of at most 8, top-4 blend: 27.1 -> 9.6 us).
__global__ void __launch_bounds__(kPriThreads) k_priority(PriArgs a) {
  __shared__ uint64_t keys[kPriMax];
  __shared__ uint16_t cand[kPriMax];   // l * 64 + j of each candidate
  __shared__ uint64_t sets[kMaxL];
  __shared__ int32_t first[kMaxL];     // candidates in the layers before
  __shared__ int32_t n_cand;
  const int tid = threadIdx.x;
  const int lane = tid % kWave;
  const int wv = tid / kWave;
  const int b = blockIdx.x;
  const int32_t* idx_b = a.idx + static_cast<int64_t>(b) * a.k;
  const float* score_b = a.score + static_cast<int64_t>(b) * a.k;
  // the match, the current layer and the layer's set load together
  const int y0 = idx_b[0];
  const int lnow = a.kind == FM_PRI_PREFETCH ? a.l_now[b] : 0;
  if (wv == 0) {
    uint64_t bits = 0ull;
    if (lane < a.L) bits = a.kind == FM_PRI_PREFETCH ? a.masks[static_cast<int64_t>(b) * a.L + lane] : a.masks[lane];
    bool live = y0 >= 0;
    if (live && y0 >= a.gv.n) {
      if (lane == 0) atomicOr(a.flags, static_cast<uint32_t>(FM_FLAG_INDEX_RANGE));
      live = false;
    }
    // the candidate sets of every layer (none after a missing match)
    const uint64_t experts = a.E == kMaxE ? ~0ull : (1ull << a.E) - 1ull;
    bits = live && lane < a.L && (a.kind != FM_PRI_PREFETCH || lane > lnow) ? bits & experts : 0ull;
    const int cnt = __popcll(bits);
    int incl = cnt;
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) {
      const int o = __shfl_up(incl, off, kWave);
      if (lane >= off) incl += o;
    }
    sets[lane] = bits;
    first[lane] = incl - cnt;
    if (lane == kWave - 1) n_cand = incl;
  }
  __syncthreads();
  const int N = n_cand;
  for (int l = wv; l < a.L; l += kPriThreads / kWave) {
    const uint64_t bits = sets[l];
    if ((bits >> lane) & 1ull)
      cand[first[l] + __popcll(bits & ((1ull << lane) - 1ull))] = static_cast<uint16_t>(l * kMaxE + lane);
  }
  __syncthreads();
  auto fill = [&](auto prob) __attribute__((always_inline)) {
    for (int i = tid; i < N; i += kPriThreads) {
      const int l = cand[i] / kMaxE;
      const int j = cand[i] % kMaxE;
      const double p = prob(l, j);
      double v;
      if (a.kind == FM_PRI_PREFETCH) {
        v = __ddiv_rn(p, static_cast<double>(l - lnow));
      } else {
        const double prod = __dmul_rn(p, static_cast<double>(a.freq[l * a.E + j]));
        v = __ddiv_rn(1.0, prod);
      }
      const uint32_t e = static_cast<uint32_t>(l * a.E + j);
      keys[i] = (static_cast<uint64_t>(ord_value(static_cast<float>(v))) << 32) | static_cast<uint32_t>(~e);
    }
  };
  // (a blend's matches are read once, not again before every candidate)
  if (a.blend == FM_BLEND_SCORE) {
    const Matches m = load_matches(a.gv.n, idx_b, score_b, a.k);
    fill([&](int l, int j) { return blended_prob(a.gv, m, l, j); });
  } else {
    fill([&](int l, int j) { return static_cast<double>(stored_prob(a.gv, y0, l, j)); });
  }
  // the places past the candidates
  for (int i = N + tid; i < a.cap; i += kPriThreads) {
    const int64_t o = static_cast<int64_t>(b) * a.cap + i;
    a.order_out[o] = -1;
    a.pri_out[o] = -__builtin_inff();
  }
  if (tid == 0) a.count_out[b] = N;
  __syncthreads();
  if (N <= kCountMax) {
    if (N <= kPriThreads) place_by_count<1>(a, keys, N, b);
    else if (N <= 2 * kPriThreads) place_by_count<2>(a, keys, N, b);
    else place_by_count<kCountMax / kPriThreads>(a, keys, N, b);
    return;
  }
  int P = 1;
  while (P < N) P <<= 1;
  for (int i = N + tid; i < P; i += kPriThreads) keys[i] = 0ull;   // padding ranks below everything
  __syncthreads();
  // bitonic sort, descending
  for (int size = 2; size <= P; size <<= 1) {
    for (int stride = size / 2; stride > 0; stride >>= 1) {
      for (int i = tid; i < P / 2; i += kPriThreads) {
        const int lo = 2 * stride * (i / stride) + (i % stride);
        const int hi = lo + stride;
        const uint64_t x = keys[lo], y = keys[hi];
        const bool desc = (lo & size) == 0;
        if (desc ? (x < y) : (x > y)) {
          keys[lo] = y;
          keys[hi] = x;
        }
      }
      __syncthreads();
    }
  }
  for (int i = tid; i < a.cap; i += kPriThreads) {
    if (i >= N) break;
    const int64_t o = static_cast<int64_t>(b) * a.cap + i;
    const uint64_t key = keys[i];
    a.order_out[o] = static_cast<int32_t>(~static_cast<uint32_t>(key));
    a.pri_out[o] = unord_score(static_cast<uint32_t>(key >> 32));
  }
}

hipError_t launch_priority(const StoreView& s, const int32_t* idx, const float* score, int32_t B, int32_t k,
                           int32_t blend, int32_t kind, const uint64_t* masks, const int32_t* l_now,
                           const float* freq, int32_t cap, int32_t* order_out, float* pri_out, int32_t* count_out,
                           hipStream_t st) {
  PriArgs a;
  a.gv = GuideView{s.planes, s.plane_elems, s.n, s.row, s.map_dtype};
  a.L = s.L;
  a.E = s.E;
  a.idx = idx;
  a.score = score;
  a.B = B;
  a.k = k;
  a.blend = blend;
  a.kind = kind;
  a.masks = masks;
  a.l_now = l_now;
  a.freq = freq;
  a.cap = cap;
  a.order_out = order_out;
  a.pri_out = pri_out;
  a.count_out = count_out;
  a.flags = s.flags;
  hipLaunchKernelGGL(k_priority, dim3(B), dim3(kPriThreads), 0, st, a);
  return hipGetLastError();
}

}  // namespace fm
