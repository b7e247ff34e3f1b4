// Semantic-based expert map search (Section 4.2.1, Eq. 4), split-k form.
//
// The contraction Q X^T of a query batch (B x d) with the stored embeddings
// (n x d), both bf16 on v_mfma_f32_16x16x32_bf16 as in k_sem_mm
// (fm_sem_mm.hip), for top-1 searches whose time is not the matrix rate: small
// stores and small batches.  (Top-2..8 lists stay on k_sem_scan: this scan's
// sums differ from a sequential one by up to 1e-6 of a cosine, and the last
// place of a list of 8 is near enough a tie in about one query of a hundred to
// change hands for it, with that query's blended sets.)
//
// A workgroup takes a group of 16 TQ queries and a range of the store's 16-map
// blocks, NB blocks per step.  Its W wavefronts split the d dimensions: each
// accumulates the whole 16 NB x 16 TQ tile over its own run of k-steps (32
// dimensions each), reading map and query operand tiles straight from memory
// into registers, D k-steps ahead.  So no operand passes through LDS, no
// barrier stands in the k loop, the serial chain of a step is d / (32 W)
// k-steps, and a store of only a few blocks still fills a workgroup per
// block.  At the end of a step the W partial tiles are summed through LDS,
// each (block, query tile) pair by one wavefront, which scales the sums by
// 1/|x| and keeps its query tile's best per lane.
//
// The dense form writes every cosine, or its weighted sum with a second
// dense matrix (the deduplicating insert's RDY), instead of keeping lists.
//
// A list ranks by dot * 1/|x|: the query's factor 1/|q| is positive (or 0 for
// a zero query, whose dots are all 0) and is applied by the merge.
//
// Measured (kernel time): 1,000 embeddings of d = 4096, 8 queries 84 us on
// k_sem_mm (128 dependent stages, one block of 32 in use) -> 7.9 us; 16,000
// of d = 2048, 8 queries 46 -> 13 us (5.0 TB/s); 60,000 of d = 2048, 8
// queries 53 -> 43 us (5.8 TB/s, the card's read rate).  With TQ = 8 a k-step
// moves as many query as map bytes into a CU, and a CU takes about 45 GB/s of
// such a mix while the map half comes from HBM (a read probe: 22 + 22 GB/s
// per CU, 113 GB/s from L2 alone), so large stores with many queries stay on
// the LDS-staged scans, which move half as much.  Three sets of operands in
// flight instead of two, one wavefront per SIMD with 128 x 128 tiles,
// streaming hints on the map loads and a k-step rotation per workgroup were
// each within 3% and are not used.
//
// TQ = 1 and 2 (groups of up to 32 queries, however many groups) read the
// caller's rows themselves and spread the query norms over the group's
// workgroups, so the search is two launches; larger groups read the tiles staged by k_sem_prep (a caller's row
// gives 64 contiguous bytes per k-step, and rows a multiple of 4 KB apart lie
// on one memory channel, which 64 and more rows feel).
#include "fm_device.h"
#include "fm_internal.h"

namespace fm {

namespace {

struct SplitArgs {
  const uint16_t* x;     // tiled embeddings
  const float* xnorm;    // [cap] |x|
  const uint16_t* q;     // RAW: [B][d] rows; else staged tiles
  float* rq;             // [b_pad] 1/|q| (RAW: written here)
  uint64_t* partial;     // [b_pad][R]: one packed key per (query, workgroup of its group)
  // dense form: the scores [B][n], or w_self * score + w_mix * mix
  float* dbg;
  const float* mix;
  double w_self, w_mix;
  int32_t vec16;         // dense rows written (and mix read) 16 bytes at a time: n % 4 == 0, aligned buffers
  int32_t n, d, ksteps, B;
  int32_t n_qg;          // query groups
  int32_t R;             // workgroups per query group
  int32_t n_blocks;      // 16-map blocks of the store
  int32_t grid;
};

template <int W, int NB, int TQ>
struct SplitShape {
  static constexpr int TC0 = W * NB * TQ <= 128 ? TQ : 128 / (W * NB);   // query tiles per reduction phase (128 KB of LDS)
  static constexpr int TC = TC0 < W ? TC0 : W;
  static constexpr int PAIRS = NB * TC;
  static constexpr int PH = TQ / TC;                  // phases
  static_assert(TQ % TC == 0 && W % TC == 0, "a wavefront sums one query tile per phase");
};

// A key that ranks any float (unlike make_key, no value stands for NaN).
__device__ __forceinline__ uint64_t split_key(float s, int32_t idx) {
  const uint32_t u = __float_as_uint(s + 0.0f);
  const uint32_t o = s != s ? 0u : ((u & 0x80000000u) ? ~u : (u | 0x80000000u));
  return (static_cast<uint64_t>(o) << 32) | static_cast<uint32_t>(~static_cast<uint32_t>(idx));
}

}  // namespace

template <int W, int NB, int TQ, int D, bool RAW, bool DENSE>
__global__ void __launch_bounds__(W * 64) __attribute__((amdgpu_waves_per_eu(W / 4, W / 4))) k_sem_split(SplitArgs a) {
  using S = SplitShape<W, NB, TQ>;
  constexpr int TC = S::TC, PAIRS = S::PAIRS, PH = S::PH;
  constexpr int QG = 16 * TQ;
  extern __shared__ __align__(16) unsigned char smem[];

  const int tid = threadIdx.x;
  const int w = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int lane = tid % kWave;
  const int g = lane / 16;
  const int c = lane % 16;

  // workgroup -> (query group, block range); the groups of a range are
  // consecutive in u, hence on one XCD, and share its map tiles in L2
  const int bid = blockIdx.x;
  const int u = (bid % 8) * (a.grid / 8) + bid / 8;
  const bool active = u < a.n_qg * a.R;
  const int qgrp = __builtin_amdgcn_readfirstlane(active ? u % a.n_qg : 0);
  const int rr = __builtin_amdgcn_readfirstlane(active ? u / a.n_qg : 0);
  const int b_begin = __builtin_amdgcn_readfirstlane(
      active ? static_cast<int>((static_cast<int64_t>(rr) * a.n_blocks) / a.R) : 0);
  const int b_end = __builtin_amdgcn_readfirstlane(
      active ? static_cast<int>((static_cast<int64_t>(rr + 1) * a.n_blocks) / a.R) : 0);
  const int n_steps = (b_end - b_begin + NB - 1) / NB;
  const int g0 = qgrp * QG;
  if (!active) return;

  uint64_t best[PH];   // best key of this lane's query of each phase
#pragma unroll
  for (int p = 0; p < PH; ++p) best[p] = 0;

  // this wavefront's k-steps [k0, k1), padded to a multiple of D (the padding
  // loads read zeros)
  const int k0 = (w * a.ksteps) / W;
  const int k1 = ((w + 1) * a.ksteps) / W;
  const int kp = ((a.ksteps + W - 1) / W + D - 1) / D * D;
  const uint32_t blk32 = static_cast<uint32_t>(a.ksteps) * 1024u;   // bytes of one 16-row block (d < 2^21)

  uint32_t vm[NB], vq[TQ];
#pragma unroll
  for (int i = 0; i < NB; ++i) vm[i] = static_cast<uint32_t>(i) * blk32 + static_cast<uint32_t>(lane * 16);
  const char* qbase;
  uint32_t qrec;
  if constexpr (RAW) {
    const int rows = a.B - g0 < QG ? a.B - g0 : QG;
    qbase = reinterpret_cast<const char*>(a.q) + static_cast<int64_t>(g0) * a.d * 2;
    qrec = static_cast<uint32_t>(rows) * static_cast<uint32_t>(a.d) * 2u;
#pragma unroll
    for (int t = 0; t < TQ; ++t) vq[t] = static_cast<uint32_t>(16 * t + c) * static_cast<uint32_t>(a.d) * 2u + static_cast<uint32_t>(g * 16);
  } else {
    qbase = reinterpret_cast<const char*>(a.q) + static_cast<int64_t>(g0 / 16) * blk32;
    qrec = static_cast<uint32_t>(TQ) * blk32;
#pragma unroll
    for (int t = 0; t < TQ; ++t) vq[t] = static_cast<uint32_t>(t) * blk32 + static_cast<uint32_t>(lane * 16);
  }

  // The loads' positions as running scalars: the query tiles' k-step, D ahead
  // of the products, and the map tiles' (D - 1 ahead) step, k-step and
  // descriptor.  A position past the wavefront's k-steps (or the last step)
  // reads zeros through an empty descriptor.
  int q_k = 0, m_k = 0;
  int c_blk = b_begin;
  uint64_t c_xbase = reinterpret_cast<uint64_t>(a.x) + static_cast<uint64_t>(static_cast<uint32_t>(b_begin)) * blk32;
  uint32_t c_rec;
  auto set_rec = [&]() __attribute__((always_inline)) {
    int nbk = b_end - c_blk;
    nbk = nbk < 0 ? 0 : (nbk > NB ? NB : nbk);
    c_rec = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(nbk) * blk32);
  };
  set_rec();
  u16x8 fm[D][NB], fq[D][TQ];
  auto load_m = [&](int s, int i) __attribute__((always_inline)) {
    const bool in = k0 + m_k < k1 && c_rec != 0;
    const uint32_t ks = in ? static_cast<uint32_t>(k0 + m_k) : 0u;
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
        reinterpret_cast<char*>(c_xbase), static_cast<short>(0), static_cast<int>(in ? c_rec : 0u), kBufWord3);
    fm[s][i] = __builtin_bit_cast(
        u16x8, __builtin_amdgcn_raw_buffer_load_b128(rs, static_cast<int>(vm[i]), static_cast<int>(ks * 1024u), 0));
  };
  auto load_q = [&](int s, int t) __attribute__((always_inline)) {
    const bool in = k0 + q_k < k1;
    const uint32_t ks = in ? static_cast<uint32_t>(k0 + q_k) : 0u;
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<char*>(qbase), static_cast<short>(0), static_cast<int>(in ? qrec : 0u), kBufWord3);
    fq[s][t] = __builtin_bit_cast(u16x8, __builtin_amdgcn_raw_buffer_load_b128(
                                             rs, static_cast<int>(vq[t]), static_cast<int>(ks * (RAW ? 64u : 1024u)), 0));
  };
  auto next_m = [&]() __attribute__((always_inline)) {
    if (++m_k == kp) {
      m_k = 0;
      c_blk += NB;
      c_xbase += static_cast<uint64_t>(NB) * blk32;
      set_rec();
    }
  };
  auto next_q = [&]() __attribute__((always_inline)) { q_k = q_k + 1 == kp ? 0 : q_k + 1; };

  floatx4 acc[NB][TQ];
#pragma unroll
  for (int i = 0; i < NB; ++i)
#pragma unroll
    for (int t = 0; t < TQ; ++t) acc[i][t] = floatx4{0.f, 0.f, 0.f, 0.f};

#pragma unroll
  for (int s = 0; s < D; ++s) {
#pragma unroll
    for (int t = 0; t < TQ; ++t) load_q(s, t);
    next_q();
    if (s < D - 1) {
#pragma unroll
      for (int i = 0; i < NB; ++i) load_m(s, i);
      next_m();
    }
  }

  if constexpr (RAW) {
    // 1/|q| (float64) of the group's queries, dealt over its workgroups and
    // their wavefronts; read by the merge only
    for (int r = rr + a.R * w; r < QG; r += a.R * W) {
      double sq = 0.0;
      if (g0 + r < a.B) {
        const uint16_t* row = a.q + static_cast<int64_t>(g0 + r) * a.d;
        for (int j0 = 8 * lane; j0 < a.d; j0 += 8 * kWave) {
          const u16x8 h = *reinterpret_cast<const u16x8*>(row + j0);
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            const double v = static_cast<double>(bf16_to_f32(h[e]));
            sq += v * v;
          }
        }
      }
#pragma unroll
      for (int m = 32; m >= 1; m >>= 1) sq += __shfl_xor(sq, m, kWave);
      if (lane == 0) {
        float v;
        if (sq != sq) v = __uint_as_float(0x7fc00000u);
        else if (sq == 0.0) v = 0.0f;
        else v = static_cast<float>(1.0 / sqrt(sq));
        a.rq[g0 + r] = v;
      }
    }
  }

  const int tt = w % TC;   // the query tile (of a phase) this wavefront sums
  for (int step = 0; step < n_steps; ++step) {
    for (int ki = 0; ki < kp; ki += D) {
#pragma unroll
      for (int s = 0; s < D; ++s) {
        // per query tile: its products, the load of its next operand into the
        // register they have just read, and a share of the map tiles that
        // replace the previous k-step's
#pragma unroll
        for (int t = 0; t < TQ; ++t) {
#pragma unroll
          for (int i = 0; i < NB; ++i) acc[i][t] = mfma_bf16(fm[s][i], fq[s][t], acc[i][t]);
          load_q(s, t);
#pragma unroll
          for (int i = t * NB / TQ; i < (t + 1) * NB / TQ; ++i) load_m((s + D - 1) % D, i);
          __builtin_amdgcn_sched_barrier(0);
        }
        next_q();
        next_m();
      }
    }
    const int blk0 = b_begin + step * NB;
#pragma unroll
    for (int ph = 0; ph < PH; ++ph) {
      // the phase's partial tiles of every wavefront: [wavefront][pair][1 KB]
#pragma unroll
      for (int i = 0; i < NB; ++i)
#pragma unroll
        for (int t = 0; t < TC; ++t)
          *reinterpret_cast<floatx4*>(smem + (((w * PAIRS) + i * TC + t) * kWave + lane) * 16) = acc[i][ph * TC + t];
      wait_lgkm0();
      raw_barrier();
      for (int p = w; p < PAIRS; p += W) {
        const int blk = blk0 + p / TC;
        if (blk < b_end) {
          floatx4 sum = *reinterpret_cast<const floatx4*>(smem + (p * kWave + lane) * 16);
#pragma unroll
          for (int ww = 1; ww < W; ++ww) sum += *reinterpret_cast<const floatx4*>(smem + ((ww * PAIRS + p) * kWave + lane) * 16);
          const int y0 = 16 * blk + 4 * g;
          float xn[4];
#pragma unroll
          for (int r = 0; r < 4; ++r) xn[r] = y0 + r < a.n ? a.xnorm[y0 + r] : 0.0f;
          float rx[4];
#pragma unroll
          for (int r = 0; r < 4; ++r) rx[r] = xn[r] > 0.0f ? __builtin_amdgcn_rcpf(xn[r]) : (xn[r] != xn[r] ? xn[r] : 0.0f);
          if constexpr (DENSE) {
            const int b = g0 + 16 * (ph * TC + tt) + c;
            if (b < a.B) {
              const float rq = a.rq[b];
              floatx4 v;
#pragma unroll
              for (int r = 0; r < 4; ++r) v[r] = sum[r] * rq * rx[r];
              store_dense4(a.dbg, a.mix, a.w_self, a.w_mix, a.vec16 != 0 && y0 + 3 < a.n,
                           static_cast<int64_t>(b) * a.n + y0, y0, a.n, v);
            }
          } else {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              const uint64_t key = y0 + r < a.n ? split_key(sum[r] * rx[r], y0 + r) : 0ull;
              best[ph] = key > best[ph] ? key : best[ph];
            }
          }
        }
      }
      wait_lgkm0();
      raw_barrier();
    }
#pragma unroll
    for (int i = 0; i < NB; ++i)
#pragma unroll
      for (int t = 0; t < TQ; ++t) acc[i][t] = floatx4{0.f, 0.f, 0.f, 0.f};
  }

  if constexpr (DENSE) return;   // no lists

  // merge: the four lane groups of a query, then the W / TC wavefronts of its tile
  uint64_t* mbuf = reinterpret_cast<uint64_t*>(smem);   // [W][PH][16]
#pragma unroll
  for (int ph = 0; ph < PH; ++ph) {
#pragma unroll
    for (int m = 16; m <= 32; m <<= 1) {
      const uint64_t o = shfl_xor_u64(best[ph], m);
      best[ph] = o > best[ph] ? o : best[ph];
    }
    if (g == 0) mbuf[(w * PH + ph) * 16 + c] = best[ph];
  }
  __syncthreads();
  for (int r = tid; r < QG; r += W * kWave) {
    const int t = r / 16;
    uint64_t m = 0;
#pragma unroll
    for (int ww = 0; ww < W / TC; ++ww) {
      const uint64_t o = mbuf[((t % TC + ww * TC) * PH + t / TC) * 16 + r % 16];
      m = o > m ? o : m;
    }
    a.partial[static_cast<int64_t>(g0 + r) * a.R + rr] = m;
  }
}

namespace {

template <int W, int NB, int TQ, int D, bool RAW, bool DENSE = false>
hipError_t split_launch(const SplitArgs& a, hipStream_t st) {
  using S = SplitShape<W, NB, TQ>;
  constexpr size_t red = static_cast<size_t>(W) * S::PAIRS * 1024;
  constexpr size_t mrg = static_cast<size_t>(W) * S::PH * 16 * 8;
  constexpr size_t lds = red > mrg ? red : mrg;
  static_assert(lds <= 160 * 1024, "LDS");
  static_assert(!(RAW && DENSE), "the dense form reads 1/|q| in the scan");
  auto kern = k_sem_split<W, NB, TQ, D, RAW, DENSE>;
  if (lds > 64 * 1024) {
    const hipError_t err = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                               hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds));
    if (err != hipSuccess) return err;
  }
  const ScanEvents& ev = scan_events();
  if (ev.start != nullptr) {
    const hipError_t err = hipEventRecord(ev.start, st);
    if (err != hipSuccess) return err;
  }
  hipLaunchKernelGGL(kern, dim3(a.grid), dim3(W * kWave), lds, st, a);
  const hipError_t err = hipGetLastError();
  if (err != hipSuccess || ev.stop == nullptr) return err;
  return hipEventRecord(ev.stop, st);
}

// The shapes: blocks per step, query tiles, whether they read the caller's
// rows, and what the choice of a scan weighs: a k-step (32 dimensions) of a
// step, the rest of a step (the reduction through LDS, which at d = 128 is most
// of it), and the bytes of embeddings per microsecond that bound a large store.
struct ShapeInfo {
  int nb, tq;
  bool raw;
  double kstep, step, rate;
};
constexpr ShapeInfo kShapes[] = {{1, 1, true, 0.06, 1.1, 5.0e6},
                                 {4, 1, true, 0.10, 1.3, 5.7e6},
                                 {4, 2, true, 0.16, 1.3, 4.6e6},
                                 {4, 4, false, 0.18, 1.9, 5.0e6},
                                 {4, 8, false, 0.26, 5.3, 5.0e6}};

hipError_t split_shape(int shape, const SplitArgs& a, hipStream_t st) {
  switch (shape) {
    case 0: return split_launch<8, 1, 1, 4, true>(a, st);
    case 1: return split_launch<8, 4, 1, 4, true>(a, st);
    case 2: return split_launch<8, 4, 2, 4, true>(a, st);
    case 3: return split_launch<8, 4, 4, 2, false>(a, st);
    case 4: return split_launch<8, 4, 8, 2, false>(a, st);
    default: return hipErrorInvalidValue;
  }
}

// Workgroups of a query group, and the blocks of the largest share.
int split_workgroups(int n_qg, int n_blocks, int nb) {
  const int units = (n_blocks + nb - 1) / nb;
  int R = 256 / n_qg;
  if (R > units) R = units;
  return R < 1 ? 1 : R;
}

constexpr double kPrep = 3.2;                     // k_sem_prep
constexpr double kMmStage128 = 1.16;              // a k-step of a k_sem_mm slice, groups of 128
constexpr double kMmStage256 = 1.24;              // ... and of 256
constexpr double kMmRate = 5.8e6;

}  // namespace

// The scan with the least estimated time: k_sem_prep where it runs, plus the
// longest workgroup's steps or slices (one costs about the same however many of
// its blocks exist), but no less than the embeddings take to read.  The weights
// (about microseconds) choose best over 1,500 random sizes, 200 to 800,000
// entries, d = 128 to 8192, 1 to 1,024 queries, each timed on k_sem_mm and on
// every shape here: 2 of them lose 2% or more against k_sem_mm (8% at most),
// and the mean call takes 0.37 of its time there.  (Without a cost per step,
// narrow embeddings of large stores went to a shape of up to 3.5 times
// k_sem_mm's time.)  Both sides, the call on k_sem_mm / on the best shape here,
// us: 1,000 entries of d = 4096, 8 queries 92.6 / 11.8; 955 of d = 768, 8
// queries 26.6 / 8.4; 3,540 of d = 2048, 109 queries 53.9 / 14.8; 3,503 of d =
// 768, 161 queries 28.8 / 13.9; and on k_sem_mm: 223,998 of d = 128, 33 queries
// 25.8 / 56.2; 107,404 of d = 384, 38 queries 26.8 / 34.5.
SemSplit sem_split_plan(int32_t Bc, int32_t n, int32_t d, bool dense) {
  const int n_blocks = (n + 15) / 16;
  const int ksteps = d / 32;
  const double bytes = 2.0 * n * d;
  // the full-width scan, k_sem_mm
  const int QG = sem_mm_group(Bc);
  const int SB = QG == 128 ? 32 : 16;
  const int R0 = split_workgroups((Bc + QG - 1) / QG, n_blocks, 1);
  const double slices = ((n_blocks + R0 - 1) / R0 + SB - 1) / SB;
  double best = slices * ksteps * (QG == 128 ? kMmStage128 : kMmStage256);
  if (best < bytes / kMmRate) best = bytes / kMmRate;
  best += kPrep;
  SemSplit p;
  for (int i = 0; i < static_cast<int>(sizeof(kShapes) / sizeof(kShapes[0])); ++i) {
    const ShapeInfo& si = kShapes[i];
    const int n_qg = (Bc + 16 * si.tq - 1) / (16 * si.tq);
    if (dense && si.raw) continue;
    const int R = split_workgroups(n_qg, n_blocks, si.nb);
    const double steps = ((n_blocks + R - 1) / R + si.nb - 1) / si.nb;
    double t = steps * (ksteps * si.kstep + si.step);
    if (t < bytes / si.rate) t = bytes / si.rate;
    if (!si.raw) t += kPrep;
    if (t < best) {
      best = t;
      p.shape = i;
      p.raw = si.raw;
      p.group = 16 * si.tq;
      p.R = R;
    }
  }
  return p;
}

const char* sem_split_name(const SemSplit& p) {
  constexpr const char* kNames[] = {"k_sem_split 1x1", "k_sem_split 4x1", "k_sem_split 4x2", "k_sem_split 4x4",
                                    "k_sem_split 4x8"};
  return kNames[p.shape];
}

hipError_t launch_sem_split(const StoreView& s, const SemSplit& p, const uint16_t* q, int32_t Bc,
                            const Workspace& ws, hipStream_t st, float* dbg, const float* mix, double w_self,
                           double w_mix) {
  SplitArgs a;
  a.dbg = dbg;
  a.mix = mix;
  a.w_self = w_self;
  a.w_mix = w_mix;
  a.vec16 = s.n % 4 == 0 && reinterpret_cast<uintptr_t>(dbg) % 16 == 0 && reinterpret_cast<uintptr_t>(mix) % 16 == 0;
  a.x = s.embs;
  a.xnorm = s.emb_norm;
  a.q = p.raw ? q : static_cast<const uint16_t*>(ws.qrows);
  a.rq = ws.rq;
  a.partial = ws.partial;
  a.n = s.n;
  a.d = s.d_emb;
  a.ksteps = s.d_emb / 32;
  a.B = Bc;
  a.n_qg = (Bc + p.group - 1) / p.group;
  a.R = p.R;
  a.n_blocks = (s.n + 15) / 16;
  a.grid = (a.n_qg * a.R + 7) / 8 * 8;
  if (dbg != nullptr) {
    if (p.shape == 3) return split_launch<8, 4, 4, 2, false, true>(a, st);
    if (p.shape == 4) return split_launch<8, 4, 8, 2, false, true>(a, st);
    return hipErrorInvalidValue;
  }
  return split_shape(p.shape, a, st);
}

}  // namespace fm
