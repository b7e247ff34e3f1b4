// Trajectory-based expert map search (Section 4.2.2, Eq. 5), split-depth form
// for small stores and batches.
//
// The general scan (fm_traj.hip) walks the layer groups of a slice one after
// the other behind a barrier each, so a store of a few slices costs 12 to 46
// dependent stages however small it is.  Here the 8 wavefronts of a workgroup
// split the k-steps of the observed layers instead: each accumulates the whole
// tile of 16 NB maps x 16 TQ queries over its own run of k-steps, reading the
// map quads and the staged query rows (k_traj_prep) straight into registers
// two k-steps ahead, with no barrier in the loop.  At the end of a step the 8
// partial tiles are summed through LDS, each (block, query tile) pair by one
// wavefront, which scales the sums by the two prefix inverse norms at the
// query's depth and keeps its query tile's best in per-lane top-K lists.  A
// query tile takes part in the layer groups that its deepest query reaches, as
// in the general scan (so a NaN or infinity stored in a deep layer stays out
// of shallower tiles); shallower queries of a tile add zeros, as their staged
// rows are zero past their depth.  Operands, products and their float16 split
// are those of the general scan.
//
// Measured (scan alone): 1,000 float32 maps of 24 x 60, 8 queries 25.5 -> 6.1
// us; of 32 x 8 9.2 -> 4.5 us; 4,000 bf16 maps of 24 x 60, 100 queries 30.3 ->
// 9.5 us.  Bound by the latency of its loads (D = 2 k-steps in flight; a
// larger store is bound by the query rows it reads again for every step, which
// the general scan keeps in LDS for 128 or 256 maps at a time).
#include <type_traits>

#include "fm_device.h"
#include "fm_internal.h"
#include "fm_traj_geo.h"

namespace fm {

namespace {

struct SplitTrajArgs {
  const char* planes;
  uint64_t plane_bytes;
  uint32_t tile_bytes;   // bytes of one 16-map tile of a plane
  const float* rnorm;    // [L][rn_stride] prefix inverse norms
  int64_t rn_stride;
  const char* qrows;     // staged query planes
  const int32_t* sdep;   // [b_pad] depth at each sorted position (0: padding)
  const float* rq;       // [b_pad] 1/|q[0:p]|
  uint64_t* partial;     // [b_pad][R][KTOP]
  int32_t n, L, row, b_pad;
  Geo geo;
  int32_t n_qg, R, n_blocks, grid;
};

constexpr int kSW = 8;   // wavefronts per workgroup
constexpr int kSD = 2;   // k-steps in flight

}  // namespace

template <bool BF, int KSG, int NB, int TQ, int KTOP>
__global__ void __launch_bounds__(kSW * 64) __attribute__((amdgpu_waves_per_eu(2, 2))) k_traj_split(SplitTrajArgs a) {
  using Raw = typename std::conditional<BF, u16x8, floatx8>::type;
  constexpr int W = kSW, D = kSD;
  constexpr int esz = BF ? 2 : 4;
  constexpr int NP = BF ? 1 : 2;
  constexpr int QG = 16 * TQ;
  constexpr int RB = 64 * KSG;
  constexpr int PAIRS = NB * TQ;
  static_assert(W % TQ == 0, "a wavefront sums one query tile");
  extern __shared__ __align__(16) unsigned char smem[];   // [W][PAIRS][1 KB]; then the merge

  const int tid = threadIdx.x;
  const int w = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int lane = tid % kWave;
  const int g = lane / 16;
  const int c = lane % 16;
  // workgroup -> (query group, block range), the groups of a range on one XCD
  const int bid = blockIdx.x;
  const int u = (bid % 8) * (a.grid / 8) + bid / 8;
  if (u >= a.n_qg * a.R) return;
  const int qgrp = __builtin_amdgcn_readfirstlane(u % a.n_qg);
  const int rr = __builtin_amdgcn_readfirstlane(u / a.n_qg);
  const int b_begin = __builtin_amdgcn_readfirstlane(static_cast<int>((static_cast<int64_t>(rr) * a.n_blocks) / a.R));
  const int b_end = __builtin_amdgcn_readfirstlane(static_cast<int>((static_cast<int64_t>(rr + 1) * a.n_blocks) / a.R));
  const int n_steps = (b_end - b_begin + NB - 1) / NB;
  const int g0 = qgrp * QG;

  TopK<KTOP> best;
  best.clear();

  // the group's k-steps (its deepest query is its first position), and this
  // wavefront's run of them, padded to a multiple of D (padding reads zeros)
  const int dg = __builtin_amdgcn_readfirstlane(a.sdep[g0]);
  const int units = ((dg + a.geo.lpg - 1) / a.geo.lpg) * KSG;
  const int u0 = (w * units) / W;
  const int u1 = ((w + 1) * units) / W;
  const int kp = ((units + W - 1) / W + D - 1) / D * D;

  // lane constants: the map quads of k position 4g.. and 16 + 4g.. of each
  // k-step of a layer group, and the query rows' units
  uint32_t moff[KSG][2], qoff[KSG];
#pragma unroll
  for (int ks = 0; ks < KSG; ++ks) {
#pragma unroll
    for (int half = 0; half < 2; ++half) {
      const int s0 = 32 * ks + 16 * half + 4 * g;
      const int li = s0 / a.geo.spl;
      const int e0 = s0 - li * a.geo.spl;
      moff[ks][half] = e0 < a.row ? static_cast<uint32_t>(li) * static_cast<uint32_t>(a.plane_bytes) +
                                        static_cast<uint32_t>(((e0 / 4) * 64 + c * 4) * esz)
                                  : kOutside;
    }
    qoff[ks] = static_cast<uint32_t>(c * RB + 16 * (KSG > 1 ? (4 * ks + g) ^ (c & 7) : 4 * ks + g));
  }

  // the loads' position, D k-steps ahead of the products
  int c_blk = b_begin;
  int c_k = 0;
  Raw fm[D][NB];
  u16x8 fq[D][NP][TQ];
  auto load = [&](int s) __attribute__((always_inline)) {
    const bool in = u0 + c_k < u1 && c_blk < b_end;
    const int un = in ? u0 + c_k : 0;
    const int lg = un / KSG;
    const int ks = un - lg * KSG;
    const int l0 = lg * a.geo.lpg;
    const int nl = a.L - l0 < a.geo.lpg ? a.L - l0 : a.geo.lpg;
    const __amdgpu_buffer_rsrc_t rs_m = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<char*>(a.planes + static_cast<uint64_t>(static_cast<uint32_t>(l0)) * a.plane_bytes),
        static_cast<short>(0), static_cast<int>(in ? static_cast<uint32_t>(nl) * static_cast<uint32_t>(a.plane_bytes) : 0u),
        kBufWord3);
    const __amdgpu_buffer_rsrc_t rs_q = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<char*>(a.qrows + (static_cast<int64_t>(lg) * a.b_pad + g0) * (NP * RB)), static_cast<short>(0),
        static_cast<int>(in ? static_cast<uint32_t>(QG * NP * RB) : 0u), kBufWord3);
    const uint32_t mlo = KSG == 1 || ks == 0 ? moff[0][0] : moff[KSG - 1][0];
    const uint32_t mhi = KSG == 1 || ks == 0 ? moff[0][1] : moff[KSG - 1][1];
    const uint32_t qo = KSG == 1 || ks == 0 ? qoff[0] : qoff[KSG - 1];
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      // (blocks past the range, and quads past the row, lie outside)
      const bool blk_in = c_blk + i < b_end;
      const uint32_t bo = static_cast<uint32_t>(c_blk + i) * a.tile_bytes;
      const uint32_t lo = blk_in && mlo != kOutside ? mlo + bo : kOutside;
      const uint32_t hi = blk_in && mhi != kOutside ? mhi + bo : kOutside;
      if constexpr (BF) {
        const uint32x2 vl = __builtin_amdgcn_raw_buffer_load_b64(rs_m, static_cast<int>(lo), 0, 0);
        const uint32x2 vh = __builtin_amdgcn_raw_buffer_load_b64(rs_m, static_cast<int>(hi), 0, 0);
        fm[s][i] = __builtin_bit_cast(u16x8, uint32x4{vl[0], vl[1], vh[0], vh[1]});
      } else {
        const uint32x4 vl = __builtin_amdgcn_raw_buffer_load_b128(rs_m, static_cast<int>(lo), 0, 0);
        const uint32x4 vh = __builtin_amdgcn_raw_buffer_load_b128(rs_m, static_cast<int>(hi), 0, 0);
        fm[s][i] = floatx8{__uint_as_float(vl[0]), __uint_as_float(vl[1]), __uint_as_float(vl[2]), __uint_as_float(vl[3]),
                           __uint_as_float(vh[0]), __uint_as_float(vh[1]), __uint_as_float(vh[2]), __uint_as_float(vh[3])};
      }
    }
#pragma unroll
    for (int pl = 0; pl < NP; ++pl)
#pragma unroll
      for (int t = 0; t < TQ; ++t)
        fq[s][pl][t] = __builtin_bit_cast(
            u16x8, __builtin_amdgcn_raw_buffer_load_b128(rs_q, static_cast<int>(qo + static_cast<uint32_t>((pl * QG + 16 * t) * RB)), 0, 0));
    if (++c_k == kp) {
      c_k = 0;
      c_blk += NB;
    }
  };

  floatx4 acc[NB][TQ];
#pragma unroll
  for (int i = 0; i < NB; ++i)
#pragma unroll
    for (int t = 0; t < TQ; ++t) acc[i][t] = floatx4{0.f, 0.f, 0.f, 0.f};

#pragma unroll
  for (int s = 0; s < D; ++s) load(s);

  // this wavefront's query tile, and this lane's query of it
  const int tt = w % TQ;
  const int p = a.sdep[g0 + 16 * tt + c];
  const float rq = a.rq[g0 + 16 * tt + c];
  const float* rrow = a.rnorm + static_cast<int64_t>(p > 0 ? p - 1 : 0) * a.rn_stride + 4 * g;

  // depth of each tile's deepest query, its first position
  int tmd[TQ];
#pragma unroll
  for (int t = 0; t < TQ; ++t) tmd[t] = __builtin_amdgcn_readfirstlane(a.sdep[g0 + 16 * t]);

  // products of the k-step in registers s for the first NT query tiles
  auto products = [&](auto nt_const, int s, const u16x8 (&ap)[NP][NB]) __attribute__((always_inline)) {
    constexpr int NT = decltype(nt_const)::value;
    if constexpr (BF) {
#pragma unroll
      for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int i = 0; i < NB; ++i) acc[i][t] = mfma_bf16(ap[0][i], fq[s][0][t], acc[i][t]);
    } else {
      // hi x lo, hi x hi, lo x hi
      constexpr int TA[3] = {0, 0, 1};
      constexpr int TB[3] = {1, 0, 0};
#pragma unroll
      for (int term = 0; term < 3; ++term)
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
          for (int i = 0; i < NB; ++i) acc[i][t] = mfma_f16(ap[TA[term]][i], fq[s][TB[term]][t], acc[i][t]);
    }
  };

  for (int step = 0; step < n_steps; ++step) {
    for (int ki = 0; ki < kp; ki += D) {
#pragma unroll
      for (int s = 0; s < D; ++s) {
        u16x8 ap[NP][NB];
#pragma unroll
        for (int i = 0; i < NB; ++i) {
          if constexpr (BF) ap[0][i] = fm[s][i];
          else split2(fm[s][i], ap[0][i], ap[NP - 1][i]);
        }
        // the tiles whose deepest query reaches this layer group (positions
        // are sorted by depth, so they come first; tile 0 always does)
        const int l_first = (u0 + ki + s) / KSG * a.geo.lpg;
        int na = 1;
#pragma unroll
        for (int t = 1; t < TQ; ++t) na += tmd[t] > l_first ? 1 : 0;
        if (TQ == 1 || na == 1) products(std::integral_constant<int, 1>{}, s, ap);
        else if (TQ == 2 || na == 2) products(std::integral_constant<int, TQ < 2 ? TQ : 2>{}, s, ap);
        else if (na == 3) products(std::integral_constant<int, TQ < 3 ? TQ : 3>{}, s, ap);
        else products(std::integral_constant<int, TQ>{}, s, ap);
        load(s);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    const int blk0 = b_begin + step * NB;
#pragma unroll
    for (int i = 0; i < NB; ++i)
#pragma unroll
      for (int t = 0; t < TQ; ++t)
        *reinterpret_cast<floatx4*>(smem + (((w * PAIRS) + i * TQ + t) * kWave + lane) * 16) = acc[i][t];
    wait_lgkm0();
    raw_barrier();
    for (int pr = w; pr < PAIRS; pr += W) {
      const int blk = blk0 + pr / TQ;
      if (blk < b_end) {
        const int y0 = 16 * blk + 4 * g;
        const floatx4 rn = *reinterpret_cast<const floatx4*>(rrow + 16 * blk);
        floatx4 sum = *reinterpret_cast<const floatx4*>(smem + (pr * kWave + lane) * 16);
#pragma unroll
        for (int ww = 1; ww < W; ++ww)
          sum += *reinterpret_cast<const floatx4*>(smem + ((ww * PAIRS + pr) * kWave + lane) * 16);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const float dot = BF ? sum[r] : sum[r] * kDotUnscale;
          if (p != 0 && y0 + r < a.n) best.push(make_key(dot * rq * rn[r], y0 + r));
        }
      }
    }
    wait_lgkm0();
    raw_barrier();
#pragma unroll
    for (int i = 0; i < NB; ++i)
#pragma unroll
      for (int t = 0; t < TQ; ++t) acc[i][t] = floatx4{0.f, 0.f, 0.f, 0.f};
  }

  // merge: the four lane groups of a query, then the W / TQ wavefronts of its tile
  uint64_t* mbuf = reinterpret_cast<uint64_t*>(smem);   // [W][16][KTOP]
#pragma unroll
  for (int m = 16; m <= 32; m <<= 1) {
    uint64_t o[KTOP];
#pragma unroll
    for (int jj = 0; jj < KTOP; ++jj) o[jj] = shfl_xor_u64(best.v[jj], m);
    best.merge(o);
  }
  if (g == 0) {
#pragma unroll
    for (int jj = 0; jj < KTOP; ++jj) mbuf[(w * 16 + c) * KTOP + jj] = best.v[jj];
  }
  __syncthreads();
  for (int r = tid; r < QG; r += W * kWave) {
    TopK<KTOP> m;
    m.clear();
#pragma unroll
    for (int ww = 0; ww < W / TQ; ++ww) m.merge(mbuf + ((r / 16 + ww * TQ) * 16 + r % 16) * KTOP);
    uint64_t* out = a.partial + (static_cast<int64_t>(g0 + r) * a.R + rr) * KTOP;
#pragma unroll
    for (int jj = 0; jj < KTOP; ++jj) out[jj] = m.v[jj];
  }
}

namespace {

template <bool BF, int KSG, int NB, int TQ, int KTOP>
hipError_t split_launch(const SplitTrajArgs& a, hipStream_t st) {
  constexpr size_t red = static_cast<size_t>(kSW) * NB * TQ * 1024;
  constexpr size_t mrg = static_cast<size_t>(kSW) * 16 * KTOP * 8;
  constexpr size_t lds = red > mrg ? red : mrg;
  static_assert(lds <= 64 * 1024, "LDS");
  const ScanEvents& ev = scan_events();
  if (ev.start != nullptr) {
    const hipError_t err = hipEventRecord(ev.start, st);
    if (err != hipSuccess) return err;
  }
  hipLaunchKernelGGL((k_traj_split<BF, KSG, NB, TQ, KTOP>), dim3(a.grid), dim3(kSW * kWave), lds, st, a);
  const hipError_t err = hipGetLastError();
  if (err != hipSuccess || ev.stop == nullptr) return err;
  return hipEventRecord(ev.stop, st);
}

template <bool BF, int KSG, int KTOP>
hipError_t split_shape(int shape, const SplitTrajArgs& a, hipStream_t st) {
  switch (shape) {
    case 0: return split_launch<BF, KSG, 1, 1, KTOP>(a, st);
    case 1: return split_launch<BF, KSG, 2, 2, KTOP>(a, st);
    case 2: return split_launch<BF, KSG, 2, 4, KTOP>(a, st);
    default: return hipErrorInvalidValue;
  }
}

template <bool BF, int KSG>
hipError_t split_k(int KTOP, int shape, const SplitTrajArgs& a, hipStream_t st) {
  if (KTOP == 1) return split_shape<BF, KSG, 1>(shape, a, st);
  if (KTOP == 4) return split_shape<BF, KSG, 4>(shape, a, st);
  return split_shape<BF, KSG, 8>(shape, a, st);
}

// The shapes: blocks per step and query tiles.
struct ShapeInfo {
  int nb, tq;
};
constexpr ShapeInfo kShapes[] = {{1, 1}, {2, 2}, {2, 4}};

// What the choice of a scan weighs (about microseconds).
struct Weights {
  double stage[4];    // a stage (layer group of a slice) of k_traj_scan with 1, 2, 4 and 8 query tiles
  double two_ksteps;  // ... times this where a layer group is two k-steps
  double slice;       // a slice of k_traj_scan
  double score[3];    // ... and the ranking of 8 (map block, query tile) pairs of it in lists of 1, 4 and 8
  double mm_stage;    // a k-step of a k_traj_mm slice
  double mm_slice;    // a slice of it
  double kstep[3];    // a k-step of a wavefront of k_traj_split, by shape
  double step[3];     // the rest of a step of it
  double lists[3];    // ... times this for lists of 1, 4 and 8
};
constexpr Weights kF32 = {{0.8, 1.05, 1.2, 1.4}, 1.5, 2.4, {3.0, 9.6, 10.2}, 0.0, 0.0,
                          {0.75, 1.35, 2.2}, {0.8, 1.3, 1.35}, {1.0, 1.05, 1.15}};
constexpr Weights kBf16 = {{1.25, 1.45, 1.75, 1.9}, 1.7, 2.7, {5.2, 9.3, 13.15}, 1.9, 5.05,
                           {1.05, 1.65, 2.45}, {0.95, 1.3, 1.45}, {1.0, 1.1, 1.65}};

constexpr double kMostSlices = 3.0;   // of the other scan, with which the split-depth scan competes
constexpr double kSplitRate = 4.0e6, kScanRate = 5.4e6;   // bytes of planes per microsecond that bound a large store

}  // namespace

// The scan with the least estimated time: the longest workgroup's dependent
// stages or k-steps and the ranking that ends a slice or step, but no less than
// the planes take to read.  The weights are fitted to 3,700 random sizes (200
// to 150,000 maps of twelve shapes, 1 to 1,024 queries, lists of 1, 4 and 8,
// depths uniform, geometric and full), each timed on the other scan and on
// every shape here: four of them lose 3% or more against the other scan (6% at
// most), and the mean call takes 0.72 of its time there.  The depths are not
// known on the host, and shallow batches of several groups are much quicker on
// the other scan than deep ones: some deep batches stay there that would gain
// here.  A scan whose workgroups walk more than three slices keeps its loads and
// stages overlapped, which the weights do not show, and stays (of 2,698 sizes
// where a shape here was 3% quicker, 10 lie there; float32 16 x 20, 79,793 maps,
// top-8 of 870 queries 323 us there, 569 here).  (Without the ranking, and with
// every stage weighed at what the first one of a scan costs, calls took up to
// 2.9 times the other scan's time.)  Both sides, the call on the other scan / on
// the best shape here, us: float32 32 x 8, 1,000 maps, 8 queries 18.6 / 14.3; 24
// x 60, 6,766 maps, 4 queries 36.3 / 15.6; bf16 61 x 33, 28,275 maps, 2 queries
// 52.0 / 23.5; and on the other scan: float32 24 x 60, 23,877 maps, 322 queries
// 98.8 / 182.8, 26 x 60, 20,420 maps, 80 queries 48.7 / 72.8.
TrajSplit traj_split_plan(bool bf, int32_t n, int32_t row, const Geo& geo, int32_t Bc, int KTOP, int nlg, int TQ,
                          int nba, bool mm) {
  const Weights& wt = bf ? kBf16 : kF32;
  const int kl = KTOP == 1 ? 0 : (KTOP == 4 ? 1 : 2);
  const int n_blocks = (n + 15) / 16;
  const double bytes = static_cast<double>(n) * nlg * geo.lpg * row * (bf ? 2 : 4);
  double best, slices;
  if (mm) {
    const int all = (n_blocks + 15) / 16 * ((Bc + traj_mm_group() - 1) / traj_mm_group());
    slices = (all + traj_mm_workgroups() - 1) / traj_mm_workgroups();
    best = slices * (nlg * geo.ksg * wt.mm_stage + wt.mm_slice);
  } else {
    const int n_qg = (Bc + 16 * TQ - 1) / (16 * TQ);
    // (one group's workgroups walk whole slices; several groups share the
    // workgroups by their cost)
    int R = 256 / n_qg;
    if (R > n_blocks) R = n_blocks;
    if (R < 1) R = 1;
    const int sw = 128 * nba;   // maps per slice
    const int maps = (n + R - 1) / R;
    slices = (maps + sw - 1) / sw;
    if (n_qg > 1) slices = static_cast<double>(n) * n_qg / (256.0 * sw);
    if (n_qg > 1 && slices < 1.0) slices = 1.0;
    const double stage = wt.stage[TQ == 1 ? 0 : (TQ == 2 ? 1 : (TQ == 4 ? 2 : 3))] * (geo.ksg == 2 ? wt.two_ksteps : 1.0);
    best = slices * (nlg * stage + wt.slice + wt.score[kl] * TQ * nba / 8.0);
  }
  if (best < bytes / kScanRate) best = bytes / kScanRate;
  const int run = ((nlg * geo.ksg + kSW - 1) / kSW + kSD - 1) / kSD * kSD;   // k-steps of a wavefront
  TrajSplit p;
  if (slices > kMostSlices) return p;
  for (int i = 0; i < static_cast<int>(sizeof(kShapes) / sizeof(kShapes[0])); ++i) {
    const ShapeInfo& si = kShapes[i];
    const int n_qg = (Bc + 16 * si.tq - 1) / (16 * si.tq);
    const int units = (n_blocks + si.nb - 1) / si.nb;
    int R = 256 / n_qg;
    if (R > units) R = units;
    if (R < 1) R = 1;
    const int steps = ((n_blocks + R - 1) / R + si.nb - 1) / si.nb;
    double t = steps * (run * wt.kstep[i] + wt.step[i] * wt.lists[kl]);
    if (t < bytes / kSplitRate) t = bytes / kSplitRate;
    if (t < best) {
      best = t;
      p.shape = i;
      p.group = 16 * si.tq;
      p.R = R;
    }
  }
  return p;
}

const char* traj_split_name(const TrajSplit& p) {
  return p.shape == 0 ? "k_traj_split 1x1" : p.shape == 1 ? "k_traj_split 2x2" : "k_traj_split 2x4";
}

hipError_t launch_traj_split(const StoreView& s, const TrajSplit& p, const Geo& geo, int32_t Bc, int32_t b_pad,
                             int KTOP, const Workspace& ws, hipStream_t st) {
  const bool bf = s.map_dtype == FM_BF16;
  const int esz = bf ? 2 : 4;
  SplitTrajArgs a;
  a.planes = static_cast<const char*>(s.planes);
  a.plane_bytes = static_cast<uint64_t>(s.plane_elems) * esz;
  a.tile_bytes = static_cast<uint32_t>(16 * s.row * esz);
  a.rnorm = s.rnorm;
  a.rn_stride = s.rn_stride;
  a.qrows = static_cast<const char*>(ws.qrows);
  a.sdep = ws.sdep;
  a.rq = ws.rq;
  a.partial = ws.partial;
  a.n = s.n;
  a.L = s.L;
  a.row = s.row;
  a.b_pad = b_pad;
  a.geo = geo;
  a.n_qg = (Bc + p.group - 1) / p.group;
  a.R = p.R;
  a.n_blocks = (s.n + 15) / 16;
  a.grid = (a.n_qg * a.R + 7) / 8 * 8;
  if (bf) return geo.ksg == 1 ? split_k<true, 1>(KTOP, p.shape, a, st) : split_k<true, 2>(KTOP, p.shape, a, st);
  return geo.ksg == 1 ? split_k<false, 1>(KTOP, p.shape, a, st) : split_k<false, 2>(KTOP, p.shape, a, st);
}

}  // namespace fm
