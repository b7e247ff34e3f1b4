// Incremental trajectory re-search (Section 4.2.2): within one pass the
// trajectory search is repeated after every newly observed layer, each time
// with the prefix grown by one layer.  The Eq. 5 cosine over the first p
// layers is dot_p / (|q[0:p]| |x[y][0:p]|) with dot_p = dot_{p-1} + the new
// layer's dot product, so a step keeps the running dot of every (query,
// stored map) pair in a caller-owned state buffer and reads one map plane
// instead of p.
//
//   k_traj_step   one 16-map tile of the store per wave: the layer's dot
//                 products by float32 MFMA (16 maps x 16 queries x 4 experts
//                 per instruction, exact float32 products), added onto the
//                 running dots, scored with the stored prefix inverse norm at
//                 depth p and the query's running float64 norm, per-lane
//                 top-K, merged per workgroup into partial lists; workgroup 0
//                 also advances the query norms and checks the state header
//                 (same store size as at layer 0, layers in order);
//   k_finalize    (shared with the scans) merges the partial lists.
#include "fm_device.h"
#include "fm_internal.h"

namespace fm {

namespace {

constexpr int kStepQ = 64;        // queries per chunk (4 query tiles)
constexpr int kStepW = 4;         // waves per workgroup
constexpr int kStepThreads = kStepW * kWave;
// partial lists of a launch at most (the match workspace's)
constexpr int kStepMaxLists = kChunkB * kMaxPartials;

struct StepHeader {
  int32_t n_begin;     // store size at layer 0
  int32_t last_layer;  // last layer added
};

// State of one chunk of kStepQ queries: [header, 256 B][query sums of squares
// after even layers: kStepQ float64][after odd layers: kStepQ float64]
// [dots: n_tiles x 4 query tiles x 64 lanes x 4 float32].  A step reads the
// sums in the previous layer's slot and workgroup 0 writes the other slot, so
// no workgroup reads a slot while it is written.
constexpr size_t kStepHead = 256 + 2 * kStepQ * 8;

struct StepArgs {
  const void* planes;
  int64_t plane_elems;
  const float* rnorm;
  int64_t rn_stride;
  int32_t n, E, row, layer, B;
  int32_t R, n_tiles;   // workgroups per chunk; 16-map tiles of the store
  const void* q;        // [B][E]
  char* state;          // the chunks' states, chunk_bytes apart
  int64_t chunk_bytes;
  uint64_t* partial;    // [B][R][KTOP]
  uint32_t* flags;
};

}  // namespace

// Lane (g, c) = (lane / 16, lane % 16).  For 4 quads of experts at a time,
// lane (g, c) loads quad 4s+g of map c of the tile (one 16-byte load: 4
// consecutive experts) and holds the same 4 experts of query c of its query
// tile; the j-th MFMA of the group takes the j-th of those experts, so the 4
// MFMAs together cover experts 16s .. 16s+15 (the k index of a product does
// not matter to the dot product).  The accumulator of lane (g, c) holds maps
// 4g .. 4g+3 of the tile for query c.
//
// A workgroup takes a contiguous range of tiles; its 4 waves split into TQ
// query tiles x (4 / TQ) phases: wave w serves query tile w % TQ and the
// tiles of the range with index = w / TQ modulo 4 / TQ.  Each wave keeps the
// loads of its next two tiles in flight: the tile loop is unrolled over the
// three register sets and every load is a buffer load without a branch (quads
// past the row, tiles past the range and the running dots of layer 0 lie
// outside their descriptors and read as zeros), so that the compiler can
// count the loads in flight.  With the set chosen by a test in the loop and
// guarded loads, it waited for all of them at every join, and prefetching any
// number of tiles ahead made no difference.  NQ: groups of 4 quads (16
// experts) of a row.
template <bool BF, int TQ, int NQ, int KTOP>
__global__ void __launch_bounds__(kStepThreads) k_traj_step(StepArgs a) {
  constexpr int NPH = kStepW / TQ;   // phases
  constexpr int P = 3;               // register buffers: current + 2 ahead
  __shared__ uint64_t mbuf[kStepW][16][KTOP];
  using T = typename std::conditional<BF, uint16_t, float>::type;
  const int tid = threadIdx.x;
  const int w = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int lane = tid % kWave;
  const int g = lane / 16;
  const int c = lane % 16;
  const int qt = w % TQ;
  const int ph = w / TQ;
  constexpr int esz = sizeof(T);
  const int nquads = a.row / 4;
  const T* plane = static_cast<const T*>(a.planes) + static_cast<int64_t>(a.layer) * a.plane_elems;
  const float* rn = a.rnorm + static_cast<int64_t>(a.layer) * a.rn_stride;
  // chunk blockIdx.y: its queries and state
  const int b0 = static_cast<int>(blockIdx.y) * kStepQ;
  const int Bc = a.B - b0 < kStepQ ? a.B - b0 : kStepQ;
  char* state = a.state + static_cast<int64_t>(blockIdx.y) * a.chunk_bytes;
  float* dots = reinterpret_cast<float*>(state + kStepHead);
  const int t_begin = static_cast<int>((static_cast<int64_t>(blockIdx.x) * a.n_tiles) / a.R);
  const int t_end = static_cast<int>((static_cast<int64_t>(blockIdx.x + 1) * a.n_tiles) / a.R);

  const uint32_t tile_bytes = static_cast<uint32_t>(16 * a.row * esz);
  uint32_t qoff[NQ];   // this lane's bytes of quad 4s + g of a tile
#pragma unroll
  for (int s = 0; s < NQ; ++s) {
    const int quad = 4 * s + g;
    qoff[s] = quad < nquads ? static_cast<uint32_t>((quad * 64 + c * 4) * esz) : kOutside;
  }
  struct Raw {
    uint32x4 av[NQ];   // bf16: two words each
    uint32x4 prev, rs;
  };
  auto load_tile = [&](int tile, Raw& r) __attribute__((always_inline)) {
    const int tl = __builtin_amdgcn_readfirstlane(tile);
    const bool in = tl < t_end;
    const uint64_t tu = static_cast<uint64_t>(static_cast<uint32_t>(in ? tl : 0));
    const __amdgpu_buffer_rsrc_t rs_p = __builtin_amdgcn_make_buffer_rsrc(
        reinterpret_cast<char*>(reinterpret_cast<uint64_t>(plane) + tu * tile_bytes), static_cast<short>(0),
        static_cast<int>(in ? tile_bytes : 0u), kBufWord3);
    const __amdgpu_buffer_rsrc_t rs_d = __builtin_amdgcn_make_buffer_rsrc(
        reinterpret_cast<char*>(reinterpret_cast<uint64_t>(dots) + tu * 4096u + static_cast<uint32_t>(qt) * 1024u),
        static_cast<short>(0), static_cast<int>(in && a.layer != 0 ? 1024u : 0u), kBufWord3);
    const __amdgpu_buffer_rsrc_t rs_n = __builtin_amdgcn_make_buffer_rsrc(
        reinterpret_cast<char*>(reinterpret_cast<uint64_t>(rn) + tu * 64u), static_cast<short>(0),
        static_cast<int>(in ? 64u : 0u), kBufWord3);
#pragma unroll
    for (int s = 0; s < NQ; ++s) {
      if constexpr (BF) {
        const uint32x2 h = __builtin_amdgcn_raw_buffer_load_b64(rs_p, static_cast<int>(qoff[s]), 0, 0);
        r.av[s] = uint32x4{h[0], h[1], 0u, 0u};
      } else {
        r.av[s] = __builtin_amdgcn_raw_buffer_load_b128(rs_p, static_cast<int>(qoff[s]), 0, 0);
      }
    }
    r.prev = __builtin_amdgcn_raw_buffer_load_b128(rs_d, lane * 16, 0, 0);
    r.rs = __builtin_amdgcn_raw_buffer_load_b128(rs_n, g * 16, 0, 0);
  };

  // the first tiles' loads go out before anything else
  Raw raw[P];
#pragma unroll
  for (int i = 0; i < P - 1; ++i) load_tile(t_begin + ph + i * NPH, raw[i]);

  // query operands of query tile qt: experts 16s + 4g .. +3 of query 16qt + c
  const int b = 16 * qt + c;
  floatx4 bq[NQ];
#pragma unroll
  for (int s = 0; s < NQ; ++s) {
    floatx4 v = floatx4{0.f, 0.f, 0.f, 0.f};
    const int e0 = 16 * s + 4 * g;
    if (b < Bc) {
      const int64_t k = static_cast<int64_t>(b0 + b) * a.E + e0;
      if (!BF && a.E % 4 == 0 && e0 < a.E) {
        v = *reinterpret_cast<const floatx4*>(static_cast<const float*>(a.q) + k);
      } else {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          if (e0 + j < a.E)
            v[j] = BF ? bf16_to_f32(static_cast<const uint16_t*>(a.q)[k + j]) : static_cast<const float*>(a.q)[k + j];
        }
      }
    }
    bq[s] = v;
  }
  // 1/|q[0:p]|: the previous layers' float64 sum of squares plus this
  // layer's (lane partials, then across the 4 lane groups of a query)
  double* qsq = reinterpret_cast<double*>(state + 256);
  double sq = 0.0;
#pragma unroll
  for (int s = 0; s < NQ; ++s)
#pragma unroll
    for (int j = 0; j < 4; ++j) sq += static_cast<double>(bq[s][j]) * static_cast<double>(bq[s][j]);
  sq += __shfl_xor(sq, 16, kWave);
  sq += __shfl_xor(sq, 32, kWave);
  const double tot = (a.layer == 0 ? 0.0 : qsq[((a.layer - 1) & 1) * kStepQ + b]) + sq;
  if (blockIdx.x == 0 && ph == 0 && g == 0) qsq[(a.layer & 1) * kStepQ + b] = tot;
  float rq;
  if (tot != tot) rq = __uint_as_float(0x7fc00000u);
  else if (tot == 0.0) rq = 0.0f;
  else rq = static_cast<float>(1.0 / sqrt(tot));
  if (blockIdx.x == 0 && tid == 0) {
    StepHeader* h = reinterpret_cast<StepHeader*>(state);
    if (a.layer == 0) {
      h->n_begin = a.n;
    } else if (h->n_begin != a.n || h->last_layer != a.layer - 1) {
      atomicOr(a.flags, static_cast<uint32_t>(FM_FLAG_STATE_STALE));
    }
    h->last_layer = a.layer;
  }

  TopK<KTOP> best;
  best.clear();
  const bool live_q = b < Bc;
  auto use_tile = [&](int tl, const Raw& r) __attribute__((always_inline)) {
    floatx4 d = __builtin_bit_cast(floatx4, r.prev);
#pragma unroll
    for (int s = 0; s < NQ; ++s) {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        float x;
        if constexpr (BF) x = __uint_as_float(j % 2 == 0 ? r.av[s][j / 2] << 16 : r.av[s][j / 2] & 0xffff0000u);
        else x = __uint_as_float(r.av[s][j]);
        d = __builtin_amdgcn_mfma_f32_16x16x4f32(x, bq[s][j], d, 0, 0, 0);
      }
    }
    *reinterpret_cast<floatx4*>(dots + (static_cast<int64_t>(tl) * 4 + qt) * 256 + lane * 4) = d;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int y = 16 * tl + 4 * g + k;
      const float sv = d[k] * rq * __uint_as_float(r.rs[k]);
      if constexpr (KTOP == 1) {
        const uint64_t key = live_q && y < a.n ? make_key(sv, y) : 0ull;   // (no branch)
        best.v[0] = key > best.v[0] ? key : best.v[0];
      } else {
        if (live_q && y < a.n) best.push(make_key(sv, y));
      }
    }
  };
  for (int tl = t_begin + ph; tl < t_end; tl += P * NPH) {
#pragma unroll
    for (int u = 0; u < P; ++u) {
      const int cur = tl + u * NPH;
      if (cur >= t_end) break;
      load_tile(cur + (P - 1) * NPH, raw[(u + P - 1) % P]);
      use_tile(cur, raw[u]);
    }
  }

  // merge the 4 lane groups, then the phases of each query tile
#pragma unroll
  for (int m = 16; m <= 32; m <<= 1) {
    uint64_t o[KTOP];
#pragma unroll
    for (int jj = 0; jj < KTOP; ++jj) o[jj] = shfl_xor_u64(best.v[jj], m);
    best.merge(o);
  }
  if (g == 0) {
#pragma unroll
    for (int jj = 0; jj < KTOP; ++jj) mbuf[w][c][jj] = best.v[jj];
  }
  __syncthreads();
  if (tid < 16 * TQ) {
    const int r = tid;
    const int rqt = r / 16;
    if (r < Bc) {
      TopK<KTOP> m;
      m.clear();
#pragma unroll
      for (int p2 = 0; p2 < NPH; ++p2) m.merge(mbuf[p2 * TQ + rqt][r % 16]);
      uint64_t* out = a.partial + (static_cast<int64_t>(b0 + r) * a.R + blockIdx.x) * KTOP;
#pragma unroll
      for (int jj = 0; jj < KTOP; ++jj) out[jj] = m.v[jj];
    }
  }
}

namespace {

size_t chunk_state_bytes(int32_t cap) {
  return kStepHead + static_cast<size_t>(round16(cap) / 16) * 4 * 256 * sizeof(float);
}

template <bool BF, int KTOP, int NQ>
void launch_step_tq(int TQ, const StepArgs& a, hipStream_t st) {
  const dim3 grid(a.R, (a.B + kStepQ - 1) / kStepQ);
  if (TQ == 1) hipLaunchKernelGGL((k_traj_step<BF, 1, NQ, KTOP>), grid, dim3(kStepThreads), 0, st, a);
  else if (TQ == 2) hipLaunchKernelGGL((k_traj_step<BF, 2, NQ, KTOP>), grid, dim3(kStepThreads), 0, st, a);
  else hipLaunchKernelGGL((k_traj_step<BF, 4, NQ, KTOP>), grid, dim3(kStepThreads), 0, st, a);
}

template <bool BF, int KTOP>
void launch_step_nq(int TQ, const StepArgs& a, hipStream_t st) {
  if (a.row <= 16) launch_step_tq<BF, KTOP, 1>(TQ, a, st);
  else if (a.row <= 32) launch_step_tq<BF, KTOP, 2>(TQ, a, st);
  else launch_step_tq<BF, KTOP, 4>(TQ, a, st);
}

// The step kernel launch, bracketed by the caller's measurement events when
// set (fm_debug_scan_events).
template <bool BF>
hipError_t launch_step(int KTOP, int TQ, const StepArgs& a, hipStream_t st) {
  const ScanEvents& ev = scan_events();
  if (ev.start != nullptr) {
    const hipError_t err = hipEventRecord(ev.start, st);
    if (err != hipSuccess) return err;
  }
  if (KTOP == 1) launch_step_nq<BF, 1>(TQ, a, st);
  else if (KTOP == 4) launch_step_nq<BF, 4>(TQ, a, st);
  else launch_step_nq<BF, 8>(TQ, a, st);
  const hipError_t err = hipGetLastError();
  if (err != hipSuccess || ev.stop == nullptr) return err;
  return hipEventRecord(ev.stop, st);
}

}  // namespace

size_t traj_state_bytes(int32_t cap, int32_t B_max) {
  const size_t chunks = static_cast<size_t>((B_max + kStepQ - 1) / kStepQ);
  return chunks * align_up(chunk_state_bytes(cap), kAlign);
}

hipError_t launch_traj_step(const StoreView& s, void* state, const void* q, int32_t layer, int32_t B, int32_t k,
                            int32_t* idx_out, float* score_out, const Workspace& ws, hipStream_t st) {
  const bool bf = s.map_dtype == FM_BF16;
  const int esz = bf ? 2 : 4;
  const int KTOP = k == 1 ? 1 : (k <= 4 ? 4 : 8);
  const int n_tiles = static_cast<int>((s.n + 15) / 16);
  const size_t cbytes = align_up(chunk_state_bytes(s.cap), kAlign);
  for (int b0 = 0; b0 < B; b0 += kChunkB) {
    const int Bc = B - b0 < kChunkB ? B - b0 : kChunkB;
    const int chunks = (Bc + kStepQ - 1) / kStepQ;
    StepArgs a;
    a.planes = s.planes;
    a.plane_elems = s.plane_elems;
    a.rnorm = s.rnorm;
    a.rn_stride = s.rn_stride;
    a.n = s.n;
    a.E = s.E;
    a.row = s.row;
    a.layer = layer;
    a.B = Bc;
    a.n_tiles = n_tiles;
    // Workgroups per chunk: a whole number per CU over the launch (one, or two
    // for top-4 and top-8 lists, whose ranking two workgroups interleave) but
    // at least 4 tiles each; an empty store still launches one, which advances
    // the query norms and the header.  50,000 x 60 float32, 64 queries, a pass
    // of 18: R = 256 289 us, 320 324, 512 293, 640 325; top-4 of 100 queries
    // of the 16-expert bf16 store R = 256 997, 512 942.
    int R = (KTOP == 1 ? 256 : 512) / chunks;
    if (R > (n_tiles + 3) / 4) R = (n_tiles + 3) / 4;
    if (R > kStepMaxLists / (kStepQ * chunks)) R = kStepMaxLists / (kStepQ * chunks);
    if (R < 1) R = 1;
    a.R = R;
    a.q = static_cast<const char*>(q) + static_cast<int64_t>(b0) * s.E * esz;
    a.state = static_cast<char*>(state) + static_cast<size_t>(b0 / kStepQ) * cbytes;
    a.chunk_bytes = static_cast<int64_t>(cbytes);
    a.partial = ws.partial;
    a.flags = s.flags;
    const int TQ = Bc <= 16 ? 1 : (Bc <= 32 ? 2 : 4);
    hipError_t err = bf ? launch_step<true>(KTOP, TQ, a, st) : launch_step<false>(KTOP, TQ, a, st);
    if (err != hipSuccess) return err;
    err = launch_finalize(ws.partial, nullptr, Bc, a.R, k, KTOP, idx_out + static_cast<int64_t>(b0) * k,
                          score_out + static_cast<int64_t>(b0) * k, st);
    if (err != hipSuccess) return err;
  }
  return hipSuccess;
}

}  // namespace fm
