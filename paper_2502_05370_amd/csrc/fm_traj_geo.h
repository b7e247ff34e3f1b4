// Slot geometry, staged-query layout and the float16 split shared by the
// trajectory scans.
#pragma once

#include "fm_device.h"
#include "fm_internal.h"

namespace fm {

typedef float floatx8 __attribute__((ext_vector_type(8)));
typedef uint16_t u16x4 __attribute__((ext_vector_type(4)));
typedef _Float16 half2v __attribute__((ext_vector_type(2)));
typedef float float2v __attribute__((ext_vector_type(2)));

// Slot geometry of a store (host-computed).
struct Geo {
  int32_t spl;   // slots per layer: E when LPG > 1, else E rounded up to 32
  int32_t lpg;   // layers per layer group
  int32_t ksg;   // 32-slot k-steps per layer group
};

// Bytes of one staged query plane row: 32*ksg 16-bit slots, in 16-byte
// units.  With ksg > 1 unit u of row r is stored at unit u ^ (r & 7) of the
// row, so the 16 rows a wave reads at one logical unit spread over 8 distinct
// 16-byte bank groups (with ksg = 1 a wave's read of 16 rows is one
// contiguous 1 KB already).
__host__ __device__ __forceinline__ int qrow_bytes(int ksg) { return 64 * ksg; }
__host__ __device__ __forceinline__ int qrow_unit(int ksg, int row, int unit) {
  return ksg > 1 ? unit ^ (row & 7) : unit;
}

inline Geo geometry(int E) {
  Geo g;
  if (E >= 8 && 32 % E == 0) {
    g.spl = E;
    g.lpg = 32 / E;
    g.ksg = 1;
  } else {
    g.spl = (E + 31) / 32 * 32;
    g.lpg = 1;
    g.ksg = g.spl / 32;
  }
  return g;
}

// float32 -> two float16 parts (bit patterns) of A = 2^12 a: hi = RN16(A),
// lo = RN16(A - hi).  A - hi is exact in float32 (one fused multiply-add of
// the widened hi); hi is finite for |a| < 16 (values above 8 are flagged
// where they enter).  Pairs convert with one packed conversion each.
constexpr float kSplitScale = 4096.0f;                        // 2^12
constexpr float kDotUnscale = 1.0f / (4096.0f * 4096.0f);     // 2^-24
constexpr float kRangeLimit = 8.0f;
__device__ __forceinline__ void split2(const floatx8& v, u16x8& h, u16x8& l) {
  uint32x4 hw, lw;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const float2v x = {v[2 * j] * kSplitScale, v[2 * j + 1] * kSplitScale};
    const half2v hb = __builtin_convertvector(x, half2v);
    float2v r;
    r[0] = __builtin_fmaf(static_cast<float>(hb[0]), -1.0f, x[0]);
    r[1] = __builtin_fmaf(static_cast<float>(hb[1]), -1.0f, x[1]);
    const half2v lb = __builtin_convertvector(r, half2v);
    hw[j] = __builtin_bit_cast(uint32_t, hb);
    lw[j] = __builtin_bit_cast(uint32_t, lb);
  }
  h = __builtin_bit_cast(u16x8, hw);
  l = __builtin_bit_cast(u16x8, lw);
}

// Split-depth scan (fm_traj_split.hip): whether and how a chunk of Bc queries
// takes it (shape < 0: it does not), and the scan itself on queries staged by
// k_traj_prep in groups of `group`; R partial lists per query.
struct TrajSplit {
  int shape = -1;
  int group = 0;
  int R = 0;
};
// (nlg: the layer groups that max_depth reaches; mm, or TQ and nba: the scan
// that would run otherwise.)
TrajSplit traj_split_plan(bool bf, int32_t n, int32_t row, const Geo& geo, int32_t Bc, int KTOP, int nlg, int TQ,
                          int nba, bool mm);
const char* traj_split_name(const TrajSplit& p);
hipError_t launch_traj_split(const StoreView& s, const TrajSplit& p, const Geo& geo, int32_t Bc, int32_t b_pad,
                             int KTOP, const Workspace& ws, hipStream_t st);

}  // namespace fm
