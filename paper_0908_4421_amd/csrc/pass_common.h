// Device helpers shared by the forward and the adjoint passes: cross-lane
// sums, buffer descriptors and loads, the solver state's words, stored values.
#pragma once

#include <cstddef>
#include <type_traits>
#include <cmath>

#include <hip/hip_ext.h>

#include "imrt_internal.h"

namespace imrt {
namespace {

// A workgroup's place in its pass: index w among the pass's G workgroups.  A
// single plan's pass has one workgroup per dispatch slot; a batched pass
// runs several plans' passes in one dispatch, each workgroup looking up its
// plan and its slot in that plan's pass, so every plan computes exactly what
// it computes alone.
struct Slot {
  int w, G;
};

// Trial point of steps 2/4: max(0, x - lambda g), evaluated in float64 and
// rounded once to float32.  NaN propagates (it is not clipped to zero).
__device__ __forceinline__ float trial_point(float x, float g, double lam) {
#pragma clang fp contract(off)
  const double t = static_cast<double>(x) - lam * static_cast<double>(g);
  return static_cast<float>(t < 0.0 ? 0.0 : t);
}

// ---- cross-lane sums ----------------------------------------------------------
// Data-parallel-primitive (DPP) moves within a wave: swaps inside quads, the
// mirrors of 8- and 16-lane rows, and the row broadcasts of lanes 15 and 31.
// Lanes a row mask leaves out receive 0.  The order of every sum is fixed.
constexpr int kDppQuadXor1 = 0xB1;     // quad_perm [1,0,3,2]
constexpr int kDppQuadXor2 = 0x4E;     // quad_perm [2,3,0,1]
constexpr int kDppRowMirror = 0x140;
constexpr int kDppRowHalfMirror = 0x141;
constexpr int kDppRowBcast15 = 0x142;
constexpr int kDppRowBcast31 = 0x143;

template <int CTRL, int ROWS>
__device__ __forceinline__ float dpp_move(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, ROWS, 0xF, false));
}

template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_move(double v) {
  const int2 w = __builtin_bit_cast(int2, v);
  int2 o;
  o.x = __builtin_amdgcn_update_dpp(0, w.x, CTRL, ROWS, 0xF, false);
  o.y = __builtin_amdgcn_update_dpp(0, w.y, CTRL, ROWS, 0xF, false);
  return __builtin_bit_cast(double, o);
}

// Sum over each aligned group of L lanes; valid in the group's last lane
// (lane % L == L - 1).
template <int L, typename T>
__device__ __forceinline__ T group_sum(T v) {
  if constexpr (L >= 2) v += dpp_move<kDppQuadXor1, 0xF>(v);
  if constexpr (L >= 4) v += dpp_move<kDppQuadXor2, 0xF>(v);
  if constexpr (L >= 8) v += dpp_move<kDppRowHalfMirror, 0xF>(v);
  if constexpr (L >= 16) v += dpp_move<kDppRowMirror, 0xF>(v);
  if constexpr (L >= 32) v += dpp_move<kDppRowBcast15, 0xA>(v);
  if constexpr (L >= 64) v += dpp_move<kDppRowBcast31, 0xC>(v);
  return v;
}

// Sum over the wave; valid in lane 63.
template <typename T>
__device__ __forceinline__ T wave_sum(T v) {
  return group_sum<64>(v);
}

// Sum of v over a workgroup of WAVES waves in a fixed order; the result is
// valid in thread 0.
template <typename T, int WAVES = kWaves>
__device__ __forceinline__ T block_sum(T v, T* sh) {
  v = wave_sum(v);
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  if (lane == 63) sh[w] = v;
  __syncthreads();
  T t = T(0);
  if (threadIdx.x == 0) {
    t = sh[0];
#pragma unroll
    for (int i = 1; i < WAVES; ++i) t += sh[i];
  }
  __syncthreads();
  return t;
}

// ---- buffer resources -----------------------------------------------------------
// A raw buffer descriptor built from a wave-uniform base address and length:
// loads take 32-bit offsets, and a lane whose offset lies past the length
// reads zeros without touching memory.  Lengths are kept multiples of the
// access size, so an access is either wholly inside or wholly outside.
using rsrc_t = __amdgpu_buffer_rsrc_t;
constexpr int kRsrcWord3 = 0x00020000;   // CDNA descriptor word 3: 32-bit data, no swizzle

__device__ __forceinline__ rsrc_t make_rsrc(const void* base, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, static_cast<int>(bytes), kRsrcWord3);
}
__device__ __forceinline__ int4 load_i4(rsrc_t r, uint32_t off) {
  return __builtin_bit_cast(int4, __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0));
}
__device__ __forceinline__ int load_i32(rsrc_t r, uint32_t off) {
  return static_cast<int>(__builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 0));
}
__device__ __forceinline__ float load_f32(rsrc_t r, uint32_t off) {
  return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 0));
}
__device__ __forceinline__ double load_f64(rsrc_t r, uint32_t off) {
  return __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, 0));
}
__device__ __forceinline__ uint32_t load_u8(rsrc_t r, uint32_t off) {
  return __builtin_amdgcn_raw_buffer_load_b8(r, off, 0, 0);
}
// Loads of the matrix streams with cache policy CP: 0 the default, 2 the
// non-temporal policy, for matrices larger than the last-level cache (a
// pass's stream would otherwise evict the vectors and tables the passes
// reuse; the values read are the same either way).
template <int CP>
__device__ __forceinline__ int4 load_i4s(rsrc_t r, uint32_t off) {
  return __builtin_bit_cast(int4, __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, CP));
}
template <int CP>
__device__ __forceinline__ float4 load_f4s(rsrc_t r, uint32_t off) {
  return __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, CP));
}
template <int CP>
__device__ __forceinline__ uint2 load_u2s(rsrc_t r, uint32_t off) {
  return __builtin_bit_cast(uint2, __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, CP));
}
__device__ __forceinline__ void store_f32(rsrc_t r, uint32_t off, float v) {
  __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, v), r, off, 0, 0);
}
__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }

__device__ __forceinline__ float* select_buf(float* const (&b)[kMaxTrials + 1], int i) {
  float* p = b[0];
  p = (i == 1) ? b[1] : p;
  p = (i == 2) ? b[2] : p;
  p = (i == 3) ? b[3] : p;
  p = (i == 4) ? b[4] : p;
  return p;
}

// Contiguous share [begin, end) of n work items for this workgroup.  With a
// grid that is a multiple of the die count, workgroup w (on die w % 8) gets
// logical slot (w % 8) * (grid / 8) + w / 8, so each die owns one contiguous
// eighth of the items.
__device__ __forceinline__ void work_range(int n, int& begin, int& end) {
  const int G = gridDim.x, w = blockIdx.x;
  const int lw = (G % kXcds == 0) ? (w % kXcds) * (G / kXcds) + w / kXcds : w;
  begin = static_cast<int>(static_cast<long long>(lw) * n / G);
  end = static_cast<int>(static_cast<long long>(lw + 1) * n / G);
}

// ---- solver state words -------------------------------------------------------------
constexpr int kStateWords = static_cast<int>(sizeof(SolverState) / sizeof(int32_t));
static_assert(kStateWords <= 64, "the state is loaded one word per lane of a wave");

// floor(i * n / parts) for wave-uniform arguments (64-bit product).
__device__ __forceinline__ int split_point(int i, int n, int parts) {
  return uniform(static_cast<int>(static_cast<long long>(i) * n / parts));
}

// Fields of a state loaded one 32-bit word per lane (lane i holds word i).
__device__ __forceinline__ int state_int(int32_t sw, size_t byte_off) {
  return __builtin_amdgcn_readlane(sw, static_cast<int>(byte_off / 4));
}
__device__ __forceinline__ double state_f64(int32_t sw, size_t byte_off) {
  const int lo = __builtin_amdgcn_readlane(sw, static_cast<int>(byte_off / 4));
  const int hi = __builtin_amdgcn_readlane(sw, static_cast<int>(byte_off / 4) + 1);
  return __builtin_bit_cast(double, (static_cast<unsigned long long>(static_cast<uint32_t>(hi)) << 32) |
                                        static_cast<uint32_t>(lo));
}

// ---- penalty ------------------------------------------------------------------------
struct RowPenalty {
  double Tu, To, wu, wo;
};

// One-sided quadratic penalty of a voxel (Eq. (1)) and its half-derivative.
__device__ __forceinline__ void penalty(const RowPenalty& p, float z, double& F, float& r) {
#pragma clang fp contract(off)
  const double zd = static_cast<double>(z);
  const double under = fmin(zd - p.Tu, 0.0);
  const double over = fmax(zd - p.To, 0.0);
  F = p.wu * under * under + p.wo * over * over;
  r = static_cast<float>(p.wu * under + p.wo * over);
}

// An s_waitcnt that waits for all loads.
constexpr int kWaitVmcnt0 = 0x0F70;   // vmcnt 0, expcnt and lgkmcnt unchecked

// ---- stored values --------------------------------------------------------------
// A lane holds its entries in groups of four: float32 storage as int4 column
// indices and float4 values, 16-bit storage as two 32-bit words of packed
// 16-bit indices or codes (entry u in the low half of word u / 2 when u is
// even, in the high half when odd); the ST_F32C16 layout pairs packed 16-bit
// indices with float4 values.
template <int ST>
__device__ __forceinline__ float code_value(uint32_t h) {
  if constexpr (ST == ST_BF16) {
    return __uint_as_float(h << 16);
  } else {
    return static_cast<float>(__builtin_bit_cast(_Float16, static_cast<uint16_t>(h)));
  }
}
__device__ __forceinline__ uint32_t half_of(const uint2& w, int u) {
  const uint32_t x = (u < 2) ? w.x : w.y;
  return (u & 1) ? (x >> 16) : (x & 0xFFFFu);
}
__device__ __forceinline__ int col_of(const int4& c, int u) {
  return u == 0 ? c.x : u == 1 ? c.y : u == 2 ? c.z : c.w;
}
__device__ __forceinline__ int col_of(const uint2& c, int u) { return static_cast<int>(half_of(c, u)); }
template <int ST>
__device__ __forceinline__ float val_of(const float4& v, int u) {
  return u == 0 ? v.x : u == 1 ? v.y : u == 2 ? v.z : v.w;
}
template <int ST>
__device__ __forceinline__ float val_of(const uint2& v, int u) {
  return code_value<ST>(half_of(v, u));
}
template <int ST>
using ColGroup = std::conditional_t<ST == ST_F32, int4, uint2>;
template <int ST>
using ValGroup = std::conditional_t<coded(ST), uint2, float4>;

}  // namespace
}  // namespace imrt
