// Adjoint pass of the gradient-projection / Armijo solver for gfx950 (an
// overview of both passes is in forward.hip).
#include <algorithm>

#include "decide.h"

namespace imrt {
namespace {

// ---- adjoint pass ----------------------------------------------------------------
// Workgroup w owns nonzeros [k0w, k1w) of the CSC arrays and walks the tiles
// covering them in rounds of 2048 entries: each thread loads two 16-byte
// vectors of row indices and of values, i.e. entries e0 + 1024 j + 64 u
// (j < 2, u < 4) of the round, where e0 = 256 * wave + lane (the tiled slot
// order of the CSC arrays); lanes past the range read zeros.  A round's
// residual gathers (each a run of 64 consecutive entries of a column across
// the wave) are issued before the next round's loads, which go to the other
// of two register stages, so one round is always in flight.  A round inside
// one column adds all its products; a round that meets a column boundary adds
// each column's share under a mask and closes every column that ends in it.
template <int ST>
struct AdjStage {
  int4 c[2];
  ValGroup<ST> v[2];
};

constexpr int kAdjStep = 8 * kThreads;   // nonzeros per round

// Logical workgroup of this dispatch slot.  With xcd_map and a grid that is a
// multiple of the die count, workgroup w (on die w % 8) gets logical slot
// (w % 8) * (grid / 8) + w / 8, so each die owns one contiguous eighth.
__device__ __forceinline__ int logical_wg(const Slot sl, bool xcd_map) {
  const int G = sl.G, w = sl.w;
  return (xcd_map && G % kXcds == 0) ? (w % kXcds) * (G / kXcds) + w / kXcds : w;
}

// The nonzeros of workgroup lw.
__device__ __forceinline__ void wg_range(const AdjArgs& a, int lw, int& k0, int& k1) {
  if (a.wg_k != nullptr) {
    k0 = uniform(a.wg_k[lw]);
    k1 = uniform(a.wg_k[lw + 1]);
  } else {
    k0 = split_point(lw, static_cast<int>(a.nnz), a.grid);
    k1 = split_point(lw + 1, static_cast<int>(a.nnz), a.grid);
  }
}

// rv covers the value array from the same entry as ri: float32 values in
// the index slots' order, or 16-bit codes in that order at half the width.
template <int ST, int CP = 0>
__device__ __forceinline__ void adj_issue(rsrc_t ri, rsrc_t rv, int round, AdjStage<ST>& S) {
  const uint32_t t = 16u * threadIdx.x;
  const uint32_t base = static_cast<uint32_t>(round) * (kAdjStep * 4u);
#pragma unroll
  for (int j = 0; j < 2; ++j) S.c[j] = load_i4s<CP>(ri, base + t + 4096u * j);
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    if constexpr (ST == ST_F32) S.v[j] = load_f4s<CP>(rv, base + t + 4096u * j);
    else S.v[j] = load_u2s<CP>(rv, base / 2 + t / 2 + 2048u * j);
  }
}

template <typename AS>
__device__ __forceinline__ void adj_gather(rsrc_t rr, const AS& S, float (&g)[8]) {
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    g[4 * j + 0] = load_f32(rr, 4u * S.c[j].x);
    g[4 * j + 1] = load_f32(rr, 4u * S.c[j].y);
    g[4 * j + 2] = load_f32(rr, 4u * S.c[j].z);
    g[4 * j + 3] = load_f32(rr, 4u * S.c[j].w);
  }
}

// Float64 sum of this thread's eight products, in a fixed order.
template <int ST>
__device__ __forceinline__ double adj_dot(const AdjStage<ST>& S, const float (&g)[8]) {
  double s = 0.0;
#pragma unroll
  for (int j = 0; j < 2; ++j) {
#pragma unroll
    for (int u = 0; u < 4; ++u) s += static_cast<double>(val_of<ST>(S.v[j], u)) * static_cast<double>(g[4 * j + u]);
  }
  return s;
}

// The same over the entries with index in [lo, hi) (e0 as above).
template <int ST>
__device__ __forceinline__ double adj_dot_masked(const AdjStage<ST>& S, const float (&g)[8], int e0, int lo, int hi) {
  double s = 0.0;
#pragma unroll
  for (int j = 0; j < 2; ++j) {
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int e = e0 + 1024 * j + 64 * u;
      const float r = (e >= lo && e < hi) ? g[4 * j + u] : 0.0f;
      s += static_cast<double>(val_of<ST>(S.v[j], u)) * static_cast<double>(r);
    }
  }
  return s;
}

// ---- an adjoint workgroup's columns ----------------------------------------------
// A workgroup walks its columns c0..c1-1 in order, kColChunk at a time: lane
// j of every wave holds column cb + j's entries of col_ptr (and its kind and
// 16-bit scale), so moving on to the next column reads a register.  Closing a
// column sums it over each wave and parks the wave's sum in lane j; when the
// chunk is full, and at the end, the waves' sums meet in LDS and wave 0 adds
// them in wave order (block_sum's order) and stores the chunk's gradient
// entries and pieces.  No workgroup barrier and no dependent global load sits
// between one column and the next.
constexpr int kColChunk = 64;

template <int ST>
struct ColChunk {
  int cb;          // first column of the chunk (uniform)
  int p0, p1;      // lane j: col_ptr[cb + j], col_ptr[cb + j + 1]
  uint32_t kind;   // lane j: col_kind[cb + j]
  float csc;       // lane j: 16-bit storage scale of column cb + j
};

template <int ST>
__device__ __forceinline__ void col_chunk_load(const AdjArgs& a, int cb, ColChunk<ST>& K) {
  const uint32_t nb = static_cast<uint32_t>(a.nb);
  const uint32_t j = static_cast<uint32_t>(cb + (threadIdx.x & 63));
  const rsrc_t rp = make_rsrc(a.col_ptr, 4u * (nb + 1));
  K.cb = cb;
  K.p0 = load_i32(rp, 4u * j);
  K.p1 = load_i32(rp, 4u * j + 4u);
  K.kind = load_u8(make_rsrc(a.col_kind, nb), j);
  K.csc = coded(ST) ? load_f32(make_rsrc(a.col_scale, 4u * nb), 4u * j) : 1.0f;
}

// Loads of a chunk after the first one: wait for them at once (vmcnt 0).
// Without this wait, the compiler cannot tell at the next column whether a
// reload is still in flight, and every column's register read would wait
// for all loads issued since, the next round's prefetch included.

template <int ST>
__device__ __forceinline__ void col_chunk_reload(const AdjArgs& a, int cb, ColChunk<ST>& K) {
  col_chunk_load(a, cb, K);
  __builtin_amdgcn_s_waitcnt(kWaitVmcnt0);
}

// Column c's entries inside the workgroup's range [k0w, k1w).
template <int ST>
__device__ __forceinline__ void col_bounds(const ColChunk<ST>& K, int c, int k0w, int k1w, int& lo, int& hi) {
  lo = max(__builtin_amdgcn_readlane(K.p0, c - K.cb), k0w);
  hi = min(__builtin_amdgcn_readlane(K.p1, c - K.cb), k1w);
}

// The wave's sum of v, parked in lane j of h.
__device__ __forceinline__ void col_park(double v, int j, double& h) {
  const uint64_t b = __builtin_bit_cast(uint64_t, wave_sum(v));
  const uint32_t lo = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(b), 63));
  const uint32_t hi = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(b >> 32), 63));
  if ((threadIdx.x & 63) == j) h = __builtin_bit_cast(double, (static_cast<uint64_t>(hi) << 32) | lo);
}

// Lane j of wave 0, column c = cb + j closed with workgroup sum t: the
// gradient entry of a column inside the range, else the workgroup's piece.
template <int ST>
__device__ __forceinline__ void col_store(const AdjArgs& aq, const ColChunk<ST>& K, int c0, int c1, int lw, int k0w,
                                          int k1w, double t) {
  const int c = K.cb + (threadIdx.x & 63);
  if (K.p0 >= k0w && K.p1 <= k1w) {
    const double f = (ST == ST_F32) ? aq.scale : aq.scale * static_cast<double>(K.csc);
    aq.out[c] = static_cast<float>(f * t);
  } else {
    if (c == c0) aq.pieces[2 * lw] = t;
    if (c == c1 - 1) aq.pieces[2 * lw + 1] = t;
    // a column shared by two workgroups also keeps its pieces side by side
    if (K.kind == 1 && aq.pieces_col != nullptr) aq.pieces_col[2 * c + (K.p0 < k0w ? 1 : 0)] = t;
  }
}

// Adjoint pass: in a solve, the decision on the preceding forward pass
// (every workgroup identically; workgroup 0 stores the new state and trace
// entry), and g = scale * D^T r over this workgroup's share of the nonzeros.
// The first two rounds' loads are issued on entry and the first round's
// residual gathers before the decision is known, from the residual buffer of
// the pass's first trial (the one an accepted step of a single-trial pass
// always lands in); if another trial is accepted they are issued again.
template <int NT, bool SOLVE, int ST, int CP = 0>
__device__ __forceinline__ void adj_pass(const AdjArgs& a, const Slot sl) {
  __shared__ double red[kWaves];
  __shared__ double colsh[kWaves * kColChunk];
  __shared__ Decision dec;
  const int tid = threadIdx.x;
  const int lw = logical_wg(sl, a.xcd_map != 0);
  int k0w, k1w;
  wg_range(a, lw, k0w, k1w);
  const int kb = k0w & ~(kTile - 1);
  const int nrounds = (k1w > kb) ? (k1w - kb + kAdjStep - 1) / kAdjStep : 0;
  // whole tiles: entries of a partial tile sit anywhere in it
  const uint32_t bytes = static_cast<uint32_t>((((k1w + kTile - 1) & ~(kTile - 1)) - kb) * 4);
  const rsrc_t ri = make_rsrc(a.row_idx + kb, bytes);
  const rsrc_t rv = (ST == ST_F32) ? make_rsrc(a.val + kb, bytes) : make_rsrc(a.val16 + kb, bytes / 2);
  // Every load of the prologue is issued at once and none sits in a branch
  // (rounds past the range read zeros out of bounds), so each wait below
  // waits for its own loads only: the decision's inputs, this workgroup's
  // columns, the first two rounds, then the gathers of the first round.
  DecideLoads<NT> DL;
  if (SOLVE) decide_start<NT>(a, DL);
  const int4 wi = load_i4(make_rsrc(a.wg_cols, 16u * static_cast<uint32_t>(a.grid)), 16u * static_cast<uint32_t>(lw));
  AdjStage<ST> A, B;
  adj_issue<ST, CP>(ri, rv, 0, A);
  adj_issue<ST, CP>(ri, rv, 1, B);
  const int c0 = uniform(wi.x), c1 = uniform(wi.y);
  int c = c0, lo = uniform(wi.z), hi = uniform(wi.w);
  ColChunk<ST> CK;
  col_chunk_load(a, c0, CK);
  // a solve gathers the residual of the first trial: the accepted one
  // unless a later trial wins
  const uint32_t rbytes = 4u * static_cast<uint32_t>(a.nv);
  rsrc_t rr = make_rsrc(SOLVE ? a.rbuf[0] : a.r, rbytes);
  float g[8];
  adj_gather(rr, A, g);
  if (SOLVE) {
    // (a finished solve passes its state through unchanged and exits here)
    decide<NT>(a.fwd_partials, a.fwd_parts, a.step_partials, a.step_parts, DL, dec, red, a.G_skip);
    if (sl.w == 0 && tid == 0) {
      *a.st_out = dec.st;
      if (dec.accepted >= 0 && a.trace != nullptr && dec.st.k - 1 < dec.st.trace_cap) {
        TraceDev e;
        e.k = dec.st.k;
        e.backtracks = dec.backtracks;
        e.lambda = dec.lam;
        e.step_sq = dec.step_sq;
        e.G = dec.st.G;
        a.trace[dec.st.k - 1] = e;
      }
    }
    if (dec.st.phase != PH_NEED_GRAD) return;
    if (dec.st.acc != 0) {
      rr = make_rsrc(select_buf(a.rbuf, dec.st.acc), rbytes);
      adj_gather(rr, A, g);
    }
  }

  double s = 0.0, h = 0.0;
  // the chunk's closed columns: the waves' sums in wave order, then stored
  auto flush = [&]() {
    colsh[(tid >> 6) * kColChunk + (tid & 63)] = h;
    __syncthreads();
    if (tid < c - CK.cb) {
      double t = colsh[tid];
#pragma unroll
      for (int w = 1; w < kWaves; ++w) t += colsh[w * kColChunk + tid];
      col_store(a, CK, c0, c1, lw, k0w, k1w, t);
    }
  };
  auto close = [&]() {
    col_park(s, c - CK.cb, h);
    s = 0.0;
    ++c;
    if (c < c1) {
      if (c - CK.cb == kColChunk) {
        flush();
        __syncthreads();   // LDS slots reused by the next chunk
        col_chunk_reload(a, c, CK);
      }
      col_bounds(CK, c, k0w, k1w, lo, hi);
    }
  };
  // distribute one round's products over the columns it meets
  auto consume = [&](const AdjStage<ST>& cur, const float (&gv)[8], int round) {
    const int base = kb + round * kAdjStep, end = base + kAdjStep;
    while (c < c1 && lo < end) {
      if (lo <= base && hi >= end) {
        s += adj_dot(cur, gv);
        if (hi == end) close();
        break;
      }
      s += adj_dot_masked(cur, gv, base + 256 * (tid >> 6) + (tid & 63), lo, hi);
      if (hi > end) break;
      close();
    }
  };
  // round 0 (its gathers and round 1's loads already issued), then the rest
  // alternating between the two register stages
  int round = 0;
  if (nrounds > 0) {
    consume(A, g, 0);
    round = 1;
    auto step = [&](const AdjStage<ST>& cur, AdjStage<ST>& nxt) {
      float gv[8];
      adj_gather(rr, cur, gv);
      // The next round's loads go out after this round's gathers and also
      // past the last round (zeros out of bounds): loads complete in issue
      // order, so either a branch here or loads moved ahead of the gathers
      // would make the wait for the gathers wait for these loads as well.
      __builtin_amdgcn_sched_barrier(0);
      adj_issue<ST, CP>(ri, rv, round + 1, nxt);
      consume(cur, gv, round);
      ++round;
      return round < nrounds;
    };
    while (round < nrounds) {
      if (!step(B, A)) break;
      if (!step(A, B)) break;
    }
  }
  // empty columns at the end of the range
  while (c < c1) close();
  if (c1 > c0) flush();
}

template <int NT, bool SOLVE, int ST, int CP = 0>
__global__ __launch_bounds__(kThreads) void adj_kernel(AdjArgs a) {
  adj_pass<NT, SOLVE, ST, CP>(a, Slot{static_cast<int>(blockIdx.x), static_cast<int>(gridDim.x)});
}

// Batched solve pass (slots as for fwd_wave_batch_kernel).
template <int NT, int ST, int CP = 0>
__global__ __launch_bounds__(kThreads) void adj_batch_kernel(const AdjArgs* __restrict__ args,
                                                             const int32_t* __restrict__ slots) {
  const int sv = uniform(slots[blockIdx.x]);
  if (sv < 0) return;
  // read in place (uniform, read-only): a local copy would live in scratch
  const AdjArgs& a = args[sv >> 16];
  adj_pass<NT, true, ST, CP>(a, Slot{sv & 0xFFFF, a.grid});
}

// Adjoint pass of n <= K solves that share one dose matrix (the same CSC
// arrays and work partition; re-plans of one resident patient): the
// matrix stream of the workgroup's range is read once, and every solve gets
// exactly the arithmetic adj_pass gives it alone -- its own decision, its
// residual gathers, its float64 column sums in the same order and the same
// workgroup-level reductions, its outputs.  plans[q] indexes args.
template <int NT, int ST, int K>
__device__ __forceinline__ void adj_multi_pass(const AdjArgs* __restrict__ args, const int32_t* plans, int n,
                                               const Slot sl) {
  __shared__ double red[kWaves];
  __shared__ double colsh[K][kWaves * kColChunk];
  __shared__ Decision dec[K];
  const AdjArgs& a = args[uniform(plans[0])];   // the shared matrix and partition
  const int tid = threadIdx.x;
  const int lw = logical_wg(sl, a.xcd_map != 0);
  int k0w, k1w;
  wg_range(a, lw, k0w, k1w);
  const int kb = k0w & ~(kTile - 1);
  const int nrounds = (k1w > kb) ? (k1w - kb + kAdjStep - 1) / kAdjStep : 0;
  const uint32_t bytes = static_cast<uint32_t>((((k1w + kTile - 1) & ~(kTile - 1)) - kb) * 4);
  const rsrc_t ri = make_rsrc(a.row_idx + kb, bytes);
  const rsrc_t rv = (ST == ST_F32) ? make_rsrc(a.val + kb, bytes) : make_rsrc(a.val16 + kb, bytes / 2);
  int pi[K];
#pragma unroll
  for (int q = 0; q < K; ++q) pi[q] = uniform(plans[q < n ? q : 0]);
  DecideLoads<NT> DL[K];
#pragma unroll
  for (int q = 0; q < K; ++q) decide_start<NT>(args[pi[q]], DL[q]);
  const int4 wi = load_i4(make_rsrc(a.wg_cols, 16u * static_cast<uint32_t>(a.grid)), 16u * static_cast<uint32_t>(lw));
  AdjStage<ST> A, B;
  adj_issue(ri, rv, 0, A);
  adj_issue(ri, rv, 1, B);
  const int c0 = uniform(wi.x), c1 = uniform(wi.y);
  int c = c0, lo = uniform(wi.z), hi = uniform(wi.w);
  ColChunk<ST> CK;
  col_chunk_load(a, c0, CK);
  const uint32_t rbytes = 4u * static_cast<uint32_t>(a.nv);
  rsrc_t rr[K];
  float g[K][8];
#pragma unroll
  for (int q = 0; q < K; ++q) {
    rr[q] = make_rsrc(q < n ? args[pi[q]].rbuf[0] : nullptr, q < n ? rbytes : 0u);
    adj_gather(rr[q], A, g[q]);
  }
  bool need[K];
  bool any = false;
#pragma unroll
  for (int q = 0; q < K; ++q) {
    need[q] = false;
    if (q < n) {
      const AdjArgs& aq = args[pi[q]];
      decide<NT>(aq.fwd_partials, aq.fwd_parts, aq.step_partials, aq.step_parts, DL[q], dec[q], red, aq.G_skip);
      if (sl.w == 0 && tid == 0) {
        *aq.st_out = dec[q].st;
        if (dec[q].accepted >= 0 && aq.trace != nullptr && dec[q].st.k - 1 < dec[q].st.trace_cap) {
          TraceDev e;
          e.k = dec[q].st.k;
          e.backtracks = dec[q].backtracks;
          e.lambda = dec[q].lam;
          e.step_sq = dec[q].step_sq;
          e.G = dec[q].st.G;
          aq.trace[dec[q].st.k - 1] = e;
        }
      }
      need[q] = dec[q].st.phase == PH_NEED_GRAD;
      if (need[q] && dec[q].st.acc != 0) {
        rr[q] = make_rsrc(select_buf(aq.rbuf, dec[q].st.acc), rbytes);
        adj_gather(rr[q], A, g[q]);
      }
      if (!need[q]) rr[q] = make_rsrc(nullptr, 0u);
      any = any || need[q];
    }
  }
  if (!any) return;

  double s[K], h[K];
#pragma unroll
  for (int q = 0; q < K; ++q) s[q] = h[q] = 0.0;
  auto flush = [&]() {
#pragma unroll
    for (int q = 0; q < K; ++q)
      if (need[q]) colsh[q][(tid >> 6) * kColChunk + (tid & 63)] = h[q];
    __syncthreads();
    if (tid < c - CK.cb) {
#pragma unroll
      for (int q = 0; q < K; ++q) {
        if (!need[q]) continue;
        double t = colsh[q][tid];
#pragma unroll
        for (int w = 1; w < kWaves; ++w) t += colsh[q][w * kColChunk + tid];
        col_store(args[pi[q]], CK, c0, c1, lw, k0w, k1w, t);
      }
    }
  };
  auto close = [&]() {
#pragma unroll
    for (int q = 0; q < K; ++q) {
      if (!need[q]) continue;
      col_park(s[q], c - CK.cb, h[q]);
      s[q] = 0.0;
    }
    ++c;
    if (c < c1) {
      if (c - CK.cb == kColChunk) {
        flush();
        __syncthreads();   // LDS slots reused by the next chunk
        col_chunk_reload(a, c, CK);
      }
      col_bounds(CK, c, k0w, k1w, lo, hi);
    }
  };
  auto consume = [&](const AdjStage<ST>& cur, const float (&gv)[K][8], int round) {
    const int base = kb + round * kAdjStep, end = base + kAdjStep;
    while (c < c1 && lo < end) {
      if (lo <= base && hi >= end) {
#pragma unroll
        for (int q = 0; q < K; ++q)
          if (need[q]) s[q] += adj_dot(cur, gv[q]);
        if (hi == end) close();
        break;
      }
      const int e0 = base + 256 * (tid >> 6) + (tid & 63);
#pragma unroll
      for (int q = 0; q < K; ++q)
        if (need[q]) s[q] += adj_dot_masked(cur, gv[q], e0, lo, hi);
      if (hi > end) break;
      close();
    }
  };
  int round = 0;
  if (nrounds > 0) {
    consume(A, g, 0);
    round = 1;
    auto step = [&](const AdjStage<ST>& cur, AdjStage<ST>& nxt) {
      float gv[K][8];
#pragma unroll
      for (int q = 0; q < K; ++q) adj_gather(rr[q], cur, gv[q]);
      // The next round's loads go out after this round's gathers and also
      // past the last round (zeros out of bounds): loads complete in issue
      // order, so either a branch here or loads moved ahead of the gathers
      // would make the wait for the gathers wait for these loads as well.
      __builtin_amdgcn_sched_barrier(0);
      adj_issue(ri, rv, round + 1, nxt);
      consume(cur, gv, round);
      ++round;
      return round < nrounds;
    };
    while (round < nrounds) {
      if (!step(B, A)) break;
      if (!step(A, B)) break;
    }
  }
  while (c < c1) close();
  if (c1 > c0) flush();
}

// Batched adjoint pass over groups of solves sharing a dose matrix:
// slots[blockIdx.x] = (group << 16) | workgroup (or -1), groups[(K + 1) g]
// = the group's size n, then its n plan indices.
template <int NT, int ST, int K>
__global__ __launch_bounds__(kThreads) void adj_multi_batch_kernel(const AdjArgs* __restrict__ args,
                                                                   const int32_t* __restrict__ groups,
                                                                   const int32_t* __restrict__ slots) {
  const int sv = uniform(slots[blockIdx.x]);
  if (sv < 0) return;
  const int32_t* gr = groups + static_cast<size_t>(sv >> 16) * (K + 1);
  const int n = uniform(gr[0]);
  adj_multi_pass<NT, ST, K>(args, gr + 1, n, Slot{sv & 0xFFFF, args[uniform(gr[1])].grid});
}

// Columns shared by several adjoint workgroups (completion not folded): the
// fixed-order sum of their pieces.  Runs after adj_kernel; in a solve only
// when that pass computed a gradient (state after the decision in `st`).
__global__ __launch_bounds__(kThreads) void adj_final_kernel(AdjArgs a, const SolverState* st) {
  if (st != nullptr && st->phase != PH_NEED_GRAD) return;
  const int c = blockIdx.x * kThreads + threadIdx.x;
  if (c >= a.nb) return;
  const int wlo = a.col_wlo[c], whi = a.col_whi[c];
  if (wlo == whi) return;
  double tot = a.pieces[2 * wlo + 1];
  for (int w = wlo + 1; w < whi; ++w) tot += a.pieces[2 * w];
  tot += a.pieces[2 * whi];
  const double f = (a.col_scale == nullptr) ? a.scale : a.scale * static_cast<double>(a.col_scale[c]);
  a.out[c] = static_cast<float>(f * tot);
}

}  // namespace

int adjoint_grid_for(const imrt_ctx* ctx, int64_t nnz, int min_nnz) {
  const int64_t cap = static_cast<int64_t>(ctx->tune.adj_grid_per_cu) * ctx->num_cu;
  // at least min_nnz nonzeros per workgroup, at least one workgroup
  const int64_t per = std::max(min_nnz, 1);
  const int64_t want = (nnz + per - 1) / per;
  return static_cast<int>(std::max<int64_t>(1, std::min(cap, want)));
}

template <int ST, int CP>
int launch_adjoint_batch_st(const AdjArgs* args, const int32_t* slots, int nslots, int ntrials, hipStream_t s) {
  const dim3 gd(nslots), bd(kThreads);
  switch (ntrials) {
    case 1: hipLaunchKernelGGL((adj_batch_kernel<1, ST, CP>), gd, bd, 0, s, args, slots); break;
    case 2: hipLaunchKernelGGL((adj_batch_kernel<2, ST, CP>), gd, bd, 0, s, args, slots); break;
    case 4: hipLaunchKernelGGL((adj_batch_kernel<4, ST, CP>), gd, bd, 0, s, args, slots); break;
    default: return set_error(IMRT_EINVAL, "trials per pass must be 1, 2 or 4");
  }
  return IMRT_OK;
}

int launch_adjoint_batch(const imrt_ctx* ctx, const AdjArgs* args, const int32_t* slots, int nslots, int ntrials,
                         int storage, int stream_cp) {
  if (nslots <= 0) return IMRT_OK;
  int rc;
  switch (storage) {
    case ST_F32:
      rc = stream_cp ? launch_adjoint_batch_st<ST_F32, 2>(args, slots, nslots, ntrials, ctx->stream)
                     : launch_adjoint_batch_st<ST_F32, 0>(args, slots, nslots, ntrials, ctx->stream);
      break;
    case ST_BF16:
      rc = stream_cp ? launch_adjoint_batch_st<ST_BF16, 2>(args, slots, nslots, ntrials, ctx->stream)
                     : launch_adjoint_batch_st<ST_BF16, 0>(args, slots, nslots, ntrials, ctx->stream);
      break;
    case ST_F16:
      rc = stream_cp ? launch_adjoint_batch_st<ST_F16, 2>(args, slots, nslots, ntrials, ctx->stream)
                     : launch_adjoint_batch_st<ST_F16, 0>(args, slots, nslots, ntrials, ctx->stream);
      break;
    default: return set_error(IMRT_EINVAL, "unknown storage");
  }
  if (rc) return rc;
  return check_launch("adj_batch_kernel");
}

template <int ST, int K>
int launch_adjoint_multi_st(const AdjArgs* args, const int32_t* groups, const int32_t* slots, int nslots,
                            int ntrials, hipStream_t s) {
  const dim3 gd(nslots), bd(kThreads);
  switch (ntrials) {
    case 1: hipLaunchKernelGGL((adj_multi_batch_kernel<1, ST, K>), gd, bd, 0, s, args, groups, slots); break;
    case 2: hipLaunchKernelGGL((adj_multi_batch_kernel<2, ST, K>), gd, bd, 0, s, args, groups, slots); break;
    case 4: hipLaunchKernelGGL((adj_multi_batch_kernel<4, ST, K>), gd, bd, 0, s, args, groups, slots); break;
    default: return set_error(IMRT_EINVAL, "trials per pass must be 1, 2 or 4");
  }
  return IMRT_OK;
}

template <int K>
int launch_adjoint_multi_k(const AdjArgs* args, const int32_t* groups, const int32_t* slots, int nslots,
                           int ntrials, int storage, hipStream_t s) {
  switch (storage) {
    case ST_F32: return launch_adjoint_multi_st<ST_F32, K>(args, groups, slots, nslots, ntrials, s);
    case ST_BF16: return launch_adjoint_multi_st<ST_BF16, K>(args, groups, slots, nslots, ntrials, s);
    case ST_F16: return launch_adjoint_multi_st<ST_F16, K>(args, groups, slots, nslots, ntrials, s);
    default: return set_error(IMRT_EINVAL, "unknown storage");
  }
}

int launch_adjoint_multi_batch(const imrt_ctx* ctx, const AdjArgs* args, const int32_t* groups, int group_k,
                               const int32_t* slots, int nslots, int ntrials, int storage) {
  if (nslots <= 0) return IMRT_OK;
  int rc;
  switch (group_k) {
    case 2: rc = launch_adjoint_multi_k<2>(args, groups, slots, nslots, ntrials, storage, ctx->stream); break;
    case 4: rc = launch_adjoint_multi_k<4>(args, groups, slots, nslots, ntrials, storage, ctx->stream); break;
    default: return set_error(IMRT_EINVAL, "shared-matrix adjoint groups hold 2 or 4 solves");
  }
  if (rc) return rc;
  return check_launch("adj_multi_batch_kernel");
}

template <int ST, int CP>
int launch_adjoint_kernel(const AdjArgs& a, int ntrials, dim3 gd, dim3 bd, hipStream_t s, hipEvent_t before,
                          hipEvent_t after) {
  switch (a.solve ? ntrials : 0) {
    case 0: hipExtLaunchKernelGGL((adj_kernel<1, false, ST>), gd, bd, 0, s, before, after, 0, a); break;
    case 1: hipExtLaunchKernelGGL((adj_kernel<1, true, ST, CP>), gd, bd, 0, s, before, after, 0, a); break;
    case 2: hipExtLaunchKernelGGL((adj_kernel<2, true, ST, CP>), gd, bd, 0, s, before, after, 0, a); break;
    case 4: hipExtLaunchKernelGGL((adj_kernel<4, true, ST, CP>), gd, bd, 0, s, before, after, 0, a); break;
    default: return set_error(IMRT_EINVAL, "trials per pass must be 1, 2 or 4");
  }
  return IMRT_OK;
}

int launch_adjoint(const imrt_ctx* ctx, const imrt_dose* D, const AdjArgs& a, int ntrials, hipEvent_t before,
                   hipEvent_t after) {
  clear_stale_error();
  const dim3 gd(a.grid), bd(kThreads);
  hipStream_t s = ctx->stream;
  if (!a.solve && ntrials != 1) return set_error(IMRT_EINVAL, "a plain adjoint pass takes one vector");
  int rc = IMRT_OK;
  switch (a.storage) {
    case ST_F32:
      rc = (a.solve && a.stream_cp) ? launch_adjoint_kernel<ST_F32, 2>(a, ntrials, gd, bd, s, before, after)
                                    : launch_adjoint_kernel<ST_F32, 0>(a, ntrials, gd, bd, s, before, after);
      break;
    case ST_BF16:
      rc = (a.solve && a.stream_cp) ? launch_adjoint_kernel<ST_BF16, 2>(a, ntrials, gd, bd, s, before, after)
                                    : launch_adjoint_kernel<ST_BF16, 0>(a, ntrials, gd, bd, s, before, after);
      break;
    case ST_F16:
      rc = (a.solve && a.stream_cp) ? launch_adjoint_kernel<ST_F16, 2>(a, ntrials, gd, bd, s, before, after)
                                    : launch_adjoint_kernel<ST_F16, 0>(a, ntrials, gd, bd, s, before, after);
      break;
    default: return set_error(IMRT_EINVAL, "unknown storage");
  }
  if (rc) return rc;
  rc = check_launch("adj_kernel");
  if (rc) return rc;
  if (!a.solve && a.wg_k == nullptr) {
    // shared columns completed here (in a solve the next forward pass
    // completes them while it stages its trial points)
    const int g2 = (a.nb + kThreads - 1) / kThreads;
    hipLaunchKernelGGL(adj_final_kernel, dim3(g2), dim3(kThreads), 0, s, a, static_cast<const SolverState*>(nullptr));
    rc = check_launch("adj_final_kernel");
  }
  (void)D;
  return rc;
}

}  // namespace imrt
