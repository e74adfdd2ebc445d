// Forward pass of the gradient-projection / Armijo solver for gfx950 (the
// adjoint pass is in adjoint.hip).
//
//  fwd_kernel / fwd_wave_kernel
//               trial points x_t = max(0, x_k - lambda g) (steps 2 and 4)
//               staged in LDS, forward dose z = D x over CSR (Section 2.1),
//               penalty residual and objective partials (Eqs. (1)-(2)), in
//               one pass over D.
//  adj_kernel   line-search decision on the preceding forward pass (Armijo
//               test of Eq. (5), stopping test of step 5), taken identically
//               by every workgroup, then the beamlet-parallel adjoint
//               g = 2 D^T r over CSC for an accepted, unfinished iterate.
//  adj_final    completes shared columns outside a solve (in a solve the
//               next forward pass completes them while staging its trials).
//
// The solver state is double-buffered: a pass reads one copy and workgroup 0
// writes the other, so no workgroup ever sees a state written during its own
// pass.  Every reduction runs in a fixed order, so results are
// bit-reproducible and independent of workgroup timing; there are no
// floating-point atomics.  (The waves of a wave-granular forward workgroup
// take row blocks from an integer counter in LDS, but a block's rows and its
// objective contribution come out the same whichever wave takes it, and the
// contributions are added in block order.)  Work is dealt to workgroups in contiguous ranges,
// consecutive ranges on the same accelerator die (workgroups are dispatched
// round-robin over the 8 dies), so neighbouring beamlet columns share that
// die's L2 for their residual gathers.
#include <algorithm>

#include "pass_common.h"

namespace imrt {
namespace {

// Lanes cooperating on one row: the largest power of two with lanes*nr <= 256, at most 64.
__device__ __forceinline__ int lanes_per_row(int nr) {
  int L = 64;
  while (L > 1 && L * nr > kThreads) L >>= 1;
  return L;
}

// Penalty of a row: the structure's entry of the LDS copy of the table, or
// per-voxel thresholds when given.
__device__ __forceinline__ RowPenalty row_penalty(const Penalties& p, int row, const PenaltyDev* tab,
                                                  uint8_t sid) {
  const PenaltyDev t = tab[sid];
  RowPenalty r{t.T_u, t.T_o, t.w_u, t.w_o};
  if (p.Tu_vox != nullptr) {
    r.Tu = static_cast<double>(p.Tu_vox[row]);
    r.To = static_cast<double>(p.To_vox[row]);
  }
  return r;
}

template <int NT>
__device__ __forceinline__ void row_epilogue(const FwdArgs& a, int row, uint8_t sid, const PenaltyDev* tab,
                                             const float (&d)[NT], double (&pacc)[NT],
                                             float* const (&rout)[NT], int ntr) {
  if (a.mode == FWD_PLAIN) {
    a.d_out[row] = d[0];
    pacc[0] += static_cast<double>(d[0]) * static_cast<double>(d[0]);
    return;
  }
  const RowPenalty p = row_penalty(a.pen, row, tab, sid);
#pragma unroll
  for (int q = 0; q < NT; ++q) {
    if (q < ntr) {
      double F;
      float r;
      penalty(p, d[q], F, r);
      pacc[q] += F;
      if (a.mode == FWD_SOLVE) {
        rout[q][row] = r;
      } else if (q == 0) {
        if (a.r_out) a.r_out[row] = r;
        if (a.d_out) a.d_out[row] = d[0];
      }
    }
  }
}

// ---- forward pass ---------------------------------------------------------------
struct BlockMeta {
  int r0, r1, k0, k1;
};

__device__ __forceinline__ BlockMeta block_meta(const FwdArgs& a, int b) {
  BlockMeta m;
  m.r0 = a.block_row[b];
  m.r1 = a.block_row[b + 1];
  m.k0 = a.block_k0[b];
  m.k1 = a.block_k0[b + 1];
  return m;
}

struct VecRegs {
  int4 c[2];
  float4 v[2];
};

// Issue the 16-byte loads covering nonzeros [base, min(base + 8*256, k1)) of
// an index/value pair of arrays.  base is a multiple of 4 and the arrays carry
// a zeroed tail, so whole vectors stay in bounds; a lane past k1 loads the
// first vector instead (never used), which keeps the loads branch-free.
__device__ __forceinline__ void issue_vec(const int32_t* idx, const float* val, int base, int k1, VecRegs& R) {
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    int e0 = base + 4 * (threadIdx.x + j * kThreads);
    e0 = (e0 < k1) ? e0 : 0;
    R.c[j] = *reinterpret_cast<const int4*>(idx + e0);
    R.v[j] = *reinterpret_cast<const float4*>(val + e0);
  }
}

// Row pointers (relative to the block's aligned start) and structure ids of
// one block, loaded ahead into registers.
struct RowRegs {
  int rp[3];
  uint8_t sid[2];
};

__device__ __forceinline__ void issue_rows(const FwdArgs& a, const BlockMeta& m, bool want_sid, RowRegs& Q) {
  const int nr = m.r1 - m.r0;
  const int t = threadIdx.x;
  const int i0 = (t <= nr) ? t : 0;
  const int i1 = (t + kThreads <= nr) ? t + kThreads : 0;
  const int i2 = (2 * kThreads <= nr) ? 2 * kThreads : 0;
  Q.rp[0] = a.row_ptr[m.r0 + i0];
  Q.rp[1] = a.row_ptr[m.r0 + i1];
  Q.rp[2] = a.row_ptr[m.r0 + i2];
  if (want_sid) {
    const int j0 = (t < nr) ? t : 0;
    const int j1 = (t + kThreads < nr) ? t + kThreads : 0;
    Q.sid[0] = a.pen.sid[m.r0 + j0];
    Q.sid[1] = a.pen.sid[m.r0 + j1];
  } else {
    Q.sid[0] = Q.sid[1] = 0;
  }
}

__device__ __forceinline__ void stage_rows(const BlockMeta& m, const RowRegs& Q, int32_t* rp, uint8_t* sid) {
  const int nr = m.r1 - m.r0;
  const int a0 = m.k0 & ~3;
  const int t = threadIdx.x;
  if (t <= nr) rp[t] = Q.rp[0] - a0;
  if (t + kThreads <= nr) rp[t + kThreads] = Q.rp[1] - a0;
  if (t == 0 && 2 * kThreads <= nr) rp[2 * kThreads] = Q.rp[2] - a0;
  if (t < nr) sid[t] = Q.sid[0];
  if (t + kThreads < nr) sid[t + kThreads] = Q.sid[1];
}

// Products D_ij * x_t^(q)_j of the block's nonzeros into LDS, written as
// whole 4-element vectors at their offset from the block's aligned start.
// Entries outside [k0, k1) (neighbouring rows or the zeroed tail, all valid
// column indices) are computed too and never read.
template <int NT>
__device__ __forceinline__ void fwd_products(const BlockMeta& m, const VecRegs& R, const float* xs, int nbp,
                                             float* prod) {
  const int a0 = m.k0 & ~3;
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int off = 4 * (threadIdx.x + j * kThreads);
    if (a0 + off < m.k1) {
#pragma unroll
      for (int q = 0; q < NT; ++q) {
        const float* xq = xs + q * nbp;
        float4 p;
        p.x = R.v[j].x * xq[R.c[j].x];
        p.y = R.v[j].y * xq[R.c[j].y];
        p.z = R.v[j].z * xq[R.c[j].z];
        p.w = R.v[j].w * xq[R.c[j].w];
        *reinterpret_cast<float4*>(prod + q * kFwdNnzMax + off) = p;
      }
    }
  }
}

// Staging of a forward pass's inputs in LDS: the penalty table and the NT
// vectors the pass multiplies by (row q of `src`, stride pad4(nb)).  The
// first round of loads (2048 entries per vector, and the table) goes to
// registers so that a caller can issue further loads before it waits for
// them; stage_finish stores them, stages the rest and ends with a barrier.
constexpr int kStageU = 8;   // entries per thread per round and vector

template <int NT>
struct StageRegs {
  float v[NT][kStageU];
  float sc[kStageU];
  double tab;
};

template <int NT, int THREADS = kThreads, int ST = ST_F32>
__device__ __forceinline__ void stage_start(const FwdArgs& a, const float* src, bool want_sid, StageRegs<NT>& R) {
  const int tid = threadIdx.x, nb = a.nb, nbp = pad4(nb);
  // (slots wholly past the last entry for this wave issue no loads)
  const int wave0 = uniform(tid - (tid & 63));
#pragma unroll
  for (int q = 0; q < NT; ++q) {
#pragma unroll
    for (int u = 0; u < kStageU; ++u) {
      const int i = tid + u * THREADS;
      R.v[q][u] = (wave0 + u * THREADS < nb) ? src[q * nbp + (i < nb ? i : 0)] : 0.0f;
    }
  }
  if constexpr (coded(ST)) {
#pragma unroll
    for (int u = 0; u < kStageU; ++u) {
      const int i = tid + u * THREADS;
      R.sc[u] = (wave0 + u * THREADS < nb) ? a.col_scale[i < nb ? i : 0] : 0.0f;
    }
  }
  // first THREADS doubles of the table (4 per structure); the rest in stage_finish
  R.tab = (want_sid && tid < 4 * a.nstruct) ? reinterpret_cast<const double*>(a.pen.table)[tid] : 0.0;
}

// With 16-bit storage the staged vector is scaled by the beamlet scales, so
// that the products use the codes directly: sum_i q_ji (s_i x_i).
template <int NT, int THREADS = kThreads, int ST = ST_F32>
__device__ __forceinline__ void stage_finish(const FwdArgs& a, const float* src, bool want_sid,
                                             const StageRegs<NT>& R, PenaltyDev* tab, float* xs) {
  const int tid = threadIdx.x, nb = a.nb, nbp = pad4(nb);
  if (want_sid) {
    double* dst = reinterpret_cast<double*>(tab);
    if (tid < 4 * a.nstruct) dst[tid] = R.tab;
    for (int i = tid + THREADS; i < 4 * a.nstruct; i += THREADS)
      dst[i] = reinterpret_cast<const double*>(a.pen.table)[i];
  }
#pragma unroll
  for (int q = 0; q < NT; ++q) {
#pragma unroll
    for (int u = 0; u < kStageU; ++u) {
      const int i = tid + u * THREADS;
      if (i < nb) xs[q * nbp + i] = !coded(ST) ? R.v[q][u] : R.v[q][u] * R.sc[u];
    }
  }
  for (int i0 = tid + kStageU * THREADS; i0 < nb; i0 += kStageU * THREADS) {
    float v[NT][kStageU];
#pragma unroll
    for (int q = 0; q < NT; ++q) {
#pragma unroll
      for (int u = 0; u < kStageU; ++u) {
        const int i = i0 + u * THREADS;
        v[q][u] = src[q * nbp + (i < nb ? i : 0)];
        if constexpr (coded(ST)) v[q][u] *= a.col_scale[i < nb ? i : 0];
      }
    }
#pragma unroll
    for (int q = 0; q < NT; ++q) {
#pragma unroll
      for (int u = 0; u < kStageU; ++u) {
        const int i = i0 + u * THREADS;
        if (i < nb) xs[q * nbp + i] = v[q][u];
      }
    }
  }
  __syncthreads();
}

// Trial staging of a solve's forward pass: for every beamlet the gradient
// entry (columns shared by two adjoint workgroups completed from their two
// float64 pieces, in order; by more, from the per-workgroup pieces), the
// iterate x_k (the state names its buffer; every candidate is loaded before
// the state arrives) and the NT trial points x_t^(q) = max(0, x_k - lambda_q g)
// (Eq. (4) with the projection of step 2), written to LDS.  The lead
// workgroup also stores the trials in their iterate buffers and reduces
// their step norms ||x_t^(q) - x_k||^2.  The initial evaluation stages x_1.
constexpr int kTrialU = 4;   // beamlets per thread per round of trial staging

template <int NT>
struct TrialRegs {
  float xc[NT + 1][kTrialU];
  float g[kTrialU];
  double p0[kTrialU], p1[kTrialU];
  uint32_t kind[kTrialU];
  float sc[kTrialU];
  double tab;
};

// Buffer loads bounded by nb: the slots of a thread past the last beamlet
// read zeros and send no request to memory.
template <int NT, int THREADS = kThreads, int ST = ST_F32>
__device__ __forceinline__ void trial_load(const FwdArgs& a, int i0, TrialRegs<NT>& R) {
  const uint32_t nb = static_cast<uint32_t>(a.nb);
  rsrc_t rx[NT + 1];
#pragma unroll
  for (int j = 0; j <= NT; ++j) rx[j] = make_rsrc(a.xbuf[j], 4u * nb);
  const rsrc_t rg = make_rsrc(a.g, 4u * nb);
  const rsrc_t rp = make_rsrc(a.pieces_col, a.pieces_col ? 16u * nb : 0u);
  const rsrc_t rk = make_rsrc(a.col_kind, nb);
  const rsrc_t rs = make_rsrc(a.col_scale, (coded(ST) && a.col_scale) ? 4u * nb : 0u);
  // a slot wholly past the last beamlet for this wave issues no loads at
  // all (out-of-range lanes cost address cycles even when they read zeros)
  const int wave0 = uniform(i0 - static_cast<int>(threadIdx.x & 63));
#pragma unroll
  for (int u = 0; u < kTrialU; ++u) {
    const uint32_t i = static_cast<uint32_t>(i0 + u * THREADS);
    if (wave0 + u * THREADS < a.nb) {
#pragma unroll
      for (int j = 0; j <= NT; ++j) R.xc[j][u] = load_f32(rx[j], 4u * i);
      R.g[u] = load_f32(rg, 4u * i);
      R.p0[u] = load_f64(rp, 16u * i);
      R.p1[u] = load_f64(rp, 16u * i + 8u);
      R.kind[u] = load_u8(rk, i);
      if constexpr (coded(ST)) R.sc[u] = load_f32(rs, 4u * i);
    } else {
#pragma unroll
      for (int j = 0; j <= NT; ++j) R.xc[j][u] = 0.0f;
      R.g[u] = 0.0f;
      R.p0[u] = R.p1[u] = 0.0;
      R.kind[u] = 0;
      R.sc[u] = 0.0f;
    }
  }
}

// Sum of the pieces of a column shared by three or more adjoint workgroups
// (16-bit storage: of the codes' products, before the beamlet scale).
__device__ __forceinline__ double pieces_sum(const FwdArgs& a, int c) {
  const int wlo = a.col_wlo[c], whi = a.col_whi[c];
  double tot = a.pieces[2 * wlo + 1];
  for (int w = wlo + 1; w < whi; ++w) tot += a.pieces[2 * w];
  tot += a.pieces[2 * whi];
  return tot;
}

struct TrialCtl {
  bool init, lead;
  int xi;
};

template <int NT, int THREADS = kThreads, int ST = ST_F32>
__device__ __forceinline__ void trial_store(const FwdArgs& a, int i0, const TrialRegs<NT>& R, const TrialCtl& T,
                                            const double (&lam)[NT], float* xs, double (&sq)[NT]) {
  const int nb = a.nb, nbp = pad4(nb);
#pragma unroll
  for (int u = 0; u < kTrialU; ++u) {
    const int i = i0 + u * THREADS;
    if (i >= nb) continue;
    float x = R.xc[0][u];
#pragma unroll
    // x_k is the candidate the state names.  Blended with exact 0/1 weights
    // rather than selected: a select among elements of the candidate array
    // becomes an indexed load from a stack copy of it (scratch memory).  The
    // candidates are finite: each solve starts with the other iterate
    // buffers zeroed, and a non-finite trial ends the solve.
    for (int j = 1; j <= NT; ++j) {
      const float c = (T.xi == j) ? 1.0f : 0.0f;
      x = x * (1.0f - c) + R.xc[j][u] * c;
    }
    if (T.init) {
#pragma unroll
      for (int q = 0; q < NT; ++q) xs[q * nbp + i] = !coded(ST) ? x : x * R.sc[u];
      continue;
    }
    const double gf = !coded(ST) ? a.g_scale : a.g_scale * static_cast<double>(R.sc[u]);
    float g = R.g[u];
    if (R.kind[u] == 1) g = static_cast<float>(gf * (R.p0[u] + R.p1[u]));
    else if (R.kind[u] > 1) g = static_cast<float>(gf * pieces_sum(a, i));
#pragma unroll
    for (int q = 0; q < NT; ++q) {
      const float t = trial_point(x, g, lam[q]);
      xs[q * nbp + i] = !coded(ST) ? t : t * R.sc[u];
      if (T.lead) {
        select_buf(a.xbuf, (T.xi + 1 + q) % (NT + 1))[i] = t;
        const double dl = static_cast<double>(t) - static_cast<double>(x);
        sq[q] += dl * dl;
      }
    }
  }
}

// After the first round (loaded by the caller): the remaining rounds, the
// lead workgroup's step norms, the penalty table; ends with a barrier.
template <int NT, int THREADS = kThreads, int ST = ST_F32>
__device__ __forceinline__ void trial_finish(const FwdArgs& a, const TrialRegs<NT>& R, const TrialCtl& T,
                                             const double (&lam)[NT], PenaltyDev* tab, float* xs, double* red,
                                             int G) {
  const int tid = threadIdx.x;
  double sq[NT];
#pragma unroll
  for (int q = 0; q < NT; ++q) sq[q] = 0.0;
  {
    double* dst = reinterpret_cast<double*>(tab);
    if (tid < 4 * a.nstruct) dst[tid] = R.tab;
    for (int i = tid + THREADS; i < 4 * a.nstruct; i += THREADS)
      dst[i] = reinterpret_cast<const double*>(a.pen.table)[i];
  }
  trial_store<NT, THREADS, ST>(a, tid, R, T, lam, xs, sq);
  for (int i0 = tid + kTrialU * THREADS; i0 < a.nb; i0 += kTrialU * THREADS) {
    TrialRegs<NT> R2;
    trial_load<NT, THREADS, ST>(a, i0, R2);
    trial_store<NT, THREADS, ST>(a, i0, R2, T, lam, xs, sq);
  }
  if (T.lead && !T.init) {
#pragma unroll
    for (int q = 0; q < NT; ++q) {
      const double t = block_sum<double, THREADS / 64>(sq[q], red);
      if (tid == 0) a.partials[NT * G + q] = t;
    }
  }
  __syncthreads();
}

template <int NT, int THREADS = kThreads>
__device__ __forceinline__ void stage_inputs(const FwdArgs& a, const float* src, PenaltyDev* tab, float* xs,
                                             bool want_sid) {
  StageRegs<NT> R;
  stage_start<NT, THREADS>(a, src, want_sid, R);
  stage_finish<NT, THREADS>(a, src, want_sid, R, tab, xs);
}

// Forward pass.  Each workgroup stages the NT trial vectors
// x_t^(q) = max(0, x_k - lambda_q g_k) and the penalty table in LDS
// (workgroup 0 also stores the trials and their step norms), then walks its
// contiguous range of row blocks (at most kFwdPartNnz nonzeros each).  The
// next block's col_idx/val (16-byte loads), row pointers and structure ids are
// in flight while the current block's rows are summed from LDS by
// lanes-per-row groups and the penalty epilogue writes r and accumulates G.
template <int NT>
__global__ __launch_bounds__(kThreads) void fwd_kernel(FwdArgs a) {
  extern __shared__ __align__(16) unsigned char smem[];
  const int nb = a.nb;
  const int nbp = pad4(nb);
  PenaltyDev* tab = reinterpret_cast<PenaltyDev*>(smem);
  float* xs = reinterpret_cast<float*>(tab + a.nstruct);
  float* prod = xs + NT * nbp;
  int32_t* rp = reinterpret_cast<int32_t*>(prod + NT * kFwdNnzMax);
  uint8_t* sidl = reinterpret_cast<uint8_t*>(rp + kFwdRowsMax + 1);
  __shared__ double red[kWaves];
  __shared__ float redf[kWaves];

  const int tid = threadIdx.x;
  const bool solve = (a.mode == FWD_SOLVE);
  const bool want_sid = (a.mode != FWD_PLAIN);
  int ntr = 1;
  float* rout[NT];
#pragma unroll
  for (int q = 0; q < NT; ++q) rout[q] = nullptr;
  TrialCtl T{true, false, 0};
  double lam[NT];
#pragma unroll
  for (int q = 0; q < NT; ++q) lam[q] = 0.0;
  if (solve) {
    const SolverState* st = a.st_in;
    // the state passes through unchanged (word copy by workgroup 0)
    constexpr int kWords = static_cast<int>(sizeof(SolverState) / sizeof(int32_t));
    if (blockIdx.x == 0 && tid < kWords)
      reinterpret_cast<int32_t*>(a.st_out)[tid] = reinterpret_cast<const int32_t*>(st)[tid];
    const int phase = st->phase;
    if (phase == PH_DONE) return;
    ntr = (phase == PH_INIT) ? 1 : NT;
    T.init = (phase == PH_INIT);
    T.lead = (blockIdx.x == 0);
    T.xi = st->xi;
    lam[0] = st->lambda;
    const double alpha = st->alpha;
#pragma unroll
    for (int q = 1; q < NT; ++q) lam[q] = lam[q - 1] / alpha;
#pragma unroll
    for (int q = 0; q < NT; ++q) rout[q] = a.rbuf[q];
  }

  int b0, b1;
  work_range(a.nblocks, b0, b1);
  // first block's data in flight while the trial vectors are staged
  VecRegs R;
  RowRegs Q;
  BlockMeta cur{0, 0, 0, 0}, nxt{0, 0, 0, 0};
  if (b0 < b1) {
    cur = block_meta(a, b0);
    if (cur.k1 - cur.k0 <= kFwdPartNnz) {
      issue_vec(a.col_idx, a.val, cur.k0 & ~3, cur.k1, R);
      issue_rows(a, cur, want_sid, Q);
    }
    if (b0 + 1 < b1) nxt = block_meta(a, b0 + 1);
  }

  if (solve) {
    TrialRegs<NT> TR;
    trial_load<NT>(a, tid, TR);
    TR.tab = (tid < 4 * a.nstruct) ? reinterpret_cast<const double*>(a.pen.table)[tid] : 0.0;
    trial_finish<NT>(a, TR, T, lam, tab, xs, red, gridDim.x);
  } else {
    stage_inputs<NT>(a, a.x, tab, xs, want_sid);
  }

  double pacc[NT];
#pragma unroll
  for (int q = 0; q < NT; ++q) pacc[q] = 0.0;

  for (int b = b0; b < b1; ++b) {
    const bool more = (b + 1 < b1);
    if (cur.k1 - cur.k0 > kFwdPartNnz) {
      // a single row longer than an LDS block: all lanes stride over it
      float s[NT];
#pragma unroll
      for (int q = 0; q < NT; ++q) s[q] = 0.f;
      for (int k = cur.k0 + tid; k < cur.k1; k += kThreads) {
        const int c = a.col_idx[k];
        const float v = a.val[k];
#pragma unroll
        for (int q = 0; q < NT; ++q) s[q] = fmaf(v, xs[q * nbp + c], s[q]);
      }
#pragma unroll
      for (int q = 0; q < NT; ++q) s[q] = block_sum(s[q], redf);
      if (tid == 0) row_epilogue<NT>(a, cur.r0, want_sid ? a.pen.sid[cur.r0] : 0, tab, s, pacc, rout, ntr);
      if (more) {
        cur = nxt;
        if (cur.k1 - cur.k0 <= kFwdPartNnz) {
          issue_vec(a.col_idx, a.val, cur.k0 & ~3, cur.k1, R);
          issue_rows(a, cur, want_sid, Q);
        }
        if (b + 2 < b1) nxt = block_meta(a, b + 2);
      }
      continue;
    }
    const int nr = cur.r1 - cur.r0;
    fwd_products<NT>(cur, R, xs, nbp, prod);
    stage_rows(cur, Q, rp, sidl);
    __syncthreads();
    const BlockMeta blk = cur;
    if (more) {
      cur = nxt;
      if (cur.k1 - cur.k0 <= kFwdPartNnz) {
        issue_vec(a.col_idx, a.val, cur.k0 & ~3, cur.k1, R);
        issue_rows(a, cur, want_sid, Q);
      }
      if (b + 2 < b1) nxt = block_meta(a, b + 2);
    }
    const int L = lanes_per_row(nr);
    const int lane = tid & (L - 1);
    for (int row = tid / L; row < nr; row += kThreads / L) {
      const int s0 = rp[row], s1 = rp[row + 1];
      float s[NT];
#pragma unroll
      for (int q = 0; q < NT; ++q) s[q] = 0.f;
      // four independent LDS reads per round; slots past the row read as 0
      for (int k = s0 + lane; k < s1; k += 4 * L) {
#pragma unroll
        for (int q = 0; q < NT; ++q) {
          const float* pq = prod + q * kFwdNnzMax;
          float v[4];
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            const int kk = k + u * L;
            const float t = pq[kk < kFwdNnzMax ? kk : kFwdNnzMax - 1];
            v[u] = (kk < s1) ? t : 0.0f;
          }
          s[q] += (v[0] + v[1]) + (v[2] + v[3]);
        }
      }
      for (int off = L >> 1; off > 0; off >>= 1) {
#pragma unroll
        for (int q = 0; q < NT; ++q) s[q] += __shfl_xor(s[q], off, 64);
      }
      if (lane == 0) row_epilogue<NT>(a, blk.r0 + row, sidl[row], tab, s, pacc, rout, ntr);
    }
    __syncthreads();
  }

#pragma unroll
  for (int q = 0; q < NT; ++q) {
    const double t = block_sum(pacc[q], red);
    if (tid == 0) a.partials[q * gridDim.x + blockIdx.x] = t;
  }
}

// ---- wave-granular forward pass --------------------------------------------------
// Each of the four waves of a workgroup streams its own contiguous range of
// small row blocks (at most wave_part_nnz nonzeros and kWaveRowsMax rows),
// an even split of the block count (a block's time is mostly latency, so
// equal counts balance better than equal bytes).
// Block bounds come from per-lane copies of the block table read with
// readlane, so all control flow and every descriptor is wave-uniform.  A
// block's column indices and values arrive as 16-byte buffer loads (lanes
// past the block read zeros), its products D_ij x_j go to the wave's LDS
// region, and groups of L lanes (the largest power of two with L * rows <= 64)
// sum one row each, reading four products per round and combining the lanes
// with DPP moves.  Row pointers and structure ids of a row are loaded by the
// lane that finishes it.  The next block's loads are issued as soon as the
// products of the current one are in LDS.
constexpr int kWaveSlack = 256;   // LDS floats after the last wave region (over-reads of masked slots)

// Groups of four entries per lane in one wave's row block: 2 (512 entries)
// with float32 storage, 3 (768) with float32 values and 16-bit indices, 4
// (1024 entries) with 16-bit storage.
template <int ST>
constexpr int wave_groups() { return wave_nnz(ST) / 256; }

template <int ST>
struct WaveStage {
  ColGroup<ST> c[wave_groups<ST>()];
  ValGroup<ST> v[wave_groups<ST>()];
  int rlo[kWavePasses], rhi[kWavePasses];
  uint32_t sid[kWavePasses];
};

// Loads of the entries base + 4 lane + 256 j + u (u < 4, j < the group count)
// of the CSR index and value arrays; base is a multiple of 4 and the arrays
// carry a zeroed tail, so whole groups stay in bounds and entries past k1
// read zeros.
template <int ST, int CP = 0>
__device__ __forceinline__ void csr_issue(const FwdArgs& a, int base, int k1, int lane,
                                          ColGroup<ST> (&c)[wave_groups<ST>()],
                                          ValGroup<ST> (&v)[wave_groups<ST>()]) {
  constexpr int G = wave_groups<ST>();
  if constexpr (ST == ST_F32) {
    const uint32_t bytes = static_cast<uint32_t>((k1 - base) * 4 + 15) & ~15u;
    const rsrc_t rc = make_rsrc(a.col_idx + base, bytes);
    const rsrc_t rv = make_rsrc(a.val + base, bytes);
#pragma unroll
    for (int j = 0; j < G; ++j) {
      c[j] = load_i4s<CP>(rc, 16 * lane + 1024 * j);
      v[j] = load_f4s<CP>(rv, 16 * lane + 1024 * j);
    }
  } else if constexpr (ST == ST_F32C16) {
    const uint32_t n = static_cast<uint32_t>(k1 - base);
    const rsrc_t rc = make_rsrc(a.col16 + base, (n * 2 + 7) & ~7u);
    const rsrc_t rv = make_rsrc(a.val + base, (n * 4 + 15) & ~15u);
#pragma unroll
    for (int j = 0; j < G; ++j) {
      c[j] = load_u2s<CP>(rc, 8 * lane + 512 * j);
      v[j] = load_f4s<CP>(rv, 16 * lane + 1024 * j);
    }
  } else {
    const uint32_t bytes = static_cast<uint32_t>((k1 - base) * 2 + 7) & ~7u;
    const rsrc_t rc = make_rsrc(a.col16 + base, bytes);
    const rsrc_t rv = make_rsrc(a.val16 + base, bytes);
#pragma unroll
    for (int j = 0; j < G; ++j) {
      c[j] = load_u2s<CP>(rc, 8 * lane + 512 * j);
      v[j] = load_u2s<CP>(rv, 8 * lane + 512 * j);
    }
  }
}

struct WaveBlock {
  int r0, r1, k0, k1;
};

__device__ __forceinline__ int log2_lanes(int nr) {
  // largest L = 2^e <= 64 with L * nr <= 64 (L = 1 beyond 64 rows)
  int e = 6;
  while (e > 0 && (nr << e) > 64) --e;
  return e;
}

// UNCOND: every row load is issued (rows past the block read zeros out of
// bounds), so that no load of the block sits in a branch and a later wait
// for an earlier load can count exactly how many were issued after it.
template <int MODE, bool UNCOND = false, int ST = ST_F32, int CP = 0>
__device__ __forceinline__ void wave_issue(const FwdArgs& a, const WaveBlock& m, int lane, WaveStage<ST>& S) {
  csr_issue<ST, CP>(a, m.k0 & ~3, m.k1, lane, S.c, S.v);
  const int nr = m.r1 - m.r0;
  const int e = log2_lanes(nr);
  const int passes = ((nr << e) + 63) >> 6;
  const rsrc_t rp = make_rsrc(a.row_ptr + m.r0, static_cast<uint32_t>(nr + 1) * 4);
  const rsrc_t rs = make_rsrc(a.pen.sid + m.r0, static_cast<uint32_t>(nr));
#pragma unroll
  for (int p = 0; p < kWavePasses; ++p) {
    S.rlo[p] = S.rhi[p] = 0;
    S.sid[p] = 0;
    if (UNCOND) {
      const int row = (p < passes) ? (p << (6 - e)) + (lane >> e) : nr + 1;
      S.rlo[p] = load_i32(rp, 4 * row);
      S.rhi[p] = load_i32(rp, 4 * row + 4);
      if (MODE != FWD_PLAIN) S.sid[p] = load_u8(rs, row);
    } else if (p < passes) {
      const int row = (p << (6 - e)) + (lane >> e);
      S.rlo[p] = load_i32(rp, 4 * row);
      S.rhi[p] = load_i32(rp, 4 * row + 4);
      if (MODE != FWD_PLAIN) S.sid[p] = load_u8(rs, row);
    }
  }
}

template <int NT, int MODE>
__device__ __forceinline__ void row_finish(const FwdArgs& a, int row, uint32_t sid, const PenaltyDev* tab,
                                           const float (&d)[NT], double (&pacc)[NT], const rsrc_t (&rout)[NT],
                                           const rsrc_t& dout, int ntr) {
#pragma clang fp contract(off)
  const uint32_t off = 4u * static_cast<uint32_t>(row);
  if (MODE == FWD_PLAIN) {
    store_f32(dout, off, d[0]);
    pacc[0] += static_cast<double>(d[0]) * static_cast<double>(d[0]);
    return;
  }
  const RowPenalty pen = row_penalty(a.pen, row, tab, static_cast<uint8_t>(sid));
#pragma unroll
  for (int q = 0; q < NT; ++q) {
    if (q < ntr) {
      double F;
      float r;
      penalty(pen, d[q], F, r);
      pacc[q] += F;
      if (MODE == FWD_SOLVE) {
        store_f32(rout[q], off, r);
      } else if (q == 0) {
        if (a.r_out) store_f32(rout[0], off, r);
        if (a.d_out) store_f32(dout, off, d[0]);
      }
    }
  }
}

// Row sums of one block with L lanes per row.
template <int L, int NT, int MODE, int NNZ, typename WS>
__device__ __forceinline__ void wave_rows(const FwdArgs& a, const float* prod, int lane, const WaveBlock& m,
                                          const WS& S, const PenaltyDev* tab, double (&pacc)[NT],
                                          const rsrc_t (&rout)[NT], const rsrc_t& dout, int ntr) {
  constexpr int kRowsPerPass = 64 / L;
  const int a0 = m.k0 & ~3;
  const int nr = m.r1 - m.r0;
  const int passes = (nr * L + 63) / 64;
  const int sub = lane & (L - 1);
#pragma unroll
  for (int p = 0; p < kWavePasses; ++p) {
    if (p < passes) {
      const int row = p * kRowsPerPass + lane / L;
      const int s1 = S.rhi[p] - a0;
      float acc[NT];
#pragma unroll
      for (int q = 0; q < NT; ++q) acc[q] = 0.f;
      // rounds of four products per lane: whole rounds first, then at most
      // one round that runs past the row's end (its tail slots read as zero)
      int k = S.rlo[p] - a0 + sub;
      for (; k + 3 * L < s1; k += 4 * L) {
#pragma unroll
        for (int q = 0; q < NT; ++q) {
          const float* pq = prod + q * NNZ + k;
          acc[q] += (pq[0] + pq[L]) + (pq[2 * L] + pq[3 * L]);
        }
      }
      if (k < s1) {
        const int left = s1 - k;
#pragma unroll
        for (int q = 0; q < NT; ++q) {
          const float* pq = prod + q * NNZ + k;
          float v[4];
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            const float t = pq[u * L];   // always in the allocation; masked below
            v[u] = (u * L < left) ? t : 0.0f;
          }
          acc[q] += (v[0] + v[1]) + (v[2] + v[3]);
        }
      }
      float d[NT];
#pragma unroll
      for (int q = 0; q < NT; ++q) d[q] = group_sum<L>(acc[q]);
      if (sub == L - 1 && row < nr) row_finish<NT, MODE>(a, m.r0 + row, S.sid[p], tab, d, pacc, rout, dout, ntr);
    }
  }
}

// Waves of a wave-granular forward workgroup: sixteen, one workgroup per
// compute unit, for a matrix solved alone; eight, up to three side by side,
// once per-plan targets are applied for dispatches that several plans share
// (one workgroup's staging -- the start of every workgroup, and of every
// plan's workgroups in a batched pass -- then overlaps the others'
// streams).  Launch bounds: 8-wave workgroups with one and two trials per
// pass keep within 80 and 128 registers per lane (six and four waves per
// SIMD); four trials take 8-wave workgroups with no such bound.
template <int NT, int WAVES>
constexpr int fwd_min_waves_per_simd() { return WAVES == 16 ? 4 : NT == 1 ? 6 : NT == 2 ? 4 : 1; }
constexpr int kMetaChunk = 256;   // row blocks whose bounds are staged in LDS at a time

template <int NT, int MODE, int WAVES, int ST, int CP = 0>
__device__ __forceinline__ void fwd_wave_pass(const FwdArgs& a, const Slot sl) {
  constexpr int THREADS = WAVES * 64;
  constexpr int NNZ = wave_nnz(ST), PART = wave_part_nnz(ST), NG = wave_groups<ST>();
  extern __shared__ __align__(16) unsigned char smem[];
  const int nb = a.nb;
  const int nbp = pad4(nb);
  PenaltyDev* tab = reinterpret_cast<PenaltyDev*>(smem);
  float* xs = reinterpret_cast<float*>(tab + a.nstruct);
  float* prod0 = xs + NT * nbp;
  int32_t* mrow = reinterpret_cast<int32_t*>(prod0 + WAVES * NT * NNZ + kWaveSlack);
  int32_t* mk0 = mrow + (kMetaChunk + 1);
  int32_t* mend = mk0 + (kMetaChunk + 1);
  double* gpart = reinterpret_cast<double*>(mend + kMetaChunk + 2);   // 8-byte aligned
  const int wv = uniform(threadIdx.x >> 6), lane = threadIdx.x & 63;
  float* prod = prod0 + wv * (NT * NNZ);
  __shared__ double red[WAVES];
  __shared__ int next_blk;

  const int tid = threadIdx.x;
  constexpr bool solve = (MODE == FWD_SOLVE);
  constexpr bool want_sid = (MODE != FWD_PLAIN);

  // This workgroup's contiguous range of row blocks; its waves take blocks
  // in turn from a counter in LDS (the first WAVES blocks one each), so a
  // wave that runs faster takes more.  Every block's objective contribution
  // goes to its own LDS slot and the workgroup adds the slots in block order,
  // so the total does not depend on which wave took which block.
  const int G = sl.G, w = sl.w;
  const int lw = (G % kXcds == 0) ? (w % kXcds) * (G / kXcds) + w / kXcds : w;
  const int B0 = split_point(lw, a.nwblocks, G);
  const int B1 = split_point(lw + 1, a.nwblocks, G);
  // Loads in the order their results are needed, none of them in a branch:
  // the first block's bounds (lanes 0 and 1), the staging inputs (a solve's
  // trial inputs before the state is known), the state (one word per lane),
  // then the first block's nonzeros.  So no wait for one of them waits for a
  // later one, and the block's loads overlap the staging.
  int b = B0 + wv;
  const bool first = b < min(B1, B0 + kMetaChunk);
  const uint32_t meta_bytes = 4u * static_cast<uint32_t>(a.nwblocks + 1);
  const uint32_t moff = 4u * static_cast<uint32_t>(b + (lane & 1));
  const int mrow0 = load_i32(make_rsrc(a.wblock_row, meta_bytes), 4u * static_cast<uint32_t>(b));
  const int mend0 = load_i32(make_rsrc(a.wblock_end, meta_bytes - 4u), 4u * static_cast<uint32_t>(b));
  const int mk00 = load_i32(make_rsrc(a.wblock_k0, meta_bytes), moff);
  // the first chunk's block bounds (thread i loads entry B0 + i), stored to
  // LDS before the staging barrier, so that no round trip and no barrier of
  // their own stand between the staging and the first block
  static_assert(THREADS > kMetaChunk, "one thread per bound of the first chunk");
  const int cfirst = min(B1, B0 + kMetaChunk) - B0;
  const uint32_t mi = 4u * static_cast<uint32_t>(B0 + tid);
  const int pre_row = load_i32(make_rsrc(a.wblock_row, meta_bytes), mi);
  const int pre_k0 = load_i32(make_rsrc(a.wblock_k0, meta_bytes), mi);
  const int pre_end = load_i32(make_rsrc(a.wblock_end, meta_bytes - 4u), mi);
  TrialRegs<NT> TR;
  StageRegs<NT> SR;
  int32_t sw = 0;
  if (solve) {
    trial_load<NT, THREADS, ST>(a, tid, TR);
    TR.tab = load_f64(make_rsrc(a.pen.table, 32u * static_cast<uint32_t>(a.nstruct)), 8u * tid);
    sw = reinterpret_cast<const int32_t*>(a.st_in)[lane < kStateWords ? lane : 0];
  } else {
    stage_start<NT, THREADS, ST>(a, a.x, want_sid, SR);
  }
  WaveBlock cur{0, 0, 0, 0};
  if (first) {
    cur.r0 = __builtin_amdgcn_readlane(mrow0, 0);
    cur.r1 = __builtin_amdgcn_readlane(mend0, 0);
    cur.k0 = __builtin_amdgcn_readlane(mk00, 0);
    cur.k1 = __builtin_amdgcn_readlane(mk00, 1);
  }
  // a row longer than a wave block is streamed in the loop instead
  const bool short_first = cur.k1 - cur.k0 <= PART;
  WaveStage<ST> S;
  wave_issue<MODE, true, ST, CP>(a, short_first ? cur : WaveBlock{0, 0, 0, 0}, lane, S);

  int ntr = 1;
  rsrc_t rout[NT];
  const uint32_t vbytes = 4u * static_cast<uint32_t>(a.nv);
#pragma unroll
  for (int q = 0; q < NT; ++q) rout[q] = make_rsrc(a.r_out, a.r_out ? vbytes : 0u);
  const rsrc_t dout = make_rsrc(a.d_out, a.d_out ? vbytes : 0u);
  TrialCtl T{true, false, 0};
  double lam[NT];
#pragma unroll
  for (int q = 0; q < NT; ++q) lam[q] = 0.0;
  if (solve) {
    if (sl.w == 0 && wv == 0 && lane < kStateWords) reinterpret_cast<int32_t*>(a.st_out)[lane] = sw;
    const int phase = state_int(sw, offsetof(SolverState, phase));
    if (phase == PH_DONE) return;
    ntr = (phase == PH_INIT) ? 1 : NT;
    T.init = (phase == PH_INIT);
    T.lead = (sl.w == 0);
    T.xi = state_int(sw, offsetof(SolverState, xi));
    lam[0] = state_f64(sw, offsetof(SolverState, lambda));
    const double alpha = state_f64(sw, offsetof(SolverState, alpha));
#pragma unroll
    for (int q = 1; q < NT; ++q) lam[q] = lam[q - 1] / alpha;
#pragma unroll
    for (int q = 0; q < NT; ++q) rout[q] = make_rsrc(a.rbuf[q], vbytes);
  }
  if (tid <= cfirst) {
    mrow[tid] = pre_row;
    mk0[tid] = pre_k0;
    if (tid < cfirst) mend[tid] = pre_end;
  }
  if (tid == 0) next_blk = B0 + WAVES;
  // (both stagings end with a barrier)
  if (solve) trial_finish<NT, THREADS, ST>(a, TR, T, lam, tab, xs, red, sl.G);
  else stage_finish<NT, THREADS, ST>(a, a.x, want_sid, SR, tab, xs);

  double gsum[NT];
#pragma unroll
  for (int q = 0; q < NT; ++q) gsum[q] = 0.0;
  for (int c0 = B0; c0 < B1; c0 += kMetaChunk) {
    const int c1 = min(c0 + kMetaChunk, B1);
    if (c0 != B0) {
      for (int i = tid; i <= c1 - c0; i += THREADS) {
        mrow[i] = a.wblock_row[c0 + i];
        mk0[i] = a.wblock_k0[c0 + i];
        if (i < c1 - c0) mend[i] = a.wblock_end[c0 + i];
      }
      if (tid == 0) next_blk = c0 + WAVES;
      __syncthreads();
    }
    auto meta = [&](int blk) {
      const int i = blk - c0;
      WaveBlock m;
      m.r0 = uniform(mrow[i]);
      m.r1 = uniform(mend[i]);
      m.k0 = uniform(mk0[i]);
      m.k1 = uniform(mk0[i + 1]);
      return m;
    };
    if (c0 != B0) {
      b = c0 + wv;
      cur = (b < c1) ? meta(b) : WaveBlock{0, 0, 0, 0};
      wave_issue<MODE, true, ST, CP>(a, (b < c1 && cur.k1 - cur.k0 <= PART) ? cur : WaveBlock{0, 0, 0, 0}, lane, S);
    }
    while (b < c1) {
      // the block after this one (taken now, its loads issued once this
      // block's products are in LDS)
      int nxt = 0;
      if (lane == 0) nxt = atomicAdd(&next_blk, 1);
      nxt = uniform(nxt);
      const WaveBlock blk = cur;
      const bool more = nxt < c1;
      if (more) cur = meta(nxt);
      double pb[NT];
#pragma unroll
      for (int q = 0; q < NT; ++q) pb[q] = 0.0;
      if (blk.k1 - blk.k0 > PART) {
        // one row longer than a wave block: the wave strides over it
        float acc[NT];
#pragma unroll
        for (int q = 0; q < NT; ++q) acc[q] = 0.f;
        for (int base = blk.k0 & ~3; base < blk.k1; base += NNZ) {
          ColGroup<ST> cg[NG];
          ValGroup<ST> vg[NG];
          csr_issue<ST, CP>(a, base, blk.k1, lane, cg, vg);
#pragma unroll
          for (int j = 0; j < NG; ++j) {
            const int e0 = base + 4 * lane + 256 * j;
#pragma unroll
            for (int q = 0; q < NT; ++q) {
#pragma unroll
              for (int u = 0; u < 4; ++u) {
                const float t = val_of<ST>(vg[j], u) * xs[q * nbp + col_of(cg[j], u)];
                acc[q] += (e0 + u >= blk.k0 && e0 + u < blk.k1) ? t : 0.0f;
              }
            }
          }
        }
        float d[NT];
#pragma unroll
        for (int q = 0; q < NT; ++q) d[q] = wave_sum(acc[q]);
        if (lane == 63) {
          const uint32_t sid = want_sid ? a.pen.sid[blk.r0] : 0;
          row_finish<NT, MODE>(a, blk.r0, sid, tab, d, pb, rout, dout, ntr);
        }
        wave_issue<MODE, true, ST, CP>(a, (more && cur.k1 - cur.k0 <= PART) ? cur : WaveBlock{0, 0, 0, 0}, lane, S);
      } else {
        // products of this block into the wave's LDS region (lanes past the
        // block hold zeros and write slots that no row reads)
#pragma unroll
        for (int j = 0; j < NG; ++j) {
          const int off = 4 * lane + 256 * j;
#pragma unroll
          for (int q = 0; q < NT; ++q) {
            const float* xq = xs + q * nbp;
            float4 p;
            p.x = val_of<ST>(S.v[j], 0) * xq[col_of(S.c[j], 0)];
            p.y = val_of<ST>(S.v[j], 1) * xq[col_of(S.c[j], 1)];
            p.z = val_of<ST>(S.v[j], 2) * xq[col_of(S.c[j], 2)];
            p.w = val_of<ST>(S.v[j], 3) * xq[col_of(S.c[j], 3)];
            *reinterpret_cast<float4*>(prod + q * NNZ + off) = p;
          }
        }
        // LDS operations of one wave complete in order; the fence only keeps
        // the compiler from moving the row reads above the product writes
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        const WaveStage<ST> R = S;   // this block's row pointers and ids (loads already waited on)
        // issued whether or not a next block follows (an empty block reads
        // zeros and touches no memory), so the loads land in the registers
        // the next products read, with no copies to merge two paths
        wave_issue<MODE, true, ST, CP>(a, (more && cur.k1 - cur.k0 <= PART) ? cur : WaveBlock{0, 0, 0, 0}, lane, S);
        switch (log2_lanes(blk.r1 - blk.r0)) {
          case 0: wave_rows<1, NT, MODE, NNZ>(a, prod, lane, blk, R, tab, pb, rout, dout, ntr); break;
          case 1: wave_rows<2, NT, MODE, NNZ>(a, prod, lane, blk, R, tab, pb, rout, dout, ntr); break;
          case 2: wave_rows<4, NT, MODE, NNZ>(a, prod, lane, blk, R, tab, pb, rout, dout, ntr); break;
          case 3: wave_rows<8, NT, MODE, NNZ>(a, prod, lane, blk, R, tab, pb, rout, dout, ntr); break;
          case 4: wave_rows<16, NT, MODE, NNZ>(a, prod, lane, blk, R, tab, pb, rout, dout, ntr); break;
          case 5: wave_rows<32, NT, MODE, NNZ>(a, prod, lane, blk, R, tab, pb, rout, dout, ntr); break;
          default: wave_rows<64, NT, MODE, NNZ>(a, prod, lane, blk, R, tab, pb, rout, dout, ntr); break;
        }
        // the next block's LDS writes must not overtake this block's reads
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      }
#pragma unroll
      for (int q = 0; q < NT; ++q) {
        const double t = wave_sum(pb[q]);
        if (lane == 63) gpart[q * kMetaChunk + (b - c0)] = t;
      }
      b = nxt;
    }
    __syncthreads();
    if (wv == 0) {
      // the chunk's block contributions in a fixed order: lane l adds blocks
      // l, l + 64, ..., then the lanes are summed
#pragma unroll
      for (int q = 0; q < NT; ++q) {
        double t = 0.0;
        for (int i = lane; i < c1 - c0; i += 64) t += gpart[q * kMetaChunk + i];
        gsum[q] += wave_sum(t);
      }
    }
    __syncthreads();
  }
  if (wv == 0 && lane == 63) {
#pragma unroll
    for (int q = 0; q < NT; ++q) a.partials[q * sl.G + sl.w] = gsum[q];
  }
}

template <int NT, int MODE, int WAVES, int ST, int CP = 0>
__global__ __launch_bounds__(WAVES * 64, (fwd_min_waves_per_simd<NT, WAVES>())) void fwd_wave_kernel(FwdArgs a) {
  fwd_wave_pass<NT, MODE, WAVES, ST, CP>(a, Slot{static_cast<int>(blockIdx.x), static_cast<int>(gridDim.x)});
}

// Batched solve pass: slots[blockIdx.x] = (plan << 16) | workgroup of that
// plan's pass, or -1 for an idle slot (plans start at multiples of the die
// count, so each plan keeps its workgroups' die placement).
template <int NT, int WAVES, int ST, int CP = 0>
__global__ __launch_bounds__(WAVES * 64, (fwd_min_waves_per_simd<NT, WAVES>())) void fwd_wave_batch_kernel(const FwdArgs* __restrict__ args,
                                                                    const int32_t* __restrict__ slots) {
  const int sv = uniform(slots[blockIdx.x]);
  if (sv < 0) return;
  const FwdArgs& a = args[sv >> 16];
  fwd_wave_pass<NT, FWD_SOLVE, WAVES, ST, CP>(a, Slot{sv & 0xFFFF, a.grid});
}

int grid_for(int items, int cap) {
  if (items <= 0) return 1;
  if (items <= cap) return items;
  return cap;
}

}  // namespace

size_t forward_lds_bytes(int nb, int ntrials, int nstruct, bool wave, int storage, int dose_waves) {
  const size_t nbp = static_cast<size_t>(pad4(nb));
  size_t bytes = static_cast<size_t>(nstruct) * sizeof(PenaltyDev) +
                 static_cast<size_t>(ntrials) * nbp * sizeof(float);
  if (wave) {
    const size_t waves = static_cast<size_t>(forward_waves(ntrials, dose_waves));
    bytes += (waves * ntrials * wave_nnz(storage) + kWaveSlack) * sizeof(float);
    bytes += (2 * (kMetaChunk + 1) + kMetaChunk + 2) * sizeof(int32_t) +
             static_cast<size_t>(ntrials) * kMetaChunk * sizeof(double);
  } else {
    bytes += static_cast<size_t>(ntrials) * kFwdNnzMax * sizeof(float) +
             static_cast<size_t>(kFwdRowsMax + 1) * sizeof(int32_t) + kFwdRowsMax;
  }
  return bytes;
}

int forward_waves(int ntrials, int dose_waves) { return (ntrials <= 2 && dose_waves == 16) ? 16 : 8; }

int forward_grid(const imrt_ctx* ctx, const imrt_dose* D, int ntrials, bool wave) {
  if (wave) return wave_grid(ctx, D->nwblocks, ntrials, D->fwd_bpw, D->nb, D->fwd_st, D->fwd_waves);
  return grid_for(D->nblocks, kWaves * ctx->tune.fwd_grid_per_cu * ctx->num_cu);
}
int forward_grid(const imrt_ctx* ctx, const imrt_dose* D, int ntrials) {
  return forward_grid(ctx, D, ntrials, ctx->tune.fwd_wave != 0);
}

// Forward workgroups per compute unit: the setting, but no more than fit
// side by side -- by registers (one 16-wave workgroup; three 8-wave ones with
// one trial per pass, two with more) and by LDS (the staged vectors grow with
// nb; a structure table of 16 entries assumed) -- since a workgroup that does
// not fit would only start once another has finished.
int wave_grid(const imrt_ctx* ctx, int nwblocks, int ntrials, int blocks_per_wave, int nb, int storage,
              int dose_waves) {
  const int waves = forward_waves(ntrials, dose_waves);
  const int64_t per = static_cast<int64_t>(waves) * std::max(blocks_per_wave, 1);
  const size_t lds = forward_lds_bytes(nb, ntrials, 16, true, storage, dose_waves);
  const int by_lds = static_cast<int>(std::max<size_t>(1, ctx->cu_lds / std::max<size_t>(lds, 1)));
  const int by_regs = (waves == 16) ? 1 : (ntrials == 1) ? 3 : 2;
  const int per_cu = std::max(1, std::min({ctx->tune.fwd_grid_per_cu, by_regs, by_lds}));
  return grid_for(static_cast<int>((nwblocks + per - 1) / per), per_cu * ctx->num_cu);
}

// Launches take optional start/stop events, recorded by the dispatch itself
// around the kernel (hipExtLaunchKernelGGL), so their elapsed time is the
// kernel's own duration.
template <int ST, int CP>
int launch_wave_solve(const FwdArgs& a, int ntrials, bool w16, dim3 gd, size_t lds, hipStream_t s, hipEvent_t before,
                      hipEvent_t after) {
  const dim3 bd16(16 * 64), bd8(8 * 64);
  switch (ntrials) {
    case 1:
      if (w16) hipExtLaunchKernelGGL((fwd_wave_kernel<1, FWD_SOLVE, 16, ST, CP>), gd, bd16, lds, s, before, after, 0, a);
      else hipExtLaunchKernelGGL((fwd_wave_kernel<1, FWD_SOLVE, 8, ST, CP>), gd, bd8, lds, s, before, after, 0, a);
      break;
    case 2:
      if (w16) hipExtLaunchKernelGGL((fwd_wave_kernel<2, FWD_SOLVE, 16, ST, CP>), gd, bd16, lds, s, before, after, 0, a);
      else hipExtLaunchKernelGGL((fwd_wave_kernel<2, FWD_SOLVE, 8, ST, CP>), gd, bd8, lds, s, before, after, 0, a);
      break;
    case 4: hipExtLaunchKernelGGL((fwd_wave_kernel<4, FWD_SOLVE, 8, ST, CP>), gd, bd8, lds, s, before, after, 0, a); break;
    default: return set_error(IMRT_EINVAL, "trials per pass must be 1, 2 or 4");
  }
  return IMRT_OK;
}

template <int ST>
int launch_wave_forward(const FwdArgs& a, int ntrials, dim3 gd, size_t lds, hipStream_t s, hipEvent_t before,
                        hipEvent_t after) {
  const dim3 bd16(16 * 64), bd8(8 * 64);
  const bool w16 = forward_waves(ntrials, a.waves) == 16;
  if (a.mode == FWD_SOLVE) {
    return a.stream_cp ? launch_wave_solve<ST, 2>(a, ntrials, w16, gd, lds, s, before, after)
                       : launch_wave_solve<ST, 0>(a, ntrials, w16, gd, lds, s, before, after);
  } else if (ntrials != 1) {
    return set_error(IMRT_EINVAL, "evaluation passes take one trial");
  } else if (a.mode == FWD_EVAL) {
    if (w16) hipExtLaunchKernelGGL((fwd_wave_kernel<1, FWD_EVAL, 16, ST>), gd, bd16, lds, s, before, after, 0, a);
    else hipExtLaunchKernelGGL((fwd_wave_kernel<1, FWD_EVAL, 8, ST>), gd, bd8, lds, s, before, after, 0, a);
  } else {
    if (w16) hipExtLaunchKernelGGL((fwd_wave_kernel<1, FWD_PLAIN, 16, ST>), gd, bd16, lds, s, before, after, 0, a);
    else hipExtLaunchKernelGGL((fwd_wave_kernel<1, FWD_PLAIN, 8, ST>), gd, bd8, lds, s, before, after, 0, a);
  }
  return IMRT_OK;
}

// Batched solve passes: one dispatch over the slot table of several plans
// (all with the same storage, forward workgroup size and trials per pass).
template <int ST, int CP>
int launch_forward_batch_st(const FwdArgs* args, const int32_t* slots, int nslots, int ntrials, int dose_waves,
                            size_t lds, hipStream_t s) {
  const dim3 gd(nslots);
  const bool w16 = forward_waves(ntrials, dose_waves) == 16;
  switch (ntrials) {
    case 1:
      if (w16) hipLaunchKernelGGL((fwd_wave_batch_kernel<1, 16, ST, CP>), gd, dim3(16 * 64), lds, s, args, slots);
      else hipLaunchKernelGGL((fwd_wave_batch_kernel<1, 8, ST, CP>), gd, dim3(8 * 64), lds, s, args, slots);
      break;
    case 2:
      if (w16) hipLaunchKernelGGL((fwd_wave_batch_kernel<2, 16, ST, CP>), gd, dim3(16 * 64), lds, s, args, slots);
      else hipLaunchKernelGGL((fwd_wave_batch_kernel<2, 8, ST, CP>), gd, dim3(8 * 64), lds, s, args, slots);
      break;
    case 4: hipLaunchKernelGGL((fwd_wave_batch_kernel<4, 8, ST, CP>), gd, dim3(8 * 64), lds, s, args, slots); break;
    default: return set_error(IMRT_EINVAL, "trials per pass must be 1, 2 or 4");
  }
  return IMRT_OK;
}

int launch_forward_batch(const imrt_ctx* ctx, const FwdArgs* args, const int32_t* slots, int nslots, int ntrials,
                         int storage, int dose_waves, size_t lds, int stream_cp) {
  if (nslots <= 0) return IMRT_OK;
  if (lds > ctx->max_lds) return set_error(IMRT_EUNSUPPORTED, "batched forward pass: LDS budget exceeded");
  int rc;
  const int w = dose_waves;
  hipStream_t s = ctx->stream;
  switch (storage) {
    case ST_F32:
      rc = stream_cp ? launch_forward_batch_st<ST_F32, 2>(args, slots, nslots, ntrials, w, lds, s)
                     : launch_forward_batch_st<ST_F32, 0>(args, slots, nslots, ntrials, w, lds, s);
      break;
    case ST_BF16:
      rc = stream_cp ? launch_forward_batch_st<ST_BF16, 2>(args, slots, nslots, ntrials, w, lds, s)
                     : launch_forward_batch_st<ST_BF16, 0>(args, slots, nslots, ntrials, w, lds, s);
      break;
    case ST_F16:
      rc = stream_cp ? launch_forward_batch_st<ST_F16, 2>(args, slots, nslots, ntrials, w, lds, s)
                     : launch_forward_batch_st<ST_F16, 0>(args, slots, nslots, ntrials, w, lds, s);
      break;
    case ST_F32C16:
      rc = stream_cp ? launch_forward_batch_st<ST_F32C16, 2>(args, slots, nslots, ntrials, w, lds, s)
                     : launch_forward_batch_st<ST_F32C16, 0>(args, slots, nslots, ntrials, w, lds, s);
      break;
    default: return set_error(IMRT_EINVAL, "unknown storage");
  }
  if (rc) return rc;
  return check_launch("fwd_wave_batch_kernel");
}

int launch_forward(const imrt_ctx* ctx, const imrt_dose* D, const FwdArgs& a, int ntrials, int grid,
                   hipEvent_t before, hipEvent_t after) {
  (void)D;
  clear_stale_error();
  const bool wave = ctx->tune.fwd_wave != 0;
  const size_t lds = forward_lds_bytes(a.nb, ntrials, a.nstruct, wave, a.storage, a.waves);
  if (lds > ctx->max_lds)
    return set_error(IMRT_EUNSUPPORTED, "forward pass: nb * trials exceeds the LDS budget");
  const dim3 gd(grid), bd(kThreads);
  hipStream_t s = ctx->stream;
  if (wave) {
    int rc = IMRT_OK;
    switch (a.storage) {
      case ST_F32: rc = launch_wave_forward<ST_F32>(a, ntrials, gd, lds, s, before, after); break;
      case ST_BF16: rc = launch_wave_forward<ST_BF16>(a, ntrials, gd, lds, s, before, after); break;
      case ST_F16: rc = launch_wave_forward<ST_F16>(a, ntrials, gd, lds, s, before, after); break;
      case ST_F32C16: rc = launch_wave_forward<ST_F32C16>(a, ntrials, gd, lds, s, before, after); break;
      default: return set_error(IMRT_EINVAL, "unknown storage");
    }
    if (rc) return rc;
  } else {
    if (coded(a.storage))   // (ST_F32C16 matrices keep their 32-bit column indices for this pass)
      return set_error(IMRT_EUNSUPPORTED, "16-bit storage needs the wave-granular forward pass (fwd_wave = 1)");
    switch (ntrials) {
      case 1: hipExtLaunchKernelGGL(fwd_kernel<1>, gd, bd, lds, s, before, after, 0, a); break;
      case 2: hipExtLaunchKernelGGL(fwd_kernel<2>, gd, bd, lds, s, before, after, 0, a); break;
      case 4: hipExtLaunchKernelGGL(fwd_kernel<4>, gd, bd, lds, s, before, after, 0, a); break;
      default: return set_error(IMRT_EINVAL, "trials per pass must be 1, 2 or 4");
    }
  }
  return check_launch("fwd_kernel");
}

}  // namespace imrt
