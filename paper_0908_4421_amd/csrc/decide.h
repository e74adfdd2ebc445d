// The line-search decision with which a solve's second pass starts (adjoint
// pass, or the step of the one-read pass).
#pragma once

#include "pass_common.h"

namespace imrt {
namespace {

// ---- line-search decision ----------------------------------------------------------
// Decision on the forward pass whose objective partials are in `partials`
// ([trial][nparts], then [trial] step norms), starting from state `in`.  All
// threads of the workgroup take part (fixed-order reductions); the new state
// and the accepted trial land in shared memory.  Every workgroup that runs it
// on the same inputs reaches the same result.
struct Decision {
  SolverState st;   // state after the decision
  int accepted;     // accepted trial, -1 if none
  int backtracks;   // reductions before the accepted trial
  double lam, step_sq;
};

// Everything the decision reads is loaded by decide_start: the first round of
// partials (four per thread and trial), the state (one 32-bit word per lane
// of every wave) and the first step-norm part of every trial.
// The loads are not combined with anything here, so that the compiler waits
// for them only where decide uses them, after the caller's later loads were
// issued.
template <int NT>
struct DecideLoads {
  double v[NT][4];
  double step0[NT];
  int32_t sw;
};

template <int NT>
__device__ __forceinline__ void decide_start(const AdjArgs& a, DecideLoads<NT>& L) {
  const int tid = threadIdx.x, lane = tid & 63;
  const int nparts = a.fwd_parts, nsteps = a.step_parts;
  const rsrc_t rp = make_rsrc(a.fwd_partials, 8u * NT * static_cast<uint32_t>(nparts));
  const rsrc_t rs = make_rsrc(a.step_partials, 8u * NT * static_cast<uint32_t>(nsteps));
  const rsrc_t rst = make_rsrc(a.st_in, static_cast<uint32_t>(sizeof(SolverState)));
#pragma unroll
  for (int q = 0; q < NT; ++q) {
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int i = tid + u * kThreads;
      L.v[q][u] = load_f64(rp, 8u * static_cast<uint32_t>(q * nparts + (i < nparts ? i : 0)));
    }
    L.step0[q] = load_f64(rs, 8u * static_cast<uint32_t>(q * nsteps));
  }
  L.sw = load_i32(rst, 4u * static_cast<uint32_t>(lane < kStateWords ? lane : 0));
}

// The decision itself, on the pass's objectives Gq and step norms sq.
struct Verdict {
  int accepted = -1, backtracks = 0;
  double lam = 0.0, step_sq = 0.0;
};

template <int NT>
__device__ __forceinline__ void decide_state(SolverState& st, const double (&Gq)[NT], const double (&sq)[NT], Verdict& v) {
#pragma clang fp contract(off)
  const bool init = (st.phase == PH_INIT);
  st.n_fwd += 1;
  if (init) {
    // (st.lambda already holds the first trial step: lambda0, or for a
    // warm-started resumed solve alpha times the step accepted last)
    const double G0 = Gq[0];
    st.G = G0;
    st.G_init = G0;
    if (!st.resume) st.G_prev = G0;
    st.acc = 0;
    st.m = 0;
    if (!isfinite(G0)) {
      st.status = IMRT_NUMERIC;
      st.phase = PH_DONE;
    } else if (st.resume && !st.fixed && (G0 == 0.0 || fabs(G0 - st.G_prev) / G0 < st.delta)) {
      st.status = IMRT_CONVERGED;   // step 5 on the pair the interrupted solve ended with
      st.phase = PH_DONE;
    } else if (st.max_iter <= 0) {
      st.status = IMRT_MAX_ITER;
      st.phase = PH_DONE;
    } else {
      st.phase = PH_NEED_GRAD;
    }
  } else {
    bool done = false;
    int accepted = -1;
    double G_acc = 0.0, s_acc = 0.0;
    double l = st.lambda;
#pragma unroll
    for (int q = 0; q < NT; ++q) {
      if (q > 0) l = l / st.alpha;
      const double s = sq[q], Gt = Gq[q];
      if (s == 0.0) {
        st.status = IMRT_STALLED;
        done = true;
        break;
      }
      if (!isfinite(Gt)) {
        st.status = IMRT_NUMERIC;
        done = true;
        break;
      }
      const double C = st.G - (st.eps / l) * s;   // Eq. (5)
      if (Gt < C) {
        accepted = q;
        G_acc = Gt;
        s_acc = s;
        break;
      }
      st.m += 1;
      if (st.m > st.max_bt) {
        st.status = IMRT_LS_FAIL;
        done = true;
        break;
      }
    }
    if (accepted >= 0) {
      v.accepted = accepted;
      v.backtracks = st.m;
      v.lam = l;
      v.step_sq = s_acc;
      st.k += 1;
      st.G_prev = st.G;
      st.G = G_acc;
      st.acc = accepted;
      st.xi = (st.xi + 1 + accepted) % (NT + 1);
      st.m = 0;
      st.lambda = st.warm ? st.alpha * l : st.lambda0;   // step 2 of the next iteration
      if (st.fixed) {
        if (st.k >= st.max_iter) {
          st.status = IMRT_MAX_ITER;
          done = true;
        }
      } else if (st.G == 0.0 || fabs(st.G - st.G_prev) / st.G < st.delta) {
        st.status = IMRT_CONVERGED;
        done = true;
      } else if (st.k >= st.max_iter) {
        st.status = IMRT_MAX_ITER;
        done = true;
      }
      st.phase = done ? PH_DONE : PH_NEED_GRAD;
    } else if (done) {
      st.phase = PH_DONE;
    } else {
      st.lambda = l / st.alpha;
      st.phase = PH_TRIAL;
    }
  }
  if (st.phase == PH_NEED_GRAD) st.n_adj += 1;
}

template <int NT>
__device__ void decide(const double* partials, int nparts, const double* steps, int nsteps,
                       const DecideLoads<NT>& L, Decision& dec, double* red, double G_add) {
#pragma clang fp contract(off)
  __shared__ double Gq[NT];
  const int tid = threadIdx.x;
  double s[NT];
#pragma unroll
  for (int q = 0; q < NT; ++q) {
    // four values per round, summed in index order
    s[q] = 0.0;
#pragma unroll
    for (int u = 0; u < 4; ++u) s[q] += (tid + u * kThreads < nparts) ? L.v[q][u] : 0.0;
    const double* pq = partials + q * nparts;
    for (int i0 = tid + 4 * kThreads; i0 < nparts; i0 += 4 * kThreads) {
      double v[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int i = i0 + u * kThreads;
        v[u] = pq[i < nparts ? i : 0];
        v[u] = (i < nparts) ? v[u] : 0.0;
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) s[q] += v[u];
    }
  }
  if (tid < kStateWords) reinterpret_cast<int32_t*>(&dec.st)[tid] = L.sw;
  if (tid == 0) dec.accepted = -1;
#pragma unroll
  for (int q = 0; q < NT; ++q) {
    const double t = block_sum(s[q], red);
    if (tid == 0) Gq[q] = t + G_add;
  }
  if (dec.st.phase == PH_DONE) return;
  if (tid == 0) {
    double sq[NT];
    for (int q = 0; q < NT; ++q) {
      double t = 0.0;
      if (nsteps > 0) t += L.step0[q];
      for (int w = 1; w < nsteps; ++w) t += steps[q * nsteps + w];
      sq[q] = t;
    }
    SolverState st = dec.st;
    Verdict v;
    decide_state<NT>(st, Gq, sq, v);
    dec.accepted = v.accepted;
    dec.backtracks = v.backtracks;
    dec.lam = v.lam;
    dec.step_sq = v.step_sq;
    dec.st = st;
  }
  __syncthreads();
}

}  // namespace
}  // namespace imrt
