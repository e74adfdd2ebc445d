// One-read pass over D for gfx950: dose, penalty and the adjoint product of
// the residual from a single read of the matrix.
//
//  quad_kernel   stages the trial points in LDS, walks the quad form of D
//                (four consecutive rows share one list of columns: an entry
//                is a 16-bit column and four values), sums the four doses of
//                each quad, evaluates the penalty, and multiplies the quad's
//                entries, still in registers, by its four residuals into the
//                workgroup's column sums in LDS.
//  step_kernel   the line-search decision on that pass (taken identically by
//                every workgroup), the gradient as the sum of the workgroups'
//                column sums, and the next trial points.
//  reduce_kernel the column sums alone (gradients and power iterations).
//
// A trial's gradient is thus computed before the trial is accepted; a
// rejected trial costs arithmetic, no memory traffic.
//
// What bounds it: the read of D, 18 bytes per entry of float32 values (10
// with 16-bit codes); at the paper's scale an entry holds 3.3 nonzeros, so
// 5.4 bytes per nonzero where the two separate passes read 6 + 8.
// Measured per iteration, two separate passes -> one read: 38.2 -> 22.0 us
// (1.33 M voxels, 2,088 beamlets, 12.1 M nonzeros, float32), 41.9 -> 29.2 us
// (the same in bfloat16 with two trials a pass), 111.6 -> 54.9 us (143 k
// voxels, 6,444 beamlets, 41.8 M nonzeros), 213 -> 113 us (32 uneven plans of
// 40.4 M nonzeros together).
//
// Column sums are 64-bit integers, in units of 2^-61 times a bound on the
// largest possible sum (from the staged vector's largest entry, the largest
// row and column sums of D and the penalties), so additions in LDS commute
// exactly: the result does not depend on which wave adds first.  A term is
// rounded to the unit, which one bound sets for every column, so the step
// checks each column on its own: where the workgroups' sums are large enough
// against the number of terms (see imprecise), the total is as close as the
// float64 sum that it replaces once rounded to float32; any other column is
// summed again in float64 from its nonzeros and the residuals.  Columns that
// received no term are told from those whose terms vanish in the unit by a
// mark in LDS.  A vector with non-finite entries, or whose residuals could
// overflow, has no unit, and all its columns are summed so.
// After such a step the next passes of a solve store their residuals (that
// step makes them from the rows); a single gradient and the power iterations
// always do.  Stored in every pass they took 95 against 85 us for 32 uneven
// plans together.  The marks and the checks cost 3 to 4% of an iteration:
// 16.4 -> 17.0 us a pass at the paper's scale, 22.0 -> 22.9 in bfloat16 with
// two trials.
#include <algorithm>

#include "decide.h"

namespace imrt {
namespace {

constexpr int kDppQuadRev = 0x1B;    // quad_perm [3,2,1,0]
constexpr int kDppRowRor8 = 0x128;

// Sum over lanes i, i ^ 4: the same bits in both.
__device__ __forceinline__ float add_xor4(float v) {
  return v + dpp_move<kDppQuadRev, 0xF>(dpp_move<kDppRowHalfMirror, 0xF>(v));
}
__device__ __forceinline__ float add_xor8(float v) { return v + dpp_move<kDppRowRor8, 0xF>(v); }
__device__ __forceinline__ float add_xor16(float v) {
  const uint32_t u = __float_as_uint(v);
  const auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ float add_xor32(float v) {
  const uint32_t u = __float_as_uint(v);
  const auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// Largest value of the wave; valid in lane 63.
template <int CTRL, int ROWS>
__device__ __forceinline__ uint32_t max_dpp(uint32_t v) {
  return max(v, static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(v), CTRL, ROWS, 0xF, false)));
}
__device__ __forceinline__ uint32_t wave_max(uint32_t v) {
  v = max_dpp<kDppQuadXor1, 0xF>(v);
  v = max_dpp<kDppQuadXor2, 0xF>(v);
  v = max_dpp<kDppRowHalfMirror, 0xF>(v);
  v = max_dpp<kDppRowMirror, 0xF>(v);
  v = max_dpp<kDppRowBcast15, 0xA>(v);
  return max_dpp<kDppRowBcast31, 0xC>(v);
}

// 2^e, -1022 <= e <= 1023
__device__ __forceinline__ double pow2(int e) {
  return __builtin_bit_cast(double, static_cast<unsigned long long>(e + 1023) << 52);
}

template <int ST>
using QuadVal = std::conditional_t<coded(ST), uint2, float4>;

// Whether a value of an entry is none of D's: an empty place of a quad holds
// -0, and a stored -0 is kept as 0.
template <int ST>
__device__ __forceinline__ bool quad_hole(const QuadVal<ST>& v, int u) {
  if constexpr (coded(ST)) return half_of(v, u) == 0x8000u;
  else return __float_as_uint(val_of<ST>(v, u)) == 0x80000000u;
}

// (NP: plans with penalties of their own)
template <int ST, int NP>
struct QuadStage {
  QuadVal<ST> v[quad_run(ST) * quad_steps(ST)];
  uint32_t c[quad_steps(ST)];   // one column or two each
  uint32_t sid[NP];
  float tu[NP], to[NP];
  uint32_t vox;   // passes that write the dose: the voxel of the lane's row
};

// The plans of a pass: one, or up to K that share the matrix (the first
// `n` of plans[], indices into args).
struct OnePlan {
  static constexpr bool kMany = false;
  const FwdArgs& a;
  __device__ __forceinline__ const FwdArgs& operator()(int) const { return a; }
  __device__ __forceinline__ bool has(int) const { return true; }
};
template <int K>
struct ManyPlans {
  static constexpr bool kMany = true;
  const FwdArgs* args;
  int plan[K], n;
  __device__ __forceinline__ const FwdArgs& operator()(int q) const { return args[plan[q]]; }
  __device__ __forceinline__ bool has(int q) const { return q < n; }
};

// Column of entry m of a lane, as the byte offset into a staged vector.
template <int ST, int NP>
__device__ __forceinline__ uint32_t quad_col(const QuadStage<ST, NP>& S, int m) {
  if constexpr (quad_run(ST) == 1) return S.c[m];
  else return (m & 1) ? S.c[m / 2] >> 16 : S.c[m / 2] & 0xFFFFu;
}
__device__ __forceinline__ float staged(const float* xs, uint32_t c) {
  return *reinterpret_cast<const float*>(reinterpret_cast<const char*>(xs) + c);
}
// The column sum of the same column.
template <typename T>
__device__ __forceinline__ T* sum_at(T* acc, uint32_t c) {
  return reinterpret_cast<T*>(reinterpret_cast<char*>(acc) + 2 * c);
}

// Loads of one block; steps past a lane's entries read zeros out of bounds
// (column code 0: none).
template <int MODE, int ST, int CP, int NP, typename Plans>
__device__ __forceinline__ void quad_issue(const Plans& P, const uint2 rec, int e0, int flags, int lane,
                                           QuadStage<ST, NP>& S) {
  const FwdArgs& a = P(0);
  constexpr int VB = coded(ST) ? 8 : 16, R = quad_run(ST);   // bytes of an entry's values
  const int e = quad_log2(flags), L = 1 << e;
  const int sub = lane & (L - 1), n = static_cast<int>(rec.x >> 16) / R;
  const uint32_t at0 = (rec.x & 0xFFFFu) / R + sub;
  // (a block ends at most kQuadPad entries after e0; the arrays are padded by as many)
  const rsrc_t rc = make_rsrc(a.q_col + e0, 2u * kQuadPad);
  const rsrc_t rv = make_rsrc(static_cast<const char*>(a.q_val) + static_cast<size_t>(e0) * VB, VB * kQuadPad);
#pragma unroll
  for (int m = 0; m < quad_steps(ST); ++m) {
    const uint32_t at = sub + m * L < n ? at0 + m * L : 0x00800000u;
    if constexpr (R == 2) {
      S.c[m] = __builtin_amdgcn_raw_buffer_load_b32(rc, 4u * at, 0, CP);
      const int4 w = load_i4s<CP>(rv, 16u * at);
      S.v[2 * m] = make_uint2(w.x, w.y);
      S.v[2 * m + 1] = make_uint2(w.z, w.w);
    } else {
      S.c[m] = __builtin_amdgcn_raw_buffer_load_b16(rc, 2u * at, 0, CP);
      S.v[m] = load_f4s<CP>(rv, 16u * at);
    }
  }
  const uint32_t row = 4u * rec.y + (lane & 3);
  const uint32_t nv = static_cast<uint32_t>(a.nv);
  if (MODE == QM_EVAL || MODE == QM_PLAIN)
    S.vox = static_cast<uint32_t>(load_i32(make_rsrc(a.vox, a.vox ? 4u * nv : 0u), 4u * row));
  if (MODE == QM_PLAIN || MODE == QM_POWER) return;
#pragma unroll
  for (int p = 0; p < NP; ++p) {
    const Penalties& pen = P(p).pen;
    S.sid[p] = load_u8(make_rsrc(pen.sid, pen.sid ? nv : 0u), row);
    const uint32_t tb = pen.Tu_vox ? 4u * nv : 0u;
    S.tu[p] = load_f32(make_rsrc(pen.Tu_vox, tb), 4u * row);
    S.to[p] = load_f32(make_rsrc(pen.To_vox, tb), 4u * row);
  }
}

// Integer nearest to t, |t| < 2^61: high 32 bits, then the exact remainder,
// each rounded by adding 1.5 * 2^52 (H. S. Warren, Hacker's Delight, 2nd ed.,
// chapter 17).
__device__ __forceinline__ unsigned long long to_fixed(double t) {
#pragma clang fp contract(off)
  constexpr double kMagic = 6755399441055744.0;   // 1.5 * 2^52
  const double A = __builtin_fma(t, 0x1p-32, kMagic);
  const double hf = A - kMagic;
  const double B = __builtin_fma(hf, -0x1p32, t) + kMagic;
  const uint32_t hi = static_cast<uint32_t>(__builtin_bit_cast(unsigned long long, A));
  const unsigned long long b = __builtin_bit_cast(unsigned long long, B);
  const uint32_t top = static_cast<uint32_t>(b >> 32) - 0x43380000u + hi;
  return (static_cast<unsigned long long>(top) << 32) | static_cast<uint32_t>(b);
}

template <int V>
__device__ __forceinline__ double quad_bcast(double v) {
  return dpp_move<V * 0x55, 0xF>(v);
}

// A column's total over workgroups: the sum of their sums; in units of 2^24, at
// most the sum of their magnitudes, which is at most that of the terms'; and
// their bits, 0 for a column that received no term (a workgroup writes a unit
// instead of a sum of 0 of terms that were not all zero).
struct ColTotal {
  unsigned long long s;
  uint32_t a, any;
};
__device__ __forceinline__ void add_part(ColTotal& T, unsigned long long v) {
  const int hi = static_cast<int>(v >> 32);
  T.s += v;
  T.a += static_cast<uint32_t>((v >> kMagnitude) ^ static_cast<unsigned long long>(static_cast<long long>(hi >> 31)));
  T.any |= static_cast<uint32_t>(hi) | static_cast<uint32_t>(v);
}
__device__ __forceinline__ void add_total(ColTotal& T, const ColTotal& U) {
  T.s += U.s;
  T.a += U.a;
  T.any |= U.any;
}

// Whether the integers are not precise enough for a column: the sums'
// magnitudes do not come to `enough` (quad_enough), or there is no unit.
// Columns far below the bound that the unit is taken from are not: one huge
// entry of x, columns or weights decades apart, residuals that nearly vanish.
__device__ __forceinline__ bool imprecise(const ColTotal& T, double unit, uint32_t enough) {
  return unit == 0.0 || (T.any != 0 && T.a < enough);
}

// Residual of a row that its pass did not store.
template <int ST>
__device__ __forceinline__ float row_residual(const Again& A, const float* x, int row) {
  double z = 0.0;
  for (int k = A.row_ptr[row]; k < A.row_ptr[row + 1]; ++k) {
    const int c = coded(ST) ? A.col16[k] : A.col_idx[k];
    const float xc = coded(ST) ? x[c] * A.col_scale[c] : x[c];
    const float v = coded(ST) ? code_value<ST>(A.val16[k]) : A.val[k];
    z += static_cast<double>(v) * static_cast<double>(xc);
  }
  const PenaltyDev t = A.pen.table[A.pen.sid[row]];
  RowPenalty p{t.T_u, t.T_o, t.w_u, t.w_o};
  if (A.pen.Tu_vox != nullptr) {
    p.Tu = static_cast<double>(A.pen.Tu_vox[row]);
    p.To = static_cast<double>(A.pen.To_vox[row]);
  }
  double F;
  float r;
  penalty(p, static_cast<float>(z), F, r);
  return r;
}

// Such a column is summed again from its nonzeros and the residuals of its
// rows (r, or where the pass did not store them (null) those of the vector x)
// in float64, in a fixed order: the share of wave i of `waves`.
template <int ST>
__device__ __forceinline__ double exact_column_of(const Again& A, const float* r, const float* x, int c, int i,
                                                  int waves) {
  constexpr int U = 4;
  const int k1 = A.col_ptr[c + 1], lane = threadIdx.x & 63;
  double s = 0.0;
  for (int k0 = A.col_ptr[c] + 64 * U * i; k0 < k1; k0 += 64 * U * waves) {
    int row[U];
    float v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int k = k0 + 64 * u + lane;
      const int64_t at = csc_slot(k < k1 ? k : k0);
      row[u] = A.row_idx[at];
      if constexpr (coded(ST)) v[u] = code_value<ST>(A.cval16[at]);
      else v[u] = A.cval[at];
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const float ru = r != nullptr ? r[row[u]] : row_residual<ST>(A, x, row[u]);
      const double t = static_cast<double>(v[u]) * static_cast<double>(ru);
      s += k0 + 64 * u + lane < k1 ? t : 0.0;
    }
  }
  const uint64_t b = __builtin_bit_cast(uint64_t, wave_sum(s));
  const uint32_t lo = __builtin_amdgcn_readlane(static_cast<int>(b), 63);
  const uint32_t hi = __builtin_amdgcn_readlane(static_cast<int>(b >> 32), 63);
  return __builtin_bit_cast(double, (static_cast<uint64_t>(hi) << 32) | lo);
}
__device__ __forceinline__ double exact_column(const Again& A, const float* r, const float* x, int c, int i,
                                               int waves) {
  if (A.storage == ST_BF16) return exact_column_of<ST_BF16>(A, r, x, c, i, waves);
  if (A.storage == ST_F16) return exact_column_of<ST_F16>(A, r, x, c, i, waves);
  return exact_column_of<ST_F32>(A, r, x, c, i, waves);
}

// A wave's sum of n float64 values: lane l adds values l, l + 64, ..., then
// the lanes are summed.  In two parts, so that the loads can be issued early;
// U rounds at once.
template <int U>
struct SumLoads {
  double v[U];
};
template <int U>
__device__ __forceinline__ void sum_start(const double* p, int n, SumLoads<U>& L) {
  const rsrc_t r = make_rsrc(p, 8u * static_cast<uint32_t>(n));
#pragma unroll
  for (int u = 0; u < U; ++u) L.v[u] = load_f64(r, 8u * ((threadIdx.x & 63) + 64u * u));
}
template <int U>
__device__ __forceinline__ double sum_finish(const double* p, int n, const SumLoads<U>& L) {
  double s = 0.0;
#pragma unroll
  for (int u = 0; u < U; ++u) s += L.v[u];
  for (int i = (threadIdx.x & 63) + 64 * U; i < n; i += 64) s += p[i];
  const uint64_t b = __builtin_bit_cast(uint64_t, wave_sum(s));
  const uint32_t lo = __builtin_amdgcn_readlane(static_cast<int>(b), 63);
  const uint32_t hi = __builtin_amdgcn_readlane(static_cast<int>(b >> 32), 63);
  return __builtin_bit_cast(double, (static_cast<uint64_t>(hi) << 32) | lo);
}

// What a small plan's launch does before its pass, in every workgroup alike:
// the decision on the last pass (first wave), this column's gradient from
// that pass's column sums, and the next trial.  Thread c takes column c.
struct Whole {
  int phase;       // after the decision
  int care;        // passes that store their residuals from this one on
  float t;         // the trial
};
constexpr int kWholeU = 12;   // column sums in flight per thread

template <int THREADS>
__device__ __forceinline__ Whole whole_step(const FwdArgs& a, const WholeArgs& W, int w, int parts, int nobj) {
  __shared__ double lam_sh;
  __shared__ int ctl[3];   // phase, accepted, a column to sum again
  __shared__ ColTotal sh[THREADS];
  static_assert(sizeof(lam_sh) + sizeof(ctl) + sizeof(sh) + kQuadFixedLds - 32 <= kWholeFixedLds, "counted by quad_fits");
  const int tid = threadIdx.x, lane = tid & 63, nb = a.nb, sg = step_grid(nb);
  // Thread (first, c) adds column c's sums of workgroups first, first + groups,
  // ...: a thread to a column leaves most threads idle and takes several
  // rounds of loads (73 workgroups of 220 columns, without the check of the
  // totals: 13.5 us an iteration, 10.9 with the sums shared out).
  int width = 64;
  while (width < nb) width *= 2;
  const int c = tid & (width - 1), first = tid / width, groups = THREADS / width;
  const rsrc_t ra = make_rsrc(W.in.acc, 8u * static_cast<uint32_t>(parts * nb));
  const uint32_t nb4 = 4u * static_cast<uint32_t>(nb), at = 4u * tid;
  float xk = load_f32(make_rsrc(W.in.xk, nb4), at), g = load_f32(make_rsrc(W.in.g, nb4), at);
  const float xt = load_f32(make_rsrc(W.in.xt, nb4), at);
  const double unit = load_f64(make_rsrc(W.in.unit, 8u), 0);
  const int was = load_i32(make_rsrc(W.in.care, W.first ? 0u : 4u), 0);
  const double factor = a.col_scale ? 2.0 * static_cast<double>(load_f32(make_rsrc(a.col_scale, nb4), at)) : 2.0;
  SumLoads<2> GL, SL;
  int32_t sw = 0;
  if (tid < 64) {
    sw = load_i32(make_rsrc(W.in.st, static_cast<uint32_t>(sizeof(SolverState))), 4u * (lane < kStateWords ? lane : 0));
    sum_start(W.in.parts, nobj, GL);
    sum_start(W.in.steps, sg, SL);
  }
  ColTotal s{0, 0, 0};
  for (int p = first; p < parts; p += groups * kWholeU) {
    unsigned long long v[kWholeU];
#pragma unroll
    for (int u = 0; u < kWholeU; ++u) {
      const int pu = p + u * groups;
      v[u] = __builtin_bit_cast(unsigned long long,
                                load_f64(ra, c < nb && pu < parts ? 8u * static_cast<uint32_t>(pu * nb + c) : 0xFFFFFFF0u));
    }
#pragma unroll
    for (int u = 0; u < kWholeU; ++u) add_part(s, v[u]);
  }
  sh[tid] = s;
  if (tid == 0) ctl[2] = 0;
  if (tid < 64) {
    int32_t words[kStateWords];
#pragma unroll
    for (int i = 0; i < kStateWords; ++i) words[i] = __builtin_amdgcn_readlane(sw, i);
    SolverState st = __builtin_bit_cast(SolverState, words);
    Verdict v;
    if (st.phase != PH_DONE && !W.first) {
      const double Gq[1] = {sum_finish(W.in.parts, nobj, GL) + W.G_skip};
      const double sq[1] = {sum_finish(W.in.steps, sg, SL)};
      decide_state<1>(st, Gq, sq, v);
    }
    st.xi = 1;
    if (lane == 0) {
      lam_sh = st.lambda;
      ctl[0] = st.phase;
      ctl[1] = v.accepted;
      if (w == 0) {
        *W.out.st = st;
        if (v.accepted >= 0 && W.trace != nullptr && st.k - 1 < st.trace_cap) {
          TraceDev e;
          e.k = st.k;
          e.backtracks = v.backtracks;
          e.lambda = v.lam;
          e.step_sq = v.step_sq;
          e.G = st.G;
          W.trace[st.k - 1] = e;
        }
      }
    }
  }
  __syncthreads();
  Whole R;
  R.phase = uniform(ctl[0]);
  if (ctl[1] >= 0) xk = xt;
  if (tid < nb)
    for (int k = 1; k < groups; ++k) add_total(s, sh[k * width + tid]);
  double total = static_cast<double>(static_cast<long long>(s.s)) * unit;
  const bool again = tid < nb && !W.first && imprecise(s, unit, W.enough);
  if (again) ctl[2] = 1;
  __syncthreads();
  const bool some = uniform(ctl[2]) != 0;
  R.care = uniform(some ? kCarePasses : max(was - 1, 0));
  if (R.phase == PH_NEED_GRAD) {
    if (some) {   // (every workgroup alike, a wave to a column)
      sh[tid].any = again;
      __syncthreads();
      for (int k = uniform(tid >> 6); k < nb; k += THREADS / 64)
        if (uniform(static_cast<int>(sh[k].any)) != 0) {
          const double t = exact_column(W.again, was > 0 ? W.in.r : nullptr, W.in.xt, k, 0, 1);
          if (lane == 0) sh[k].s = __builtin_bit_cast(unsigned long long, t);
        }
      __syncthreads();
      if (again) total = __builtin_bit_cast(double, sh[tid].s);
    }
    g = static_cast<float>(factor * total);
  }
  R.t = W.first ? xt : trial_point(xk, g, lam_sh);
  if (w == 0) {
    if (tid == 0) *W.out.care = R.care;
    if (tid < nb) {
      W.out.xk[tid] = xk;
      W.out.g[tid] = g;
      W.out.xt[tid] = R.t;
    }
    const double dl = static_cast<double>(R.t) - static_cast<double>(xk);
    const double sq = group_sum<kStepCols>(tid < nb ? dl * dl : 0.0);
    if ((tid & (kStepCols - 1)) == kStepCols - 1 && tid / kStepCols < sg) W.out.steps[tid / kStepCols] = sq;
  }
  return R;
}

// NT vectors: the trials of one plan, or one trial of each of NT plans (nst:
// LDS places of a plan's penalty table).
template <int NT, int MODE, int WAVES, int ST, int CP, typename Plans>
__device__ __forceinline__ void quad_pass(const Plans& P, const Slot sl, int nst, const WholeArgs* W = nullptr) {
  constexpr int NP = Plans::kMany ? NT : 1;
  const FwdArgs& a = P(0);
  constexpr int THREADS = WAVES * 64, M = quad_run(ST) * quad_steps(ST), U = WAVES == 16 ? 4 : 8;
  constexpr bool GRAD = quad_grad(MODE);
  constexpr bool PEN = MODE != QM_PLAIN && MODE != QM_POWER;
  extern __shared__ __align__(16) unsigned char smem[];
  const int nb = a.nb, nbs = quad_stride(nb);
  unsigned char* mark = smem;   // columns that received a term
  auto* acc = reinterpret_cast<unsigned long long*>(smem + (GRAD ? quad_mark_bytes(nb, NP) : 0));
  PenaltyDev* tab = reinterpret_cast<PenaltyDev*>(acc + (GRAD ? NT * nbs : 0));
  float* xs = reinterpret_cast<float*>(tab + NP * nst);
  __shared__ double red[WAVES];
  __shared__ uint32_t mx[NT][WAVES];
  __shared__ double gsum[NT][WAVES];
  static_assert(sizeof(red) + sizeof(mx) + sizeof(gsum) <= kQuadFixedLds, "counted by quad_fits");
  const int tid = threadIdx.x, wv = uniform(tid >> 6), lane = tid & 63;

  // this wave's blocks: heads (lane i: block i) and the first two blocks' records
  const int kmax = a.q_kmax, blk0 = (sl.w * WAVES + wv) * kmax;
  const uint32_t nblk = static_cast<uint32_t>(a.q_nblocks);
  const rsrc_t rh = make_rsrc(a.q_head, 8u * nblk);
  const rsrc_t rr = make_rsrc(a.q_rec + static_cast<size_t>(blk0) * 16, 128u * static_cast<uint32_t>(kmax));
  auto load_head = [&](int i) {
    return __builtin_bit_cast(uint2, __builtin_amdgcn_raw_buffer_load_b64(rh, 8u * static_cast<uint32_t>(i), 0, 0));
  };
  auto load_rec = [&](int i) {
    return __builtin_bit_cast(
        uint2, __builtin_amdgcn_raw_buffer_load_b64(rr, 128u * static_cast<uint32_t>(i) + 8u * (lane >> 2), 0, 0));
  };
  uint2 heads = load_head(lane < kmax ? blk0 + lane : static_cast<int>(nblk));
  uint2 rec0 = load_rec(0), rec1 = load_rec(1);

  // the vectors this pass multiplies by, and the state
  auto vec = [&](int q) -> const float* {
    return MODE != QM_SOLVE ? a.x : Plans::kMany ? P(q).xbuf[0] : a.xbuf[q];
  };
  float xr[NT][U], sc[U];
  rsrc_t rx[NT];
#pragma unroll
  for (int q = 0; q < NT; ++q) rx[q] = make_rsrc(vec(q), 4u * static_cast<uint32_t>(nb));
  const rsrc_t rsc = make_rsrc(a.col_scale, (coded(ST) && a.col_scale) ? 4u * static_cast<uint32_t>(nb) : 0u);
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const uint32_t i = static_cast<uint32_t>(tid + u * THREADS);
#pragma unroll
    for (int q = 0; q < NT; ++q) xr[q][u] = MODE == QM_WHOLE ? 0.0f : load_f32(rx[q], 4u * i);
    sc[u] = coded(ST) ? load_f32(rsc, 4u * i) : 1.0f;
  }
  double tab0[NP];
  int32_t sw[NP];
#pragma unroll
  for (int p = 0; p < NP; ++p) {
    tab0[p] = PEN ? load_f64(make_rsrc(P(p).pen.table, 32u * static_cast<uint32_t>(P(p).nstruct)), 8u * tid) : 0.0;
    sw[p] = MODE == QM_SOLVE ? reinterpret_cast<const int32_t*>(P(p).st_in)[lane < kStateWords ? lane : 0] : 0;
  }
  double np = 0.0;
  if (MODE == QM_POWER)
    for (int i = tid; i < a.norm_parts; i += THREADS) np += a.norm[i];

  auto head_e0 = [&](int i) { return __builtin_amdgcn_readlane(static_cast<int>(heads.x), i & 63); };
  auto head_fl = [&](int i) { return __builtin_amdgcn_readlane(static_cast<int>(heads.y), i & 63); };
  QuadStage<ST, NP> A, B;
  int e0 = head_e0(0), fl = head_fl(0);
  quad_issue<MODE, ST, CP>(P, rec0, e0, fl, lane, A);

  int keep = GRAD;   // residuals are stored
  if constexpr (MODE == QM_WHOLE) {
    static_assert(NT == 1 && U >= 1 && !Plans::kMany, "one column per thread");
    const Whole R = whole_step<THREADS>(a, *W, sl.w, sl.G, sl.G * (WAVES / 8));
    if (R.phase == PH_DONE) return;
    xr[0][0] = R.t;
    keep = R.care;
  }
  if (MODE == QM_EVAL || MODE == QM_PLAIN)
    for (int i = sl.w * THREADS + tid; i < a.nzero; i += sl.G * THREADS) a.d_out[a.zero[i]] = 0.0f;

  int care[NP];   // (a solve's plans each have their own)
#pragma unroll
  for (int p = 0; p < NP; ++p)
    care[p] = MODE != QM_SOLVE ? keep
              : state_int(sw[p], offsetof(SolverState, again)) == state_int(sw[p], offsetof(SolverState, n_fwd))
                  ? kCarePasses
                  : max(state_int(sw[p], offsetof(SolverState, stored)) - 1, 0);

  bool on[NP];   // plans that are not done
#pragma unroll
  for (int p = 0; p < NP; ++p) on[p] = true;
  if (MODE == QM_SOLVE) {
    bool any = false;
#pragma unroll
    for (int p = 0; p < NP; ++p) {
      on[p] = P.has(p) && state_int(sw[p], offsetof(SolverState, phase)) != PH_DONE;
      any = any || on[p];
      if (P.has(p) && sl.w == 0 && wv == 0 && lane < kStateWords)
        reinterpret_cast<int32_t*>(P(p).st_out)[lane] = lane == static_cast<int>(offsetof(SolverState, stored) / 4) ? care[p] : sw[p];
    }
    if (!any) return;
    // the last step's norms, moved to where the next step reads them
    if (sl.w == 0) {
      const int n = (Plans::kMany ? 1 : NT) * step_grid(nb);
#pragma unroll
      for (int p = 0; p < NP; ++p)
        if (on[p])
          for (int i = tid; i < n; i += THREADS) P(p).q_steps[i] = P(p).q_steps[n + i];
    }
  }
  auto active = [&](int q) { return on[Plans::kMany ? q : 0]; };
  // power iterations multiply by v = w / ||w||
  double nrm = 1.0;
  if (MODE == QM_POWER && a.norm_parts > 0) {
    const double s = block_sum<double, WAVES>(np, red);
    if (tid == 0) red[0] = sqrt(s);
    __syncthreads();
    nrm = red[0];
    __syncthreads();
  }
  if (PEN) {
#pragma unroll
    for (int p = 0; p < NP; ++p) {
      double* dst = reinterpret_cast<double*>(tab + p * nst);
      const int n = 4 * P(p).nstruct;
      if (tid < n) dst[tid] = tab0[p];
      for (int i = tid + THREADS; i < n; i += THREADS) dst[i] = reinterpret_cast<const double*>(P(p).pen.table)[i];
    }
  }
  // staged vectors at [1, nb]; slot 0 (idle lanes) is zero.  With 16-bit
  // storage they are scaled by the beamlet scales and multiply the codes.
  uint32_t big[NT];   // largest magnitude's bits (orders NaN above infinity)
#pragma unroll
  for (int q = 0; q < NT; ++q) big[q] = 0;
  auto copy_of = [&](int q) { return P(q).q_x + (Plans::kMany ? 0 : static_cast<size_t>(q) * nb); };
  auto put = [&](int q, int i, float x, float s) {
    if (MODE == QM_POWER && a.norm_parts > 0)
      x = nrm > 0.0 ? static_cast<float>(static_cast<double>(x) / nrm) : 0.0f;
    if (coded(ST)) x *= s;
    xs[q * nbs + i + 1] = x;
    big[q] = max(big[q], __float_as_uint(x) & 0x7FFFFFFFu);
  };
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int i = tid + u * THREADS;
    if (i < nb) {
#pragma unroll
      for (int q = 0; q < NT; ++q) {
        put(q, i, xr[q][u], sc[u]);
        if (MODE == QM_SOLVE && active(q) && min(u, sl.G - 1) == sl.w) copy_of(q)[i] = xr[q][u];
      }
    }
  }
  for (int i = tid + U * THREADS, u = U; i < nb && MODE != QM_WHOLE; i += THREADS, ++u)
#pragma unroll
    for (int q = 0; q < NT; ++q) {
      const float x = vec(q)[i];
      put(q, i, x, coded(ST) ? a.col_scale[i] : 1.0f);
      if (MODE == QM_SOLVE && active(q) && min(u, sl.G - 1) == sl.w) copy_of(q)[i] = x;
    }
  if (tid < NT) xs[tid * nbs] = 0.0f;
  if (GRAD) {
    for (int i = tid; i < NT * nbs; i += THREADS) acc[i] = 0;
    for (int i = tid; i < NP * nbs / 4; i += THREADS) reinterpret_cast<uint32_t*>(mark)[i] = 0;
  }
#pragma unroll
  for (int q = 0; q < NT; ++q) {
    big[q] = wave_max(big[q]);
    if (lane == 63) mx[q][wv] = big[q];
  }
  __syncthreads();

  // the unit of each vector's column sums
  double up[NT];    // residuals times up: in units
  bool wild[NT];    // no integer sums: the step sums every column from the residuals
  bool any_wild = false;
#pragma unroll
  for (int q = 0; q < NT; ++q) {
    uint32_t b = 0;
#pragma unroll
    for (int k = 0; k < WAVES; ++k) b = max(b, mx[q][k]);
    const FwdArgs& aq = P(q);
    const double zmax = a.q_rowsum * static_cast<double>(__uint_as_float(b));
    const double R = PEN ? aq.pen_w * zmax + aq.pen_r0 : zmax;
    wild[q] = uniform(R < 1e38 && zmax < 1e38 ? 0 : 1) != 0;
    any_wild = any_wild || wild[q];
    const double bound = fmax(R * a.q_colsum, 1e-200);
    // bound < 2^ex
    const int ex = wild[q] ? 61 : static_cast<int>(__builtin_bit_cast(unsigned long long, bound) >> 52) - 1022;
    up[q] = pow2(61 - ex);
    if (GRAD && sl.w == 0 && tid == 0 && active(q))
      *(MODE == QM_WHOLE ? W->out.unit : Plans::kMany ? aq.q_unit : aq.q_unit + q) = wild[q] ? 0.0 : pow2(ex - 61);
  }

  const uint32_t vbytes = 4u * static_cast<uint32_t>(a.nv);
  const rsrc_t dout = make_rsrc(a.d_out, a.d_out ? vbytes : 0u);
  rsrc_t rout[NT];
#pragma unroll
  for (int q = 0; q < NT; ++q)
    rout[q] = make_rsrc(MODE == QM_WHOLE ? W->out.r : P(q).rbuf[Plans::kMany ? 0 : q], active(q) ? vbytes : 0u);
  double pacc[NT];
  float z[NT][4];
  double rd[NT];    // residual of the lane's voxel, in units
  bool live[NT];
#pragma unroll
  for (int q = 0; q < NT; ++q) {
    pacc[q] = 0.0;
    live[q] = false;
    rd[q] = 0.0;
#pragma unroll
    for (int u = 0; u < 4; ++u) z[q][u] = 0.0f;
  }

  // The doses of a block's quads (summed over each quad's lanes; a lane keeps
  // its own voxel, row lane & 3), their objective and residuals.
  auto finish = [&](int q, const float (&zq)[4], int e, const uint2 rec, const RowPenalty& pen, uint32_t vox) {
    const uint32_t row = 4u * rec.y + (lane & 3);
    const bool own = rec.x != 0 && row < static_cast<uint32_t>(a.nv);
    const bool count = own && (lane & ((1 << e) - 1)) < 4;
    const bool b0 = lane & 1, b1 = lane & 2;
    const float lo = (b0 ? zq[1] : zq[0]) + dpp_move<kDppQuadXor1, 0xF>(b0 ? zq[0] : zq[1]);
    const float hi = (b0 ? zq[3] : zq[2]) + dpp_move<kDppQuadXor1, 0xF>(b0 ? zq[2] : zq[3]);
    float d = (b1 ? hi : lo) + dpp_move<kDppQuadXor2, 0xF>(b1 ? lo : hi);
    if (e >= 3) d = add_xor4(d);
    if (e >= 4) d = add_xor8(d);
    if (e >= 5) d = add_xor16(d);
    if (e >= 6) d = add_xor32(d);
    double F;
    float r;
    if (PEN) {
      penalty(pen, d, F, r);
    } else {
      F = static_cast<double>(d) * static_cast<double>(d);
      r = d;
    }
    pacc[q] += count ? F : 0.0;
    if (MODE == QM_EVAL || MODE == QM_PLAIN) {
      if (q == 0 && count) store_f32(dout, 4u * (a.vox ? vox : row), d);
    }
    if (GRAD && care[Plans::kMany ? q : 0] > 0 && count) store_f32(rout[q], 4u * row, r);
    return own ? r : 0.0f;
  };
  auto penalty_of = [&](int p, uint32_t sid, float tu, float to) {
    const PenaltyDev t = tab[p * nst + sid];
    RowPenalty pen{t.T_u, t.T_o, t.w_u, t.w_o};
    if (P(p).pen.Tu_vox != nullptr) {
      pen.Tu = static_cast<double>(tu);
      pen.To = static_cast<double>(to);
    }
    return pen;
  };

  auto add_fixed = [&](int q, uint32_t c, double t) {
    __hip_atomic_fetch_add(sum_at(acc + q * nbs, c), to_fixed(t), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  };
  auto add_term = [&](int q, uint32_t c, double t) {
    if (t == 0.0) return;
    add_fixed(q, c, t);
    mark[(Plans::kMany ? q * nbs : 0) + (c >> 2)] = 1;
  };

  auto compute = [&](const QuadStage<ST, NP>& S, const uint2 rec, int flags) {
    if (flags & kQuadFirst) {
#pragma unroll
      for (int q = 0; q < NT; ++q)
#pragma unroll
        for (int u = 0; u < 4; ++u) z[q][u] = 0.0f;
    }
    if (flags & kQuadDose) {
      // (idle lanes multiply zeros)
#pragma unroll
      for (int q = 0; q < NT; ++q) {
        float x[M];
#pragma unroll
        for (int m = 0; m < M; ++m) x[m] = staged(xs + q * nbs, quad_col(S, m));
#pragma unroll
        for (int m = 0; m < M; ++m)
#pragma unroll
          for (int u = 0; u < 4; ++u) z[q][u] = fmaf(val_of<ST>(S.v[m], u), x[m], z[q][u]);
      }
    }
    __builtin_amdgcn_sched_barrier(0);   // (interleaving the phases costs registers)
    if (flags & kQuadFinish) {
      RowPenalty pen{0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int q = 0; q < NT; ++q) {
        if (PEN && q < NP) pen = penalty_of(q, S.sid[q], S.tu[q], S.to[q]);
        const float r = finish(q, z[q], quad_log2(flags), rec, pen, S.vox);
        if (GRAD) {
          live[q] = active(q) && __ballot(r != 0.0f) != 0;
          rd[q] = static_cast<double>(r) * up[q];
        }
      }
    }
    __builtin_amdgcn_sched_barrier(0);
    bool some = false;
#pragma unroll
    for (int q = 0; q < NT; ++q) some = some || live[q];
    if (GRAD && (flags & kQuadAdjoint) && some) {
      double r4[NT][4];
#pragma unroll
      for (int q = 0; q < NT; ++q) {
        r4[q][0] = quad_bcast<0>(rd[q]);
        r4[q][1] = quad_bcast<1>(rd[q]);
        r4[q][2] = quad_bcast<2>(rd[q]);
        r4[q][3] = quad_bcast<3>(rd[q]);
      }
#pragma unroll
      for (int m = 0; m < M; ++m) {
        const uint32_t c = quad_col(S, m);
        if (c != 0) {   // (steps that no lane takes are passed over)
          QuadVal<ST> v = S.v[m];
          // (codes are decoded again: keeping the dose's floats costs registers)
          if constexpr (coded(ST)) asm("" : "+v"(v.x), "+v"(v.y));
          bool term = false;
#pragma unroll
          for (int q = 0; q < NT; ++q) {
            if (NT > 1 && !live[q]) continue;
            double t = static_cast<double>(val_of<ST>(v, 0)) * r4[q][0];
#pragma unroll
            for (int u = 1; u < 4; ++u) t = __builtin_fma(static_cast<double>(val_of<ST>(v, u)), r4[q][u], t);
            if (Plans::kMany || NT == 1) {
              add_term(q, c, t);
            } else {
              add_fixed(q, c, t);
              term = term || t != 0.0;
            }
          }
          if (!Plans::kMany && NT > 1 && term) mark[c >> 2] = 1;
        }
      }
    }
  };

  // A vector that is wild, or staged beside one that is: entry by entry, the
  // places without a nonzero left out (infinity times their zero is not 0).
  auto slow = [&](int q) {
    float zq[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    double r4[4] = {0.0, 0.0, 0.0, 0.0};
    for (int b = 0; b < kmax; ++b) {
      const uint2 hd = load_head(blk0 + b), rec = load_rec(b);
      const int flags = uniform(static_cast<int>(hd.y)), e = quad_log2(flags);
      if (flags == 0) break;
      const int sub = lane & ((1 << e) - 1), n = static_cast<int>(rec.x >> 16);
      const size_t at = static_cast<size_t>(uniform(static_cast<int>(hd.x))) + (rec.x & 0xFFFFu);
      const auto* ev = static_cast<const QuadVal<ST>*>(a.q_val) + at;
      const uint16_t* ec = a.q_col + at;
      if (flags & kQuadFirst) zq[0] = zq[1] = zq[2] = zq[3] = 0.0f;
      constexpr int R = quad_run(ST);   // (the lanes' entries in their steps' order)
      if (flags & kQuadDose)
        for (int j = sub; j < n / R; j += 1 << e)
          for (int k = R * j; k < R * j + R; ++k) {
            const QuadVal<ST> v = ev[k];
            const float x = staged(xs + q * nbs, ec[k]);
#pragma unroll
            for (int u = 0; u < 4; ++u)
              if (!quad_hole<ST>(v, u)) zq[u] = fmaf(val_of<ST>(v, u), x, zq[u]);
          }
      if (flags & kQuadFinish) {
        const int p = Plans::kMany ? q : 0;
        RowPenalty pen{0.0, 0.0, 0.0, 0.0};
        const uint32_t row = 4u * rec.y + (lane & 3);
        const uint32_t vox = a.vox && row < static_cast<uint32_t>(a.nv) ? a.vox[row] : row;
        if (PEN && row < static_cast<uint32_t>(a.nv)) {
          const Penalties& pp = P(p).pen;
          pen = penalty_of(p, pp.sid[row], pp.Tu_vox ? pp.Tu_vox[row] : 0.0f, pp.To_vox ? pp.To_vox[row] : 0.0f);
        }
        const double r = static_cast<double>(finish(q, zq, e, rec, pen, vox)) * up[q];
        r4[0] = quad_bcast<0>(r);
        r4[1] = quad_bcast<1>(r);
        r4[2] = quad_bcast<2>(r);
        r4[3] = quad_bcast<3>(r);
      }
      if (GRAD && (flags & kQuadAdjoint) && !wild[q])
        for (int j = sub; j < n / R; j += 1 << e)
          for (int k = R * j; k < R * j + R; ++k) {
            const QuadVal<ST> v = ev[k];
            double t = 0.0;
#pragma unroll
            for (int u = 0; u < 4; ++u)
              if (!quad_hole<ST>(v, u)) t = __builtin_fma(static_cast<double>(val_of<ST>(v, u)), r4[u], t);
            add_term(q, ec[k], t);
          }
    }
  };

  if (!any_wild) {
    // Block i is in A; block i + 1's loads are issued into B before block i's
    // arithmetic, and the record of block i + 2 with them.
    int i = 0;
    auto turn = [&](const QuadStage<ST, NP>& cur, QuadStage<ST, NP>& nxt) {
      const uint2 rc = rec0;
      const int f = fl;
      ++i;
      if ((i & 63) == 0) {   // the next 64 heads
        heads = load_head(i + lane < kmax ? blk0 + i + lane : static_cast<int>(nblk));
        __builtin_amdgcn_s_waitcnt(kWaitVmcnt0);
      }
      e0 = head_e0(i);
      fl = head_fl(i);
      rec0 = rec1;
      quad_issue<MODE, ST, CP>(P, rec0, e0, fl, lane, nxt);
      rec1 = load_rec(i + 1);
      __builtin_amdgcn_sched_barrier(0);
      compute(cur, rc, f);
      return fl != 0;
    };
    for (bool more = fl != 0; more;) {
      if (!turn(A, B)) break;
      more = turn(B, A);
    }
  } else {
#pragma unroll
    for (int q = 0; q < NT; ++q)
      if (active(q)) slow(q);
  }

  // objective partials, one of every eight waves: the same whether a
  // workgroup has eight or sixteen
  constexpr int kHalves = WAVES / 8;
#pragma unroll
  for (int q = 0; q < NT; ++q) {
    const double t = wave_sum(pacc[q]);
    if (lane == 63) gsum[q][wv] = t;
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < NT; ++q)
    if (tid < kHalves && active(q)) {
      double t = gsum[q][8 * tid];
#pragma unroll
      for (int k = 1; k < 8; ++k) t += gsum[q][8 * tid + k];
      double* parts = MODE == QM_WHOLE ? W->out.parts : P(q).partials;
      parts[(Plans::kMany ? 0 : q * sl.G * kHalves) + sl.w * kHalves + tid] = t;
    }
  if (GRAD) {
    // (the barrier also ends the waves' additions)
#pragma unroll
    for (int q = 0; q < NT; ++q) {
      if (!active(q)) continue;
      unsigned long long* out = (MODE == QM_WHOLE ? W->out.acc : P(q).q_acc) + static_cast<size_t>(Plans::kMany ? sl.w : sl.w * NT + q) * nb;
      for (int c = tid; c < nb; c += THREADS) {
        const unsigned long long s = acc[q * nbs + c + 1];
        out[c] = s == 0 ? mark[(Plans::kMany ? q * nbs : 0) + c + 1] : s;
      }
    }
  }
}

// Sixteen waves a workgroup leave 128 registers per lane; eight-wave
// workgroups run two side by side.
template <int NT, int WAVES>
constexpr int quad_waves_per_simd() { return WAVES == 16 || NT <= 2 ? 4 : 2; }

template <int NT, int MODE, int WAVES, int ST, int CP = 0>
__global__ __launch_bounds__(WAVES * 64, (quad_waves_per_simd<NT, WAVES>())) void quad_kernel(FwdArgs a) {
  quad_pass<NT, MODE, WAVES, ST, CP>(OnePlan{a}, Slot{static_cast<int>(blockIdx.x), static_cast<int>(gridDim.x)},
                                     a.nstruct);
}

// A small plan's iteration in one launch: every workgroup repeats the step
// for all columns (they are at most one per thread, and the pass's column
// sums few) instead of waiting for a launch that does it once.  What bounds
// it: two chains of dependent loads, with a barrier between; 11.2 us an
// iteration in two launches, 10.1 in one (32,000 voxels, 160 beamlets).
template <int ST>
__global__ __launch_bounds__(16 * 64, 4) void whole_kernel(FwdArgs a, WholeArgs w) {
  quad_pass<1, QM_WHOLE, 16, ST, 0>(OnePlan{a}, Slot{static_cast<int>(blockIdx.x), static_cast<int>(gridDim.x)},
                                    a.nstruct, &w);
}

// Batched solve pass over a slot table (see fwd_wave_batch_kernel).
template <int NT, int WAVES, int ST, int CP = 0>
__global__ __launch_bounds__(WAVES * 64, (quad_waves_per_simd<NT, WAVES>())) void quad_batch_kernel(
    const FwdArgs* __restrict__ args, const int32_t* __restrict__ slots) {
  const int sv = uniform(slots[blockIdx.x]);
  if (sv < 0) return;
  const FwdArgs& a = args[sv >> 16];
  quad_pass<NT, QM_SOLVE, WAVES, ST, CP>(OnePlan{a}, Slot{sv & 0xFFFF, a.grid}, a.nstruct);
}

// The same over groups of solves that share a matrix, one trial each (slots
// and groups as for adj_multi_batch_kernel): its entries are read once for
// all of them, and every solve gets the arithmetic it gets alone.
template <int K, int WAVES, int ST>
__global__ __launch_bounds__(WAVES * 64, (quad_waves_per_simd<K, WAVES>())) void quad_shared_kernel(
    const FwdArgs* __restrict__ args, const int32_t* __restrict__ groups, const int32_t* __restrict__ slots, int nst) {
  const int sv = uniform(slots[blockIdx.x]);
  if (sv < 0) return;
  const int32_t* gr = groups + static_cast<size_t>(sv >> 16) * (K + 1);
  ManyPlans<K> P;
  P.args = args;
  P.n = uniform(gr[0]);
#pragma unroll
  for (int q = 0; q < K; ++q) P.plan[q] = uniform(gr[1 + (q < P.n ? q : 0)]);
  quad_pass<K, QM_SOLVE, WAVES, ST, 0>(P, Slot{sv & 0xFFFF, P(0).grid}, nst);
}

// ---- step ---------------------------------------------------------------------------
// A workgroup takes kStepCols columns: thread (p, c) adds the column sums of
// workgroups p, p + 32, ... of the pass (128-byte runs), the 32 partial sums
// meet in LDS and the first wave completes them.  A column's total is exact
// whatever the order; only the float64 sums of a wild vector depend on it,
// and it is fixed here.
//
// What bounds it: latency.  So every load is issued on entry, the decision is
// taken by whole waves in registers (no barrier: the first wave alone, or
// every wave where the accepted trial picks the column sums to add), and one
// barrier separates the partial sums from the totals.
constexpr int kStepRows = kStepThreads / kStepCols, kStepWaves = kStepThreads / 64;
constexpr int kStepU = 8;    // column sums per thread and round

struct ColParts {
  unsigned long long v[kStepU];
};

// Byte offset of workgroup p's sum of column c and trial q; rows and columns
// past the last read zeros out of bounds.
__device__ __forceinline__ void col_load(const AdjArgs& a, rsrc_t r, int nt, int q, int c, int p0, ColParts& P) {
#pragma unroll
  for (int u = 0; u < kStepU; ++u) {
    const int p = p0 + u * kStepRows;
    const uint32_t off = p < a.q_parts && c < a.nb ? 8u * static_cast<uint32_t>((p * nt + q) * a.nb + c) : 0xFFFFFFF0u;
    P.v[u] = __builtin_bit_cast(unsigned long long, load_f64(r, off));
  }
}

__device__ __forceinline__ ColTotal col_sum(const AdjArgs& a, rsrc_t r, int nt, int q, int c, int p0,
                                            const ColParts& P) {
  ColTotal s{0, 0, 0};
#pragma unroll
  for (int u = 0; u < kStepU; ++u) add_part(s, P.v[u]);
  for (int p = p0 + kStepU * kStepRows; p < a.q_parts; p += kStepU * kStepRows) {
    ColParts R;
    col_load(a, r, nt, q, c, p, R);
#pragma unroll
    for (int u = 0; u < kStepU; ++u) add_part(s, R.v[u]);
  }
  return s;
}

__device__ __forceinline__ rsrc_t acc_rsrc(const AdjArgs& a, int nt) {
  return make_rsrc(a.q_acc, 8u * static_cast<uint32_t>(a.q_parts) * static_cast<uint32_t>(nt * a.nb));
}

// Partial totals of a workgroup's columns in LDS.  w: `a`, saturated, above
// six bits that count the partial totals with `any` set (32 at most).
struct StepSums {
  unsigned long long s[kStepThreads];
  uint32_t w[kStepThreads];
  double exact[kStepWaves][kStepCols];
  uint32_t bad;
};
__device__ __forceinline__ void put_sum(StepSums& sh, const ColTotal& T) {
  sh.s[threadIdx.x] = T.s;
  sh.w[threadIdx.x] = min(T.a, 1u << 20) << 6 | (T.any != 0);
}

// After put_sum by all, in the first wave: the total of column c = sl.w * 16 +
// lane % 16 in every lane, in the products' own scale.  Columns whose integers
// are not precise enough (again: there are some) are summed again by all
// waves, where the totals are wanted.
__device__ __forceinline__ double col_total(const AdjArgs& a, StepSums& sh, double unit, const float* r, const float* x,
                                            int c, bool want, bool& again) {
  const int lane = threadIdx.x & 63, wv = uniform(threadIdx.x >> 6), i = lane & (kStepCols - 1), p0 = lane / kStepCols;
  __syncthreads();
  bool bad = false;
  double total = 0.0;
  if (wv == 0) {
    unsigned long long s = 0;
    uint32_t w = 0;
#pragma unroll
    for (int p = 0; p < kStepRows; p += 64 / kStepCols) {
      s += sh.s[(p + p0) * kStepCols + i];
      w += sh.w[(p + p0) * kStepCols + i];
    }
#pragma unroll
    for (int d = kStepCols; d < 64; d <<= 1) {
      s += __shfl_xor(s, d);
      w += __shfl_xor(w, d);
    }
    bad = c < a.nb && imprecise(ColTotal{s, w >> 6, w & 63}, unit, a.enough);
    total = static_cast<double>(static_cast<long long>(s)) * unit;
    const uint64_t mask = __ballot(bad);
    again = mask != 0;
    if (lane == 0) sh.bad = want ? static_cast<uint32_t>(mask) & ((1u << kStepCols) - 1) : 0;
  }
  __syncthreads();
  const uint32_t mask = uniform(static_cast<int>(sh.bad));
  if (mask != 0) {
    for (int k = 0; k < kStepCols; ++k)
      if (mask >> k & 1) {
        const double t = exact_column(a.again, r, x, c - i + k, wv, kStepWaves);
        if (lane == 0) sh.exact[wv][k] = t;
      }
    __syncthreads();
    if (bad) {
      total = 0.0;
      for (int k = 0; k < kStepWaves; ++k) total += sh.exact[k][i];
    }
  }
  return total;
}

__device__ __forceinline__ double col_factor(const AdjArgs& a, int c) {
  return a.col_scale ? a.scale * static_cast<double>(load_f32(make_rsrc(a.col_scale, 4u * a.nb), 4u * c)) : a.scale;
}

// The sum that the step takes of a pass's objectives.
__global__ __launch_bounds__(64) void wave_sum_kernel(const double* parts, int n, double* out, double add) {
  SumLoads<8> L;
  sum_start(parts, n, L);
  const double s = sum_finish(parts, n, L);
  if (threadIdx.x == 0) *out = s + add;
}

// The state but for `again`, which another workgroup may be writing.
__device__ __forceinline__ void put_state(SolverState* to, const SolverState& st) {
  struct Words {
    int32_t w[kStateWords];
  };
  const Words v = __builtin_bit_cast(Words, st);
#pragma unroll
  for (int i = 0; i < kStateWords; ++i)
    if (i != static_cast<int>(offsetof(SolverState, again) / 4)) reinterpret_cast<int32_t*>(to)[i] = v.w[i];
}

template <int NT>
__device__ __forceinline__ void step_pass(const AdjArgs& a, const Slot sl) {
  __shared__ StepSums sh;
  const int tid = threadIdx.x, lane = tid & 63, wv = uniform(tid >> 6);
  const int c = sl.w * kStepCols + (tid & (kStepCols - 1)), p0 = tid / kStepCols;
  const bool decides = NT > 1 || wv == 0;
  const rsrc_t ra = acc_rsrc(a, NT);
  int32_t sw = 0;
  SumLoads<8> GL[NT];
  SumLoads<4> SL[NT];
  float xt[NT], xk = 0.0f, g = 0.0f;
  double unit[NT], factor = 1.0;
  if (decides) {
    sw = load_i32(make_rsrc(a.st_in, static_cast<uint32_t>(sizeof(SolverState))), 4u * (lane < kStateWords ? lane : 0));
#pragma unroll
    for (int q = 0; q < NT; ++q) {
      sum_start(a.fwd_partials + q * a.fwd_parts, a.fwd_parts, GL[q]);
      sum_start(a.q_steps + q * sl.G, sl.G, SL[q]);
    }
  }
  ColParts CP;
  col_load(a, ra, NT, 0, c, p0, CP);
  const rsrc_t ru = make_rsrc(a.q_unit, 8u * NT);
#pragma unroll
  for (int q = 0; q < NT; ++q) unit[q] = load_f64(ru, 8u * q);
  const int stored = load_i32(make_rsrc(a.st_in, static_cast<uint32_t>(sizeof(SolverState))), offsetof(SolverState, stored));
  if (wv == 0) {
    const uint32_t nb4 = 4u * static_cast<uint32_t>(a.nb), at = 4u * static_cast<uint32_t>(c);
    xk = load_f32(make_rsrc(a.xbuf[NT], nb4), at);
    g = load_f32(make_rsrc(a.out, nb4), at);
#pragma unroll
    for (int q = 0; q < NT; ++q) xt[q] = load_f32(make_rsrc(a.xbuf[q], nb4), at);
    factor = col_factor(a, c);
  }
  SolverState st;
  Verdict v;
  bool was_done = false;
  if (decides) {
    int32_t w[kStateWords];
#pragma unroll
    for (int i = 0; i < kStateWords; ++i) w[i] = __builtin_amdgcn_readlane(sw, i);
    st = __builtin_bit_cast(SolverState, w);
    was_done = st.phase == PH_DONE;
    if (!was_done) {
      double Gq[NT], sq[NT];
#pragma unroll
      for (int q = 0; q < NT; ++q) {
        Gq[q] = sum_finish(a.fwd_partials + q * a.fwd_parts, a.fwd_parts, GL[q]) + a.G_skip;
        sq[q] = sum_finish(a.q_steps + q * sl.G, sl.G, SL[q]);
      }
      decide_state<NT>(st, Gq, sq, v);
    }
    st.xi = NT;   // x_k has a buffer of its own
  }
  // (the initial evaluation accepts nothing: trial 0 is x_1)
  int q = 0;
  if (NT > 1) {
    q = uniform(max(v.accepted, 0));
    if (q != 0 && !was_done) col_load(a, ra, NT, q, c, p0, CP);
  }
  double u = unit[0];
#pragma unroll
  for (int k = 1; k < NT; ++k) u = (q == k) ? unit[k] : u;
  const float* r = a.rbuf[0];
#pragma unroll
  for (int k = 1; k < NT; ++k) r = (q == k) ? a.rbuf[k] : r;
  put_sum(sh, col_sum(a, ra, NT, q, c, p0, CP));
  bool again = false;
  const double total = col_total(a, sh, u, uniform(stored) > 0 ? r : nullptr, a.q_x + static_cast<size_t>(q) * a.nb, c,
                                 decides && !was_done && st.phase == PH_NEED_GRAD, again);
  if (wv != 0) return;
  if (again && lane == 0) a.st_out->again = st.n_fwd;   // (the passes decided on so far)
  if (sl.w == 0 && lane == 0) {
    put_state(a.st_out, st);
    if (v.accepted >= 0 && a.trace != nullptr && st.k - 1 < st.trace_cap) {
      TraceDev e;
      e.k = st.k;
      e.backtracks = v.backtracks;
      e.lambda = v.lam;
      e.step_sq = v.step_sq;
      e.G = st.G;
      a.trace[st.k - 1] = e;
    }
  }
  if (was_done) return;
  const bool mine = lane < kStepCols && c < a.nb;
  if (v.accepted >= 0) {
#pragma unroll
    for (int k = 0; k < NT; ++k) xk = (v.accepted == k) ? xt[k] : xk;
    if (mine) a.xbuf[NT][c] = xk;
  }
  if (st.phase == PH_DONE) return;
  if (st.phase == PH_NEED_GRAD) {
    g = static_cast<float>(factor * total);
    if (mine) a.out[c] = g;
  }
  double lam = st.lambda;
#pragma unroll
  for (int k = 0; k < NT; ++k) {
    if (k > 0) lam = lam / st.alpha;
    double sq = 0.0;
    if (mine) {
      const float t = trial_point(xk, g, lam);
      a.xbuf[k][c] = t;
      const double dl = static_cast<double>(t) - static_cast<double>(xk);
      sq = dl * dl;
    }
    sq = group_sum<kStepCols>(sq);
    // (read by the next step from the copy that the next pass makes)
    if (lane == kStepCols - 1) a.q_steps[(NT + k) * sl.G + sl.w] = sq;
  }
}

// (one trial: 64 registers, so that four workgroups run side by side; with the
// 72 that the compiler would take, 32 plans' steps took 9.5 against 8.5 us)
template <int NT>
constexpr int step_waves() { return NT == 1 ? 8 : 1; }

template <int NT>
__global__ __launch_bounds__(kStepThreads, step_waves<NT>()) void step_kernel(AdjArgs a) {
  step_pass<NT>(a, Slot{static_cast<int>(blockIdx.x), static_cast<int>(gridDim.x)});
}

template <int NT>
__global__ __launch_bounds__(kStepThreads, step_waves<NT>()) void step_batch_kernel(const AdjArgs* __restrict__ args,
                                                                  const int32_t* __restrict__ slots) {
  const int sv = uniform(slots[blockIdx.x]);
  if (sv < 0) return;
  const AdjArgs& a = args[sv >> 16];
  step_pass<NT>(a, Slot{sv & 0xFFFF, step_grid(a.nb)});
}

// out = scale * D^T r from a pass's column sums; norm (nullable): each
// workgroup's sum of squares of its entries.
// With `sum` one more workgroup adds parts[0..n) as wave_sum_kernel does.
__global__ __launch_bounds__(kStepThreads) void reduce_kernel(AdjArgs a, double* norm, double* sum,
                                                              const double* parts, int n, double add) {
  __shared__ StepSums sh;
  if (static_cast<int>(blockIdx.x) == step_grid(a.nb)) {
    if (threadIdx.x >= 64) return;
    SumLoads<8> L;
    sum_start(parts, n, L);
    const double s = sum_finish(parts, n, L);
    if (threadIdx.x == 0) *sum = s + add;
    return;
  }
  const int tid = threadIdx.x, c = blockIdx.x * kStepCols + (tid & (kStepCols - 1)), p0 = tid / kStepCols;
  const rsrc_t ra = acc_rsrc(a, 1);
  ColParts CP;
  col_load(a, ra, 1, 0, c, p0, CP);
  const double unit = load_f64(make_rsrc(a.q_unit, 8u), 0);
  const double factor = col_factor(a, c);
  put_sum(sh, col_sum(a, ra, 1, 0, c, p0, CP));
  bool again = false;
  const double total = col_total(a, sh, unit, a.rbuf[0], nullptr, c, true, again);
  if (tid >= 64) return;
  const float g = static_cast<float>(factor * total);
  double sq = 0.0;
  if (tid < kStepCols && c < a.nb) {
    a.out[c] = g;
    sq = static_cast<double>(g) * static_cast<double>(g);
  }
  if (norm == nullptr) return;
  sq = group_sum<kStepCols>(sq);
  if (tid == kStepCols - 1) norm[blockIdx.x] = sq;
}

template <int MODE, int WAVES, int ST>
void launch_quad_one(const FwdArgs& a, dim3 gd, size_t lds, hipStream_t s) {
  hipLaunchKernelGGL((quad_kernel<1, MODE, WAVES, ST>), gd, dim3(WAVES * 64), lds, s, a);
}

template <int ST, int CP>
int launch_quad_solve(const FwdArgs& a, int nt, int waves, dim3 gd, size_t lds, hipStream_t s, hipEvent_t b,
                      hipEvent_t e) {
  const dim3 t16(16 * 64), t8(8 * 64);
  const bool w16 = waves == 16;
  switch (nt) {
    case 1:
      if (w16) hipExtLaunchKernelGGL((quad_kernel<1, QM_SOLVE, 16, ST, CP>), gd, t16, lds, s, b, e, 0, a);
      else hipExtLaunchKernelGGL((quad_kernel<1, QM_SOLVE, 8, ST, CP>), gd, t8, lds, s, b, e, 0, a);
      break;
    case 2:
      if (w16) hipExtLaunchKernelGGL((quad_kernel<2, QM_SOLVE, 16, ST, CP>), gd, t16, lds, s, b, e, 0, a);
      else hipExtLaunchKernelGGL((quad_kernel<2, QM_SOLVE, 8, ST, CP>), gd, t8, lds, s, b, e, 0, a);
      break;
    case 4: hipExtLaunchKernelGGL((quad_kernel<4, QM_SOLVE, 8, ST, CP>), gd, t8, lds, s, b, e, 0, a); break;
    default: return set_error(IMRT_EINVAL, "trials per pass must be 1, 2 or 4");
  }
  return IMRT_OK;
}

template <int ST>
int launch_quad_st(const FwdArgs& a, int nt, int waves, dim3 gd, size_t lds, hipStream_t s, hipEvent_t b,
                   hipEvent_t e) {
  const bool w16 = waves == 16;
  switch (a.mode) {
    case QM_SOLVE:
      return a.stream_cp ? launch_quad_solve<ST, 2>(a, nt, waves, gd, lds, s, b, e)
                         : launch_quad_solve<ST, 0>(a, nt, waves, gd, lds, s, b, e);
    case QM_EVAL: w16 ? launch_quad_one<QM_EVAL, 16, ST>(a, gd, lds, s) : launch_quad_one<QM_EVAL, 8, ST>(a, gd, lds, s); break;
    case QM_GRAD: w16 ? launch_quad_one<QM_GRAD, 16, ST>(a, gd, lds, s) : launch_quad_one<QM_GRAD, 8, ST>(a, gd, lds, s); break;
    case QM_PLAIN: w16 ? launch_quad_one<QM_PLAIN, 16, ST>(a, gd, lds, s) : launch_quad_one<QM_PLAIN, 8, ST>(a, gd, lds, s); break;
    default: w16 ? launch_quad_one<QM_POWER, 16, ST>(a, gd, lds, s) : launch_quad_one<QM_POWER, 8, ST>(a, gd, lds, s); break;
  }
  return IMRT_OK;
}

template <int ST, int CP>
int launch_quad_batch_st(const FwdArgs* args, const int32_t* slots, int nslots, int nt, int waves, size_t lds,
                         hipStream_t s) {
  const dim3 gd(nslots);
  const bool w16 = waves == 16;
  switch (nt) {
    case 1:
      if (w16) hipLaunchKernelGGL((quad_batch_kernel<1, 16, ST, CP>), gd, dim3(16 * 64), lds, s, args, slots);
      else hipLaunchKernelGGL((quad_batch_kernel<1, 8, ST, CP>), gd, dim3(8 * 64), lds, s, args, slots);
      break;
    case 2:
      if (w16) hipLaunchKernelGGL((quad_batch_kernel<2, 16, ST, CP>), gd, dim3(16 * 64), lds, s, args, slots);
      else hipLaunchKernelGGL((quad_batch_kernel<2, 8, ST, CP>), gd, dim3(8 * 64), lds, s, args, slots);
      break;
    case 4: hipLaunchKernelGGL((quad_batch_kernel<4, 8, ST, CP>), gd, dim3(8 * 64), lds, s, args, slots); break;
    default: return set_error(IMRT_EINVAL, "trials per pass must be 1, 2 or 4");
  }
  return IMRT_OK;
}

}  // namespace

int launch_quad(const imrt_ctx* ctx, const FwdArgs& a, int ntrials, int waves, int grid, hipEvent_t before,
                hipEvent_t after) {
  clear_stale_error();
  const size_t lds = quad_lds_bytes(a.nb, ntrials, a.nstruct, a.mode);
  if (!quad_fits(ctx->max_lds, lds)) return set_error(IMRT_EUNSUPPORTED, "one-read pass: LDS budget exceeded");
  if (a.mode != QM_SOLVE && ntrials != 1) return set_error(IMRT_EINVAL, "evaluation passes take one trial");
  int rc;
  switch (a.storage) {
    case ST_F32: rc = launch_quad_st<ST_F32>(a, ntrials, waves, dim3(grid), lds, ctx->stream, before, after); break;
    case ST_BF16: rc = launch_quad_st<ST_BF16>(a, ntrials, waves, dim3(grid), lds, ctx->stream, before, after); break;
    case ST_F16: rc = launch_quad_st<ST_F16>(a, ntrials, waves, dim3(grid), lds, ctx->stream, before, after); break;
    default: return set_error(IMRT_EINVAL, "unknown storage");
  }
  return rc ? rc : check_launch("quad_kernel");
}

int launch_quad_batch(const imrt_ctx* ctx, const FwdArgs* args, const int32_t* slots, int nslots, int ntrials,
                      int storage, int waves, size_t lds, int stream_cp) {
  if (nslots <= 0) return IMRT_OK;
  if (!quad_fits(ctx->max_lds, lds)) return set_error(IMRT_EUNSUPPORTED, "batched one-read pass: LDS budget exceeded");
  hipStream_t s = ctx->stream;
  int rc;
  switch (storage) {
    case ST_F32:
      rc = stream_cp ? launch_quad_batch_st<ST_F32, 2>(args, slots, nslots, ntrials, waves, lds, s)
                     : launch_quad_batch_st<ST_F32, 0>(args, slots, nslots, ntrials, waves, lds, s);
      break;
    case ST_BF16:
      rc = stream_cp ? launch_quad_batch_st<ST_BF16, 2>(args, slots, nslots, ntrials, waves, lds, s)
                     : launch_quad_batch_st<ST_BF16, 0>(args, slots, nslots, ntrials, waves, lds, s);
      break;
    case ST_F16:
      rc = stream_cp ? launch_quad_batch_st<ST_F16, 2>(args, slots, nslots, ntrials, waves, lds, s)
                     : launch_quad_batch_st<ST_F16, 0>(args, slots, nslots, ntrials, waves, lds, s);
      break;
    default: return set_error(IMRT_EINVAL, "unknown storage");
  }
  return rc ? rc : check_launch("quad_batch_kernel");
}

int launch_quad_shared(const imrt_ctx* ctx, const FwdArgs* args, const int32_t* groups, int group_k,
                       const int32_t* slots, int nslots, int storage, int nb, int nstruct) {
  if (nslots <= 0) return IMRT_OK;
  const size_t lds = quad_lds_bytes(nb, group_k, group_k * nstruct, QM_SOLVE, group_k);
  if (!quad_fits(ctx->max_lds, lds)) return set_error(IMRT_EUNSUPPORTED, "shared one-read pass: LDS budget exceeded");
  if (group_k != 2 && group_k != 4) return set_error(IMRT_EINVAL, "shared-matrix groups hold 2 or 4 solves");
  const dim3 gd(nslots), bd(8 * 64);
  hipStream_t s = ctx->stream;
  auto go = [&](auto k2, auto k4) {
    if (group_k == 2) hipLaunchKernelGGL(k2, gd, bd, lds, s, args, groups, slots, nstruct);
    else hipLaunchKernelGGL(k4, gd, bd, lds, s, args, groups, slots, nstruct);
  };
  switch (storage) {
    case ST_F32: go(quad_shared_kernel<2, 8, ST_F32>, quad_shared_kernel<4, 8, ST_F32>); break;
    case ST_BF16: go(quad_shared_kernel<2, 8, ST_BF16>, quad_shared_kernel<4, 8, ST_BF16>); break;
    case ST_F16: go(quad_shared_kernel<2, 8, ST_F16>, quad_shared_kernel<4, 8, ST_F16>); break;
    default: return set_error(IMRT_EINVAL, "unknown storage");
  }
  return check_launch("quad_shared_kernel");
}

int launch_whole(const imrt_ctx* ctx, const FwdArgs& a, const WholeArgs& w, int grid) {
  clear_stale_error();
  const size_t lds = quad_lds_bytes(a.nb, 1, a.nstruct, QM_SOLVE);
  if (!quad_fits(ctx->max_lds, lds, QM_WHOLE)) return set_error(IMRT_EUNSUPPORTED, "one-read pass: LDS budget exceeded");
  if (a.nb > 16 * 64) return set_error(IMRT_EINVAL, "internal: more columns than threads");
  const dim3 gd(grid), bd(16 * 64);
  hipStream_t s = ctx->stream;
  switch (a.storage) {
    case ST_F32: hipLaunchKernelGGL(whole_kernel<ST_F32>, gd, bd, lds, s, a, w); break;
    case ST_BF16: hipLaunchKernelGGL(whole_kernel<ST_BF16>, gd, bd, lds, s, a, w); break;
    case ST_F16: hipLaunchKernelGGL(whole_kernel<ST_F16>, gd, bd, lds, s, a, w); break;
    default: return set_error(IMRT_EINVAL, "unknown storage");
  }
  return check_launch("whole_kernel");
}

int launch_step(const imrt_ctx* ctx, const AdjArgs& a, int ntrials, hipEvent_t before, hipEvent_t after) {
  clear_stale_error();
  const dim3 gd(step_grid(a.nb)), bd(kStepThreads);
  hipStream_t s = ctx->stream;
  switch (ntrials) {
    case 1: hipExtLaunchKernelGGL((step_kernel<1>), gd, bd, 0, s, before, after, 0, a); break;
    case 2: hipExtLaunchKernelGGL((step_kernel<2>), gd, bd, 0, s, before, after, 0, a); break;
    case 4: hipExtLaunchKernelGGL((step_kernel<4>), gd, bd, 0, s, before, after, 0, a); break;
    default: return set_error(IMRT_EINVAL, "trials per pass must be 1, 2 or 4");
  }
  return check_launch("step_kernel");
}

int launch_step_batch(const imrt_ctx* ctx, const AdjArgs* args, const int32_t* slots, int nslots, int ntrials) {
  if (nslots <= 0) return IMRT_OK;
  const dim3 gd(nslots), bd(kStepThreads);
  hipStream_t s = ctx->stream;
  switch (ntrials) {
    case 1: hipLaunchKernelGGL((step_batch_kernel<1>), gd, bd, 0, s, args, slots); break;
    case 2: hipLaunchKernelGGL((step_batch_kernel<2>), gd, bd, 0, s, args, slots); break;
    case 4: hipLaunchKernelGGL((step_batch_kernel<4>), gd, bd, 0, s, args, slots); break;
    default: return set_error(IMRT_EINVAL, "trials per pass must be 1, 2 or 4");
  }
  return check_launch("step_batch_kernel");
}

int launch_wave_sum(const imrt_ctx* ctx, const double* parts, int n, double* out, double add) {
  clear_stale_error();
  hipLaunchKernelGGL(wave_sum_kernel, dim3(1), dim3(64), 0, ctx->stream, parts, n, out, add);
  return check_launch("wave_sum_kernel");
}

int launch_reduce(const imrt_ctx* ctx, const AdjArgs& a, double* norm, double* sum, const double* parts, int n,
                  double add) {
  clear_stale_error();
  hipLaunchKernelGGL(reduce_kernel, dim3(step_grid(a.nb) + (sum ? 1 : 0)), dim3(kStepThreads), 0, ctx->stream, a, norm,
                     sum, parts, n, add);
  return check_launch("reduce_kernel");
}

}  // namespace imrt
