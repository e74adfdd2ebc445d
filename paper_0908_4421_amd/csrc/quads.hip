// The quad form of a dose matrix, which the one-read pass walks (see
// imrt_internal.h for its layout): built on the device from the CSR arrays,
// its work partition on the host.
#include <algorithm>
#include <new>

#include "pass_common.h"

namespace imrt {
namespace {

// The four rows of a quad merged by column, in ascending order: visit(column,
// values, mask of the rows that hold it).
template <typename Col, typename Visit>
__device__ __forceinline__ void merge_rows(const int32_t* row_ptr, const Col* col, int nv, int quad, Visit visit) {
  int at[4], end[4], c[4];
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int r = 4 * quad + u;
    at[u] = r < nv ? row_ptr[r] : 0;
    end[u] = r < nv ? row_ptr[r + 1] : 0;
    c[u] = at[u] < end[u] ? static_cast<int>(col[at[u]]) : 0x7FFFFFFF;
  }
  for (;;) {
    const int lo = min(min(c[0], c[1]), min(c[2], c[3]));
    if (lo == 0x7FFFFFFF) return;
    int k[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) k[u] = c[u] == lo ? at[u] : -1;
    visit(lo, k);
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (c[u] == lo) {
        ++at[u];
        c[u] = at[u] < end[u] ? static_cast<int>(col[at[u]]) : 0x7FFFFFFF;
      }
  }
}

// sums[0]: the largest row sum (bits of a float64 >= 0, which order as integers)
__device__ __forceinline__ void atomic_max_f64(unsigned long long* p, double v) {
  atomicMax(p, static_cast<unsigned long long>(__double_as_longlong(v)));
}

template <typename Col>
__global__ __launch_bounds__(kThreads) void quad_count_kernel(const int32_t* row_ptr, const Col* col, int nv, int nq,
                                                              int32_t* counts) {
  const int q = blockIdx.x * kThreads + threadIdx.x;
  if (q >= nq) return;
  int n = 0;
  merge_rows(row_ptr, col, nv, q, [&](int, const int (&)[4]) { ++n; });
  counts[q] = n;
}

// Voxels (in the caller's order) of the rows of empty quads, in any order.
// A workgroup counts its share of the rows first: one atomic each (one per
// wave took 5 ms of a 1.33 M row matrix's build on their one address).
__global__ __launch_bounds__(kThreads) void quad_empty_kernel(const int32_t* counts, int nv, const int32_t* vox,
                                                              int32_t* zero, int32_t* nzero) {
  __shared__ int32_t place;
  int r0, r1;
  work_range(nv, r0, r1);
  auto empty = [&](int row) { return row < r1 && counts[row / 4] == 0; };
  if (threadIdx.x == 0) place = 0;
  __syncthreads();
  int mine = 0;
  for (int row = r0 + threadIdx.x; row < r1; row += kThreads) mine += empty(row);
  const int at = atomicAdd(&place, mine);
  __syncthreads();
  if (threadIdx.x == 0) place = atomicAdd(nzero, place);
  __syncthreads();
  int to = place + at;
  for (int row = r0 + threadIdx.x; row < r1; row += kThreads)
    if (empty(row)) zero[to++] = vox ? vox[row] : row;
}

template <int ST>
__device__ __forceinline__ double stored(const float* val, const uint16_t* val16, int64_t k) {
  if constexpr (coded(ST)) return static_cast<double>(code_value<ST>(val16[k]));
  else return static_cast<double>(val[k]);
}

// Entries of the quads in their final order: quad rows qrow[i], first entry
// ptr[i] (ptr[nq]: their number).
template <int ST, typename Col>
__global__ __launch_bounds__(kThreads) void quad_fill_kernel(const int32_t* row_ptr, const Col* col, const float* val,
                                                             const uint16_t* val16, int nv, int nq,
                                                             const int32_t* qrow, const int32_t* ptr, uint16_t* q_col,
                                                             void* q_val, unsigned long long* sums) {
  const int i = blockIdx.x * kThreads + threadIdx.x;
  double rs[4] = {0.0, 0.0, 0.0, 0.0};
  if (i < nq) {
    const int e0 = ptr[i], n = ptr[i + 1] - e0, full = quad_full(ST);
    const int before = quad_parts_before(n, full);
    int r = 0, part = 0, p0 = 0, p1 = quad_part(n, full, before, 1);
    // place of entry r of the part [p0, p1): in column order, or in pairs
    auto place = [&]() {
      if (quad_run(ST) == 1) return e0 + r;
      if (r == p1) {
        ++part;
        p0 = p1;
        p1 = quad_part(n, full, before, part + 1);
      }
      const int h = (p1 - p0) / 2, j = r - p0;
      return e0 + p0 + (j < h ? 2 * j : 2 * (j - h) + 1);
    };
    merge_rows(row_ptr, col, nv, qrow[i], [&](int c, const int (&k)[4]) {
      const int e = place();
      q_col[e] = static_cast<uint16_t>(4 * (c + 1));
      if constexpr (coded(ST)) {
        uint32_t h[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          h[u] = k[u] >= 0 ? val16[k[u]] : 0x8000u;
          if (k[u] >= 0 && h[u] == 0x8000u) h[u] = 0;   // (a stored -0 is no hole)
          if (k[u] >= 0) rs[u] += stored<ST>(val, val16, k[u]);
        }
        static_cast<uint2*>(q_val)[e] = make_uint2(h[0] | (h[1] << 16), h[2] | (h[3] << 16));
      } else {
        float v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          v[u] = k[u] >= 0 ? val[k[u]] + 0.0f : -0.0f;   // (a stored -0 is no hole)
          if (k[u] >= 0) rs[u] += static_cast<double>(v[u]);
        }
        static_cast<float4*>(q_val)[e] = make_float4(v[0], v[1], v[2], v[3]);
      }
      ++r;
    });
    if (coded(ST) && r < n) {
      const int e = place();
      q_col[e] = 0;
      static_cast<uint2*>(q_val)[e] = make_uint2(0x80008000u, 0x80008000u);
    }
  }
  double m = fmax(fmax(rs[0], rs[1]), fmax(rs[2], rs[3]));
  for (int d = 1; d < 64; d <<= 1) m = fmax(m, __shfl_xor(m, d));
  if ((threadIdx.x & 63) == 0) atomic_max_f64(sums, m);
}

// sums[1]: the largest column sum; a wave per column.
template <int ST>
__global__ __launch_bounds__(kThreads) void column_sum_kernel(const int32_t* col_ptr, const float* cval,
                                                              const uint16_t* cval16, int nb,
                                                              unsigned long long* sums) {
  const int c = blockIdx.x * kWaves + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  double s = 0.0;
  if (c < nb)
    for (int k = col_ptr[c] + lane; k < col_ptr[c + 1]; k += 64) s += stored<ST>(cval, cval16, csc_slot(k));
  s = wave_sum(s);
  if (lane == 63) atomic_max_f64(sums + 1, s);
}

struct Scratch {
  void* p = nullptr;
  ~Scratch() {
    if (p) (void)hipFree(p);
  }
};

int alloc(void** p, size_t bytes) {
  const hipError_t e = hipMalloc(p, std::max<size_t>(bytes, 16));
  if (e == hipErrorOutOfMemory) return set_error(IMRT_ENOMEM, "hipMalloc: out of device memory");
  return e == hipSuccess ? IMRT_OK : hip_error(e, "hipMalloc(quad form)");
}

// Quads are ordered by falling size within windows of so many, so that the
// quads of a block are of one size and its lanes take equally many steps.
constexpr int kWindow = 512;

int lanes_for(int n, int storage) {
  int L = 4;
  while (L < 64 && L * quad_full(storage) < 64 * n) L *= 2;
  return L;
}

}  // namespace

// Whether a pass of nt trials over D is the one-read pass: the matrix keeps
// its quad form, and the trials with their column sums fit LDS.
bool one_read(const imrt_ctx* C, const imrt_dose* D, int nt, int nstruct) {
  return D->q_waves > 0 && C->tune.fwd_wave != 0 && quad_fits(C->max_lds, quad_lds_bytes(D->nb, nt, nstruct, QM_SOLVE));
}

int quad_grid(const imrt_dose* D, int nt) { return D->q_waves / forward_waves(nt, D->fwd_waves); }

// Bytes of the entries that a one-read pass reads.
int64_t quad_bytes(const imrt_dose* D) { return D->nent * (D->storage == ST_F32 ? 18 : 10); }

// The matrix without its quad form: the two separate passes.
void drop_quads(imrt_dose* D) {
  for (void* p : {static_cast<void*>(D->q_col), D->q_val, static_cast<void*>(D->q_head), static_cast<void*>(D->q_rec),
                  static_cast<void*>(D->q_zero)})
    if (p) (void)hipFree(p);
  D->q_col = nullptr;
  D->q_val = nullptr;
  D->q_head = nullptr;
  D->q_rec = nullptr;
  D->q_zero = nullptr;
  D->nent = 0;
  D->nzero = 0;
  D->q_nblocks = D->q_kmax = D->q_waves = 0;
  D->qn.clear();
  D->qrow.clear();
  D->qgaps.clear();
  D->quad_epoch += 1;
}

namespace {

// Waits for a stream's copies from and to what was declared before it, also
// where an exception ends the function.
struct Drain {
  hipStream_t s;
  ~Drain() { (void)hipStreamSynchronize(s); }
};

// The form is extra: a matrix whose device has no room for it goes without.
template <typename Make>
int quads_or_none(imrt_dose* D, Make make) {
  int rc;
  try {
    rc = make();
  } catch (const std::bad_alloc&) {
    rc = IMRT_ENOMEM;
  }
  if (rc != IMRT_ENOMEM) return rc;
  (void)hipGetLastError();
  drop_quads(D);
  return IMRT_OK;
}

int place_quads(imrt_dose* D);

int make_quads(imrt_dose* D) {
  if (!D->ctx->tune.one_read || D->nb > 8191 || D->nv >= (1 << 30) || D->nnz == 0 || (D->storage == ST_F32 && D->fwd_st != ST_F32C16))
    return IMRT_OK;
  if (!quad_fits(D->ctx->max_lds, quad_lds_bytes(D->nb, 1, kMaxStruct, QM_SOLVE))) return IMRT_OK;
  hipStream_t s = D->ctx->stream;
  const int nqa = (D->nv + 3) / 4;
  Scratch cnt, ord, sums;
  int rc;
  if ((rc = alloc(&cnt.p, sizeof(int32_t) * nqa)) || (rc = alloc(&sums.p, 2 * sizeof(unsigned long long)))) return rc;
  auto* d_cnt = static_cast<int32_t*>(cnt.p);
  auto* d_sums = static_cast<unsigned long long*>(sums.p);
  const dim3 gq((nqa + kThreads - 1) / kThreads), bd(kThreads), gc((D->nb + kWaves - 1) / kWaves);
  const bool c16 = D->storage != ST_F32;
  if (c16) hipLaunchKernelGGL(quad_count_kernel<uint16_t>, gq, bd, 0, s, D->row_ptr, D->col16, D->nv, nqa, d_cnt);
  else hipLaunchKernelGGL(quad_count_kernel<int32_t>, gq, bd, 0, s, D->row_ptr, D->col_idx, D->nv, nqa, d_cnt);
  IMRT_HIP(hipGetLastError());
  std::vector<int32_t> n(nqa);
  IMRT_HIP(hipMemcpyAsync(n.data(), d_cnt, sizeof(int32_t) * nqa, hipMemcpyDeviceToHost, s));
  IMRT_HIP(hipMemsetAsync(d_sums, 0, 2 * sizeof(unsigned long long), s));
  IMRT_HIP(hipStreamSynchronize(s));
  int64_t nent = 0;
  for (int32_t& v : n) {
    v += v % quad_run(D->storage);
    nent += v;
  }
  // The rule: the quad form where its one read is fewer bytes than the two
  // passes' reads together.
  const int64_t per = c16 ? 10 : 18, two = c16 ? 10 : 14;
  if (nent >= (int64_t(1) << 31) - kQuadPad) return IMRT_OK;
  if (D->ctx->tune.one_read < 2 && nent * per > D->nnz * two) return IMRT_OK;
  std::vector<int32_t> qrow(nqa);
  std::vector<std::pair<int32_t, int32_t>> gaps;
  size_t some = 0;
  for (int q = 0; q < nqa;) {
    if (n[q] > 0) {
      qrow[some++] = q++;
      continue;
    }
    const int q0 = q;
    while (q < nqa && n[q] == 0) ++q;
    gaps.emplace_back(4 * q0, std::min(4 * q, D->nv));
  }
  qrow.resize(some);
  const int nq = static_cast<int>(qrow.size());
  for (const auto& gap : gaps) D->nzero += gap.second - gap.first;
  if (D->nzero > 0) {
    if ((rc = alloc(reinterpret_cast<void**>(&D->q_zero), sizeof(int32_t) * D->nzero))) return rc;
    auto* counter = reinterpret_cast<int32_t*>(d_sums);
    hipLaunchKernelGGL(quad_empty_kernel, dim3(std::min((D->nv + 1023) / 1024, 512)), bd, 0, s, d_cnt, D->nv, D->vox,
                       D->q_zero, counter);
    IMRT_HIP(hipGetLastError());
    IMRT_HIP(hipMemsetAsync(d_sums, 0, 2 * sizeof(unsigned long long), s));
  }
  {
    std::vector<int32_t> first(static_cast<size_t>(D->nb) + 3), tmp(kWindow);
    for (int w0 = 0; w0 < nq; w0 += kWindow) {
      const int w1 = std::min(nq, w0 + kWindow);
      int top = 0;
      for (int i = w0; i < w1; ++i) top = std::max(top, n[qrow[i]]);
      std::fill(first.begin(), first.begin() + top + 2, 0);
      for (int i = w0; i < w1; ++i) ++first[top - n[qrow[i]] + 1];
      for (int k = 1; k <= top; ++k) first[k] += first[k - 1];
      for (int i = w0; i < w1; ++i) tmp[first[top - n[qrow[i]]]++] = qrow[i];
      std::copy(tmp.begin(), tmp.begin() + (w1 - w0), qrow.begin() + w0);
    }
  }
  std::vector<int32_t> order(2 * static_cast<size_t>(nq) + 1);   // rows, first entries
  std::vector<int32_t> qn(nq);
  int64_t at = 0;
  for (int i = 0; i < nq; ++i) {
    qn[i] = n[qrow[i]];
    order[i] = qrow[i];
    order[static_cast<size_t>(nq) + i] = static_cast<int32_t>(at);
    at += qn[i];
  }
  order.back() = static_cast<int32_t>(at);
  const size_t ents = static_cast<size_t>(nent) + kQuadPad, vb = c16 ? 8 : 16;
  if ((rc = alloc(&ord.p, sizeof(int32_t) * order.size())) ||
      (rc = alloc(reinterpret_cast<void**>(&D->q_col), 2 * ents)) || (rc = alloc(&D->q_val, vb * ents)))
    return rc;
  auto* d_row = static_cast<int32_t*>(ord.p);
  unsigned long long bits[2] = {0, 0};
  const Drain drain{s};
  IMRT_HIP(hipMemcpyAsync(d_row, order.data(), sizeof(int32_t) * order.size(), hipMemcpyHostToDevice, s));
  IMRT_HIP(hipMemsetAsync(D->q_col + nent, 0, 2 * kQuadPad, s));
  IMRT_HIP(hipMemsetAsync(static_cast<char*>(D->q_val) + vb * nent, 0, vb * kQuadPad, s));
  const dim3 gf((nq + kThreads - 1) / kThreads);
  auto fill = [&](auto kernel, auto col, auto sum) {
    hipLaunchKernelGGL(kernel, gf, bd, 0, s, D->row_ptr, col, D->val, D->val16, D->nv, nq, d_row, d_row + nq, D->q_col,
                       D->q_val, d_sums);
    hipLaunchKernelGGL(sum, gc, bd, 0, s, D->col_ptr, D->cval, D->cval16, D->nb, d_sums);
  };
  if (D->storage == ST_F32) fill(quad_fill_kernel<ST_F32, int32_t>, D->col_idx, column_sum_kernel<ST_F32>);
  else if (D->storage == ST_BF16) fill(quad_fill_kernel<ST_BF16, uint16_t>, D->col16, column_sum_kernel<ST_BF16>);
  else fill(quad_fill_kernel<ST_F16, uint16_t>, D->col16, column_sum_kernel<ST_F16>);
  IMRT_HIP(hipGetLastError());
  IMRT_HIP(hipMemcpyAsync(bits, d_sums, sizeof(bits), hipMemcpyDeviceToHost, s));
  D->nent = nent;
  D->qn.swap(qn);
  D->qrow.swap(qrow);
  D->qgaps.swap(gaps);
  D->quad_epoch += 1;
  rc = place_quads(D);
  IMRT_HIP(hipStreamSynchronize(s));
  // (a little over the sums: they are rounded)
  D->q_rowsum = __builtin_bit_cast(double, bits[0]) * (1.0 + 1e-9);
  D->q_colsum = __builtin_bit_cast(double, bits[1]) * (1.0 + 1e-9);
  return rc;
}

// Waves get runs of quads of about equal cost; each wave's run is cut into
// blocks.  As in the wave forward, a matrix solved alone spreads over up to
// 16 waves of every compute unit, one with per-plan targets over fewer.
int place_quads(imrt_dose* D) {
  const int full = quad_full(D->storage), run = quad_run(D->storage), nq = static_cast<int>(D->qn.size());
  const std::vector<int32_t>& qn = D->qn;
  constexpr int kQuadCost = 8;   // of a quad beside its entries, in entries
  int64_t total = 0, slots = 0;
  for (int32_t n : qn) {
    total += n + kQuadCost;
    const int step = run * lanes_for(n, D->storage);
    slots += static_cast<int64_t>(step) * ((n + step - 1) / step);
  }
  // two steps a wave at least when alone, fwd_bpw blocks in shared dispatches
  const int64_t per = D->fwd_waves == 16 ? 128 : static_cast<int64_t>(full) * D->fwd_bpw;
  int64_t waves = std::min<int64_t>((slots + per - 1) / per, static_cast<int64_t>(16) * D->ctx->num_cu);
  // (the column sums of a pass have to fit the static scratch of the entry
  // point that allocates nothing)
  const int64_t groups = std::max<int64_t>(1, ((16 << 20) - (1 << 17)) / (8 * static_cast<int64_t>(D->nb)));
  waves = std::min(waves, groups * D->fwd_waves);
  waves = std::max<int64_t>(1, waves / 16 + (waves % 16 != 0)) * 16;
  if (waves > groups * D->fwd_waves) waves = std::max<int64_t>(16, groups * D->fwd_waves / 16 * 16);
  std::vector<int2> head;
  std::vector<uint2> rec;
  std::vector<int32_t> first(static_cast<size_t>(waves) + 1, 0);
  int32_t e0 = 0;
  auto block = [&](int flags, int q, int nqb, int L, int start, int count) {
    // nqb quads from q on (or entries [start, start + count) of one)
    int rel = 0;
    uint2 r[16];
    for (int g = 0; g < 16; ++g) r[g] = make_uint2(0, 0);
    for (int j = 0; j < nqb; ++j) {
      const int n = count > 0 ? count : qn[q + j];
      for (int g = j * L / 4; g < (j + 1) * L / 4; ++g)
        r[g] = make_uint2(static_cast<uint32_t>(rel) | (static_cast<uint32_t>(n) << 16),
                          static_cast<uint32_t>(D->qrow[q + j]));
      rel += n;
    }
    int e = 2;
    while ((1 << e) < L) ++e;
    head.push_back(make_int2(e0 + start, flags | (e << 8)));
    rec.insert(rec.end(), r, r + 16);
  };
  constexpr int kAll = kQuadFirst | kQuadDose | kQuadFinish | kQuadAdjoint;
  int q = 0;
  int64_t spent = 0;
  for (int64_t w = 0; w < waves; ++w) {
    first[w] = static_cast<int32_t>(head.size());
    int qe = q;
    const int64_t until = total * (w + 1) / waves;
    while (qe < nq && spent + (qn[qe] + kQuadCost) / 2 < until) spent += qn[qe++] + kQuadCost;
    if (w == waves - 1) qe = nq;
    while (q < qe) {
      if (qn[q] > full) {
        const int n = qn[q], parts = quad_parts_before(n, full);   // before the last one, which is full
        auto part = [&](int k) { return quad_part(n, full, parts, k); };
        for (int k = 0; k < parts; ++k)
          block(kQuadDose | (k == 0 ? kQuadFirst : 0), q, 1, 64, part(k), part(k + 1) - part(k));
        block(kQuadDose | kQuadFinish | kQuadAdjoint, q, 1, 64, n - full, full);
        for (int k = 0; k < parts; ++k) block(kQuadAdjoint, q, 1, 64, part(k), part(k + 1) - part(k));
        e0 += n;
        ++q;
        continue;
      }
      int c = 1, L = lanes_for(qn[q], D->storage);
      while (q + c < qe && qn[q + c] <= full) {
        const int Ln = std::max(L, lanes_for(qn[q + c], D->storage));
        if ((c + 1) * Ln > 64) break;
        L = Ln;
        ++c;
      }
      while (2 * c * L <= 64) L *= 2;
      block(kAll, q, c, L, 0, 0);
      for (int j = 0; j < c; ++j) e0 += qn[q + j];
      q += c;
    }
  }
  first[waves] = static_cast<int32_t>(head.size());
  int kmax = 1;
  for (int64_t w = 0; w < waves; ++w) kmax = std::max(kmax, first[w + 1] - first[w]);
  const size_t nblk = static_cast<size_t>(waves) * kmax;
  std::vector<uint2> ph(nblk, make_uint2(0, 0)), pr(nblk * 16, make_uint2(0, 0));
  for (int64_t w = 0; w < waves; ++w)
    for (int b = first[w]; b < first[w + 1]; ++b) {
      const size_t to = static_cast<size_t>(w) * kmax + (b - first[w]);
      ph[to] = make_uint2(static_cast<uint32_t>(head[b].x), static_cast<uint32_t>(head[b].y));
      std::copy(rec.begin() + 16 * static_cast<size_t>(b), rec.begin() + 16 * static_cast<size_t>(b) + 16,
                pr.begin() + 16 * to);
    }
  hipStream_t s = D->ctx->stream;
  if (D->q_head) IMRT_HIP(hipFree(D->q_head));
  D->q_head = nullptr;
  if (D->q_rec) IMRT_HIP(hipFree(D->q_rec));
  D->q_rec = nullptr;
  D->q_waves = 0;
  int rc;
  if ((rc = alloc(reinterpret_cast<void**>(&D->q_head), sizeof(uint2) * ph.size())) ||
      (rc = alloc(reinterpret_cast<void**>(&D->q_rec), sizeof(uint2) * pr.size())))
    return rc;
  IMRT_HIP(hipMemcpyAsync(D->q_head, ph.data(), sizeof(uint2) * ph.size(), hipMemcpyHostToDevice, s));
  IMRT_HIP(hipMemcpyAsync(D->q_rec, pr.data(), sizeof(uint2) * pr.size(), hipMemcpyHostToDevice, s));
  IMRT_HIP(hipStreamSynchronize(s));
  D->q_nblocks = static_cast<int32_t>(nblk);
  D->q_kmax = kmax;
  D->q_waves = static_cast<int32_t>(waves);
  return IMRT_OK;
}

}  // namespace

int build_quads(imrt_dose* D) {
  return quads_or_none(D, [&] { return make_quads(D); });
}

int partition_quads(imrt_dose* D) {
  return quads_or_none(D, [&] { return place_quads(D); });
}

}  // namespace imrt
