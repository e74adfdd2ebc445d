// Synthetic prostate-shaped phantom and its dose-deposition matrix D, built on
// the device.  D plays the role of the dose deposition coefficients of
// Section 2.1 (dose to voxel j from beamlet i at unit intensity); the paper
// takes it from a clinical dose engine, here a pencil-beam model stands in.
//
// Every float64 expression is evaluated in one fixed order with contraction
// off (this file is compiled with -ffp-contract=off as well), so the sparsity
// pattern is a deterministic function of the geometry:
//   voxel centre   p_a = (i_a + 0.5)*h - (n_a*h)/2
//   depth          -max over in-plane axes with dir_a != 0 of
//                  min((lo_a - p_a)/dir_a, (hi_a - p_a)/dir_a)
//   lateral        u = (-sin)*x + cos*y,  v = z
//   exponent       e = (mu*depth) + (((u-u_c)^2 + (v-v_c)^2) / ((2*sigma)*sigma))
//   kept           e <= e_min(beamlet) + log(1/tau), e_min over every grid voxel
//   value          float32(exp(-e))
// Beam angles' cosines/sines and log(1/tau) are computed once on the host.
//
// Unspecified tissue at twice the voxel size (Section 3.1): with
// coarse_normal, every aligned, complete 2x2x2 block of grid voxels that are
// all normal tissue becomes one voxel centred at
//   c_a = (2*b_a + 1)*h - (n_a*h)/2
// of structure "normal".  The voxels crossing the API are then the remaining
// grid voxels (grid index ascending) followed by the coarse voxels (block
// index bx + (nx/2)*(by + (ny/2)*bz) ascending).
#pragma clang fp contract(off)

#include <algorithm>
#include <cmath>
#include <vector>

#include "imrt_internal.h"

namespace imrt {
namespace {

struct Geo {
  int nx, ny, nz;
  int ngrid, nv;               // grid voxels; rows of D (the layout's voxels)
  int cx, cy;                  // coarse blocks per x row and per y column (nx/2, ny/2)
  double h, hx, hy;            // half extents (n*h)/2 in x and y
  double r_ptv, r_rectum, r_bladder;
  double mu, two_sig2;         // (2*sigma)*sigma
  double keep_log;             // log(1/tau)
  int nbeam;
};

struct BeamletDev {
  int32_t beam;
  int32_t pad;
  double u_c, v_c;
};

__device__ __forceinline__ double centre(int i, int n, double h) {
  return (static_cast<double>(i) + 0.5) * h - (static_cast<double>(n) * h) / 2.0;
}

__device__ __forceinline__ void voxel_xyz(const Geo& g, int j, double& x, double& y, double& z) {
  const int ix = j % g.nx;
  const int t = j / g.nx;
  const int iy = t % g.ny;
  const int iz = t / g.ny;
  x = centre(ix, g.nx, g.h);
  y = centre(iy, g.ny, g.h);
  z = centre(iz, g.nz, g.h);
}

__device__ __forceinline__ double coarse_centre(int b, int n, double h) {
  return (2.0 * static_cast<double>(b) + 1.0) * h - (static_cast<double>(n) * h) / 2.0;
}

__device__ __forceinline__ void depth_u(const Geo& g, double x, double y, double c, double s,
                                        double& depth, double& u) {
  double t = 0.0;
  bool have = false;
  if (c != 0.0) {
    t = fmin((-g.hx - x) / c, (g.hx - x) / c);
    have = true;
  }
  if (s != 0.0) {
    const double ty = fmin((-g.hy - y) / s, (g.hy - y) / s);
    t = have ? fmax(t, ty) : ty;
  }
  depth = -t;
  u = (-s) * x + c * y;
}

// Rows of D follow the internal voxel order: row p is the voxel with point
// code code[p] (grid voxel p itself when code is NULL).
__device__ __forceinline__ int code_of(const int32_t* code, int p) { return code ? code[p] : p; }

// Structure id of rows [0, n): coarse voxels are normal tissue.
__global__ __launch_bounds__(kThreads) void structure_kernel(Geo g, int n, const int32_t* code, uint8_t* sid) {
  const int p = blockIdx.x * kThreads + threadIdx.x;
  if (p >= n) return;
  const int c = code_of(code, p);
  if (c < 0) {
    sid[p] = 0;
    return;
  }
  double x, y, z;
  voxel_xyz(g, c, x, y, z);
  uint8_t s = 0;
  const double cb = g.r_ptv + g.r_bladder;
  const double dyb = y - cb;
  if ((x * x + dyb * dyb) + z * z <= g.r_bladder * g.r_bladder) s = 3;
  const double cr = -(g.r_ptv + g.r_rectum);
  const double dyr = y - cr;
  if (x * x + dyr * dyr <= g.r_rectum * g.r_rectum) s = 2;
  if ((x * x + y * y) + z * z <= g.r_ptv * g.r_ptv) s = 1;
  sid[p] = s;
}

// Voxel order of a uniform grid: tiles of 4 x 4 x 2 voxels in x, y, z order,
// inside a tile squares of 2 x 2 (cut tiles leave out what lies outside).
__device__ __forceinline__ int tile_rank(int x, int y, int z) {
  return (x & 1) | (y & 1) << 1 | (x & 2) << 1 | (y & 2) << 2 | z << 4;
}
__global__ __launch_bounds__(kThreads) void tile_order_kernel(int nx, int ny, int nz, int32_t* vox) {
  const int j = blockIdx.x * kThreads + threadIdx.x;
  if (j >= nx * ny * nz) return;
  const int x = j % nx, y = j / nx % ny, z = j / nx / ny;
  const int x0 = x & ~3, y0 = y & ~3, z0 = z & ~1;
  const int tx = min(4, nx - x0), ty = min(4, ny - y0), tz = min(2, nz - z0);
  const int own = tile_rank(x - x0, y - y0, z - z0);
  int rank = own;
  if (tx < 4 || ty < 4) {   // the places before it that the grid holds
    rank = 0;
    for (int i = 0; i < own; ++i)
      rank += (i & 1) + ((i >> 1) & 2) < tx && ((i >> 1) & 1) + ((i >> 2) & 2) < ty;
  }
  vox[nx * ny * z0 + nx * tz * y0 + ty * tz * x0 + rank] = j;
}

// Exclusive prefix sums of n counts: sums of runs of kScanRun, their prefix
// sums by one workgroup, then the runs.
constexpr int kScanRun = 16 * kThreads;

__global__ __launch_bounds__(kThreads) void scan_runs_kernel(const int32_t* counts, int n, long long* sums) {
  __shared__ long long red[kWaves];
  const int64_t i0 = static_cast<int64_t>(blockIdx.x) * kScanRun;
  long long s = 0;
  for (int64_t i = i0 + threadIdx.x; i < min(i0 + kScanRun, static_cast<int64_t>(n)); i += kThreads) s += counts[i];
  for (int d = 1; d < 64; d <<= 1) s += __shfl_xor(s, d);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0) {
    s = 0;
    for (int w = 0; w < kWaves; ++w) s += red[w];
    sums[blockIdx.x] = s;
  }
}

// sums[0..nrun) to their exclusive prefix sums, the total to sums[nrun].
__global__ __launch_bounds__(64) void scan_sums_kernel(long long* sums, int nrun) {
  const int lane = threadIdx.x;
  long long base = 0;
  for (int i0 = 0; i0 < nrun; i0 += 64) {
    const long long v = i0 + lane < nrun ? sums[i0 + lane] : 0;
    long long t = v;
    for (int d = 1; d < 64; d <<= 1) {
      const long long u = __shfl_up(t, d);
      if (lane >= d) t += u;
    }
    if (i0 + lane < nrun) sums[i0 + lane] = base + t - v;
    base += __shfl(t, 63);
  }
  if (lane == 0) sums[nrun] = base;
}

__global__ __launch_bounds__(kThreads) void scan_fill_kernel(const int32_t* counts, int n, const long long* sums,
                                                             int nrun, int32_t* ptr) {
  __shared__ int32_t part[kWaves];
  const int64_t i0 = static_cast<int64_t>(blockIdx.x) * kScanRun + 16 * threadIdx.x;
  int32_t v[16], s = 0;
  for (int u = 0; u < 16; ++u) {
    v[u] = i0 + u < n ? counts[i0 + u] : 0;
    s += v[u];
  }
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  int32_t t = s;
  for (int d = 1; d < 64; d <<= 1) {
    const int32_t u = __shfl_up(t, d);
    if (lane >= d) t += u;
  }
  if (lane == 63) part[w] = t;
  __syncthreads();
  int32_t at = static_cast<int32_t>(sums[blockIdx.x]) + t - s;
  for (int k = 0; k < w; ++k) at += part[k];
  for (int u = 0; u < 16; ++u) {
    if (i0 + u < n) ptr[i0 + u] = at;
    at += v[u];
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) ptr[n] = static_cast<int32_t>(sums[nrun]);
}

// ---- tables of the builder ----------------------------------------------------------
// A beam is parallel to the x-y plane, so a voxel's depth and lateral
// coordinate depend on (x, y) alone.  plane[beam][t] holds (mu*depth, u) of
// in-plane position t: t = ix + nx*iy for the grid, then nx*ny + bx + cx*by
// for coarse blocks.  The four float64 divisions of a depth are done once
// per beam and position instead of once per (voxel, beamlet) pair.
struct Point {
  int t;      // in-plane position
  double z;
};

__device__ __forceinline__ Point point_of(const Geo& g, int c) {
  Point p;
  if (c >= 0) {
    const int iz = c / (g.nx * g.ny);
    p.t = c - iz * (g.nx * g.ny);
    p.z = centre(iz, g.nz, g.h);
  } else {
    const int b = -1 - c;
    const int bz = b / (g.cx * g.cy);
    p.t = g.nx * g.ny + (b - bz * (g.cx * g.cy));
    p.z = coarse_centre(bz, g.nz, g.h);
  }
  return p;
}

__device__ __forceinline__ double exponent(const Geo& g, double mu_depth, double u, double z, double uc, double vc) {
  const double du = u - uc;
  const double dv = z - vc;
  const double r2 = du * du + dv * dv;
  return mu_depth + (r2 / g.two_sig2);
}

__global__ __launch_bounds__(kThreads) void plane_kernel(Geo g, const double2* dirs, int nt, double2* plane) {
  const int blocks = (nt + kThreads - 1) / kThreads, beam = blockIdx.x / blocks;
  const int t = (blockIdx.x - beam * blocks) * kThreads + threadIdx.x;
  if (t >= nt) return;
  double x, y;
  if (t < g.nx * g.ny) {
    x = centre(t % g.nx, g.nx, g.h);
    y = centre(t / g.nx, g.ny, g.h);
  } else {
    const int b = t - g.nx * g.ny;
    x = coarse_centre(b % g.cx, g.nx, g.h);
    y = coarse_centre(b / g.cx, g.ny, g.h);
  }
  const double2 d = dirs[beam];
  double depth, u;
  depth_u(g, x, y, d.x, d.y, depth, u);
  plane[static_cast<size_t>(beam) * nt + t] = make_double2(g.mu * depth, u);
}

// One workgroup per beamlet: minimum exponent over every grid voxel.  Every
// operation after dv = z - v_c rounds monotonically in dv*dv, so at a fixed
// (x, y) the smallest exponent is the one at the z with the smallest
// rounded dv*dv: nx*ny evaluations instead of nx*ny*nz, the same float64
// minimum bit for bit.  Also the largest minimum of all beamlets (as the bit
// pattern of a nonnegative double), which bounds every beamlet's reach.
// The build of the paper-scale matrix (1.33 M voxels x 2,088 beamlets) took
// 11.6 ms here when every voxel was evaluated, 0.05 ms now.
__global__ __launch_bounds__(kThreads) void emin_kernel(Geo g, const BeamletDev* bl, const double2* plane, int nt,
                                                        double* emin, unsigned long long* emin_max) {
  const int i = blockIdx.x;
  const BeamletDev b = bl[i];
  const double2* pl = plane + static_cast<size_t>(b.beam) * nt;
  __shared__ double sh[kThreads];
  auto min_all = [&](double m) {
    sh[threadIdx.x] = m;
    __syncthreads();
    for (int s = kThreads / 2; s > 0; s >>= 1) {
      if (threadIdx.x < s) sh[threadIdx.x] = fmin(sh[threadIdx.x], sh[threadIdx.x + s]);
      __syncthreads();
    }
    const double r = sh[0];
    __syncthreads();
    return r;
  };
  double m = INFINITY;
  for (int iz = threadIdx.x; iz < g.nz; iz += kThreads) {
    const double dv = centre(iz, g.nz, g.h) - b.v_c;
    m = fmin(m, dv * dv);
  }
  const double dv2 = min_all(m);
  m = INFINITY;
  for (int t = threadIdx.x; t < g.nx * g.ny; t += kThreads) {
    const double2 p = pl[t];
    const double du = p.y - b.u_c;
    const double r2 = du * du + dv2;
    m = fmin(m, p.x + (r2 / g.two_sig2));
  }
  m = min_all(m);
  if (threadIdx.x == 0) {
    emin[i] = m;
    atomicMax(emin_max, static_cast<unsigned long long>(__double_as_longlong(fmax(m, 0.0))));
  }
}

// ---- culling --------------------------------------------------------------------------
// A voxel can only be kept when r^2 <= 2 sigma^2 (limit - mu*depth), and
// mu*depth >= 0.  The bound is widened by far more than the rounding of the
// exponent, so it never drops a voxel that the exact test keeps; every voxel
// it lets through still takes the exact test.
__device__ __forceinline__ double reach_sq(const Geo& g, double limit) {
  return g.two_sig2 * (limit + 1e-6 * (1.0 + fabs(limit)));
}

// Boxes (u and z ranges) of runs of kRun consecutive rows, and of kRun runs:
// box level 0 per beam and run, level 1 per beam and group of kRun runs.
constexpr int kRun = 64;

__device__ __forceinline__ double wave_min(double v) {
  for (int off = 32; off > 0; off >>= 1) v = fmin(v, __shfl_xor(v, off, 64));
  return v;
}
__device__ __forceinline__ double wave_max(double v) {
  for (int off = 32; off > 0; off >>= 1) v = fmax(v, __shfl_xor(v, off, 64));
  return v;
}

// One wave per run.
__global__ __launch_bounds__(kThreads) void run_box_kernel(Geo g, const int32_t* code, const double2* plane, int nt,
                                                           int nrun, double2* ubox, double2* zbox) {
  const int q = blockIdx.x * kWaves + static_cast<int>(threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (q >= nrun) return;
  const int p = min(q * kRun + lane, g.nv - 1);   // (the last run repeats its last row)
  const Point pt = point_of(g, code_of(code, p));
  const double zl = wave_min(pt.z), zh = wave_max(pt.z);
  if (lane == 0) zbox[q] = make_double2(zl, zh);
  for (int b = 0; b < g.nbeam; ++b) {
    const double u = plane[static_cast<size_t>(b) * nt + pt.t].y;
    const double ul = wave_min(u), uh = wave_max(u);
    if (lane == 0) ubox[static_cast<size_t>(b) * nrun + q] = make_double2(ul, uh);
  }
}

// One wave per group of runs of each beam's u boxes, then of the z boxes (b == nbeam).
__global__ __launch_bounds__(kThreads) void group_box_kernel(int nbeam, int nrun, int ngroup, const double2* ubox,
                                                             const double2* zbox, double2* gubox, double2* gzbox) {
  const int blocks = (ngroup + kWaves - 1) / kWaves, b = blockIdx.x / blocks;
  const int s = (blockIdx.x - b * blocks) * kWaves + static_cast<int>(threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (s >= ngroup) return;
  const double2* in = b < nbeam ? ubox + static_cast<size_t>(b) * nrun : zbox;
  const double2 v = in[min(s * kRun + lane, nrun - 1)];
  const double lo = wave_min(v.x), hi = wave_max(v.y);
  if (lane == 0) (b < nbeam ? gubox + static_cast<size_t>(b) * ngroup : gzbox)[s] = make_double2(lo, hi);
}

__device__ __forceinline__ bool box_near(const double2 u, const double2 z, const BeamletDev& b, double r2) {
  const double du = fmax(0.0, fmax(u.x - b.u_c, b.u_c - u.y));
  const double dv = fmax(0.0, fmax(z.x - b.v_c, b.v_c - z.y));
  return !(du * du + dv * dv > r2);   // (a bound that is not a number culls nothing)
}

// One workgroup per beamlet: ordered compaction of the kept voxels (CSC).
// With FILL false only the count is produced.  The runs of rows near the
// beamlet are listed in row order in LDS (groups of runs first, kGroups
// groups at a time), each wave takes a contiguous quarter of the list, and
// the kept rows' ballots of that list give every wave its place in the
// column.  What bounds it: the dependent loads of a run (code, plane entry),
// hidden by eight workgroups a compute unit.  A pass over every (voxel,
// beamlet) pair took 14.0 ms at paper scale, the near runs 0.11 ms (count)
// and 0.26 ms (fill).
constexpr int kGroups = 16;   // groups of runs listed at a time: 1,024 runs, 12 KB of LDS

template <bool FILL>
__global__ __launch_bounds__(kThreads) void column_kernel(Geo g, const int32_t* code, const BeamletDev* bl,
                                                          const double2* plane, int nt, const double* emin, int nrun,
                                                          int ngroup, const double2* ubox, const double2* zbox,
                                                          const double2* gubox, const double2* gzbox, int32_t* counts,
                                                          const int32_t* col_ptr, int32_t* row_idx, float* cval) {
  const int i = blockIdx.x;
  const BeamletDev b = bl[i];
  const double limit = emin[i] + g.keep_log;
  const double r2 = reach_sq(g, limit);
  const double2* pl = plane + static_cast<size_t>(b.beam) * nt;
  ubox += static_cast<size_t>(b.beam) * nrun;
  gubox += static_cast<size_t>(b.beam) * ngroup;
  __shared__ int near_group[kThreads];
  __shared__ unsigned long long group_mask[kThreads / 64];
  __shared__ unsigned long long run_mask[kGroups];
  __shared__ int list[kGroups * kRun];
  __shared__ unsigned long long keep_mask[kGroups * kRun];
  __shared__ int wave_cnt[kWaves];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const unsigned long long below = (1ull << lane) - 1ull;
  int base = FILL ? col_ptr[i] : 0;
  for (int s0 = 0; s0 < ngroup; s0 += kThreads) {
    // near groups of this window, in order
    const int s = s0 + threadIdx.x;
    const bool gn = s < ngroup && box_near(gubox[s], gzbox[s], b, r2);
    const unsigned long long gm = __ballot(gn);
    if (lane == 0) group_mask[w] = gm;
    __syncthreads();
    int at = __popcll(gm & below), ng = 0;
    for (int k = 0; k < kWaves; ++k) {
      const int n = __popcll(group_mask[k]);
      at += k < w ? n : 0;
      ng += n;
    }
    if (gn) near_group[at] = s;
    __syncthreads();
    for (int g0 = 0; g0 < ng; g0 += kGroups) {
      const int gn_here = min(kGroups, ng - g0);
      // near runs of these groups, in order
      for (int k = w; k < gn_here; k += kWaves) {
        const int q = near_group[g0 + k] * kRun + lane;
        const bool rn = q < nrun && box_near(ubox[q], zbox[q], b, r2);
        const unsigned long long m = __ballot(rn);
        if (lane == 0) run_mask[k] = m;
      }
      __syncthreads();
      int nlist = 0;
      for (int k = 0; k < gn_here; ++k) {
        const unsigned long long m = run_mask[k];
        if ((k & (kWaves - 1)) == w && (m >> lane & 1ull))
          list[nlist + __popcll(m & below)] = near_group[g0 + k] * kRun + lane;
        nlist += __popcll(m);
      }
      __syncthreads();
      // this wave's quarter of the list
      const int l0 = w * nlist / kWaves, l1 = (w + 1) * nlist / kWaves;
      int cnt = 0;
      for (int l = l0; l < l1; ++l) {
        const int p = list[l] * kRun + lane;
        bool keep = false;
        if (p < g.nv) {
          const Point pt = point_of(g, code_of(code, p));
          const double2 du = pl[pt.t];
          keep = exponent(g, du.x, du.y, pt.z, b.u_c, b.v_c) <= limit;
        }
        const unsigned long long m = __ballot(keep);
        if (FILL && lane == 0) keep_mask[l] = m;
        cnt += __popcll(m);
      }
      if (lane == 0) wave_cnt[w] = cnt;
      __syncthreads();
      int before = base, total = 0;
      for (int k = 0; k < kWaves; ++k) {
        before += k < w ? wave_cnt[k] : 0;
        total += wave_cnt[k];
      }
      if (FILL) {
        for (int l = l0; l < l1; ++l) {
          const unsigned long long m = keep_mask[l];
          if (m >> lane & 1ull) {
            const int p = list[l] * kRun + lane;
            const Point pt = point_of(g, code_of(code, p));
            const double2 du = pl[pt.t];
            const double e = exponent(g, du.x, du.y, pt.z, b.u_c, b.v_c);
            const int64_t pos = csc_slot(before + __popcll(m & below));
            row_idx[pos] = p;
            cval[pos] = static_cast<float>(exp(-e));
          }
          before += __popcll(m);
        }
      }
      base += total;
      __syncthreads();   // the lists are rewritten
    }
  }
  if (!FILL && threadIdx.x == 0) counts[i] = base;
}

// One thread per voxel: kept beamlets in ascending column order (CSR).  Every
// beam has the same beamlets: lateral index m in [-kmax, kmax) ascending,
// for each the axial indices lat[m + kmax] = {first n, count, index of the
// first}.  Only the (m, n) rectangle within the reach of the voxel is
// tested.  2.2 ms a pass at paper scale with every beamlet tested, now 0.18 ms
// (count) and 0.30 ms (fill).
template <bool FILL>
__global__ __launch_bounds__(kThreads) void row_kernel(Geo g, const int32_t* code, const BeamletDev* bl,
                                                       const int32_t* beam_first, const int4* lat, int kmax, double w,
                                                       const double2* plane, int nt, const double* emin,
                                                       const unsigned long long* emin_max, int32_t* counts,
                                                       const int32_t* row_ptr, int32_t* col_idx, float* val) {
  const int p = blockIdx.x * kThreads + threadIdx.x;
  if (p >= g.nv) return;
  const Point pt = point_of(g, code_of(code, p));
  const double top = __longlong_as_double(static_cast<long long>(*emin_max)) + g.keep_log;
  int pos = FILL ? row_ptr[p] : 0;
  for (int beam = 0; beam < g.nbeam; ++beam) {
    const double2 du = plane[static_cast<size_t>(beam) * nt + pt.t];
    const double r2 = reach_sq(g, top) - g.two_sig2 * du.x;
    if (r2 < 0.0) continue;
    // (m + 0.5) w within the reach of u: one index of margin on either side
    const double r = sqrt(r2);
    const int m0 = static_cast<int>(fmax(floor((du.y - r) / w) - 1.0, static_cast<double>(-kmax)));
    const int m1 = static_cast<int>(fmin(floor((du.y + r) / w) + 1.0, static_cast<double>(kmax - 1)));
    const int nlo = static_cast<int>(fmax(floor((pt.z - r) / w) - 1.0, static_cast<double>(-kmax)));
    const int nhi = static_cast<int>(fmin(floor((pt.z + r) / w) + 1.0, static_cast<double>(kmax - 1)));
    for (int m = m0; m <= m1; ++m) {
      const int4 L = lat[m + kmax];
      const int i0 = beam_first[beam] + L.z - L.x;   // index of axial index n: i0 + n
      const int n1 = min(nhi, L.x + L.y - 1);
      for (int n = max(nlo, L.x); n <= n1; ++n) {
        const int i = i0 + n;
        const double e = exponent(g, du.x, du.y, pt.z, bl[i].u_c, bl[i].v_c);
        if (e <= emin[i] + g.keep_log) {
          if (FILL) {
            col_idx[pos] = i;
            val[pos] = static_cast<float>(exp(-e));
          }
          ++pos;
        }
      }
    }
  }
  if (!FILL) counts[p] = pos;
}

struct DevBuf {
  void* p = nullptr;
  ~DevBuf() {
    if (p) (void)hipFree(p);
  }
};

// ---- 16-bit storage ---------------------------------------------------------------
// Code of a nonnegative float64 quotient v = D_ij / s_i in bfloat16 (8
// significand bits, smallest normal exponent -126) or binary16 (11, -14):
// with 2^e <= v < 2^(e+1), the quantum is 2^(max(e, emin) - p + 1); v divided
// by it is exact, rint rounds it to nearest with ties to even, and the rounded
// value is representable in float32 and in the 16-bit format.  The float64
// quotient of two float32 numbers never lands on (or across) a tie of these
// formats unless the exact quotient does, so this is the rounding of the
// exact quotient.
template <int ST>
__device__ uint16_t code16(double v) {
  if (!(v > 0.0)) return 0;
  constexpr int p = (ST == ST_BF16) ? 8 : 11;
  constexpr int emin = (ST == ST_BF16) ? -126 : -14;
  int E = 0;
  (void)frexp(v, &E);   // v = m 2^E, 1/2 <= m < 1
  const int qe = max(E - 1, emin) - (p - 1);
  const float f = static_cast<float>(ldexp(rint(ldexp(v, -qe)), qe));
  if (ST == ST_BF16) return static_cast<uint16_t>(__float_as_uint(f) >> 16);
  return __builtin_bit_cast(uint16_t, static_cast<_Float16>(f));
}

// One wave per column: s = the largest value (1 when none is positive), then
// the codes of the column's entries in CSC slot order.
template <int ST>
__global__ __launch_bounds__(kThreads) void quantize_columns_kernel(const int32_t* col_ptr, const float* cval,
                                                                     int nb, float* scale, uint16_t* cval16) {
  const int c = blockIdx.x * kWaves + static_cast<int>(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (c >= nb) return;
  const int k0 = col_ptr[c], k1 = col_ptr[c + 1];
  float m = 0.0f;
  for (int k = k0 + lane; k < k1; k += 64) m = fmaxf(m, cval[csc_slot(k)]);
  for (int off = 32; off > 0; off >>= 1) m = fmaxf(m, __shfl_xor(m, off, 64));
  const float sc = (m > 0.0f) ? m : 1.0f;
  if (lane == 0) scale[c] = sc;
  for (int k = k0 + lane; k < k1; k += 64) {
    const int64_t slot = csc_slot(k);
    cval16[slot] = code16<ST>(static_cast<double>(cval[slot]) / static_cast<double>(sc));
  }
}

// CSR codes and 16-bit column indices.
template <int ST>
__global__ __launch_bounds__(kThreads) void quantize_rows_kernel(const int32_t* col_idx, const float* val, int64_t nnz,
                                                                  const float* scale, uint16_t* col16,
                                                                  uint16_t* val16) {
  for (int64_t k = blockIdx.x * static_cast<int64_t>(kThreads) + threadIdx.x; k < nnz;
       k += static_cast<int64_t>(gridDim.x) * kThreads) {
    const int c = col_idx[k];
    col16[k] = static_cast<uint16_t>(c);
    val16[k] = code16<ST>(static_cast<double>(val[k]) / static_cast<double>(scale[c]));
  }
}

__global__ __launch_bounds__(kThreads) void narrow_columns_kernel(const int32_t* col_idx, int64_t nnz,
                                                                   uint16_t* col16) {
  for (int64_t k = blockIdx.x * static_cast<int64_t>(kThreads) + threadIdx.x; k < nnz;
       k += static_cast<int64_t>(gridDim.x) * kThreads)
    col16[k] = static_cast<uint16_t>(col_idx[k]);
}

// float32 storage read by the forward pass through 16-bit column indices
// (nb <= 65536): a 16-bit copy of the CSR column indices beside the 32-bit
// ones, which the other passes and the export keep using.
int narrow_columns(imrt_dose* D) {
  const size_t nz = static_cast<size_t>(D->nnz) + kPad;
  const hipError_t e = hipMalloc(reinterpret_cast<void**>(&D->col16), 2 * nz);
  if (e == hipErrorOutOfMemory) return set_error(IMRT_ENOMEM, "hipMalloc: out of device memory");
  if (e != hipSuccess) return hip_error(e, "hipMalloc(16-bit column indices)");
  hipStream_t s = D->ctx->stream;
  IMRT_HIP(hipMemsetAsync(D->col16, 0, 2 * nz, s));
  const int gr = static_cast<int>(std::max<int64_t>(1, std::min<int64_t>((D->nnz + kThreads - 1) / kThreads, 8192)));
  hipLaunchKernelGGL(narrow_columns_kernel, dim3(gr), dim3(kThreads), 0, s, D->col_idx, D->nnz, D->col16);
  IMRT_HIP(hipGetLastError());
  IMRT_HIP(hipStreamSynchronize(s));
  return IMRT_OK;
}

}  // namespace

int store16(imrt_dose* D, int storage) {
  if (storage == ST_F32) return D->fwd_st == ST_F32C16 ? narrow_columns(D) : IMRT_OK;
  if (storage != ST_BF16 && storage != ST_F16) return set_error(IMRT_EINVAL, "unknown storage");
  if (D->nb > 65536) return set_error(IMRT_EUNSUPPORTED, "16-bit storage needs nb <= 65536 (16-bit column indices)");
  const size_t nz = static_cast<size_t>(D->nnz) + kPad, nzc = csc_alloc(D->nnz);
  auto alloc = [](void** p, size_t bytes) -> int {
    const hipError_t e = hipMalloc(p, bytes < 1 ? 1 : bytes);
    if (e == hipErrorOutOfMemory) return set_error(IMRT_ENOMEM, "hipMalloc: out of device memory");
    if (e != hipSuccess) return hip_error(e, "hipMalloc(16-bit storage)");
    return IMRT_OK;
  };
  int rc;
  if ((rc = alloc(reinterpret_cast<void**>(&D->col_scale), sizeof(float) * std::max(D->nb, 1))) ||
      (rc = alloc(reinterpret_cast<void**>(&D->col16), 2 * nz)) ||
      (rc = alloc(reinterpret_cast<void**>(&D->val16), 2 * nz)) ||
      (rc = alloc(reinterpret_cast<void**>(&D->cval16), 2 * nzc)))
    return rc;
  hipStream_t s = D->ctx->stream;
  IMRT_HIP(hipMemsetAsync(D->col16, 0, 2 * nz, s));
  IMRT_HIP(hipMemsetAsync(D->val16, 0, 2 * nz, s));
  IMRT_HIP(hipMemsetAsync(D->cval16, 0, 2 * nzc, s));
  const int gc = std::max(1, (D->nb + kWaves - 1) / kWaves);
  const int gr = static_cast<int>(std::max<int64_t>(1, std::min<int64_t>((D->nnz + kThreads - 1) / kThreads, 8192)));
  if (storage == ST_BF16) {
    hipLaunchKernelGGL(quantize_columns_kernel<ST_BF16>, dim3(gc), dim3(kThreads), 0, s, D->col_ptr, D->cval, D->nb,
                       D->col_scale, D->cval16);
    hipLaunchKernelGGL(quantize_rows_kernel<ST_BF16>, dim3(gr), dim3(kThreads), 0, s, D->col_idx, D->val, D->nnz,
                       D->col_scale, D->col16, D->val16);
  } else {
    hipLaunchKernelGGL(quantize_columns_kernel<ST_F16>, dim3(gc), dim3(kThreads), 0, s, D->col_ptr, D->cval, D->nb,
                       D->col_scale, D->cval16);
    hipLaunchKernelGGL(quantize_rows_kernel<ST_F16>, dim3(gr), dim3(kThreads), 0, s, D->col_idx, D->val, D->nnz,
                       D->col_scale, D->col16, D->val16);
  }
  IMRT_HIP(hipGetLastError());
  IMRT_HIP(hipStreamSynchronize(s));
  // the float32 values and indices are not kept
  IMRT_HIP(hipFree(D->col_idx));
  IMRT_HIP(hipFree(D->val));
  IMRT_HIP(hipFree(D->cval));
  D->col_idx = nullptr;
  D->val = nullptr;
  D->cval = nullptr;
  D->storage = storage;
  return IMRT_OK;
}

int build_phantom(imrt_ctx* ctx, const imrt_geometry* G, imrt_dose* D) {
  if (G->nx <= 0 || G->ny <= 0 || G->nz <= 0 || G->n_beams <= 0)
    return set_error(IMRT_EINVAL, "geometry: grid sizes and beam count must be positive");
  const int64_t nv64 = static_cast<int64_t>(G->nx) * G->ny * G->nz;
  if (nv64 >= (int64_t(1) << 31)) return set_error(IMRT_EINVAL, "geometry: too many voxels");
  if (!(G->h > 0) || !(G->beamlet > 0) || !(G->sigma > 0) || !(G->tau > 0 && G->tau <= 1) ||
      !(G->mu >= 0) || !(G->r_ptv > 0) || !(G->r_rectum >= 0) || !(G->r_bladder >= 0) || !(G->margin >= 0))
    return set_error(IMRT_EINVAL, "geometry: lengths, sigma, tau or mu out of range");
  if (G->coarse_normal != 0 && G->coarse_normal != 1) return set_error(IMRT_EINVAL, "geometry: coarse_normal must be 0 or 1");
  const int ngrid = static_cast<int>(nv64);

  // Beam directions and beamlets on the host (libm cos/sin, exact integer scans).
  std::vector<double2> dirs(G->n_beams);
  for (int b = 0; b < G->n_beams; ++b) {
    const double theta = (2.0 * M_PI * b) / G->n_beams;
    dirs[b] = make_double2(std::cos(theta), std::sin(theta));
  }
  const double w = G->beamlet;
  const double reach = G->r_ptv + G->margin;
  const int kmax = static_cast<int>(std::ceil(reach / w)) + 1;
  std::vector<BeamletDev> bls;
  std::vector<int32_t> beam_first(G->n_beams + 1, 0);
  std::vector<int4> lat(2 * static_cast<size_t>(kmax), make_int4(0, 0, 0, 0));   // the same for every beam
  for (int b = 0; b < G->n_beams; ++b) {
    beam_first[b] = static_cast<int32_t>(bls.size());
    for (int m = -kmax; m < kmax; ++m) {
      const double lo_u = m * w, hi_u = (m + 1) * w;
      const double cu = std::min(std::max(0.0, lo_u), hi_u);
      for (int n = -kmax; n < kmax; ++n) {
        const double lo_v = n * w, hi_v = (n + 1) * w;
        const double cv = std::min(std::max(0.0, lo_v), hi_v);
        if (cu * cu + cv * cv <= reach * reach) {
          if (b == 0) {
            int4& L = lat[m + kmax];
            if (L.y == 0) L = make_int4(n, 0, static_cast<int>(bls.size()), 0);
            L.y += 1;
          }
          bls.push_back({b, 0, (m + 0.5) * w, (n + 0.5) * w});
        }
      }
    }
  }
  beam_first[G->n_beams] = static_cast<int32_t>(bls.size());
  const int nb = static_cast<int>(bls.size());
  if (nb == 0) return set_error(IMRT_EINVAL, "geometry: no beamlets");

  Geo g;
  g.nx = G->nx; g.ny = G->ny; g.nz = G->nz;
  g.ngrid = ngrid;
  g.nv = ngrid;
  g.cx = G->nx / 2;
  g.cy = G->ny / 2;
  g.h = G->h;
  g.hx = (static_cast<double>(G->nx) * G->h) / 2.0;
  g.hy = (static_cast<double>(G->ny) * G->h) / 2.0;
  g.r_ptv = G->r_ptv; g.r_rectum = G->r_rectum; g.r_bladder = G->r_bladder;
  g.mu = G->mu;
  g.two_sig2 = (2.0 * G->sigma) * G->sigma;
  g.keep_log = std::log(1.0 / G->tau);
  g.nbeam = G->n_beams;

  hipStream_t s = ctx->stream;
  (void)hipGetLastError();  // drop an error left by an unrelated earlier call
  DevBuf d_bl, d_first, d_dirs, d_emin, d_cnt_c, d_cnt_r, d_code;
  IMRT_HIP(hipMalloc(&d_bl.p, sizeof(BeamletDev) * nb));
  IMRT_HIP(hipMalloc(&d_first.p, sizeof(int32_t) * (G->n_beams + 1)));
  IMRT_HIP(hipMalloc(&d_dirs.p, sizeof(double2) * G->n_beams));
  IMRT_HIP(hipMalloc(&d_emin.p, sizeof(double) * nb));
  IMRT_HIP(hipMalloc(&d_cnt_c.p, sizeof(int32_t) * nb));
  IMRT_HIP(hipMemcpyAsync(d_bl.p, bls.data(), sizeof(BeamletDev) * nb, hipMemcpyHostToDevice, s));
  IMRT_HIP(hipMemcpyAsync(d_first.p, beam_first.data(), sizeof(int32_t) * (G->n_beams + 1),
                          hipMemcpyHostToDevice, s));
  IMRT_HIP(hipMemcpyAsync(d_dirs.p, dirs.data(), sizeof(double2) * G->n_beams, hipMemcpyHostToDevice, s));

  // Voxel layout.  api_code[a] is the point code of the voxel with API index
  // a (empty for a uniform grid, where the API index is the grid index);
  // fine_api and block_api give the API index of a grid voxel and of a
  // coarse block (-1: merged into a block, or not coarse).
  std::vector<int32_t> api_code, fine_api, block_api;
  int nv = ngrid;
  if (G->coarse_normal) {
    DevBuf d_gsid;
    IMRT_HIP(hipMalloc(&d_gsid.p, static_cast<size_t>(ngrid)));
    hipLaunchKernelGGL(structure_kernel, dim3((ngrid + kThreads - 1) / kThreads), dim3(kThreads), 0, s, g, ngrid,
                       static_cast<const int32_t*>(nullptr), static_cast<uint8_t*>(d_gsid.p));
    IMRT_HIP(hipGetLastError());
    std::vector<uint8_t> gsid(static_cast<size_t>(ngrid));
    IMRT_HIP(hipMemcpyAsync(gsid.data(), d_gsid.p, static_cast<size_t>(ngrid), hipMemcpyDeviceToHost, s));
    IMRT_HIP(hipStreamSynchronize(s));
    const int cx = g.cx, cy = g.cy, cz = G->nz / 2;
    std::vector<uint8_t> merged(static_cast<size_t>(ngrid), 0);
    std::vector<int32_t> blocks;
    block_api.assign(static_cast<size_t>(cx) * cy * cz, -1);
    for (int bz = 0; bz < cz; ++bz)
      for (int by = 0; by < cy; ++by)
        for (int bx = 0; bx < cx; ++bx) {
          bool normal = true;
          for (int d = 0; d < 8 && normal; ++d) {
            const int j = (2 * bx + (d & 1)) + G->nx * ((2 * by + ((d >> 1) & 1)) + G->ny * (2 * bz + (d >> 2)));
            normal = gsid[j] == 0;
          }
          if (!normal) continue;
          blocks.push_back(bx + cx * (by + cy * bz));
          for (int d = 0; d < 8; ++d)
            merged[(2 * bx + (d & 1)) + G->nx * ((2 * by + ((d >> 1) & 1)) + G->ny * (2 * bz + (d >> 2)))] = 1;
        }
    fine_api.assign(static_cast<size_t>(ngrid), -1);
    api_code.reserve(static_cast<size_t>(ngrid));
    for (int j = 0; j < ngrid; ++j)
      if (!merged[j]) {
        fine_api[j] = static_cast<int32_t>(api_code.size());
        api_code.push_back(j);
      }
    for (int32_t b : blocks) {
      block_api[b] = static_cast<int32_t>(api_code.size());
      api_code.push_back(-1 - b);
    }
    nv = static_cast<int>(api_code.size());
  }
  g.nv = nv;

  // Internal voxel order: tiles of 4 x 4 x 2 grid voxels (tiles in x, y, z
  // order; a tile's coarse voxels after its grid voxels; inside a tile
  // squares of 2 x 2 voxels, the quads of the one-read pass: of all groups of
  // four they share the most columns, 0.83 of a quad's entries at the paper's
  // scale against 0.79 for four voxels along x), so that the voxels a beamlet crosses sit close together in
  // memory whatever the beam direction.  Row p of D is the voxel with API
  // index vox[p] and point code codes[p].
  std::vector<int32_t> codes;
  if (ctx->tune.voxel_tiles && api_code.empty()) {
    // the uniform grid's order is a closed form, and its point codes are the
    // API indices: made on the device (on the host it took 2.2 ms of a
    // 1.33 M voxel matrix's build)
    IMRT_HIP(hipMalloc(&D->vox, sizeof(int32_t) * nv));
    hipLaunchKernelGGL(tile_order_kernel, dim3((nv + kThreads - 1) / kThreads), dim3(kThreads), 0, s, G->nx, G->ny,
                       G->nz, D->vox);
    IMRT_HIP(hipGetLastError());
  } else if (ctx->tune.voxel_tiles) {
    constexpr int tx = 4, ty = 4, tz = 2;
    D->vox_host.resize(static_cast<size_t>(nv));
    codes.resize(static_cast<size_t>(nv));
    int64_t p = 0;
    for (int z0 = 0; z0 < G->nz; z0 += tz)
      for (int y0 = 0; y0 < G->ny; y0 += ty)
        for (int x0 = 0; x0 < G->nx; x0 += tx) {
          for (int i = 0; i < tx * ty * tz; ++i) {
            const int x = x0 + (i & 1) + ((i >> 1) & 2), y = y0 + ((i >> 1) & 1) + ((i >> 2) & 2), z = z0 + (i >> 4);
            if (x >= G->nx || y >= G->ny || z >= G->nz) continue;
            const int j = x + G->nx * (y + G->ny * z);
            const int a = fine_api[j];
            if (a < 0) continue;
            if (p >= nv) return set_error(IMRT_EINVAL, "internal: voxel tiles overrun the layout");
            D->vox_host[p] = a;
            codes[p] = j;
            ++p;
          }
          const int bz = z0 / 2;
          if (bz >= G->nz / 2) continue;
          for (int by = y0 / 2; by < std::min(y0 / 2 + ty / 2, g.cy); ++by)
            for (int bx = x0 / 2; bx < std::min(x0 / 2 + tx / 2, g.cx); ++bx) {
              const int b = bx + g.cx * (by + g.cy * bz);
              const int a = block_api[b];
              if (a < 0) continue;
              if (p >= nv) return set_error(IMRT_EINVAL, "internal: voxel tiles overrun the layout");
              D->vox_host[p] = a;
              codes[p] = -1 - b;
              ++p;
            }
        }
    if (p != nv) return set_error(IMRT_EINVAL, "internal: voxel tiles do not cover the layout");
    IMRT_HIP(hipMalloc(&D->vox, sizeof(int32_t) * nv));
    IMRT_HIP(hipMemcpyAsync(D->vox, D->vox_host.data(), sizeof(int32_t) * nv, hipMemcpyHostToDevice, s));
  } else if (!api_code.empty()) {
    codes = api_code;   // rows in API order
  }
  if (!codes.empty()) {
    IMRT_HIP(hipMalloc(&d_code.p, sizeof(int32_t) * nv));
    IMRT_HIP(hipMemcpyAsync(d_code.p, codes.data(), sizeof(int32_t) * nv, hipMemcpyHostToDevice, s));
  }
  const int32_t* code = codes.empty() ? D->vox : static_cast<const int32_t*>(d_code.p);
  IMRT_HIP(hipMalloc(&d_cnt_r.p, sizeof(int32_t) * nv));
  IMRT_HIP(hipMalloc(&D->sid, nv));
  const int vgrid = (nv + kThreads - 1) / kThreads;
  hipLaunchKernelGGL(structure_kernel, dim3(vgrid), dim3(kThreads), 0, s, g, nv, code, D->sid);
  IMRT_HIP(hipGetLastError());
  const auto* blp = static_cast<const BeamletDev*>(d_bl.p);
  const auto* dp = static_cast<const double2*>(d_dirs.p);
  auto* em = static_cast<double*>(d_emin.p);
  // one allocation for the builder's tables (see the kernels)
  const int nt = g.nx * g.ny + (G->coarse_normal ? g.cx * g.cy : 0);
  const int nrun = (nv + kRun - 1) / kRun, ngroup = (nrun + kRun - 1) / kRun;
  const size_t nbeam = static_cast<size_t>(G->n_beams);
  DevBuf d_tab;
  IMRT_HIP(hipMalloc(&d_tab.p, sizeof(double2) * (nbeam * nt + (nbeam + 1) * (static_cast<size_t>(nrun) + ngroup)) +
                                   sizeof(int4) * lat.size() + sizeof(unsigned long long)));
  auto* plane = static_cast<double2*>(d_tab.p);
  double2* ubox = plane + nbeam * nt;
  double2* zbox = ubox + nbeam * nrun;
  double2* gubox = zbox + nrun;
  double2* gzbox = gubox + nbeam * ngroup;
  auto* d_lat = reinterpret_cast<int4*>(gzbox + ngroup);
  auto* emax = reinterpret_cast<unsigned long long*>(d_lat + lat.size());
  IMRT_HIP(hipMemcpyAsync(d_lat, lat.data(), sizeof(int4) * lat.size(), hipMemcpyHostToDevice, s));
  IMRT_HIP(hipMemsetAsync(emax, 0, sizeof(unsigned long long), s));
  hipLaunchKernelGGL(plane_kernel, dim3((nt + kThreads - 1) / kThreads * G->n_beams), dim3(kThreads), 0, s, g, dp, nt,
                     plane);
  IMRT_HIP(hipGetLastError());
  hipLaunchKernelGGL(run_box_kernel, dim3((nrun + kWaves - 1) / kWaves), dim3(kThreads), 0, s, g, code, plane, nt, nrun,
                     ubox, zbox);
  IMRT_HIP(hipGetLastError());
  hipLaunchKernelGGL(group_box_kernel, dim3((ngroup + kWaves - 1) / kWaves * (G->n_beams + 1)), dim3(kThreads), 0, s,
                     G->n_beams, nrun, ngroup, ubox, zbox, gubox, gzbox);
  IMRT_HIP(hipGetLastError());
  hipLaunchKernelGGL(emin_kernel, dim3(nb), dim3(kThreads), 0, s, g, blp, plane, nt, em, emax);
  IMRT_HIP(hipGetLastError());
  auto columns = [&](auto kernel, int32_t* counts, const int32_t* col_ptr, int32_t* row_idx, float* cval) {
    hipLaunchKernelGGL(kernel, dim3(nb), dim3(kThreads), 0, s, g, code, blp, plane, nt, em, nrun, ngroup, ubox, zbox,
                       gubox, gzbox, counts, col_ptr, row_idx, cval);
    return hipGetLastError();
  };
  auto rows = [&](auto kernel, int32_t* counts, const int32_t* row_ptr, int32_t* col_idx, float* val) {
    hipLaunchKernelGGL(kernel, dim3(vgrid), dim3(kThreads), 0, s, g, code, blp,
                       static_cast<const int32_t*>(d_first.p), d_lat, kmax, w, plane, nt, em, emax, counts, row_ptr,
                       col_idx, val);
    return hipGetLastError();
  };
  IMRT_HIP(columns(column_kernel<false>, static_cast<int32_t*>(d_cnt_c.p), nullptr, nullptr, nullptr));
  IMRT_HIP(rows(row_kernel<false>, static_cast<int32_t*>(d_cnt_r.p), nullptr, nullptr, nullptr));

  // row pointers by a scan on the device, column pointers on the host
  const int nscan = (nv + kScanRun - 1) / kScanRun;
  DevBuf d_scan;
  IMRT_HIP(hipMalloc(&d_scan.p, sizeof(long long) * (static_cast<size_t>(nscan) + 1)));
  auto* scan = static_cast<long long*>(d_scan.p);
  const auto* rcount = static_cast<const int32_t*>(d_cnt_r.p);
  hipLaunchKernelGGL(scan_runs_kernel, dim3(nscan), dim3(kThreads), 0, s, rcount, nv, scan);
  hipLaunchKernelGGL(scan_sums_kernel, dim3(1), dim3(64), 0, s, scan, nscan);
  IMRT_HIP(hipGetLastError());
  std::vector<int32_t> ccount(nb);
  long long tot_r = 0;
  IMRT_HIP(hipMemcpyAsync(ccount.data(), d_cnt_c.p, sizeof(int32_t) * nb, hipMemcpyDeviceToHost, s));
  IMRT_HIP(hipMemcpyAsync(&tot_r, scan + nscan, sizeof(tot_r), hipMemcpyDeviceToHost, s));
  IMRT_HIP(hipStreamSynchronize(s));
  std::vector<int32_t> col_ptr(nb + 1, 0);
  int64_t tot_c = 0;
  for (int i = 0; i < nb; ++i) {
    tot_c += ccount[i];
    if (tot_c >= (int64_t(1) << 31)) return set_error(IMRT_EUNSUPPORTED, "D has 2^31 or more nonzeros");
    col_ptr[i + 1] = static_cast<int32_t>(tot_c);
  }
  if (tot_c != tot_r) return set_error(IMRT_EINVAL, "internal: CSR and CSC nonzero counts differ");

  D->nv = nv;
  D->nb = nb;
  D->nnz = tot_r;
  const int arc = alloc_nonzeros(D);
  if (arc) return arc;
  hipLaunchKernelGGL(scan_fill_kernel, dim3(nscan), dim3(kThreads), 0, s, rcount, nv, scan, nscan, D->row_ptr);
  IMRT_HIP(hipGetLastError());
  IMRT_HIP(hipMemcpyAsync(D->col_ptr, col_ptr.data(), sizeof(int32_t) * (nb + 1), hipMemcpyHostToDevice, s));
  IMRT_HIP(columns(column_kernel<true>, nullptr, D->col_ptr, D->row_idx, D->cval));
  IMRT_HIP(rows(row_kernel<true>, nullptr, D->row_ptr, D->col_idx, D->val));
  IMRT_HIP(hipStreamSynchronize(s));
  apply_partition_targets(ctx, D);
  return finish_columns(D, col_ptr);
}

}  // namespace imrt
