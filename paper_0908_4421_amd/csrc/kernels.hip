// Small kernels beside the two passes: fixed-order sums, zero fill, projection,
// normalisation, voxel permutation.
#include <algorithm>

#include "pass_common.h"

namespace imrt {
namespace {

// ---- small utility kernels ----------------------------------------------------------
__global__ __launch_bounds__(kThreads) void sum_kernel(const double* parts, int n, double* out, double add) {
  __shared__ double red[kWaves];
  double s = 0.0;
  for (int i = threadIdx.x; i < n; i += kThreads) s += parts[i];
  s = block_sum(s, red);
  if (threadIdx.x == 0) *out = s + add;
}

__global__ __launch_bounds__(kThreads) void zero_kernel(float* p, int n) {
  for (int i = blockIdx.x * kThreads + threadIdx.x; i < n; i += gridDim.x * kThreads) p[i] = 0.0f;
}

__global__ __launch_bounds__(kThreads) void project_kernel(const float* x, const float* g, double lam,
                                                           int nb, float* x_out, double* s_out) {
  __shared__ double red[kWaves];
  double s = 0.0;
  for (int i = threadIdx.x; i < nb; i += kThreads) {
    const float xi = x[i];
    const float t = trial_point(xi, g[i], lam);
    x_out[i] = t;
    const double dl = static_cast<double>(t) - static_cast<double>(xi);
    s += dl * dl;
  }
  s = block_sum(s, red);
  if (threadIdx.x == 0) *s_out = s;
}

__global__ __launch_bounds__(kThreads) void normalize_kernel(const float* w, int nb, float* v,
                                                             double* norm_out) {
  __shared__ double red[kWaves];
  __shared__ double nrm;
  double s = 0.0;
  for (int i = threadIdx.x; i < nb; i += kThreads) {
    const double wi = static_cast<double>(w[i]);
    s += wi * wi;
  }
  s = block_sum(s, red);
  if (threadIdx.x == 0) {
    nrm = sqrt(s);
    *norm_out = nrm;
  }
  __syncthreads();
  const double n = nrm;
  for (int i = threadIdx.x; i < nb; i += kThreads)
    v[i] = n > 0.0 ? static_cast<float>(static_cast<double>(w[i]) / n) : 0.0f;
}

__global__ __launch_bounds__(kThreads) void permute_kernel(const float* in, const int32_t* vox, int n, float* out,
                                                           int scatter) {
  const int p = blockIdx.x * kThreads + threadIdx.x;
  if (p >= n) return;
  if (scatter) out[vox[p]] = in[p];
  else out[p] = in[vox[p]];
}

int grid_for(int items, int cap) {
  if (items <= 0) return 1;
  if (items <= cap) return items;
  return cap;
}

}  // namespace

int check_launch(const char* what) {
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return hip_error(e, what);
  return IMRT_OK;
}

// Drop an error left behind by an unrelated earlier runtime call on this
// thread, so that check_launch reports only the launch that follows.
void clear_stale_error() { (void)hipGetLastError(); }

int launch_sum(const imrt_ctx* ctx, const double* parts, int n, double* out, double add) {
  clear_stale_error();
  hipLaunchKernelGGL(sum_kernel, dim3(1), dim3(kThreads), 0, ctx->stream, parts, n, out, add);
  return check_launch("sum_kernel");
}

int launch_zero(const imrt_ctx* ctx, float* p, int n) {
  if (n <= 0) return IMRT_OK;
  clear_stale_error();
  const int g = std::min((n + kThreads - 1) / kThreads, 4096);
  hipLaunchKernelGGL(zero_kernel, dim3(g), dim3(kThreads), 0, ctx->stream, p, n);
  return check_launch("zero_kernel");
}

int launch_project(const imrt_ctx* ctx, const float* x, const float* g, double lambda, int nb,
                   float* x_out, double* s_out) {
  clear_stale_error();
  hipLaunchKernelGGL(project_kernel, dim3(1), dim3(kThreads), 0, ctx->stream, x, g, lambda, nb, x_out, s_out);
  return check_launch("project_kernel");
}

int launch_permute(const imrt_ctx* ctx, const float* in, const int32_t* vox, int n, float* out, bool scatter) {
  clear_stale_error();
  hipLaunchKernelGGL(permute_kernel, dim3(grid_for((n + kThreads - 1) / kThreads, 1 << 30)), dim3(kThreads), 0,
                     ctx->stream, in, vox, n, out, scatter ? 1 : 0);
  return check_launch("permute_kernel");
}

int launch_normalize(const imrt_ctx* ctx, const float* w, int nb, float* v_out, double* norm_out) {
  clear_stale_error();
  hipLaunchKernelGGL(normalize_kernel, dim3(1), dim3(kThreads), 0, ctx->stream, w, nb, v_out, norm_out);
  return check_launch("normalize_kernel");
}

}  // namespace imrt
