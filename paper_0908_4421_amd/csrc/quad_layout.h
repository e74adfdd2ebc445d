// LDS of the one-read pass (onepass.hip).  No device code: also compiled by
// host tests.
#pragma once

#include <cstddef>
#include <cstdint>

namespace imrt {

enum QuadMode : int32_t {
  QM_SOLVE = 0,   // trials of a solve, with their gradients
  QM_EVAL = 1,    // objective of x, dose optional
  QM_GRAD = 2,    // objective and gradient of x
  QM_PLAIN = 3,   // dose of x, partials of sum d^2
  QM_POWER = 4,   // D^T D of w / ||w||, partials of sum d^2
  QM_WHOLE = 5    // a small plan's step and pass in one
};
constexpr bool quad_grad(int mode) { return mode != QM_EVAL && mode != QM_PLAIN; }

// LDS stride of a staged vector or of a trial's column sums (slot 0: no column)
constexpr int quad_stride(int nb) { return (nb + 1 + 3) & ~3; }

constexpr size_t kPenaltyBytes = 32;   // of a structure's thresholds and weights

// Bytes that the launch asks for: penalty tables (nstruct: of all plans
// together), staged vectors and column sums.
constexpr size_t quad_lds_bytes(int nb, int ntrials, int nstruct, int mode) {
  return static_cast<size_t>(nstruct) * kPenaltyBytes +
         static_cast<size_t>(ntrials) * static_cast<size_t>(quad_stride(nb)) * (quad_grad(mode) ? 12 : 4);
}

// What the kernels hold beside them: the waves' partial sums and maxima, 384
// bytes at most (two trials of sixteen waves, four of eight).  A small plan's
// launch also exchanges its sums there, for 1,024 columns at most.
constexpr size_t kQuadFixedLds = 512;
constexpr size_t kWholeFixedLds = 8192 + 512;

// A workgroup's LDS holds both: two trials of 6,800 to 6,823 beamlets are beyond
// 160 KB only with the second, and keep the two separate passes.
constexpr bool quad_fits(size_t max_lds, size_t lds_bytes, int mode = QM_SOLVE) {
  return lds_bytes + (mode == QM_WHOLE ? kWholeFixedLds : kQuadFixedLds) <= max_lds;
}

}  // namespace imrt
