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

// Bytes that the launch asks for: column marks (a byte each, shared by a
// plan's trials), column sums, penalty tables (nstruct: of all plans together)
// and staged vectors.
constexpr size_t quad_mark_bytes(int nb, int plans) {
  return (static_cast<size_t>(plans) * static_cast<size_t>(quad_stride(nb)) + 15) & ~static_cast<size_t>(15);
}
constexpr size_t quad_lds_bytes(int nb, int ntrials, int nstruct, int mode, int plans = 1) {
  return static_cast<size_t>(nstruct) * kPenaltyBytes + (quad_grad(mode) ? quad_mark_bytes(nb, plans) : 0) +
         static_cast<size_t>(ntrials) * static_cast<size_t>(quad_stride(nb)) * (quad_grad(mode) ? 12 : 4);
}

// What the kernels hold beside them: the waves' partial sums and maxima, 384
// bytes at most (two trials of sixteen waves, four of eight).  A small plan's
// launch also exchanges its sums there, for 1,024 columns at most.
constexpr size_t kQuadFixedLds = 512;
constexpr size_t kWholeFixedLds = 16384 + 512;

// A workgroup's LDS holds both: two trials of about 6,530 beamlets are beyond
// 160 KB only with the second, and keep the two separate passes.
constexpr bool quad_fits(size_t max_lds, size_t lds_bytes, int mode = QM_SOLVE) {
  return lds_bytes + (mode == QM_WHOLE ? kWholeFixedLds : kQuadFixedLds) <= max_lds;
}

// When the integers that a column's terms are rounded to (by half a unit each,
// and a workgroup's sum moved by a unit at most) are precise enough: the
// workgroups' sums have to come, in magnitude and in units of 2^24, to this
// for columns of n nonzeros at most.  Roundings of either sign then move the
// total by about 2^-28 of that (sqrt(n) / 2 units of 2^27 sqrt(n)), and at
// worst, if all were of one sign, by 2^-21; one rounding of the result to float32 is
// 2^-24.
constexpr int kMagnitude = 24;
inline uint32_t quad_enough(int32_t n) {
  double root = 1.0;
  while (root * root < n) root *= 1.0905077326652577;   // 2^(1/8)
  const double by_chance = 8.0 * root, at_worst = n / 12.0;
  return static_cast<uint32_t>(by_chance > at_worst ? by_chance : at_worst) + 1;
}

}  // namespace imrt
