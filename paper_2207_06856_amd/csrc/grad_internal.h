// Split-operand form of the gradient reduction (grad_split.hip), chosen and
// finished by grad.hip.
#pragma once

#include "internal.h"

namespace gpmi {
namespace grad {

constexpr int kGradSplitMaxDim = 16;
// Points from which this form is taken.  Its five extra launches cost about 18 us;
// what it saves per entry depends on how the S_m are summed (grad_split.hip).  The
// call in us, difference form against this one (R = 16):
//   d >= 9: n = 2000 125 against 133, 2500 145 against 133, 6000 259 against 160;
//   d = 5 to 8: n = 4000 127 against 129, 6000 154 against 147, 32,000 698 against
//     630 (Matern-5/2: 16,000 308 against 309, 24,000 514 against 497);
//   d <= 4: n = 20,000 256 against 273, 32,000 471 against 456;
//   one lengthscale: d <= 5 n = 20,000 196 against 207, 28,000 281 against 273;
//     d >= 6 n = 12,000 162 against 161, 16,384 208 against 189.
inline int64_t split_min_points(int d, bool iso) {
  if (iso) return d <= 5 ? 24576 : 16384;
  return d <= 4 ? 28672 : d <= 8 ? 6144 : 2250;
}

struct SplitWork {
  split::Plan p;               // point operands
  int64_t rblocks;
  int nsplit, width;
  _Float16* H;                 // n_pad x 4 x 16 parts of U and C
  double* Zb;                  // n_pad x width coordinates b
};
// whether the gradient over `rows` rows of n takes this form (the inputs' range
// is checked on the device: Info::ok)
bool use_split(int kind, int64_t n, int d, bool iso, int r, int64_t rows);
SplitWork split_plan(int64_t n, int d, bool iso);
size_t split_bytes(const SplitWork& w, int d);
gp_status split_carve(SplitWork& w, int d, Arena& ar);
// part[rblocks * nsplit][nacc + 1] (nacc = 1 or d); point operands and scl are
// ready on the stream.
gp_status split_launch(const SplitWork& w, const KParams& kp, bool iso, const float* X, int64_t n,
                       const float* U, const float* B, int r, float inv2m, const float* scl,
                       double* part, hipStream_t s);

}  // namespace grad
}  // namespace gpmi
