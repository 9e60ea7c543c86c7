// Split-operand form of the gradient reduction (grad_split.hip), chosen and
// finished by grad.hip.
#pragma once

#include "internal.h"

namespace gpmi {
namespace grad {

constexpr int kGradSplitMaxDim = 16;
// Its five extra launches cost about 18 us.  With one lengthscale per input the
// difference form's work is n^2 (3 d + 12): at 4e8 (N = 3000, d = 12) 161 us
// against 131, at 5e7 (N = 1500, d = 3) 101 against 119.  One isotropic
// lengthscale leaves only the distance and W to gain on: N = 10,000 129 us
// against 140, N = 60,000 1050 against 930.
constexpr double kGradSplitMinWork = 2e8;
constexpr int64_t kGradSplitMinIso = 16384;

struct SplitWork {
  split::Plan p;               // point operands
  int64_t rblocks;
  int nsplit, comps;
  _Float16* H;                 // n_pad x 4 x 16 parts of U and C
  _Float16* Zt;                // 2 x comps x n_pad parts of [b | b^2]
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
