// Float64-accumulated product on split operands (the solver's true residual):
// the float32 entry k(x_i, x_j) from the fine distances of split_tile.h, widened,
// and every product k v summed in float64 -- the sums of valu_tile.h's aug64_rows
// with its distance MFMAs replaced.  Those take T = ceil((d + 2) / 4) float64 MFMAs
// of 64 cycles per 16 x 16 entries, three quarters of the time the sums themselves
// take at d = 8; KC binary16 MFMAs of 16 cycles and two additions give r^2 with the
// two roundings that the float64 distance takes as a float32 argument, and the
// diagonal exactly: the residual's error is the float64 distances' to 5% (n = 8400,
// d = 2 to 12, boxes and clusters of radius 4 to 31, all three kernels; the coarser
// operands of the float32 product doubled it at d = 12 and lost the last digits of
// residuals near 1e-8 on wide boxes).
//
// With the entries' lane layout (row l16, columns 4 g + v) product MFMA v takes
// the columns {4 g + v}: A is the entry, B the right-hand side l16 of that
// column.  That MFMA is 16 wide in right-hand sides and runs at the vector
// unit's float64 rate, so up to eight right-hand sides (RT > 0) are summed by
// float64 FMAs instead, R of them per entry rather than 16.  One residual on the
// float64 distances and on these: N = 100,000, d = 8, R = 16 9.75 ms and 7.60 (5.95
// of them the product MFMAs); N = 40,000, d = 8, R = 5 1.54 and 0.95, R = 1 1.53 and
// 0.50.

#include <algorithm>

#include "split_tile.h"

namespace gpmi {
namespace split {

typedef double d4 __attribute__((ext_vector_type(4)));
constexpr int JT = kStageCols;

template <int KIND, int KC, int RT>
__global__ __launch_bounds__(256) void f64_kernel(const _Float16* __restrict__ Xr,
                                                  const _Float16* __restrict__ Xc,
                                                  const float* __restrict__ V, int r, int c0,
                                                  int64_t n1, int64_t n2, double* __restrict__ part,
                                                  int nsplit, const Info* __restrict__ info) {
  if (!info->ok) return;
  constexpr int NSUB = subtiles(KC, true);
  constexpr int KP = 32 * KC, XS = KP + 8;
  constexpr int RW = RT ? RT : 16;             // right-hand sides staged
  constexpr int XPT = JT * KP / 8 / 256, VPT = (JT * RW + 255) / 256;
  __shared__ __attribute__((aligned(16))) _Float16 sX[2][JT * XS];
  __shared__ __attribute__((aligned(16))) double sV[2][JT * RW];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, g = lane >> 4, l16 = lane & 15;
  const int split = blockIdx.x % nsplit;
  const int64_t row0 = (int64_t)(blockIdx.x / nsplit) * (64 * NSUB) + wave * 16 * NSUB;
  const int64_t nstage = ceil_div(n2, (int64_t)JT);
  const int64_t sb = split * nstage / nsplit, se = (split + 1) * nstage / nsplit;
  const float cs = info->cs;
  const int rc = min(RW, r - c0);

  h8 bi[NSUB][KC];
#pragma unroll
  for (int q = 0; q < NSUB; ++q)
#pragma unroll
    for (int kc = 0; kc < KC; ++kc)
      bi[q][kc] = *reinterpret_cast<const h8*>(Xr + (row0 + q * 16 + l16) * KP + kc * 32 + g * 8);
  d4 acc[NSUB];
  double sum[NSUB][RT ? RT : 1];
#pragma unroll
  for (int q = 0; q < NSUB; ++q) {
    acc[q] = d4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int c = 0; c < RT; ++c) sum[q][c] = 0.0;
  }

  h8 xreg[XPT];
  float vreg[VPT];
  auto gload = [&](int64_t st) {
    const int64_t j0 = st * JT;
#pragma unroll
    for (int e = 0; e < XPT; ++e) {
      const int ch = tid + e * 256, row = ch / (KP / 8), col = ch % (KP / 8);
      xreg[e] = *reinterpret_cast<const h8*>(Xc + (j0 + row) * KP + col * 8);
    }
#pragma unroll
    for (int e = 0; e < VPT; ++e) {
      const int ch = tid + e * 256, jj = ch / RW, c = ch % RW;
      vreg[e] = (c < rc && jj < JT && j0 + jj < n2) ? V[(j0 + jj) * r + c0 + c] : 0.0f;
    }
  };
  auto lstore = [&](int buf) {
#pragma unroll
    for (int e = 0; e < XPT; ++e) {
      const int ch = tid + e * 256, row = ch / (KP / 8), col = ch % (KP / 8);
      *reinterpret_cast<h8*>(&sX[buf][row * XS + col * 8]) = xreg[e];
    }
#pragma unroll
    for (int e = 0; e < VPT; ++e) {
      const int ch = tid + e * 256;
      if (ch < JT * RW) sV[buf][ch] = (double)vreg[e];
    }
  };

  if (sb < se) {
    gload(sb);
    lstore(0);
  }
  __syncthreads();
  for (int64_t st = sb; st < se; ++st) {
    const int buf = (int)((st - sb) & 1);
    const bool more = st + 1 < se;
    if (more) gload(st + 1);
    const _Float16* X = sX[buf];
    const double* Vs = sV[buf];
#pragma unroll 1
    for (int jb = 0; jb < JT / 16; ++jb) {
      h8 a[KC];
#pragma unroll
      for (int kc = 0; kc < KC; ++kc)
        a[kc] = *reinterpret_cast<const h8*>(X + (jb * 16 + l16) * XS + kc * 32 + g * 8);
      float k[NSUB][4];
#pragma unroll
      for (int q = 0; q < NSUB; ++q) {
        const f4 s = sqdist_fine<KC>(a, bi[q]);
#pragma unroll
        for (int v = 0; v < 4; ++v) k[q][v] = kval<KIND>(s[v], cs);
      }
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const double* vr = Vs + (jb * 16 + 4 * g + v) * RW;
        if constexpr (RT == 0) {
          const double b = vr[l16];
#pragma unroll
          for (int q = 0; q < NSUB; ++q)
            acc[q] = __builtin_amdgcn_mfma_f64_16x16x4f64((double)k[q][v], b, acc[q], 0, 0, 0);
        } else {
          double b[RT ? RT : 1];
#pragma unroll
          for (int c = 0; c < RT; ++c) b[c] = vr[c];
#pragma unroll
          for (int q = 0; q < NSUB; ++q) {
            const double kd = (double)k[q][v];
#pragma unroll
            for (int c = 0; c < RT; ++c) sum[q][c] = fma(kd, b[c], sum[q][c]);
          }
        }
      }
    }
    if (more) lstore(buf ^ 1);
    __syncthreads();
  }
  // The diagonal's entry is 1, not the kernel of T's rounding (a Matern value near 0
  // rounds to 3e-8 of 1): the split that summed it adds (1 - k) v, k from the same
  // operations.  (A second loop for the stages that hold the wave's rows took the
  // registers of the right-hand sides' sums: one wave per SIMD at d <= 10 with five to
  // eight of them, 1.49 ms a residual at N = 40,000, d = 8, R = 5, for 0.95 ms.)
#pragma unroll
  for (int q = 0; q < NSUB; ++q) {
    const int64_t i0 = row0 + q * 16;
    if (i0 >= n1 || i0 / JT < sb || i0 / JT >= se) continue;    // wave-uniform
    h8 a[KC];
#pragma unroll
    for (int kc = 0; kc < KC; ++kc)
      a[kc] = *reinterpret_cast<const h8*>(Xc + (i0 + l16) * KP + kc * 32 + g * 8);
    const f4 s = sqdist_fine<KC>(a, bi[q]);
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int64_t j = i0 + 4 * g + v;
      const double e = l16 == 4 * g + v ? 1.0 - (double)kval<KIND>(s[v], cs) : 0.0;
      // nothing to add to a sum that is not finite
      auto rhs = [&](int c) {
        const float x = j < n2 && c < rc ? V[j * r + c0 + c] : 0.0f;
        return isfinite(x) ? (double)x : 0.0;
      };
      if constexpr (RT == 0) {
        acc[q] = __builtin_amdgcn_mfma_f64_16x16x4f64(e, rhs(l16), acc[q], 0, 0, 0);
      } else if (l16 == 4 * g + v) {
#pragma unroll
        for (int c = 0; c < RT; ++c) sum[q][c] = fma(e, rhs(c), sum[q][c]);
      }
    }
  }
  double* P = part + (int64_t)split * n1 * r;
#pragma unroll
  for (int q = 0; q < NSUB; ++q) {
    if constexpr (RT == 0) {
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int64_t i = row0 + q * 16 + g + 4 * v;
        if (i < n1 && l16 < rc) P[i * r + c0 + l16] = acc[q][v];
      }
    } else {
      const int64_t i = row0 + q * 16 + l16;
#pragma unroll
      for (int c = 0; c < RT; ++c) {
        double t = sum[q][c];
        t += __shfl_xor(t, 16);
        t += __shfl_xor(t, 32);
        if (g == 0 && i < n1 && c < rc) P[i * r + c0 + c] = t;
      }
    }
  }
}

typedef void (*F64Fn)(const _Float16*, const _Float16*, const float*, int, int, int64_t, int64_t,
                      double*, int, const Info*);
template <int KIND, int RT>
static F64Fn f64_fn(int kc) {
  switch (kc) {
    case 3: return &f64_kernel<KIND, 3, RT>;
    case 4: return &f64_kernel<KIND, 4, RT>;
    case 5: return &f64_kernel<KIND, 5, RT>;
    case 6: return &f64_kernel<KIND, 6, RT>;
    case 7: return &f64_kernel<KIND, 7, RT>;
    case 8: return &f64_kernel<KIND, 8, RT>;
  }
  return nullptr;
}
template <int KIND>
static F64Fn f64_fn(int kc, int rt) {
  switch (rt) {
    case 1: return f64_fn<KIND, 1>(kc);
    case 4: return f64_fn<KIND, 4>(kc);
    case 8: return f64_fn<KIND, 8>(kc);
  }
  return f64_fn<KIND, 0>(kc);
}

// Right-hand sides of one FMA launch, 0 for the 16-wide MFMA form.
static int fma_rhs(int r) { return r == 1 ? 1 : r <= 4 ? 4 : r <= 8 ? 8 : 0; }

gp_status partial64(const Plan& p, const KParams& kp, int64_t n, const float* V, int r,
                    double* part, int nsplit, hipStream_t s) {
  const int rt = fma_rhs(r), step = rt ? rt : 16;
  const F64Fn fn = kp.kind == GP_KERNEL_RBF        ? f64_fn<GP_KERNEL_RBF>(p.kc, rt)
                   : kp.kind == GP_KERNEL_MATERN52 ? f64_fn<GP_KERNEL_MATERN52>(p.kc, rt)
                   : kp.kind == GP_KERNEL_MATERN32 ? f64_fn<GP_KERNEL_MATERN32>(p.kc, rt)
                                                   : nullptr;
  if (!fn) return set_error(GP_ERR_ARG, "internal: no split product for this kernel");
  const int64_t blocks = p.n1_pad / (64 * subtiles(p.kc, true)) * nsplit;
  for (int c0 = 0; c0 < r; c0 += step) {
    fn<<<(unsigned)blocks, 256, 0, s>>>(p.Xr, p.Xc, V, r, c0, n, n, part, nsplit, p.info);
    GP_HIP(hipGetLastError());
  }
  return GP_OK;
}

// The fewest column splits within 1% of the best rounds per unit of work.
int choose_splits64(const Plan& p, int r) {
  const int rt = fma_rhs(r), rw = rt ? rt : 16;
  const int lds = 2 * (2 * JT * (32 * p.kc + 8) + 8 * JT * rw);
  const int64_t resident = 256 * std::max(1, std::min(3, 160 * 1024 / (lds + 512)));
  const int64_t rblocks = p.n1_pad / (64 * subtiles(p.kc, true));
  const int64_t smax = std::max<int64_t>(1, std::min<int64_t>(64, p.n2_pad / JT / 4));
  auto cost = [&](int64_t sp) { return (double)ceil_div(rblocks * sp, resident) / (double)sp; };
  double best = 1e300;
  for (int64_t sp = 1; sp <= smax; ++sp) best = std::min(best, cost(sp));
  for (int64_t sp = 1; sp <= smax; ++sp)
    if (cost(sp) <= best * 1.01) return (int)sp;
  return 1;
}

bool use64(int kind, int64_t n, int d) {
  return kind != GP_KERNEL_MATERN12 && d <= kSplitMaxDim && n >= kSplit64MinPoints;
}

}  // namespace split
}  // namespace gpmi
