// Gradient reduction (grad.hip's sums, over the whole row range) on split
// operands.  Per entry the vector unit forms the kernel value, P = G W~ and
// its binary16 parts; everything that grows with d is on the matrix cores:
//   * r^2 from exact integer products (split_tile.h);
//   * W~ = W + W^T from the binary16 split of U and C, as in grad.hip, at a
//     scale that keeps |P| below 2^15;
//   * S_m = sum_ij P_ij (a_im - b_jm)^2 = sum_i [a_im^2 p_i - 2 a_im Z_im + Y_im],
//     p_i = sum_j P_ij, Z = P b, Y = P b^2: P and the operands [b | b^2] in two
//     binary16 parts each (22 bits), three products, float32 sums over a work
//     group's columns, float64 beyond.
// Coordinates are taken from the centre of the points' box (a, b = (x - c) / l),
// so a^2 and b^2 exceed the squared differences they cancel to by the square of
// the points' spread in lengthscales; where the box is wide (kSplitMaxRadius)
// or an input is not finite, grad.hip's kernel, which takes the differences
// themselves, runs instead.
//
// Bound by issue at two waves per SIMD: 360 cycles of a SIMD per 256 evaluated
// entries at N = 100,000, d = 8, R = 16 (RBF, one lengthscale per input), of
// which matrix cores 136 and vector unit 125; the difference form took 704.  The
// whole call 5.62 -> 2.96 ms, N = 30,000, d = 16 (Matern-5/2) 1.61 -> 0.85,
// N = 60,000, d = 4 1.43 -> 1.07 (RBF), 1.74 -> 1.36 (Matern-3/2); the error
// against float64 is that of the difference form or below.

#include <math.h>

#include <algorithm>

#include "device_common.h"
#include "grad_internal.h"
#include "split_tile.h"

namespace gpmi {
namespace grad {

using f16::f4;
using f16::h4;
using f16::h8;
using split::Info;

namespace {

// [b | b^2] are scaled so that their largest values (|b| <= kSplitMaxRadius) stay
// below 2^15 and the low parts of ordinary ones clear binary16's smallest normal
constexpr double kCoordScale = 128.0, kSquareScale = 32.0;
static_assert(split::kSplitMaxRadius * kCoordScale <= 32768.0 &&
                  split::kSplitMaxRadius * split::kSplitMaxRadius * kSquareScale <= 32768.0,
              "binary16 range of the coordinate operands");
// 16-row subtiles per wave: four where their operands leave two waves per SIMD
__host__ __device__ constexpr int row_subtiles(int kc, int nb) {
  return nb == 0 && kc == 2 ? 4 : 2;
}
constexpr int kStage = split::kStageCols;        // 64 columns per LDS stage
constexpr int kHS = 64 + 8;                      // LDS row stride of the U, C parts (halfs)
constexpr int kZS = kStage + 4;                  // LDS row stride of the [b | b^2] parts

// The binary16 parts of the scaled U (hi, lo) and C (hi, lo) of one row, 16
// halfs each; a thread writes 8 halfs.  Rows n .. n_pad - 1 are zero.
__global__ __launch_bounds__(256) void parts_kernel(const float* __restrict__ U,
                                                    const float* __restrict__ B, int64_t n,
                                                    int64_t n_pad, int r, float inv2m,
                                                    const float* __restrict__ scl,
                                                    const Info* __restrict__ info,
                                                    _Float16* __restrict__ H) {
  if (!info->ok) return;
  const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int64_t i = t >> 3;
  if (i >= n_pad) return;
  const int w = (int)(t & 7) >> 1, c0 = (int)(t & 1) * 8;
  h8 o;
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    const int c = c0 + k;
    float v = 0.0f;
    if (i < n && c < r)
      v = w < 2 ? U[i * r + c] * scl[c]
                : (c == 0 ? -0.5f * U[i * r] : inv2m * B[i * r + c]) * scl[64 + c];
    const _Float16 h = (_Float16)v;
    o[k] = (w & 1) ? (_Float16)(v - (float)h) : h;
  }
  *reinterpret_cast<h8*>(H + i * 64 + w * 16 + c0) = o;
}

// Zt[part][component][n_pad]: b_m (components 0 .. d - 1) and b_m^2 (d .. 2d - 1)
// in two binary16 parts, zero elsewhere.
__global__ __launch_bounds__(256) void coord_kernel(const float* __restrict__ X, int64_t n,
                                                    int64_t n_pad, KParams kp, int comps,
                                                    const Info* __restrict__ info,
                                                    _Float16* __restrict__ Zt) {
  if (!info->ok) return;
  const int64_t j = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (j >= n_pad) return;
  const int d = kp.d, c = blockIdx.y;
  const int m = c < d ? c : c - d;
  double v = 0.0;
  if (j < n && c < 2 * d) {
    v = ((double)X[j * d + m] - info->centre[m]) / (double)kp.ls[m];
    v = c < d ? v * kCoordScale : v * v * kSquareScale;
  }
  // five leading bits, then two binary16 parts of the rest
  int e;
  (void)frexp(v, &e);
  const double z0 = ldexp(rint(ldexp(v, 5 - e)), e - 5);
  const _Float16 z1 = (_Float16)(float)(v - z0);
  Zt[(int64_t)c * n_pad + j] = (_Float16)(float)z0;
  Zt[(int64_t)(comps + c) * n_pad + j] = z1;
  Zt[(int64_t)(2 * comps + c) * n_pad + j] = (_Float16)(float)(v - z0 - (double)(float)z1);
}

// kappa and G from D = r^2 / u^2.
template <int KIND>
__device__ __forceinline__ void kval_deriv_split(float D, float cs, float& kap, float& G) {
  constexpr float kLn2f = 0.6931471805599453f;
  if constexpr (KIND == GP_KERNEL_RBF) {
    kap = __builtin_amdgcn_exp2f(D * cs);
    G = kap;
  } else {
    const float sp = __builtin_amdgcn_sqrtf(fabsf(D * cs));
    const float e = __builtin_amdgcn_exp2f(-sp);
    const float l = fmaf(sp, kLn2f, 1.0f);                  // 1 + t, t = sqrt(nu') r
    if constexpr (KIND == GP_KERNEL_MATERN32) {
      kap = l * e;
      G = 3.0f * e;
    } else {
      kap = fmaf(sp * sp, kLn2f * kLn2f / 3.0f, l) * e;
      G = (5.0f / 3.0f) * l * e;
    }
  }
}

__device__ __forceinline__ double wave_sum64(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// NB: 16-component blocks of [b | b^2] (0: one isotropic lengthscale, whose sum
// is P r^2).  A work group of 4 waves owns 64 NSUB rows and a run of column
// stages from its own first row on; past its own rows W takes the mirrored
// products as well.  Lane layout of every tile: row l16, columns 4 g + v (the
// A operand is the column side), which is the A layout of P [b | b^2].  MFMA sums
// are about 0.02 ulp low on average; the odd subtiles' U and C rows are negated,
// so that they carry -W and -P and the two halves' shares cancel in the sums.
template <int KIND, int KC, int NB>
__global__ __launch_bounds__(256) void grad_split_kernel(
    const _Float16* __restrict__ Xr, const _Float16* __restrict__ Xc,
    const _Float16* __restrict__ H, const _Float16* __restrict__ Zt, const float* __restrict__ X,
    const Info* __restrict__ info, const float* __restrict__ scl, int64_t n, int64_t n_pad,
    KParams kp, double* __restrict__ part, int nsplit) {
  if (!info->ok) return;
  constexpr bool ISO = NB == 0;
  constexpr int NSUB = row_subtiles(KC, NB);
  constexpr int KP = 32 * KC, XS = KP + 8, RB = 64 * NSUB;
  constexpr int NZ = ISO ? 1 : NB;
  constexpr int XPT = kStage * KP / 8 / 256;     // 16-byte chunks per thread
  constexpr int HPT = kStage * 64 / 8 / 256;
  // the RBF instantiations have the registers for both 32-column halves of a
  // stage at once (6% faster); the Matern ones spill
  constexpr int kUnroll = KIND == GP_KERNEL_RBF && NB < 2 ? 2 : 1;
  constexpr int ZPT = (3 * 16 * NB * kStage / 8 + 255) / 256;
  __shared__ __attribute__((aligned(16))) _Float16 sX[2][kStage * XS];
  __shared__ __attribute__((aligned(16))) _Float16 sH[2][kStage * kHS];
  __shared__ __attribute__((aligned(16))) _Float16 sZ[2][ISO ? 8 : 3 * 16 * NB * kZS];
  __shared__ double sRed[4][2 * 16 + 2];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, g = lane >> 4, l16 = lane & 15;
  const int gl = g & 1, gh = g >> 1;
  const int spl = blockIdx.x % nsplit;
  const int64_t rowb = (int64_t)(blockIdx.x / nsplit) * RB;
  const int64_t row0 = rowb + wave * 16 * NSUB;
  const float cs = info->cs;
  const h8 z8 = h8{0, 0, 0, 0, 0, 0, 0, 0};

  h8 bi[NSUB][KC], aw[NSUB][3];
#pragma unroll
  for (int q = 0; q < NSUB; ++q) {
    const int64_t i = row0 + q * 16 + l16;
#pragma unroll
    for (int kc = 0; kc < KC; ++kc)
      bi[q][kc] = *reinterpret_cast<const h8*>(Xr + i * KP + kc * 32 + g * 8);
    // [U_hi | U_lo], [U_hi | C_hi], [C_lo | C_hi]
    const _Float16* Hr = H + i * 64 + 8 * gl;
    aw[q][0] = *reinterpret_cast<const h8*>(Hr + (gh ? 16 : 0));
    aw[q][1] = *reinterpret_cast<const h8*>(Hr + (gh ? 32 : 0));
    aw[q][2] = *reinterpret_cast<const h8*>(Hr + (gh ? 32 : 48));
    if (q & 1)
#pragma unroll
      for (int w = 0; w < 3; ++w) aw[q][w] = -aw[q][w];
  }
  f4 acc[NSUB][NZ];
  float p[NSUB];
  float acck = 0.0f, accr = 0.0f;
#pragma unroll
  for (int q = 0; q < NSUB; ++q) {
    p[q] = 0.0f;
#pragma unroll
    for (int z = 0; z < NZ; ++z) acc[q][z] = f4{0.f, 0.f, 0.f, 0.f};
  }

  const int64_t nstage = n_pad / kStage;
  const int64_t s0 = rowb / kStage, own_end = s0 + RB / kStage;
  const int64_t sb = s0 + spl * (nstage - s0) / nsplit, se = s0 + (spl + 1) * (nstage - s0) / nsplit;
  h8 xreg[XPT], hreg[HPT], zreg[ISO ? 1 : ZPT];
  auto gload = [&](int64_t st) {
    const int64_t j0 = st * kStage;
#pragma unroll
    for (int e = 0; e < XPT; ++e) {
      const int ch = tid + e * 256, row = ch / (KP / 8), col = ch % (KP / 8);
      xreg[e] = *reinterpret_cast<const h8*>(Xc + (j0 + row) * KP + col * 8);
    }
#pragma unroll
    for (int e = 0; e < HPT; ++e) {
      const int ch = tid + e * 256, row = ch / 8, col = ch % 8;
      hreg[e] = *reinterpret_cast<const h8*>(H + (j0 + row) * 64 + col * 8);
    }
#pragma unroll
    for (int e = 0; e < ZPT; ++e) {
      const int ch = tid + e * 256, c = ch / (kStage / 8), col = ch % (kStage / 8);
      if (ch < 3 * 16 * NB * kStage / 8) zreg[e] = *reinterpret_cast<const h8*>(Zt + (int64_t)c * n_pad + j0 + col * 8);
    }
  };
  auto lstore = [&](int buf) {
#pragma unroll
    for (int e = 0; e < XPT; ++e) {
      const int ch = tid + e * 256, row = ch / (KP / 8), col = ch % (KP / 8);
      *reinterpret_cast<h8*>(&sX[buf][row * XS + col * 8]) = xreg[e];
    }
#pragma unroll
    for (int e = 0; e < HPT; ++e) {
      const int ch = tid + e * 256, row = ch / 8, col = ch % 8;
      *reinterpret_cast<h8*>(&sH[buf][row * kHS + col * 8]) = hreg[e];
    }
#pragma unroll
    for (int e = 0; e < ZPT; ++e) {
      const int ch = tid + e * 256, c = ch / (kStage / 8), col = ch % (kStage / 8);
      if (ch >= 3 * 16 * NB * kStage / 8) continue;
      _Float16* dst = &sZ[buf][c * kZS + col * 8];
      *reinterpret_cast<h4*>(dst) = h4{zreg[e][0], zreg[e][1], zreg[e][2], zreg[e][3]};
      *reinterpret_cast<h4*>(dst + 4) = h4{zreg[e][4], zreg[e][5], zreg[e][6], zreg[e][7]};
    }
  };

  if (sb < se) {
    gload(sb);
    lstore(0);
  }
  __syncthreads();
  for (int64_t st = sb; st < se; ++st) {
    const int buf = (int)((st - sb) & 1);
    const bool more = st + 1 < se, mirror = st >= own_end;
    if (more) gload(st + 1);
    const _Float16* Xs = sX[buf];
    const _Float16* Hs = sH[buf];
#pragma unroll kUnroll
    for (int jb = 0; jb < kStage / 32; ++jb) {
      h8 a[2][KC], bw[2][3];
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int col = jb * 32 + h * 16 + l16;
#pragma unroll
        for (int kc = 0; kc < KC; ++kc)
          a[h][kc] = *reinterpret_cast<const h8*>(Xs + col * XS + kc * 32 + g * 8);
        // [C_hi ; C_hi], [C_lo ; U_hi] (second half mirror only), [U_hi ; U_lo] (mirror only)
        const _Float16* Hc = Hs + col * kHS + 8 * gl;
        bw[h][0] = *reinterpret_cast<const h8*>(Hc + 32);
        bw[h][1] = (gh && !mirror) ? z8 : *reinterpret_cast<const h8*>(Hc + (gh ? 0 : 48));
        bw[h][2] = *reinterpret_cast<const h8*>(Hc + (gh ? 16 : 0));
      }
      h8 zb[NZ][3];
#pragma unroll
      for (int z = 0; z < NB; ++z)
#pragma unroll
        for (int w = 0; w < 3; ++w) {
          const _Float16* zr = &sZ[buf][((w * NB + z) * 16 + l16) * kZS + jb * 32 + g * 4];
          const h4 lo = *reinterpret_cast<const h4*>(zr);
          const h4 hi = *reinterpret_cast<const h4*>(zr + 16);
          zb[z][w] = h8{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
        }
#pragma unroll
      for (int q = 0; q < NSUB; ++q) {
        h8 ph, pl;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const f4 D = split::sqdist<KC>(a[h], bi[q]);
          f4 W = f4{0.f, 0.f, 0.f, 0.f};
          W = f16::mfma32<_Float16>(bw[h][0], aw[q][0], W);
          W = f16::mfma32<_Float16>(bw[h][1], aw[q][1], W);
          if (mirror) {
            W = f16::mfma32<_Float16>(bw[h][2], aw[q][2], W);
          } else {
            // the diagonal adds nothing to the S_m but would dominate p, Z, Y
            // and their roundings; its kappa(0) W_ii is added at the end
            const int off = (int)(row0 - st * kStage) + q * 16 + l16 - (jb * 32 + h * 16 + 4 * g);
#pragma unroll
            for (int v = 0; v < 4; ++v) W[v] = off == v ? 0.0f : W[v];
          }
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            float kap, G;
            kval_deriv_split<KIND>(D[v], cs, kap, G);
            // P is rounded to float32 once, here: a conversion to binary16 that
            // takes the product unrounded (v_fma_mixlo_f16) in only one of its
            // two uses below would leave parts that do not add up to P
            float P = G * W[v];
            asm("" : "+v"(P));
            if constexpr (KIND != GP_KERNEL_RBF) acck = fmaf(q & 1 ? -kap : kap, W[v], acck);
            if constexpr (!ISO || KIND == GP_KERNEL_RBF) p[q] += P;
            if constexpr (ISO) {
              accr = q & 1 ? fmaf(-P, D[v], accr) : fmaf(P, D[v], accr);
            } else {
              const _Float16 hp = (_Float16)P;
              ph[4 * h + v] = hp;
              pl[4 * h + v] = (_Float16)(P - (float)hp);
            }
          }
        }
        if constexpr (!ISO) {
#pragma unroll
          for (int z = 0; z < NZ; ++z) {
            // 32 columns from zero, then one vector add: an MFMA cuts the low
            // bits of products far below its accumulator
            f4 t = f4{0.f, 0.f, 0.f, 0.f};
            t = f16::mfma32<_Float16>(ph, zb[z][0], t);
            t = f16::mfma32<_Float16>(ph, zb[z][1], t);
            t = f16::mfma32<_Float16>(ph, zb[z][2], t);
            t = f16::mfma32<_Float16>(pl, zb[z][0], t);
            t = f16::mfma32<_Float16>(pl, zb[z][1], t);
#pragma unroll
            for (int v = 0; v < 4; ++v) acc[q][z][v] += t[v];
          }
        }
      }
    }
    if (more) lstore(buf ^ 1);
    __syncthreads();
  }

  // float64: a^2 p - 2 a Z + Y per row and component, lanes, then the waves
  const int d = kp.d;
  const double unscale = (double)scl[128];
  double kk = (double)acck;
  if constexpr (KIND == GP_KERNEL_RBF)
#pragma unroll
    for (int q = 0; q < NSUB; ++q) kk += q & 1 ? -(double)p[q] : (double)p[q];
  kk = wave_sum64(kk);
  if (lane == 0) sRed[wave][2 * 16] = kk;
  if constexpr (ISO) {
    const double s = wave_sum64((double)accr);
    if (lane == 0) sRed[wave][0] = s;
  } else {
    auto coord = [&](int64_t i, int m) {
      return i < n ? ((double)X[i * d + m] - info->centre[m]) / (double)kp.ls[m] : 0.0;
    };
#pragma unroll
    for (int z = 0; z < NZ; ++z) {
      const int c = 16 * z + l16;
      double s = 0.0;
#pragma unroll
      for (int q = 0; q < NSUB; ++q)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const double t = q & 1 ? -(double)acc[q][z][v] : (double)acc[q][z][v];
          if (c < d)
            s -= 2.0 / kCoordScale * coord(row0 + q * 16 + 4 * g + v, c) * t;
          else
            s += t / kSquareScale;
        }
      s += __shfl_xor(s, 16);
      s += __shfl_xor(s, 32);
      if (g == 0) sRed[wave][c] = s;
    }
    __syncthreads();
    double ps[NSUB];
#pragma unroll
    for (int q = 0; q < NSUB; ++q) {
      ps[q] = q & 1 ? -(double)p[q] : (double)p[q];
      ps[q] += __shfl_xor(ps[q], 16);
      ps[q] += __shfl_xor(ps[q], 32);
    }
    // lane group g takes dimensions g, g + 4, ...; its 16 lanes are 16 rows
    for (int m = g; m < ((d + 3) & ~3); m += 4) {
      double s = 0.0;
#pragma unroll
      for (int q = 0; q < NSUB; ++q) {
        const double x = m < d ? coord(row0 + q * 16 + l16, m) : 0.0;
        s += x * x * ps[q];
      }
#pragma unroll
      for (int o = 8; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
      if (m < d && l16 == 0) sRed[wave][m] += s + sRed[wave][d + m];
    }
  }
  __syncthreads();
  const int nacc = ISO ? 1 : d;
  if (tid <= nacc) {
    const int k = tid < nacc ? tid : 2 * 16;
    double s = ((sRed[0][k] + sRed[1][k]) + sRed[2][k]) + sRed[3][k];
    if (ISO && tid == 0) s /= info->inv_u * info->inv_u;
    part[(int64_t)blockIdx.x * (nacc + 1) + tid] = s * unscale;
  }
}

typedef void (*GradFn)(const _Float16*, const _Float16*, const _Float16*, const _Float16*,
                       const float*, const Info*, const float*, int64_t, int64_t, KParams, double*,
                       int);
template <int KIND>
GradFn grad_fn(int d, bool iso) {
  const int kc = split::operand_chunks(d);
  if (iso)
    return kc == 2 ? &grad_split_kernel<KIND, 2, 0>
                   : kc == 3 ? &grad_split_kernel<KIND, 3, 0> : &grad_split_kernel<KIND, 4, 0>;
  if (kc == 2) return &grad_split_kernel<KIND, 2, 1>;
  if (kc == 3) return d <= 8 ? &grad_split_kernel<KIND, 3, 1> : &grad_split_kernel<KIND, 3, 2>;
  return &grad_split_kernel<KIND, 4, 2>;
}

int comps_of(int d, bool iso) { return iso ? 0 : d <= 8 ? 16 : 32; }

}  // namespace

bool use_split(int kind, int64_t n, int d, bool iso, int r, int64_t rows) {
  if (kind == GP_KERNEL_MATERN12 || d > kGradSplitMaxDim || r > 16 || rows != n) return false;
  return iso ? n >= kGradSplitMinIso : (double)n * (double)n * (3 * d + 12) >= kGradSplitMinWork;
}

SplitWork split_plan(int64_t n, int d, bool iso) {
  SplitWork w{};
  w.p = split::plan(n, n, d, 1, true, 1);
  const int64_t rb = w.p.n1_pad / (64 * row_subtiles(w.p.kc, comps_of(d, iso) / 16));
  w.rblocks = rb;
  // about 3000 work groups of at least two stages on average
  const int64_t most = std::max<int64_t>(1, w.p.n2_pad / kStage / 4);
  w.nsplit = (int)std::max<int64_t>(1, std::min<int64_t>(std::min<int64_t>(64, ceil_div(3072, rb)), most));
  w.comps = comps_of(d, iso);
  return w;
}

size_t split_bytes(const SplitWork& w, int d) {
  return split::operand_bytes(w.p, d) + 2 * (size_t)w.p.n1_pad * 64 +
         2 * 3 * (size_t)w.comps * w.p.n1_pad + 4 * 256;
}

gp_status split_carve(SplitWork& w, int d, Arena& ar) {
  GP_TRY(split::carve(w.p, d, ar));
  w.H = ar.take<_Float16>((size_t)w.p.n1_pad * 64);
  w.Zt = w.comps ? ar.take<_Float16>(3 * (size_t)w.comps * w.p.n1_pad) : nullptr;
  if (!w.H || (w.comps && !w.Zt)) return set_error(GP_ERR_NOMEM, "internal: gradient workspace sizing");
  return GP_OK;
}

gp_status split_launch(const SplitWork& w, const KParams& kp, bool iso, const float* X, int64_t n,
                       const float* U, const float* B, int r, float inv2m, const float* scl,
                       double* part, hipStream_t s) {
  const int64_t n_pad = w.p.n1_pad;
  parts_kernel<<<(unsigned)ceil_div(n_pad * 8, (int64_t)256), 256, 0, s>>>(U, B, n, n_pad, r, inv2m,
                                                                           scl, w.p.info, w.H);
  GP_HIP(hipGetLastError());
  if (w.comps) {
    coord_kernel<<<dim3((unsigned)ceil_div(n_pad, (int64_t)256), w.comps), 256, 0, s>>>(
        X, n, n_pad, kp, w.comps, w.p.info, w.Zt);
    GP_HIP(hipGetLastError());
  }
  const GradFn fn = kp.kind == GP_KERNEL_RBF        ? grad_fn<GP_KERNEL_RBF>(kp.d, iso)
                    : kp.kind == GP_KERNEL_MATERN52 ? grad_fn<GP_KERNEL_MATERN52>(kp.d, iso)
                                                    : grad_fn<GP_KERNEL_MATERN32>(kp.d, iso);
  fn<<<(unsigned)(w.rblocks * w.nsplit), 256, 0, s>>>(w.p.Xr, w.p.Xc, w.H, w.Zt, X, w.p.info, scl,
                                                     n, n_pad, kp, part, w.nsplit);
  GP_HIP(hipGetLastError());
  return GP_OK;
}

}  // namespace grad
}  // namespace gpmi
