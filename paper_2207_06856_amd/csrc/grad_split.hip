// Gradient reduction (grad.hip's sums, over the whole row range) on split
// operands.  Per entry the vector unit forms the kernel value and P = G W~ in
// float32; what grows with d is on the matrix cores:
//   * r^2 from exact integer products (split_tile.h);
//   * W~ = W + W^T from the binary16 split of U and C, as in grad.hip;
//   * S_m = sum_ij P_ij (a_im - b_jm)^2 = sum_i [a_im^2 p_i - 2 a_im Z_im + Y_im],
//     p_i = sum_j P_ij, Z = P b, Y = P b^2, in float64 throughout: the float32 P
//     is widened, b = (x - c) / l about the centre c of the points' box is held
//     in float64, and every product is summed there.
// The squares cancel by (|a| / |a - b|)^2, whatever the box: for clustered points
// far from the centre that is 10^6 and more, which no 16-bit parts and no float32
// sum can carry.  In float64 it costs 2^-53 (|a| / |a - b|)^2 of a term, where the
// difference form's float32 coordinates cost 2^-24 |a| / |a - b|: less down to
// |a - b| of 2^-29 |a|, where both have lost the difference.  Up to four inputs the
// sixteen-wide float64 products would be mostly padding, and P (a - b)^2 is summed
// from differences of centred float32 coordinates, as in grad.hip.  The error
// against float64 is below the difference form's on spreads from 1 to 30
// lengthscales, tight clusters and one large target among ordinary ones (2e-7 and
// less of sum |dK||W|, where that form reaches 5e-5 on Matern-3/2 clusters); equal,
// near 1e-8, on standard normal points.
// Where the box is wide (kSplitMaxRadius) or an input is not finite, grad.hip's
// kernel runs instead.
//
// Bound by issue: of 600 cycles of a SIMD per 256 evaluated entries at N = 100,000,
// d = 8, R = 16 (RBF, one lengthscale per input) the float64 products take 256, during
// which nothing else proceeds (interleaving them with the next tile's vector work by
// hand changed nothing).  The whole call against the difference form: 4.80 ms for 5.62;
// N = 60,000 1.25 for 1.43 (d = 4) and 2.67 for 4.89 (d = 12); N = 20,000, Matern-5/2,
// 0.51 for 0.92 (d = 16).

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

typedef double d2 __attribute__((ext_vector_type(2)));
typedef double d4 __attribute__((ext_vector_type(4)));

namespace {

// 16-row subtiles per wave: four where their operands leave two waves per SIMD
__host__ __device__ constexpr int row_subtiles(int kc, int zw) {
  return zw < 8 && kc == 2 ? 4 : 2;
}
constexpr int kStage = split::kStageCols;        // 64 columns per LDS stage
constexpr int kHS = 64 + 8;                      // LDS row stride of the U, C parts (halfs)

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

// Zb[j][m] = b_jm for m < d, zero elsewhere.
template <typename T>
__global__ __launch_bounds__(256) void coord_kernel(const float* __restrict__ X, int64_t n,
                                                    int64_t n_pad, KParams kp, int width,
                                                    const Info* __restrict__ info,
                                                    T* __restrict__ Zb) {
  if (!info->ok) return;
  const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int64_t j = t / width;
  const int m = (int)(t - j * width), d = kp.d;
  if (j >= n_pad) return;
  Zb[t] = j < n && m < d ? (T)(((double)X[j * d + m] - info->centre[m]) / (double)kp.ls[m]) : (T)0;
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

// ZW: the coordinates held of a point, d at least.  0: one isotropic lengthscale,
// whose sum is P r^2; 4: differences of float32 coordinates; 8: one block of float64
// products, b in its lower eight components and b^2 in the others; 16: two blocks,
// b and b^2.  A work group of 4 waves owns 64 NSUB rows and a run of column stages
// from its own first row on; past its own rows W takes the mirrored products as
// well.  Lane layout of every tile: row l16, columns 4 g + v (the A operand is the
// column side), and float64 product v takes the columns {4 g + v}: A is P, B
// component l16 of that column, D row g + 4 v, component l16.  MFMA sums are about
// 0.02 ulp low on average; the odd subtiles' U and C rows are negated, so that they
// carry -W and -P and the two halves' shares cancel in the sums.
template <int KIND, int KC, int ZW>
__global__ __launch_bounds__(256, 2) void grad_split_kernel(
    const _Float16* __restrict__ Xr, const _Float16* __restrict__ Xc,
    const _Float16* __restrict__ H, const void* __restrict__ Zv, const Info* __restrict__ info,
    const float* __restrict__ scl, int64_t n_pad, KParams kp, double* __restrict__ part,
    int nsplit) {
  if (!info->ok) return;
  constexpr bool ISO = ZW == 0, DIFF = ZW == 4, F64 = ZW >= 8;
  constexpr int NSUB = row_subtiles(KC, ZW);
  constexpr int KP = 32 * KC, XS = KP + 8, RB = 64 * NSUB;
  constexpr int NZ = ZW == 16 ? 2 : 1;
  constexpr int ZS = ZW + 4;                     // LDS stride of a column's coordinates
  constexpr int CS = kStage + 4;                 // and of one input's in the difference form
  constexpr int XPT = kStage * KP / 8 / 256;     // 16-byte chunks per thread
  constexpr int HPT = kStage * 64 / 8 / 256;
  constexpr int ZPT = F64 ? kStage * ZW / 2 / 256 : 1;
  // 16-column tiles in flight: two where the registers hold them
  constexpr int kUnroll = ISO || (F64 && KIND == GP_KERNEL_RBF) ? 2 : 1;
  const double* Zb = static_cast<const double*>(Zv);
  __shared__ __attribute__((aligned(16))) _Float16 sX[2][kStage * XS];
  __shared__ __attribute__((aligned(16))) _Float16 sH[2][kStage * kHS];
  __shared__ __attribute__((aligned(16))) double sZ[2][F64 ? kStage * ZS : 2];
  __shared__ __attribute__((aligned(16))) float sC[2][DIFF ? 4 * CS : 4];
  __shared__ double sRed[4][16 + 1];
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
  d4 acc[NSUB][NZ];
  double p[NSUB];
  float ac[NSUB][4], dm[4];                      // difference form: row coordinates, sums
  float pk = 0.0f, acck = 0.0f, accr = 0.0f;
#pragma unroll
  for (int m = 0; m < 4; ++m) {
    dm[m] = 0.0f;
    if constexpr (DIFF)
#pragma unroll
      for (int q = 0; q < NSUB; ++q)
        ac[q][m] = static_cast<const float*>(Zv)[(row0 + q * 16 + l16) * 4 + m];
  }
#pragma unroll
  for (int q = 0; q < NSUB; ++q) {
    p[q] = 0.0;
#pragma unroll
    for (int z = 0; z < NZ; ++z) acc[q][z] = d4{0.0, 0.0, 0.0, 0.0};
  }

  const int64_t nstage = n_pad / kStage;
  const int64_t s0 = rowb / kStage, own_end = s0 + RB / kStage;
  const int64_t sb = s0 + spl * (nstage - s0) / nsplit, se = s0 + (spl + 1) * (nstage - s0) / nsplit;
  h8 xreg[XPT], hreg[HPT];
  d2 zreg[ZPT];
  float creg;
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
    if constexpr (F64) {
#pragma unroll
      for (int e = 0; e < ZPT; ++e)
        zreg[e] = *reinterpret_cast<const d2*>(Zb + j0 * ZW + 2 * (tid + e * 256));
    }
    if constexpr (DIFF) creg = static_cast<const float*>(Zv)[j0 * 4 + tid];
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
    if constexpr (DIFF) sC[buf][(tid & 3) * CS + (tid >> 2)] = creg;
    if constexpr (F64) {
#pragma unroll
      for (int e = 0; e < ZPT; ++e) {
        const int ch = tid + e * 256, row = ch / (ZW / 2), col = ch % (ZW / 2);
        *reinterpret_cast<d2*>(&sZ[buf][row * ZS + 2 * col]) = zreg[e];
      }
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
    for (int jb = 0; jb < kStage / 16; ++jb) {
      const int col = jb * 16 + l16;
      h8 a[KC], bw[3];
#pragma unroll
      for (int kc = 0; kc < KC; ++kc)
        a[kc] = *reinterpret_cast<const h8*>(Xs + col * XS + kc * 32 + g * 8);
      // [C_hi ; C_hi], [C_lo ; U_hi] (second half mirror only), [U_hi ; U_lo] (mirror only)
      const _Float16* Hc = Hs + col * kHS + 8 * gl;
      bw[0] = *reinterpret_cast<const h8*>(Hc + 32);
      bw[1] = (gh && !mirror) ? z8 : *reinterpret_cast<const h8*>(Hc + (gh ? 0 : 48));
      bw[2] = *reinterpret_cast<const h8*>(Hc + (gh ? 16 : 0));
      double zb[NZ][4];
      f4 bc[4];
      if constexpr (DIFF)
#pragma unroll
        for (int m = 0; m < 4; ++m)
          bc[m] = *reinterpret_cast<const f4*>(&sC[buf][m * CS + jb * 16 + 4 * g]);
      if constexpr (F64) {
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const double b = sZ[buf][(jb * 16 + 4 * g + v) * ZS + (l16 & (ZW - 1))];
          if constexpr (ZW == 8) {
            zb[0][v] = b * (l16 < 8 ? 1.0 : b);
          } else {
            zb[0][v] = b;
            zb[NZ - 1][v] = b * b;
          }
        }
      }
#pragma unroll
      for (int q = 0; q < NSUB; ++q) {
        const f4 D = split::sqdist<KC>(a, bi[q]);
        f4 W = f4{0.f, 0.f, 0.f, 0.f};
        W = f16::mfma32<_Float16>(bw[0], aw[q][0], W);
        W = f16::mfma32<_Float16>(bw[1], aw[q][1], W);
        if (mirror) {
          W = f16::mfma32<_Float16>(bw[2], aw[q][2], W);
        } else {
          // the diagonal adds nothing to the S_m; its kappa(0) W_ii is added at the end
          const int off = (int)(row0 - st * kStage) + q * 16 + l16 - (jb * 16 + 4 * g);
#pragma unroll
          for (int v = 0; v < 4; ++v) W[v] = off == v ? 0.0f : W[v];
        }
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          float kap, G;
          kval_deriv_split<KIND>(D[v], cs, kap, G);
          const float P = G * W[v];
          if constexpr (KIND != GP_KERNEL_RBF) acck = fmaf(q & 1 ? -kap : kap, W[v], acck);
          if constexpr (!F64 && KIND == GP_KERNEL_RBF) pk = q & 1 ? pk - P : pk + P;
          if constexpr (ISO) accr = q & 1 ? fmaf(-P, D[v], accr) : fmaf(P, D[v], accr);
          if constexpr (DIFF) {
#pragma unroll
            for (int m = 0; m < 4; ++m) {
              const float dl = ac[q][m] - bc[m][v], t = P * dl;
              dm[m] = q & 1 ? fmaf(-t, dl, dm[m]) : fmaf(t, dl, dm[m]);
            }
          }
          if constexpr (F64) {
            const double Pd = (double)P;
            p[q] += Pd;
#pragma unroll
            for (int z = 0; z < NZ; ++z)
              acc[q][z] = __builtin_amdgcn_mfma_f64_16x16x4f64(Pd, zb[z][v], acc[q][z], 0, 0, 0);
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
  double kk = (double)acck + (double)pk;
  if constexpr (KIND == GP_KERNEL_RBF && F64)
#pragma unroll
    for (int q = 0; q < NSUB; ++q) kk += q & 1 ? -p[q] : p[q];
  kk = wave_sum64(kk);
  if (lane == 0) sRed[wave][16] = kk;
  if constexpr (ISO) {
    const double s = wave_sum64((double)accr);
    if (lane == 0) sRed[wave][0] = s;
  } else if constexpr (DIFF) {
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      const double s = wave_sum64((double)dm[m]);
      if (lane == 0) sRed[wave][m] = s;
    }
  } else {
    auto coord = [&](int64_t i, int m) { return m < d ? Zb[i * ZW + m] : 0.0; };
    const int c = l16 & (ZW - 1);
    const bool square = ZW == 8 && l16 >= 8;     // this lane's block-0 component is b^2
    double s = 0.0;
#pragma unroll
    for (int q = 0; q < NSUB; ++q)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const double sg = q & 1 ? -1.0 : 1.0;
        const double f = square ? 1.0 : -2.0 * coord(row0 + q * 16 + g + 4 * v, c);
        s += sg * f * acc[q][0][v];
        if constexpr (ZW == 16) s += sg * acc[q][NZ - 1][v];
      }
    if constexpr (ZW == 8) s += __shfl_xor(s, 8);
    s += __shfl_xor(s, 16);
    s += __shfl_xor(s, 32);
    if (lane < d) sRed[wave][lane] = s;
    __syncthreads();
    double ps[NSUB];
#pragma unroll
    for (int q = 0; q < NSUB; ++q) {
      ps[q] = q & 1 ? -p[q] : p[q];
      ps[q] += __shfl_xor(ps[q], 16);
      ps[q] += __shfl_xor(ps[q], 32);
    }
    // lane group g takes dimensions g, g + 4, ...; its 16 lanes are 16 rows
    for (int m = g; m < ((d + 3) & ~3); m += 4) {
      double t = 0.0;
#pragma unroll
      for (int q = 0; q < NSUB; ++q) {
        const double x = coord(row0 + q * 16 + l16, m);
        t += x * x * ps[q];
      }
#pragma unroll
      for (int o = 8; o > 0; o >>= 1) t += __shfl_xor(t, o, 64);
      if (m < d && l16 == 0) sRed[wave][m] += t;
    }
  }
  __syncthreads();
  const int nacc = ISO ? 1 : d;
  if (tid <= nacc) {
    const int k = tid < nacc ? tid : 16;
    double s = ((sRed[0][k] + sRed[1][k]) + sRed[2][k]) + sRed[3][k];
    if (ISO && tid == 0) s /= info->inv_u * info->inv_u;
    part[(int64_t)blockIdx.x * (nacc + 1) + tid] = s * unscale;
  }
}

typedef void (*GradFn)(const _Float16*, const _Float16*, const _Float16*, const void*,
                       const Info*, const float*, int64_t, KParams, double*, int);
template <int KIND>
GradFn grad_fn(int d, bool iso) {
  const int kc = split::operand_chunks(d);
  if (iso)
    return kc == 2 ? &grad_split_kernel<KIND, 2, 0>
                   : kc == 3 ? &grad_split_kernel<KIND, 3, 0> : &grad_split_kernel<KIND, 4, 0>;
  if (d <= 4) return &grad_split_kernel<KIND, 2, 4>;
  if (kc == 2) return &grad_split_kernel<KIND, 2, 8>;
  if (kc == 3) return d <= 8 ? &grad_split_kernel<KIND, 3, 8> : &grad_split_kernel<KIND, 3, 16>;
  return &grad_split_kernel<KIND, 4, 16>;
}

int width_of(int d, bool iso) { return iso ? 0 : d <= 4 ? 4 : d <= 8 ? 8 : 16; }

}  // namespace

bool use_split(int kind, int64_t n, int d, bool iso, int r, int64_t rows) {
  if (kind == GP_KERNEL_MATERN12 || d > kGradSplitMaxDim || r > 16 || rows != n) return false;
  return n >= split_min_points(d, iso);
}

SplitWork split_plan(int64_t n, int d, bool iso) {
  SplitWork w{};
  w.p = split::plan(n, n, d, 1, true, 1, split::kSplitMaxRadius);
  const int64_t rb = w.p.n1_pad / (64 * row_subtiles(w.p.kc, width_of(d, iso)));
  w.rblocks = rb;
  // about 3000 work groups of at least two stages on average
  const int64_t most = std::max<int64_t>(1, w.p.n2_pad / kStage / 4);
  w.nsplit = (int)std::max<int64_t>(1, std::min<int64_t>(std::min<int64_t>(64, ceil_div(3072, rb)), most));
  w.width = width_of(d, iso);
  return w;
}

size_t split_bytes(const SplitWork& w, int d) {
  return split::operand_bytes(w.p, d) + 2 * (size_t)w.p.n1_pad * 64 +
         8 * (size_t)w.width * w.p.n1_pad + 4 * 256;
}

gp_status split_carve(SplitWork& w, int d, Arena& ar) {
  GP_TRY(split::carve(w.p, d, ar));
  w.H = ar.take<_Float16>((size_t)w.p.n1_pad * 64);
  w.Zb = w.width ? ar.take<double>((size_t)w.width * w.p.n1_pad) : nullptr;
  if (!w.H || (w.width && !w.Zb)) return set_error(GP_ERR_NOMEM, "internal: gradient workspace sizing");
  return GP_OK;
}

gp_status split_launch(const SplitWork& w, const KParams& kp, bool iso, const float* X, int64_t n,
                       const float* U, const float* B, int r, float inv2m, const float* scl,
                       double* part, hipStream_t s) {
  const int64_t n_pad = w.p.n1_pad;
  parts_kernel<<<(unsigned)ceil_div(n_pad * 8, (int64_t)256), 256, 0, s>>>(U, B, n, n_pad, r, inv2m,
                                                                           scl, w.p.info, w.H);
  GP_HIP(hipGetLastError());
  if (w.width) {
    const unsigned blocks = (unsigned)ceil_div(n_pad * w.width, (int64_t)256);
    if (w.width == 4)
      coord_kernel<<<blocks, 256, 0, s>>>(X, n, n_pad, kp, w.width, w.p.info,
                                          reinterpret_cast<float*>(w.Zb));
    else
      coord_kernel<<<blocks, 256, 0, s>>>(X, n, n_pad, kp, w.width, w.p.info, w.Zb);
    GP_HIP(hipGetLastError());
  }
  const GradFn fn = kp.kind == GP_KERNEL_RBF        ? grad_fn<GP_KERNEL_RBF>(kp.d, iso)
                    : kp.kind == GP_KERNEL_MATERN52 ? grad_fn<GP_KERNEL_MATERN52>(kp.d, iso)
                                                    : grad_fn<GP_KERNEL_MATERN32>(kp.d, iso);
  fn<<<(unsigned)(w.rblocks * w.nsplit), 256, 0, s>>>(w.p.Xr, w.p.Xc, w.H, w.Zb, w.p.info, scl,
                                                     n_pad, kp, part, w.nsplit);
  GP_HIP(hipGetLastError());
  return GP_OK;
}

}  // namespace grad
}  // namespace gpmi
