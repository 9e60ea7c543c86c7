// Float32 kernel-matrix product on the matrix cores (GP_PREC_FP32; Eq. mvm):
// float32 kernel entries, float32 products and sums, as the vector-unit form in
// kmvm_valu.hip, with both contractions moved to 16-bit MFMAs that lose nothing:
//   * the squared distances come from exact integer products plus a small
//     remainder (split_tile.h);
//   * the entry k and the right-hand side v are cut into three bfloat16 parts of 8
//     bits each that hold all 24 bits, k's by truncation, v's each the nearest to
//     what is left: k v = k1 v1 + k1 v2 + k2 v1 + k1 v3 + k2 v2 + k3 v1 leaves out
//     k3 v2 + k2 v3 + k3 v3, at most 1.5 2^-23 of k v and of the sign of v2 and v3,
//     which differs from column to column.  (With v cut off too it is 2^-21 and
//     always in one direction, 6e-8 of a same-sign sum; with k rounded too, 2^-24
//     for 6% of the launch.)  bfloat16 has float32's range, so no scaling is needed;
//     the third part is normal, and the 24 bits whole, from about 2^-110 on.
// Per 16 x 16 tile of entries that is KC + 3 RB MFMAs of 16 cycles and, per
// entry, the addition of the distance's two sums, one multiplication, the
// exponential and 5.5 operations for the parts, against 2 d + 16 RB vector
// operations and the library expf of the vector form.  With at most four
// right-hand sides the parts cost more than the sums they feed, and each lane adds
// its entries' products by float32 FMAs instead.
// Bound by issue: at N = 40,011, d = 8, R = 16 (RBF) the launch takes 285 cycles
// of a SIMD per 256 entries, where the matrix cores' 96 and the vector unit's
// 157 add up to 253.  Product calls there, against the vector form: 0.76 ms
// from 1.85 (d = 8, R = 16), 0.31 from 1.02 (d = 3, R = 1), 1.14 from 3.55
// (Matern-5/2, d = 16, R = 16); N = 20,000: 0.38 from 1.75 (d = 12, R = 32).  The
// relative error against float64 falls from 7.3e-7 to 3.9e-7: a lane's chain of
// sums is a thirty-second as long.

#include <math.h>

#include <algorithm>
#include <type_traits>

#include "device_common.h"
#include "split_tile.h"

namespace gpmi {
namespace split {

typedef __bf16 b8 __attribute__((ext_vector_type(8)));
typedef __bf16 b4 __attribute__((ext_vector_type(4)));
typedef uint32_t u4 __attribute__((ext_vector_type(4)));

// ---- bounding box, unit and operands ----------------------------------------
// Per-group minimum and maximum of every input over the two sets (groups
// [0, g1) read X1, the rest X2); a non-finite input makes the maximum NaN.
__global__ __launch_bounds__(256) void box_kernel(const float* __restrict__ X1, int64_t n1,
                                                  const float* __restrict__ X2, int64_t n2, int d,
                                                  int g1, float* __restrict__ part) {
  __shared__ float lo[256], hi[256];
  const bool first = (int)blockIdx.x < g1;
  const float* X = first ? X1 : X2;
  const int64_t n = first ? n1 : n2;
  const int64_t grp = first ? blockIdx.x : blockIdx.x - g1;
  const int64_t groups = first ? g1 : gridDim.x - g1;
  const int rows = 256 / d;                     // rows per pass of the group
  const int m = threadIdx.x % d, ro = threadIdx.x / d;
  float mn = INFINITY, mx = -INFINITY;
  if (ro < rows) {
    for (int64_t i = grp * rows + ro; i < n; i += groups * rows) {
      const float x = X[i * d + m];
      mn = x < mn ? x : mn;
      mx = isfinite(x) && !isnan(mx) ? (x > mx ? x : mx) : NAN;
    }
  }
  lo[threadIdx.x] = mn;
  hi[threadIdx.x] = mx;
  __syncthreads();
  if ((int)threadIdx.x < d) {
    for (int q = 1; q < rows; ++q) {
      const float a = lo[q * d + threadIdx.x], b = hi[q * d + threadIdx.x];
      mn = a < mn ? a : mn;
      mx = !isnan(b) && !isnan(mx) ? (b > mx ? b : mx) : NAN;
    }
    part[(int64_t)blockIdx.x * 2 * d + threadIdx.x] = mn;
    part[(int64_t)blockIdx.x * 2 * d + d + threadIdx.x] = mx;
  }
}

// One group: the box's centre, the unit u and the exponent scale; ok = 0 when
// the inputs are not finite or the box is too wide for this form.
__global__ __launch_bounds__(256) void info_kernel(const float* __restrict__ part, int groups,
                                                   KParams kp, double arg, float radius,
                                                   Info* __restrict__ o) {
  __shared__ float lo[4][kMaxDim], hi[4][kMaxDim];
  __shared__ double half2[kMaxDim];
  const int m = threadIdx.x & 63, q = threadIdx.x >> 6, d = kp.d;
  float mn = INFINITY, mx = -INFINITY;
  if (m < d) {
#pragma unroll 8
    for (int b = q; b < groups; b += 4) {
      const float a = part[(int64_t)b * 2 * d + m], c = part[(int64_t)b * 2 * d + d + m];
      mn = a < mn ? a : mn;
      mx = !isnan(c) && !isnan(mx) ? (c > mx ? c : mx) : NAN;
    }
  }
  lo[q][m] = mn;
  hi[q][m] = mx;
  __syncthreads();
  if (q == 0 && m < d) {
    for (int w = 1; w < 4; ++w) {
      mn = lo[w][m] < mn ? lo[w][m] : mn;
      mx = !isnan(hi[w][m]) && !isnan(mx) ? (hi[w][m] > mx ? hi[w][m] : mx) : NAN;
    }
    o->centre[m] = 0.5 * ((double)mn + (double)mx);
    const double h = 0.5 * ((double)mx - (double)mn) / (double)kp.ls[m];
    half2[m] = h * h;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    double r2 = 0.0;
    for (int k = 0; k < d; ++k) r2 += half2[k];
    const bool ok = r2 <= (double)radius * radius;   // false for NaN
    // |arg| u^2 is a power of two >= |arg| (R / 2000)^2: the exponent argument
    // is then an exact multiple of r^2 / u^2
    int e = -100;
    if (ok && r2 > 0.0) {
      const double f = frexp(fabs(arg) * r2 / 4e6, &e);  // f 2^e, f in [1/2, 1)
      if (f == 0.5) --e;
      if (e < -100) e = -100;                            // all points (nearly) equal
    }
    o->inv_u = sqrt(ldexp(fabs(arg), -e));
    o->cs = copysignf(ldexpf(1.0f, e), (float)arg);
    o->ok = ok ? 1 : 0;
  }
}

constexpr int kPrepPoints = 32;

// Operand rows of 32 points: out0 as output rows, out1 as columns (either may
// be null).  Rows n .. n_pad - 1 are zero.
__global__ __launch_bounds__(256) void prep_kernel(const float* __restrict__ X, int64_t n,
                                                   int64_t n_pad, KParams kp, int width,
                                                   const Info* __restrict__ info,
                                                   _Float16* __restrict__ out0,
                                                   _Float16* __restrict__ out1) {
  if (!info->ok) return;
  __shared__ double f[kPrepPoints][kSplitMaxDim];
  __shared__ float q[kPrepPoints][kSplitMaxDim];
  __shared__ _Float16 f1[kPrepPoints][kSplitMaxDim], f2[kPrepPoints][kSplitMaxDim];
  __shared__ float nq[kPrepPoints][2];
  __shared__ _Float16 gp[kPrepPoints][3];
  const int d = kp.d;
  const int64_t i0 = (int64_t)blockIdx.x * kPrepPoints;
  const double inv_u = info->inv_u;
  for (int e = threadIdx.x; e < kPrepPoints * d; e += 256) {
    const int p = e / d, m = e - p * d;
    double a = 0.0;
    if (i0 + p < n) a = ((double)X[(i0 + p) * d + m] - info->centre[m]) / (double)kp.ls[m] * inv_u;
    const double qi = rint(a), fr = a - qi;
    q[p][m] = (float)qi;
    f[p][m] = fr;
    const _Float16 h = (_Float16)(float)fr;
    f1[p][m] = h;
    f2[p][m] = (_Float16)(float)(fr - (double)(float)h);
  }
  __syncthreads();
  if (threadIdx.x < kPrepPoints) {
    const int p = threadIdx.x;
    int N = 0;
    double G = 0.0;
    for (int m = 0; m < d; ++m) {
      const double qi = (double)q[p][m], fr = f[p][m];
      N += (int)q[p][m] * (int)q[p][m];
      G += fr * (2.0 * qi + fr);
    }
    nq[p][0] = (float)(N & 2047);
    nq[p][1] = (float)(N >> 11);
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      const _Float16 h = (_Float16)(float)G;
      gp[p][k] = h;
      G -= (double)(float)h;
    }
  }
  __syncthreads();
  const int chunks = width / 8;
  for (int e = threadIdx.x; e < kPrepPoints * chunks; e += 256) {
    const int p = e / chunks, c = e - p * chunks;
    const int64_t i = i0 + p;
    if (i >= n_pad) continue;
    h8 o0, o1;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const int s = c * 8 + k;
      float v0 = 0.0f, v1 = 0.0f;
      if (i < n) {
        if (s < d) {
          v0 = q[p][s];
          v1 = -2.0f * v0;
        } else if (s < d + 4) {
          const int w = s - d;
          v0 = w == 0 ? 1.0f : w == 1 ? 2048.0f : nq[p][w - 2];
          v1 = w == 2 ? 1.0f : w == 3 ? 2048.0f : nq[p][w];
        } else if (s >= 32) {
          const int t = s - 32;
          if (t < 5 * d) {
            const int b = t / d, m = t - b * d;
            v0 = b < 2 ? q[p][m] : b == 3 ? (float)f2[p][m] : (float)f1[p][m];
            v1 = -2.0f * (b == 2 || b == 3 ? q[p][m] : b == 1 ? (float)f2[p][m] : (float)f1[p][m]);
          } else if (t < 5 * d + 6) {
            const int w = t - 5 * d;
            v0 = w < 3 ? 1.0f : (float)gp[p][w - 3];
            v1 = w < 3 ? (float)gp[p][w] : 1.0f;
          }
        }
      }
      o0[k] = (_Float16)v0;
      o1[k] = (_Float16)v1;
    }
    if (out0) *reinterpret_cast<h8*>(out0 + i * width + c * 8) = o0;
    if (out1) *reinterpret_cast<h8*>(out1 + i * width + c * 8) = o1;
  }
}

// The same in the fine form.
__global__ __launch_bounds__(256) void prep_fine_kernel(const float* __restrict__ X, int64_t n,
                                                        int64_t n_pad, KParams kp, int width,
                                                   const Info* __restrict__ info,
                                                   _Float16* __restrict__ out0,
                                                   _Float16* __restrict__ out1) {
  if (!info->ok) return;
  __shared__ float q[kPrepPoints][kSplitMaxDim], f[kPrepPoints][kSplitMaxDim];
  __shared__ float E[kPrepPoints][kSplitMaxDim];
  __shared__ float nq[kPrepPoints][2];
  __shared__ _Float16 hp[kPrepPoints][3];
  const int d = kp.d;
  const int64_t i0 = (int64_t)blockIdx.x * kPrepPoints;
  const double inv_u = info->inv_u;
  for (int e = threadIdx.x; e < kPrepPoints * d; e += 256) {
    const int p = e / d, m = e - p * d;
    double a = 0.0;
    if (i0 + p < n) a = ((double)X[(i0 + p) * d + m] - info->centre[m]) / (double)kp.ls[m] * inv_u;
    const double qi = rint(a), fi = rint((a - qi) * 1024.0) / 1024.0;
    q[p][m] = (float)qi;
    f[p][m] = (float)fi;
    E[p][m] = (float)(_Float16)(float)((a - qi - fi) * 2048.0);
  }
  __syncthreads();
  if (threadIdx.x < kPrepPoints) {
    const int p = threadIdx.x;
    int N = 0;
    double G = 0.0, H = 0.0;
    for (int m = 0; m < d; ++m) {
      const double qi = (double)q[p][m], fi = (double)f[p][m], ei = (double)E[p][m] / 2048.0;
      N += (int)q[p][m] * (int)q[p][m];
      G += 2.0 * qi * fi;
      H += 2.0 * qi * ei + fi * (fi + 2.0 * ei);
    }
    const double Gi = rint(G);
    H += G - Gi;
    N += (int)Gi;                                // >= -|f|^2: |q + f|^2 is not negative
    nq[p][0] = (float)(N & 2047);
    nq[p][1] = (float)(N >> 11);
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      const _Float16 h = (_Float16)(float)H;
      hp[p][k] = h;
      H -= (double)(float)h;
    }
  }
  __syncthreads();
  const int chunks = width / 8, rest = 32 * (1 + f_chunks(d));
  for (int e = threadIdx.x; e < kPrepPoints * chunks; e += 256) {
    const int p = e / chunks, c = e - p * chunks;
    const int64_t i = i0 + p;
    if (i >= n_pad) continue;
    h8 o0, o1;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const int s = c * 8 + k;
      float v0 = 0.0f, v1 = 0.0f;
      if (i < n) {
        if (s < d) {
          v0 = q[p][s];
          v1 = -2.0f * v0;
        } else if (s < d + 4) {
          const int w = s - d;
          v0 = w == 0 ? 1.0f : w == 1 ? 2048.0f : nq[p][w - 2];
          v1 = w == 2 ? 1.0f : w == 3 ? 2048.0f : nq[p][w];
        } else if (s >= 32 && s < rest) {
          const int t = s - 32, m = t < d ? t : t - d;
          if (t < 2 * d) {
            v0 = t < d ? q[p][m] : f[p][m];
            v1 = -2.0f * (t < d ? f[p][m] : q[p][m]);
          }
        } else if (s >= rest) {
          const int t = s - rest;
          if (t < 5 * d) {
            const int b = t / d, m = t - b * d;
            const float q2 = q[p][m] / 2048.0f, f5 = f[p][m] / 32.0f, e6 = E[p][m] / 64.0f;
            v0 = b == 0 ? q2 : b == 1 ? E[p][m] : b == 2 ? f[p][m] : b == 3 ? f5 : e6;
            v1 = -2.0f * (b == 0 ? E[p][m] : b == 1 ? q2 : b == 2 ? f[p][m] : b == 3 ? e6 : f5);
          } else if (t < 5 * d + 6) {
            const int w = t - 5 * d;
            v0 = w < 3 ? 1.0f : (float)hp[p][w - 3];
            v1 = w < 3 ? (float)hp[p][w] : 1.0f;
          }
        }
      }
      o0[k] = (_Float16)v0;
      o1[k] = (_Float16)v1;
    }
    if (out0) *reinterpret_cast<h8*>(out0 + i * width + c * 8) = o0;
    if (out1) *reinterpret_cast<h8*>(out1 + i * width + c * 8) = o1;
  }
}

// ---- the fused product -------------------------------------------------------
constexpr int JT = kStageCols;
constexpr int kVS = JT + 4;                    // LDS row stride of a right-hand-side part

// three truncated 8-bit parts of eight non-negative floats
__device__ __forceinline__ void parts3(const float (&k)[8], b8 (&o)[3]) {
  uint32_t a[8], b[8], c[8];
#pragma unroll
  for (int v = 0; v < 8; ++v) {
    a[v] = __float_as_uint(k[v]);
    const float r = k[v] - __uint_as_float(a[v] & 0xffff0000u);
    b[v] = __float_as_uint(r);
    c[v] = __float_as_uint(r - __uint_as_float(b[v] & 0xffff0000u));
  }
  u4 p[3];
#pragma unroll
  for (int h = 0; h < 4; ++h) {
    p[0][h] = __builtin_amdgcn_perm(a[2 * h + 1], a[2 * h], 0x07060302u);
    p[1][h] = __builtin_amdgcn_perm(b[2 * h + 1], b[2 * h], 0x07060302u);
    p[2][h] = __builtin_amdgcn_perm(c[2 * h + 1], c[2 * h], 0x07060302u);
  }
#pragma unroll
  for (int q = 0; q < 3; ++q) o[q] = __builtin_bit_cast(b8, p[q]);
}

// A work group of 4 waves owns 64 NSUB rows (operands in registers) and a run
// of 64-column stages; columns and right-hand sides go through two LDS stages,
// the right-hand sides cut into parts as they are staged.  An infinite
// right-hand side only multiplies the first part of the entry (the others may
// be zero): once a stage has held one, the other products take 0 for it.
// Partial sums to part[split][row][16 RB].
// RB = 0: RT <= 4 right-hand sides by FMAs; each lane sums the columns
// 4 g + v of its row, the four lanes of a row are added at the end, and the
// partial sums are part[split][row][RT].
template <int KIND, int KC, int RB, int RT>
__global__ __launch_bounds__(256, 2) void main_kernel(const _Float16* __restrict__ Xr,
                                                   const _Float16* __restrict__ Xc,
                                                   const float* __restrict__ V, int r, int c0,
                                                   int64_t n2, float* __restrict__ part,
                                                   int64_t n1_pad, int nsplit, int64_t nstage,
                                                   const Info* __restrict__ info, int same,
                                                   const int* __restrict__ live) {
  if (live && *live == 0) return;
  if (!info->ok) return;
  constexpr int NSUB = subtiles(KC);
  constexpr int KP = 32 * KC, XS = KP + 8, RP = RB ? 16 * RB : RT;
  constexpr int XPT = JT * KP / 8 / 256;       // 16-byte chunks of a column stage per thread
  constexpr int VPT = (JT * RP + 255) / 256;   // right-hand-side values per thread
  __shared__ __attribute__((aligned(16))) _Float16 sX[2][JT * XS];
  __shared__ __attribute__((aligned(16))) __bf16 sV[2][3][RB ? RP * kVS : 1];
  __shared__ __attribute__((aligned(16))) float sF[2][RB ? 1 : RP * kVS];
  __shared__ int sInf;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, g = lane >> 4, l16 = lane & 15;
  const int split = blockIdx.x % nsplit;
  const int64_t row0 = (int64_t)(blockIdx.x / nsplit) * (64 * NSUB) + wave * 16 * NSUB;
  const int64_t sb = split * nstage / nsplit, se = (split + 1) * nstage / nsplit;
  const float cs = info->cs;
  const int rc = min(RP, r - c0);

  h8 bi[NSUB][KC];
#pragma unroll
  for (int q = 0; q < NSUB; ++q)
#pragma unroll
    for (int kc = 0; kc < KC; ++kc)
      bi[q][kc] = *reinterpret_cast<const h8*>(Xr + (row0 + q * 16 + l16) * KP + kc * 32 + g * 8);
  f4 acc[NSUB][RB ? RB : 1];
  float sum[NSUB][RT ? RT : 1];
#pragma unroll
  for (int q = 0; q < NSUB; ++q) {
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) acc[q][rb] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int c = 0; c < RT; ++c) sum[q][c] = 0.0f;
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
      const int ch = tid + e * 256, jj = ch / RP, c = ch % RP;
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
      const int ch = tid + e * 256, jj = ch / RP, c = ch % RP;
      const float v = vreg[e];
      if constexpr (RB == 0) {
        if (ch < JT * RP) sF[buf][c * kVS + jj] = v;
        continue;
      }
      __bf16 v1 = (__bf16)v;
      float r1 = v - (float)v1;
      const uint32_t a = __float_as_uint(v) & 0x7fffffffu;
      if (__builtin_expect(a >= 0x7f7f8000u, 0)) {
        if (a == 0x7f800000u) {
          r1 = 0.0f;
          sInf = 1;
        } else if (a < 0x7f800000u) {            // no infinite part of a finite value
          v1 = __builtin_bit_cast(__bf16, (unsigned short)(__float_as_uint(v) >> 16));
          r1 = v - (float)v1;
        }
      }
      const __bf16 v2 = (__bf16)r1;
      const int at = c * kVS + jj;
      sV[buf][0][at] = v1;
      sV[buf][1][at] = v2;
      sV[buf][2][at] = (__bf16)(r1 - (float)v2);
    }
  };

  if (tid == 0) sInf = 0;
  __syncthreads();
  if (sb < se) {
    gload(sb);
    lstore(0);
  }
  __syncthreads();
  for (int64_t st = sb; st < se; ++st) {
    const int buf = (int)((st - sb) & 1);
    const bool more = st + 1 < se;
    if (more) gload(st + 1);
    const bool has_inf = sInf != 0;
    const _Float16* X = sX[buf];
    const int off = __builtin_amdgcn_readfirstlane((int)(row0 - st * JT));   // wave-uniform
    auto columns = [&](auto diag) {
      constexpr bool DIAG = decltype(diag)::value;
      // the rare copy must not set the registers (R = 32, d = 12: 378 us, unrolled 549)
      constexpr int kUnroll = DIAG && (RB == 2 || KC > 4) ? 1 : JT / 32;
#pragma unroll kUnroll
      for (int jb = 0; jb < JT / 32; ++jb) {
        h8 a0[KC], a1[KC];
#pragma unroll
        for (int kc = 0; kc < KC; ++kc) {
          a0[kc] = *reinterpret_cast<const h8*>(X + (jb * 32 + l16) * XS + kc * 32 + g * 8);
          a1[kc] = *reinterpret_cast<const h8*>(X + (jb * 32 + 16 + l16) * XS + kc * 32 + g * 8);
        }
        f4 fv[RT ? RT : 1][2];
#pragma unroll
        for (int c = 0; c < RT; ++c)
#pragma unroll
          for (int h = 0; h < 2; ++h)
            fv[c][h] = *reinterpret_cast<const f4*>(&sF[buf][c * kVS + jb * 32 + 16 * h + g * 4]);
        b8 bv[RB ? RB : 1][3], bf[RB ? RB : 1];
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
#pragma unroll
          for (int p = 0; p < 3; ++p) {
            const __bf16* vr = &sV[buf][p][(rb * 16 + l16) * kVS + jb * 32 + g * 4];
            const b4 lo = *reinterpret_cast<const b4*>(vr);
            const b4 hi = *reinterpret_cast<const b4*>(vr + 16);
            bv[rb][p] = b8{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
          }
          bf[rb] = bv[rb][0];
          if (has_inf) {
#pragma unroll
            for (int e = 0; e < 8; ++e) {
              const unsigned short w = __builtin_bit_cast(unsigned short, bv[rb][0][e]);
              if ((w & 0x7fff) == 0x7f80) bf[rb][e] = (__bf16)0.0f;
            }
          }
        }
#pragma unroll
        for (int q = 0; q < NSUB; ++q) {
          f4 s0 = sqdist<KC>(a0, bi[q]);
          f4 s1 = sqdist<KC>(a1, bi[q]);
          if constexpr (DIAG) {
            // the diagonal's distance is 0, not its expansion's roundings
            const int at = off + (q - 2 * jb) * 16 + l16 - 4 * g;
#pragma unroll
            for (int v = 0; v < 4; ++v) {
              s0[v] = at == v ? 0.0f : s0[v];
              s1[v] = at - 16 == v ? 0.0f : s1[v];
            }
          }
          float k[8];
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            k[v] = kval<KIND>(s0[v], cs);
            k[4 + v] = kval<KIND>(s1[v], cs);
          }
          if constexpr (RB == 0) {
#pragma unroll
            for (int c = 0; c < RT; ++c)
#pragma unroll
              for (int v = 0; v < 8; ++v) sum[q][c] = fmaf(k[v], fv[c][v / 4][v % 4], sum[q][c]);
            continue;
          }
          b8 kp[3];
          parts3(k, kp);
#pragma unroll
          for (int rb = 0; rb < RB; ++rb) {
            // 32 columns from zero, smallest products first, then one vector add:
            // an MFMA cuts the low bits of products far below its accumulator, so
            // a long chain on one accumulator falls short of a same-sign sum
            // (2e-6 of it over 40,000 columns; 3% of the launch buys that back)
            f4 t = f4{0.f, 0.f, 0.f, 0.f};
            t = f16::mfma32<__bf16>(kp[2], bf[rb], t);
            t = f16::mfma32<__bf16>(kp[1], bv[rb][1], t);
            t = f16::mfma32<__bf16>(kp[0], bv[rb][2], t);
            t = f16::mfma32<__bf16>(kp[1], bf[rb], t);
            t = f16::mfma32<__bf16>(kp[0], bv[rb][1], t);
            t = f16::mfma32<__bf16>(kp[0], bv[rb][0], t);
#pragma unroll
            for (int v = 0; v < 4; ++v) acc[q][rb][v] += t[v];
          }
        }
      }
    };
    if (same && off > -JT * NSUB / 4 && off < JT)    // a stage that holds some of the wave's rows
      columns(std::true_type{});
    else
      columns(std::false_type{});
    if (more) lstore(buf ^ 1);
    __syncthreads();
  }
  float* P = part + (int64_t)split * n1_pad * RP;
#pragma unroll
  for (int q = 0; q < NSUB; ++q)
#pragma unroll
    for (int c = 0; c < RT; ++c) {
      float t = sum[q][c];
      t += __shfl_xor(t, 16);
      t += __shfl_xor(t, 32);
      if (g == 0) P[(row0 + q * 16 + l16) * RP + c] = t;
    }
#pragma unroll
  for (int q = 0; q < NSUB; ++q)
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
      for (int v = 0; v < 4; ++v)
        P[(row0 + q * 16 + 4 * g + v) * RP + rb * 16 + l16] = acc[q][rb][v];
}

// out = a2 * sum of the split partials (+ s2 V), from this form's partials or,
// when it did not run (info->ok == 0), from the vector form's [split][n1][r].
__global__ __launch_bounds__(256) void reduce_kernel(const float* __restrict__ part, int nsplit,
                                                     int64_t n1_pad, int rp,
                                                     const float* __restrict__ vpart, int vsplit,
                                                     int64_t n1, int r, int c0, int rc, float a2,
                                                     float s2, const float* __restrict__ V,
                                                     float* __restrict__ out,
                                                     const Info* __restrict__ info,
                                                     const int* __restrict__ live) {
  if (live && *live == 0) return;
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= n1 * rc) return;
  const int64_t i = e / rc;
  const int c = (int)(e - i * rc);
  const int64_t at = i * r + c0 + c;
  const float acc = info->ok ? ordered_split_sum(part + i * rp + c, nsplit, n1_pad * rp, 0.0f)
                             : ordered_split_sum(vpart + at, vsplit, n1 * r, 0.0f);
  float o = a2 * acc;
  if (V) o = fmaf(s2, V[at], o);
  out[at] = o;
}

// ---- host side ----------------------------------------------------------------
// The instantiation's function for (kind, KC, RB).
typedef void (*MainFn)(const _Float16*, const _Float16*, const float*, int, int, int64_t, float*,
                       int64_t, int, int64_t, const Info*, int, const int*);
template <int KIND, int RB, int RT>
static MainFn main_fn(int kc) {
  switch (kc) {
    case 2: return &main_kernel<KIND, 2, RB, RT>;
    case 3: return &main_kernel<KIND, 3, RB, RT>;
    case 4: return &main_kernel<KIND, 4, RB, RT>;
    case 5: return &main_kernel<KIND, 5, RB, RT>;
    case 6: return &main_kernel<KIND, 6, RB, RT>;
  }
  return nullptr;
}
template <int KIND>
static MainFn main_fn(int kc, int rp) {
  switch (rp) {
    case 1: return main_fn<KIND, 0, 1>(kc);
    case 4: return main_fn<KIND, 0, 4>(kc);
    case 16: return main_fn<KIND, 1, 0>(kc);
    case 32: return main_fn<KIND, 2, 0>(kc);
  }
  return nullptr;
}
static MainFn main_fn(int kind, int kc, int rp) {
  switch (kind) {
    case GP_KERNEL_RBF: return main_fn<GP_KERNEL_RBF>(kc, rp);
    case GP_KERNEL_MATERN52: return main_fn<GP_KERNEL_MATERN52>(kc, rp);
    case GP_KERNEL_MATERN32: return main_fn<GP_KERNEL_MATERN32>(kc, rp);
  }
  return nullptr;
}

bool use(int kind, int64_t n1, int64_t n2, int d, int r) {
  return kind != GP_KERNEL_MATERN12 && d <= kSplitMaxDim && n1 >= kSplitMinRows &&
         n2 >= kSplitMinRows && (double)n1 * (double)n2 * (2 * d + r + 12) >= kSplitMinWork;
}

// Work groups resident per compute unit: the 160 KB of LDS, and three waves per SIMD
// (two of the widest instantiations' registers: their grids' rounds are then a guess).
constexpr int kCus = 256;
static int groups_per_cu(int kc, int rb) {
  const int lds = 2 * (2 * JT * (32 * kc + 8) + 3 * 2 * 16 * rb * kVS);
  return std::max(1, std::min(3, 160 * 1024 / (lds + 512)));
}

// Column splits: the fewest whose grid's rounds per unit of work are within 2%
// of the best (a grid just above a multiple of the resident groups idles most
// compute units in its last round).
static int choose_splits(int kc, int rb, int64_t rblocks, int64_t nstage, int most) {
  const int64_t resident = (int64_t)kCus * groups_per_cu(kc, rb);
  const int64_t smax = std::max<int64_t>(1, std::min<int64_t>(most, nstage / 4));
  auto cost = [&](int64_t sp) { return (double)ceil_div(rblocks * sp, resident) / (double)sp; };
  double best = 1e300;
  for (int64_t sp = 1; sp <= smax; ++sp) best = std::min(best, cost(sp));
  for (int64_t sp = 1; sp <= smax; ++sp)
    if (cost(sp) <= best * 1.02) return (int)sp;
  return 1;
}

Plan plan(int64_t n1, int64_t n2, int d, int r, bool same, int most_splits, float radius,
          bool fine) {
  Plan p{};
  p.kc = fine ? fine_chunks(d) : operand_chunks(d);
  p.fine = fine;
  p.radius = radius;
  p.same = same;
  const int rows = 64 * subtiles(p.kc, fine);
  p.n1_pad = round_up(n1, rows);
  p.n2_pad = round_up(n2, JT);
  if (same) p.n1_pad = p.n2_pad = round_up(n1, std::max(rows, JT));
  p.rp = r == 1 ? 1 : r <= 4 ? 4 : r <= 16 ? 16 : 32;
  p.nsplit = choose_splits(p.kc, p.rp / 16, p.n1_pad / rows, p.n2_pad / JT, most_splits);
  p.groups1 = (int)std::max<int64_t>(1, std::min<int64_t>(128, ceil_div(n1 * d, 2048)));
  p.groups2 = same ? 0 : (int)std::max<int64_t>(1, std::min<int64_t>(128, ceil_div(n2 * d, 2048)));
  return p;
}

static size_t pad256(size_t b) { return (b + 255) & ~size_t(255); }

size_t operand_bytes(const Plan& p, int d) {
  return pad256(2 * (size_t)p.n1_pad * 32 * p.kc) + pad256(2 * (size_t)p.n2_pad * 32 * p.kc) +
         pad256(sizeof(Info)) + pad256(4 * (size_t)(p.groups1 + p.groups2) * 2 * d);
}
size_t part_bytes(const Plan& p) { return pad256(4 * (size_t)p.nsplit * p.n1_pad * p.rp); }

gp_status carve(Plan& p, int d, Arena& ar) {
  p.Xr = ar.take<_Float16>((size_t)p.n1_pad * 32 * p.kc);
  p.Xc = ar.take<_Float16>((size_t)p.n2_pad * 32 * p.kc);
  p.info = ar.take<Info>(1);
  p.box = ar.take<float>((size_t)(p.groups1 + p.groups2) * 2 * d);
  if (!p.box) return set_error(GP_ERR_NOMEM, "internal: workspace sizing");
  return GP_OK;
}

gp_status measure(const Plan& p, const KParams& kp, const float* X1, int64_t n1, const float* X2,
                  int64_t n2, hipStream_t s, const float* box) {
  // v_sqrt_f32 falls short of the root by 1.2e-8 of it on average (16M arguments
  // in [1, 4), worst 9.3e-8), which every entry of a Matern sum would share:
  // its argument is raised by twice that
  constexpr double kLog2e = 1.4426950408889634074, kSqrtBias = 1.2e-8;
  const double arg = kp.kind == GP_KERNEL_RBF
                         ? -0.5 * kLog2e
                         : (kp.kind == GP_KERNEL_MATERN52 ? 5.0 : 3.0) * kLog2e * kLog2e *
                               (1.0 + 2.0 * kSqrtBias);
  if (!box) {
    box_kernel<<<(unsigned)(p.groups1 + p.groups2), 256, 0, s>>>(X1, n1, X2, n2, kp.d, p.groups1,
                                                                 p.box);
    GP_HIP(hipGetLastError());
  }
  info_kernel<<<1, 256, 0, s>>>(box ? box : p.box, p.groups1 + p.groups2, kp, arg, p.radius, p.info);
  GP_HIP(hipGetLastError());
  return GP_OK;
}

gp_status prepare(const Plan& p, const KParams& kp, const float* X1, int64_t n1, const float* X2,
                  int64_t n2, hipStream_t s, bool measured) {
  if (!measured) GP_TRY(measure(p, kp, X1, n1, X2, n2, s));
  const int w = 32 * p.kc;
  const auto prep = p.fine ? &prep_fine_kernel : &prep_kernel;
  prep<<<(unsigned)ceil_div(p.n1_pad, (int64_t)kPrepPoints), 256, 0, s>>>(
      X1, n1, p.n1_pad, kp, w, p.info, p.Xr, p.same ? p.Xc : nullptr);
  GP_HIP(hipGetLastError());
  if (!p.same) {
    prep<<<(unsigned)ceil_div(p.n2_pad, (int64_t)kPrepPoints), 256, 0, s>>>(
        X2, n2, p.n2_pad, kp, w, p.info, nullptr, p.Xc);
    GP_HIP(hipGetLastError());
  }
  return GP_OK;
}

gp_status product(const Plan& p, const KParams& kp, const float* X1, int64_t n1, const float* X2,
                  int64_t n2, const float* V, int r, float* part, float* vpart, int vsplit,
                  bool add_noise, float* out, const int* live, hipStream_t s) {
  const int rows = 64 * subtiles(p.kc);
  const int64_t nstage = p.n2_pad / JT;
  if (vpart)
    GP_TRY(valu::launch_partial(kp, X1, n1, X2, n2, V, r, vpart, false, vsplit, live, s,
                                &p.info->ok));
  for (int c0 = 0; c0 < r; c0 += p.rp) {
    const int rc = std::min(p.rp, r - c0);
    const MainFn fn = main_fn(kp.kind, p.kc, p.rp);
    if (!fn) return set_error(GP_ERR_ARG, "internal: unsupported operand width %d", 32 * p.kc);
    fn<<<(unsigned)(p.n1_pad / rows * p.nsplit), 256, 0, s>>>(p.Xr, p.Xc, V, r, c0, n2, part,
                                                              p.n1_pad, p.nsplit, nstage, p.info,
                                                              p.same ? 1 : 0, live);
    GP_HIP(hipGetLastError());
    reduce_kernel<<<(unsigned)ceil_div(n1 * rc, (int64_t)256), 256, 0, s>>>(
        part, p.nsplit, p.n1_pad, p.rp, vpart, vsplit, n1, r, c0, rc, kp.a2, kp.s2,
        add_noise ? V : nullptr, out, p.info, live);
    GP_HIP(hipGetLastError());
  }
  return GP_OK;
}

}  // namespace split
}  // namespace gpmi
