// Device pieces of the preconditioner apply (Sec. 5.2, Eq. woodbury), shared
// by the single-problem and batched kernels:
//   T = L^T w   skinny product with a huge reduction dimension, on the
//               float32 matrix cores (v_mfma_f32_16x16x4f32);
//   z = s^-2 w - s^-4 L Y   two threads per row, Y staged in LDS.
// L is rank x n (each pivot column contiguous), w and z are n x r.
#pragma once

#include "internal.h"

namespace gpmi {
namespace pc {

typedef float pf4 __attribute__((ext_vector_type(4)));

constexpr int kLtMaxChunks = 1024;  // row chunks of the single-problem L^T w
constexpr int kLtChunkRows = 128;   // rows per chunk of the single-problem L^T w
constexpr int kLtResidentChunks = 512;  // 2 work groups x 256 compute units

// Work group (256 threads): out[m * r + c] = sum_{i0 <= i < i1} L[m][i] w[i][c]
// for m < k, c < r, in 16x16x4 products, wave w owning pivot tiles w and w + 4.
// Operands come straight from memory.  A operand (lane l): L[tile + l % 16][row],
// B operand: w[row][ctile + l % 16], row = t0 + 4 * u + l / 16 for product u; D:
// lane l, element v holds pivot tile + 4 * (l / 16) + v, column ctile + l % 16.
// The loads of the next 4 U rows are issued before the products of the current
// ones.  Bound by the loads' latency: staged through LDS in 32-row tiles, two
// barriers each, 48 problems of rank 20 and 220,000 rows (20 MB of L) took 34 us,
// 17 now; 100,000 rows at rank 100, R = 16 (40 MB) 25 us both ways.  Eight rows in a
// row per lane would take 12 and 17, but sum in another order, and a float32 ulp
// of z flips binary16 roundings of the next direction.
// CT: column tiles (1, 2 or 4; r <= 16 CT).
template <int CT>
__device__ __forceinline__ void lt_chunk_mfma(const float* __restrict__ L, int64_t n, int k,
                                              const float* __restrict__ w, int r, int64_t i0,
                                              int64_t i1, float* __restrict__ out) {
  constexpr int U = CT == 1 ? 16 : 8;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int l16 = lane & 15, g = lane >> 4;
  const int kt = (k + 15) / 16;
  if (wave >= kt) return;
  pf4 acc[2][CT];
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int t = 0; t < CT; ++t) acc[a][t] = pf4{0.f, 0.f, 0.f, 0.f};
  float la[2][U], lw[CT][U];
  auto load = [&](int64_t t0) {
    const bool full = t0 + 4 * U <= i1;                // the same for the whole wave
#pragma unroll
    for (int a = 0; a < 2; ++a) {
      if (wave + 4 * a >= kt) continue;
      const int m = 16 * (wave + 4 * a) + l16;
      const float* p = L + (int64_t)(m < k ? m : k - 1) * n + t0 + g;  // past k: unused sums
#pragma unroll
      for (int u = 0; u < U; ++u) la[a][u] = full || t0 + g + 4 * u < i1 ? p[4 * u] : 0.0f;
    }
#pragma unroll
    for (int t = 0; t < CT; ++t) {
      const int c = 16 * t + l16;
      const float* p = w + (t0 + g) * r + c;
#pragma unroll
      for (int u = 0; u < U; ++u)
        lw[t][u] = c < r && (full || t0 + g + 4 * u < i1) ? p[4 * u * r] : 0.0f;
    }
  };
  if (i0 < i1) load(i0);
  for (int64_t t0 = i0; t0 < i1;) {
    float ca[2][U], cw[CT][U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
#pragma unroll
      for (int a = 0; a < 2; ++a) ca[a][u] = la[a][u];
#pragma unroll
      for (int t = 0; t < CT; ++t) cw[t][u] = lw[t][u];
    }
    t0 += 4 * U;
    if (t0 < i1) load(t0);
#pragma unroll
    for (int a = 0; a < 2; ++a) {
      if (wave + 4 * a >= kt) continue;
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int t = 0; t < CT; ++t)
          acc[a][t] = __builtin_amdgcn_mfma_f32_16x16x4f32(ca[a][u], cw[t][u], acc[a][t], 0, 0, 0);
    }
  }
#pragma unroll
  for (int a = 0; a < 2; ++a) {
    const int mt = wave + 4 * a;
    if (mt >= kt) continue;
#pragma unroll
    for (int t = 0; t < CT; ++t) {
      const int c = t * 16 + l16;
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int mm = mt * 16 + 4 * g + v;
        if (mm < k && c < r) out[mm * r + c] = acc[a][t][v];
      }
    }
  }
}

// sum_{g0 <= q < g1} base[q * stride] in float64, in increasing q, with the
// loads issued eight at a time.
__device__ __forceinline__ double sum_strided(const float* __restrict__ base, int64_t stride,
                                              int g0, int g1) {
  double acc = 0.0;
  int q = g0;
  for (; q + 8 <= g1; q += 8) {
    float v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = base[(int64_t)(q + u) * stride];
#pragma unroll
    for (int u = 0; u < 8; ++u) acc += (double)v[u];
  }
  for (; q < g1; ++q) acc += (double)base[(int64_t)q * stride];
  return acc;
}

// (value, index) argmax with the lowest index winning ties; NaN never wins.
__device__ inline bool better(double v, int64_t i, double bv, int64_t bi) {
  if (isnan(v)) return false;
  if (isnan(bv)) return true;
  return v > bv || (v == bv && i < bi);
}

struct Best {
  double v;
  int64_t i;
  double sum;
};

__device__ __forceinline__ Best best_of(const Best& a, const Best& b) {
  const bool take = better(b.v, b.i, a.v, a.i);
  return Best{take ? b.v : a.v, take ? b.i : a.i, a.sum + b.sum};
}

// Argmax (lowest index on ties) and sum over a wave, then over the work
// group's waves, in a fixed order; every thread returns the result.
__device__ __forceinline__ Best group_best(Best x) {
  constexpr int kMaxWaves = 16;
  __shared__ Best sw[kMaxWaves];
#pragma unroll
  for (int o = 32; o > 0; o >>= 1)
    x = best_of(x, Best{__shfl_xor(x.v, o, 64), __shfl_xor(x.i, o, 64), __shfl_xor(x.sum, o, 64)});
  const int waves = blockDim.x >> 6;
  __syncthreads();
  if ((threadIdx.x & 63) == 0) sw[threadIdx.x >> 6] = x;
  __syncthreads();
  Best r = sw[0];
  for (int w = 1; w < waves; ++w) r = best_of(r, sw[w]);
  return r;
}

// Fixed-order merge of nparts argmax partials by one work group: the largest
// residual diagonal (lowest index on ties), its index and the residual trace,
// returned to every thread.
__device__ __forceinline__ Best merge_partials(const double* __restrict__ pv,
                                               const int64_t* __restrict__ pi,
                                               const double* __restrict__ psum, int nparts) {
  Best x{-INFINITY, INT64_MAX, 0.0};
  for (int g = threadIdx.x; g < nparts; g += blockDim.x) x = best_of(x, Best{pv[g], pi[g], psum[g]});
  return group_best(x);
}

// acc - sum_{t < m} L[t][i] lp[t] in increasing t (one FMA each), with sixteen
// loads of L in flight ahead of their FMAs.
__device__ __forceinline__ double sub_lrow(const double* __restrict__ L, int64_t n, int64_t i,
                                           const double* __restrict__ lp, int m, double acc) {
  int t = 0;
  for (; t + 16 <= m; t += 16) {
    double v[16];
#pragma unroll
    for (int u = 0; u < 16; ++u) v[u] = L[(int64_t)(t + u) * n + i];
#pragma unroll
    for (int u = 0; u < 16; ++u) acc = fma(-v[u], lp[t + u], acc);
  }
  // the rest (fewer than sixteen) as one batch, repeating the last column where
  // there is none
  if (t < m) {
    double v[16];
#pragma unroll
    for (int u = 0; u < 16; ++u) v[u] = L[(int64_t)(t + u < m ? t + u : m - 1) * n + i];
#pragma unroll
    for (int u = 0; u < 16; ++u)
      if (t + u < m) acc = fma(-v[u], lp[t + u], acc);
  }
  return acc;
}

// sy[m * rp + c] = Y[m * r + c] (zero for r <= c < rp); rp a multiple of 16.
__device__ __forceinline__ void stage_y(const float* __restrict__ Y, int k, int r, int rp,
                                        float* __restrict__ sy) {
  for (int e = threadIdx.x; e < k * rp; e += blockDim.x) {
    const int m = e / rp, c = e % rp;
    sy[e] = c < r ? Y[m * r + c] : 0.0f;
  }
}

// z[i][c] = s^-2 w[i][c] - s^-4 sum_m L[m][i] Y[m][c] for one row i and the
// columns c0 .. c0 + 7 of every sixteen.  Two threads share a row (c0 = 0 and 8):
// twice the waves of one thread per row, so twice the loads of L in flight (the
// pair's loads of L[m][i] are one address).
__device__ __forceinline__ void z_row(const float* __restrict__ L, int64_t n, int k,
                                      const float* __restrict__ sy, int rp,
                                      const float* __restrict__ w, float* __restrict__ z, int r,
                                      int64_t i, int c0, float inv_s2, float inv_s4) {
  for (; c0 < r; c0 += 16) {
    float acc[8];
#pragma unroll
    for (int c = 0; c < 8; ++c) acc[c] = 0.0f;
    auto step = [&](float l, int m) {
      const pf4* y4 = reinterpret_cast<const pf4*>(sy + m * rp + c0);
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        const pf4 y = y4[q];
        acc[4 * q + 0] = fmaf(l, y[0], acc[4 * q + 0]);
        acc[4 * q + 1] = fmaf(l, y[1], acc[4 * q + 1]);
        acc[4 * q + 2] = fmaf(l, y[2], acc[4 * q + 2]);
        acc[4 * q + 3] = fmaf(l, y[3], acc[4 * q + 3]);
      }
    };
    // sixteen loads of L in flight before their (in-order) accumulation
    int m = 0;
    for (; m + 16 <= k; m += 16) {
      float l[16];
#pragma unroll
      for (int u = 0; u < 16; ++u) l[u] = L[(int64_t)(m + u) * n + i];
#pragma unroll
      for (int u = 0; u < 16; ++u) step(l[u], m + u);
    }
    for (; m < k; ++m) step(L[(int64_t)m * n + i], m);
#pragma unroll
    for (int c = 0; c < 8; ++c)
      if (c0 + c < r) z[i * r + c0 + c] = inv_s2 * w[i * r + c0 + c] - inv_s4 * acc[c];
  }
}

// Cholesky factorisation C = L L^T of a k x k float64 matrix (k <= kMaxRank)
// and its inverse C^-1 = M^T M, M = L^-1, by one work group (a multiple of 64
// threads) with the matrix held in LDS (A: kCholLds doubles, rows of odd
// length ld so that a column's entries lie in distinct banks; dinv: kMaxRank).
// The work is a few hundred thousand operations: what it costs is barriers and
// serial chains.  Right-looking factorisation in blocks of 16 columns, a
// block's columns within one wave (no group barrier between them), the
// trailing update by the whole group; then M, eight lanes a column holding it
// in registers, with no barrier (column c goes to row c of the free upper
// triangle); then C^-1, each entry a sum
// over b >= max(a, c) in one order for (a, c) and (c, a), so the result is
// exactly symmetric.  352 us -> 139 at k = 100 (one barrier per row and three
// per column before).  *not_pd is set when a pivot is not > 0.
constexpr int kCholBlock = 16;
constexpr int kCholLds = kMaxRank * (kMaxRank + 1);
__device__ __forceinline__ double readlane64(double v, int lane) {
  const uint64_t u = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = __builtin_amdgcn_readlane((uint32_t)u, lane);
  const uint32_t hi = __builtin_amdgcn_readlane((uint32_t)(u >> 32), lane);
  return __builtin_bit_cast(double, (uint64_t)hi << 32 | lo);
}
// v moved by a DPP control (0xB1, 0x4E: lane ^ 1, ^ 2; 0x141: mirrored in its eight)
template <int CTRL>
__device__ __forceinline__ double dpp64(double v) {
  const uint64_t u = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = __builtin_amdgcn_update_dpp(0u, (uint32_t)u, CTRL, 0xf, 0xf, true);
  const uint32_t hi = __builtin_amdgcn_update_dpp(0u, (uint32_t)(u >> 32), CTRL, 0xf, 0xf, true);
  return __builtin_bit_cast(double, (uint64_t)hi << 32 | lo);
}
__device__ __forceinline__ double sum8(double v) {
  v += dpp64<0xB1>(v);
  v += dpp64<0x4E>(v);
  return v + dpp64<0x141>(v);
}

__device__ __forceinline__ void chol_inverse(const double* __restrict__ C,
                                             double* __restrict__ Cinv, int k, double* A,
                                             double* dinv, int* not_pd) {
  const int t = threadIdx.x, nt = blockDim.x, lane = t & 63;
  const int ld = k | 1;
  for (int e = t; e < k * k; e += nt) A[(e / k) * ld + e % k] = C[e];
  __syncthreads();
  for (int j0 = 0; j0 < k; j0 += kCholBlock) {
    const int j1 = k - j0 < kCholBlock ? k : j0 + kCholBlock;
    if (t < 64) {
      // the block's 16 columns in registers, rows lane and lane + 64
      const bool up = j0 >= 64;                 // the block's own rows are the second ones
      double v[2][kCholBlock];
#pragma unroll
      for (int r = 0; r < 2; ++r) {
        const int i = lane + 64 * r;
#pragma unroll
        for (int c = 0; c < kCholBlock; ++c)
          v[r][c] = i < k && j0 + c < j1 && i >= j0 ? A[i * ld + j0 + c] : 0.0;
      }
#pragma unroll
      for (int c = 0; c < kCholBlock; ++c) {
        const int j = j0 + c;
        __builtin_amdgcn_sched_barrier(0);      // keeps the columns' registers apart
        if (j < j1) {
          const double dj = readlane64(up ? v[1][c] : v[0][c], j & 63);
          if (!(dj > 0.0) && lane == 0) *not_pd = 1;
          const double root = sqrt(fmax(dj, 1e-300)), inv = 1.0 / root;
          if (lane == 0) dinv[j] = inv;
#pragma unroll
          for (int r = 0; r < 2; ++r) v[r][c] = lane + 64 * r == j ? root : v[r][c] * inv;
#pragma unroll
          for (int q = c + 1; q < kCholBlock; ++q) {
            const double x = readlane64(up ? v[1][c] : v[0][c], (j0 + q) & 63);
#pragma unroll
            for (int r = 0; r < 2; ++r) v[r][q] = fma(-v[r][c], x, v[r][q]);
          }
        }
      }
#pragma unroll
      for (int r = 0; r < 2; ++r) {
        const int i = lane + 64 * r;
#pragma unroll
        for (int c = 0; c < kCholBlock; ++c)
          if (i < k && j0 + c <= i && j0 + c < j1) A[i * ld + j0 + c] = v[r][c];
      }
    }
    __syncthreads();
    const int m = k - j1;
    for (int e = t; e < m * m; e += nt) {
      const int i = j1 + e / m, l = j1 + e % m;
      if (l <= i) {
        double acc = A[i * ld + l];
#pragma unroll 8
        for (int j = j0; j < j1; ++j) acc = fma(-A[i * ld + j], A[l * ld + j], acc);
        A[i * ld + l] = acc;
      }
    }
    __syncthreads();
  }
  // lane sub of column c's eight keeps M_mc for m = sub mod 8 in registers
  // (zero until row m is done, so the sums need no bounds)
  const int sub = t & 7;
  constexpr int kSlots = kMaxRank / 8;
  for (int c0 = 0; c0 < k; c0 += nt / 8) {
    const int c = c0 + t / 8;
    double M[kSlots];
#pragma unroll
    for (int u = 0; u < kSlots; ++u) M[u] = 0.0;
#pragma unroll
    for (int w = 0; w < kSlots; ++w) {
      if (8 * w >= k) break;
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll 1
      for (int x = 0; x < 8; ++x) {
        const int i = 8 * w + x;
        if (i >= k) break;
        double s = 0.0;
#pragma unroll
        for (int u = 0; u <= w; ++u) {
          const int m = 8 * u + sub;
          s = fma(A[i * ld + (m < i ? m : 0)], m < i ? M[u] : 0.0, s);
        }
        s = sum8(s);
        const double val = i == c ? dinv[i] : i > c ? -s * dinv[i] : 0.0;
        if (x == sub) M[w] = val;
      }
    }
#pragma unroll
    for (int u = 0; u < kSlots; ++u) {
      const int m = 8 * u + sub;
      if (c < k && m < k && m > c) A[c * ld + m] = M[u];   // the strict upper triangle
    }
  }
  __syncthreads();
  for (int e = t; e < k * k; e += nt) {
    const int a = e / k, c = e % k;
    const int hi = a > c ? a : c, lo = a > c ? c : a;
    double s = dinv[hi] * (hi == lo ? dinv[lo] : A[lo * ld + hi]);
#pragma unroll 4
    for (int b = hi + 1; b < k; ++b) s = fma(A[a * ld + b], A[c * ld + b], s);
    Cinv[e] = s;
  }
}

}  // namespace pc
}  // namespace gpmi
