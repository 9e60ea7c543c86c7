// Fused, never-materialised kernel matrix x multi-vector product on the
// gfx950 matrix cores (Sec. 5.1, Eq. mvm; binary16 tiles with single-precision
// block summation).
//
// For an output-row tile I and a column tile J the product needs
//   S_IJ  = the kernel's exponent argument for every pair (i, j),
//   K_IJ  = kappa(S_IJ) rounded to binary16,
//   acc_I += K_IJ V_J.
// Both contractions run on v_mfma_f32_16x16x32_f16 with float32 accumulation.
// The exponent argument is produced by the first MFMA directly: the operands
// are augmented rows (built once by operands) whose dot product is
//   alpha * <x_i, x_j> + beta * (n_i + n_j),        n = ||x_hat||^2,
// with (alpha, beta) = (c, -c/2) for the RBF kernel (so S = -c r^2 / 2 and
// K = exp2(S), c = log2 e) and (-2c, c) for the Matern family (S = c r^2 with
// c = nu' (log2 e)^2, so sqrt|S| is the scaled distance).  The column-side
// factors alpha*x and beta*n are split into binary16 hi + lo pairs so that the
// argument keeps float32 accuracy although the operands are binary16.  This
// leaves one v_exp_f32 (RBF) or one v_sqrt_f32 + one v_exp_f32 (Matern) and a
// packed conversion per entry on the vector units, which bound the kernel.
//
// The accumulator layout of S^T (lane holds column i = lane%16 and rows
// j = 4*(lane/16) + v) is reused, without an LDS round trip, as the A operand
// of K V: two adjacent 16-column subtiles give each lane the 8 reduction
// slots the second MFMA consumes, and the matching rows of V are gathered from
// LDS in the same order.
//
// Work split: a grid of (row block of 256, column split) work groups; the
// column split equals blockIdx % nsplit, so with 8 splits every XCD (work
// groups are dealt round-robin to the 8 XCDs) streams only its own eighth of
// the column points through its L2.  Partial sums are reduced in a fixed
// order by kmvm_reduce, which also applies a^2, the column scale and s^2 V.

#include <math.h>

#include "fused_tile.h"
#include "internal.h"

namespace gpmi {
namespace f16 {

// ---- a1: augmented 16-bit operands --------------------------------------
// Side 0 = row points (B operand of the first MFMA), side 1 = column points (A
// operand), ax = alpha x, bn = beta n:
//   binary16, side 1: [hi(ax), lo(ax), hi(bn), lo(bn), 1, 1, 0...]
//   binary16, side 0: [x, x, 1, 1, hi(bn), lo(bn), 0...]
//   bfloat16: three parts instead of two, widths as in kmvm_bf16.hip.
//
// The two sides and the right-hand sides' column maxima do not depend on each
// other: work groups of one launch take them.  A product of a few hundred
// points costs its launches (seven took 34 us, three take 20), and a row's
// inputs are divided by the lengthscales once per side, not once per 16-byte
// chunk: at 10,000 points, d = 16, R = 8, 5.8 us for the 12.2 + 5.0 + 2.9 of
// separate sides, maxima and clearing.  Bound by latency: one pass of loads,
// the serial norm, the stores.
// Points: kPrepRows rows a group, scaled inputs and norm parts in LDS, then one
// thread per 16-byte chunk.  Maxima: each group writes its own row of pmax,
// folded by quant_kernel, so that nothing is cleared first; of few right-hand
// sides every group takes them all, and no second launch is needed.
constexpr int kPrepRows = 32;

template <typename T>
__device__ __forceinline__ float round_to(float x) { return (float)(T)x; }

struct PrepSide {
  const float* X;
  int64_t n;
  int groups;        // of kPrepRows padded rows
  void* out;
};

template <typename T>
__device__ __forceinline__ void prep_rows(const PrepSide& ps, const KParams& kp, int side, int w,
                                          float alpha, float beta, int64_t r0,
                                          float (*sh)[kMaxDim + 1], float (*sn)[3]) {
  typedef typename Vec<T>::v8 v8;
  constexpr int NP = __is_same(T, _Float16) ? 2 : 3;   // parts of a column-side factor
  const int d = kp.d, tid = threadIdx.x;
  for (int e = tid; e < kPrepRows * d; e += 256) {
    const int row = e / d, m = e - row * d;
    sh[row][m] = r0 + row < ps.n ? round_to<T>(ps.X[r0 * d + e] / kp.ls[m]) : 0.0f;
  }
  __syncthreads();
  if (tid < kPrepRows) {
    float nrm = 0.0f;
    for (int m = 0; m < d; ++m) nrm = fmaf(sh[tid][m], sh[tid][m], nrm);
    float rest = beta * nrm;
#pragma unroll
    for (int q = 0; q < NP; ++q) {
      sn[tid][q] = round_to<T>(rest);
      rest -= sn[tid][q];
    }
  }
  __syncthreads();
  const int chunks = w / 8;
  T* out = static_cast<T*>(ps.out);
  for (int e = tid; e < kPrepRows * chunks; e += 256) {
    const int row = e / chunks, c = e - row * chunks;
    v8 o;
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const int p = c * 8 + q;
      float v = 0.0f;
      if (p < NP * d) {
        const int part = p < d ? 0 : p < 2 * d ? 1 : 2;
        const float h = sh[row][p - part * d];
        if (side == 0) {
          v = h;
        } else {
          const float ax = alpha * h;
          const float a0 = round_to<T>(ax);
          v = part == 0 ? a0 : ax - a0;
          if (part == 2) v -= round_to<T>(v);
        }
      } else if (p < NP * d + 2 * NP) {
        const int f = p - NP * d;
        const bool norm_slot = (f < NP) == (side == 1);
        v = norm_slot ? sn[row][f < NP ? f : f - NP] : 1.0f;
      }
      o[q] = (T)v;
    }
    if (r0 + row >= ps.n)
#pragma unroll
      for (int q = 0; q < 8; ++q) o[q] = (T)0.0f;
    *reinterpret_cast<v8*>(out + (r0 + row) * w + c * 8) = o;
  }
}

// ---- right-hand-side quantisation -----------------------------------------
__device__ inline void pow2_scale(uint32_t maxbits, float* s, float* inv) {
  const float m = __uint_as_float(maxbits);
  if (!(m > 0.0f) || !isfinite(m)) {
    *s = 1.0f;
    *inv = 1.0f;
    return;
  }
  int e;
  frexpf(m, &e);                       // m = f 2^e, f in [0.5, 1)
  *s = ldexpf(1.0f, 15 - e);
  *inv = ldexpf(1.0f, e - 15);
}

// Per-column max |v| as float bits (non-negative floats order like uint32) of
// the rows group g of `groups` strides over, in smax; r <= 64, so that each
// thread keeps a column.
__device__ __forceinline__ void group_max(const float* __restrict__ V, int64_t n, int r,
                                          int64_t ld, int g, int groups, uint32_t* smax) {
  const int tid = threadIdx.x;
  if (tid < 64) smax[tid] = 0u;
  __syncthreads();
  const int per = 256 / r, c = tid % r, row = tid / r;
  uint32_t m = 0u;
  if (row < per) {
    const int64_t step = (int64_t)groups * per;
    for (int64_t i = (int64_t)g * per + row; i < n; i += 8 * step) {
      uint32_t x[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int64_t k = i + u * step;
        x[u] = __float_as_uint(fabsf(V[(k < n ? k : i) * ld + c]));
      }
#pragma unroll
      for (int u = 0; u < 8; ++u) m = max(m, x[u]);
    }
    if (m) atomicMax(&smax[c], m);
  }
  __syncthreads();
}

// Vt[c][i] = T(V[i][c] * s_c) for c < r, i < n; zero padding elsewhere (T is
// binary16 or bfloat16), s_c from the maxima in smax.  A tiled transpose: a work
// group reads kQRows rows of V (all rp columns, row-contiguous) into LDS, then
// each thread writes eight consecutive rows of one column.  rp <= 64.
constexpr int kQRows = 128;
template <typename T>
__device__ __forceinline__ void quant_rows(const Rhs<T>& q, int g, const uint32_t* smax,
                                           float (*sv)[64 + 1], float* ss) {
  typedef typename Vec<T>::v8 v8;
  const int64_t r0 = (int64_t)g * kQRows;
  const int rp = q.rp, r = q.r;
  if ((int)threadIdx.x < rp) {
    const int c = threadIdx.x;
    float sc = 1.0f, inv = 1.0f;
    if (c < r) {
      if (q.scale_mode == 1) {
        sc = q.fixed_scale;
        inv = q.fixed_inv;
      } else {
        pow2_scale(smax[c], &sc, &inv);
      }
      if (g == 0) {
        q.scale[c] = sc;
        q.inv_scale[c] = inv;
      }
    }
    ss[c] = sc;
  }
  __syncthreads();
  for (int e = threadIdx.x; e < kQRows * rp; e += 256) {
    const int row = e / rp, c = e % rp;
    const int64_t i = r0 + row;
    sv[row][c] = (c < r && i < q.n) ? q.V[i * q.ld + c] * ss[c] : 0.0f;
  }
  __syncthreads();
  for (int e = threadIdx.x; e < (kQRows / 8) * rp; e += 256) {
    const int c = e / (kQRows / 8), q0 = (e % (kQRows / 8)) * 8;
    const int64_t i0 = r0 + q0;
    if (i0 >= q.n_pad) continue;
    v8 o;
#pragma unroll
    for (int u = 0; u < 8; ++u) o[u] = (T)sv[q0 + u][c];
    *reinterpret_cast<v8*>(q.Vt + (int64_t)c * q.n_pad + i0) = o;
  }
}

// Each group folds the `groups` rows of maxima (scale_mode 0) first.
template <typename T>
__global__ __launch_bounds__(256) void quant_kernel(Rhs<T> q, int groups,
                                                    const int* __restrict__ live) {
  if (live && *live == 0) return;
  __shared__ float sv[kQRows][64 + 1];
  __shared__ float ss[64];
  __shared__ uint32_t smax[64];
  if (q.scale_mode == 0) {
    if (threadIdx.x < 64) smax[threadIdx.x] = 0u;
    __syncthreads();
    const int per = 256 / q.r, c = threadIdx.x % q.r, g0 = threadIdx.x / q.r;
    uint32_t m = 0u;
    if (g0 < per) {
#pragma unroll 8
      for (int g = g0; g < groups; g += per) m = max(m, q.pmax[g * q.r + c]);
      if (m) atomicMax(&smax[c], m);
    }
    __syncthreads();
  }
  quant_rows(q, (int)blockIdx.x, smax, sv, ss);
}

// SMALL: right-hand sides of at most kSmallRhs entries, whose every group takes
// all the maxima itself and quantises kQRows rows at once.
template <typename T, bool SMALL>
__global__ __launch_bounds__(256) void operands_kernel(PrepSide rows, PrepSide cols, KParams kp,
                                                       int w, float alpha, float beta, Rhs<T> q,
                                                       int vgroups) {
  __shared__ float sh[kPrepRows][kMaxDim + 1], sn[kPrepRows][3];
  __shared__ uint32_t smax[64];
  int b = blockIdx.x;
  if (b < vgroups) {
    if constexpr (SMALL) {
      __shared__ float sv[kQRows][64 + 1];
      __shared__ float ss[64];
      if (q.scale_mode == 0) group_max(q.V, q.n, q.r, q.ld, 0, 1, smax);
      quant_rows(q, b, smax, sv, ss);
    } else {
      group_max(q.V, q.n, q.r, q.ld, b, vgroups, smax);
      if ((int)threadIdx.x < q.r) q.pmax[(int64_t)b * q.r + threadIdx.x] = smax[threadIdx.x];
    }
    return;
  }
  b -= vgroups;
  if (b < rows.groups)
    prep_rows<T>(rows, kp, 0, w, alpha, beta, (int64_t)b * kPrepRows, sh, sn);
  else
    prep_rows<T>(cols, kp, 1, w, alpha, beta, (int64_t)(b - rows.groups) * kPrepRows, sh, sn);
}

// Where the line lies: every group reads all of them, 64 loads a thread here.  One
// launch instead of two: n = 1000, R = 16 22.8 -> 20.3 us, n = 16,000, R = 1 51.8 ->
// 49.4; at 64,000 entries n = 4000, R = 16 22.4 -> 24.4, n = 16,000, R = 4 52.2 -> 58.2.
constexpr int64_t kSmallRhs = 16384;

template <typename T>
gp_status quant(const Rhs<T>& q, int groups, const int* live, hipStream_t s) {
  if (q.rp > 64 || q.r < 1 || q.r > q.rp)
    return set_error(GP_ERR_ARG, "internal: %d padded right-hand sides (max 64)", q.rp);
  if (q.n_pad == 0) return GP_OK;
  quant_kernel<T><<<(unsigned)ceil_div(q.n_pad, (int64_t)kQRows), 256, 0, s>>>(q, groups, live);
  GP_HIP(hipGetLastError());
  return GP_OK;
}

template <typename T>
gp_status operands(const float* X1, int64_t n1, int64_t n1_pad, T* Xr, const float* X2, int64_t n2,
                   int64_t n2_pad, T* Xc, const KParams& kp, const Rhs<T>* rhs, hipStream_t s) {
  const Rhs<T> q = rhs ? *rhs : Rhs<T>{};
  if (rhs && (q.rp > 64 || q.r < 1 || q.r > q.rp))
    return set_error(GP_ERR_ARG, "internal: %d padded right-hand sides (max 64)", q.rp);
  if ((Xr && n1_pad % kPrepRows) || (Xc && n2_pad % kPrepRows))
    return set_error(GP_ERR_ARG, "internal: operand rows not padded");
  const int w = __is_same(T, _Float16) ? aug_width(kp.d) : aug_width_bf16(kp.d);
  const float c = arg_scale(kp.kind);
  const float alpha = kp.kind == GP_KERNEL_RBF ? c : -2.0f * c;
  const float beta = kp.kind == GP_KERNEL_RBF ? -0.5f * c : c;
  const PrepSide rows{X1, n1, Xr ? (int)(n1_pad / kPrepRows) : 0, Xr};
  const PrepSide cols{X2, n2, Xc ? (int)(n2_pad / kPrepRows) : 0, Xc};
  const bool small = rhs && q.n * q.r <= kSmallRhs;
  // maxima: eight loads a thread, at most one group per compute unit
  const int vgroups =
      !rhs ? 0
      : small ? (int)ceil_div(q.n_pad, (int64_t)kQRows)
      : q.scale_mode == 0 ? (int)std::min<int64_t>(kMaxGroups, ceil_div(q.n * q.r, 2048)) : 0;
  const unsigned grid = (unsigned)(rows.groups + cols.groups + vgroups);
  if (grid > 0) {
    if (small)
      operands_kernel<T, true><<<grid, 256, 0, s>>>(rows, cols, kp, w, alpha, beta, q, vgroups);
    else
      operands_kernel<T, false><<<grid, 256, 0, s>>>(rows, cols, kp, w, alpha, beta, q, vgroups);
    GP_HIP(hipGetLastError());
  }
  return rhs && !small ? quant(q, vgroups, nullptr, s) : GP_OK;
}

template gp_status quant<_Float16>(const Rhs<_Float16>&, int, const int*, hipStream_t);
template gp_status quant<__bf16>(const Rhs<__bf16>&, int, const int*, hipStream_t);
template gp_status operands<_Float16>(const float*, int64_t, int64_t, _Float16*, const float*,
                                      int64_t, int64_t, _Float16*, const KParams&,
                                      const Rhs<_Float16>*, hipStream_t);
template gp_status operands<__bf16>(const float*, int64_t, int64_t, __bf16*, const float*, int64_t,
                                    int64_t, __bf16*, const KParams&, const Rhs<__bf16>*,
                                    hipStream_t);

// ---- a2: fused product ------------------------------------------------------
// First position p in [0, cnt) with list[p] >= v (list increasing).
__device__ __forceinline__ int lower_pos(const int* __restrict__ list, int cnt, int64_t v) {
  int lo = 0, hi = cnt;
  while (lo < hi) {
    const int mid = (lo + hi) >> 1;
    if (list[mid] < v)
      lo = mid + 1;
    else
      hi = mid;
  }
  return lo;
}

// LIST: row block b visits only the stages lists[b * list_ld + p], p < counts[b]
// (increasing), of its split's stage range (the truncated product).
template <int KIND, int KC, int RB, bool LIST>
__global__ __launch_bounds__(256) void kmvm_f16_main(const _Float16* __restrict__ Xr,
                                                     const _Float16* __restrict__ Xc,
                                                     const _Float16* __restrict__ Vt,
                                                     float* __restrict__ part, int64_t n1_pad,
                                                     int64_t n2_pad, int nsplit,
                                                     const int* __restrict__ live,
                                                     const int* __restrict__ lists,
                                                     const int* __restrict__ counts,
                                                     int64_t list_ld) {
  if (live && *live == 0) return;
  __shared__ __attribute__((aligned(16))) _Float16 sX[2 * x_stage_halfs<KC>()];
  __shared__ __attribute__((aligned(16))) _Float16 sV[2 * v_stage_halfs<RB>()];
  const int split = blockIdx.x % nsplit;
  const int64_t rblk = blockIdx.x / nsplit;
  const int64_t nstage = n2_pad / JT;
  const int64_t sb = split * nstage / nsplit;
  const int64_t se = (split + 1) * nstage / nsplit;
  float* P = part + ((int64_t)split * n1_pad) * (16 * RB);
  if constexpr (LIST) {
    const int* li = lists + rblk * list_ld;
    const int cnt = counts[rblk];
    const int pb = lower_pos(li, cnt, sb), pe = lower_pos(li, cnt, se);
    fused_rows<KIND, KC, RB>(Xr, Xc, Vt, n2_pad, P, rblk * kRowsPerBlock, pb, pe, sX, sV, li);
  } else {
    fused_rows<KIND, KC, RB>(Xr, Xc, Vt, n2_pad, P, rblk * kRowsPerBlock, sb, se, sX, sV);
  }
}

template <int KIND, int KC, int RB>
static gp_status launch_t(const _Float16* Xr, const _Float16* Xc, const _Float16* Vt, float* part,
                          int64_t n1_pad, int64_t n2_pad, int nsplit, const int* live,
                          const StageLists* sl, hipStream_t s) {
  const int64_t blocks = (n1_pad / kRowsPerBlock) * nsplit;
  if (sl)
    kmvm_f16_main<KIND, KC, RB, true><<<(unsigned)blocks, 256, 0, s>>>(
        Xr, Xc, Vt, part, n1_pad, n2_pad, nsplit, live, sl->lists, sl->counts, sl->ld);
  else
    kmvm_f16_main<KIND, KC, RB, false><<<(unsigned)blocks, 256, 0, s>>>(
        Xr, Xc, Vt, part, n1_pad, n2_pad, nsplit, live, nullptr, nullptr, 0);
  GP_HIP(hipGetLastError());
  return GP_OK;
}

template <int KIND, int KC>
static gp_status launch_rb(int rb, const _Float16* Xr, const _Float16* Xc, const _Float16* Vt,
                           float* part, int64_t n1_pad, int64_t n2_pad, int nsplit, const int* live,
                           const StageLists* sl, hipStream_t s) {
  switch (rb) {
    case 1: return launch_t<KIND, KC, 1>(Xr, Xc, Vt, part, n1_pad, n2_pad, nsplit, live, sl, s);
    case 2: return launch_t<KIND, KC, 2>(Xr, Xc, Vt, part, n1_pad, n2_pad, nsplit, live, sl, s);
    case 3: return launch_t<KIND, KC, 3>(Xr, Xc, Vt, part, n1_pad, n2_pad, nsplit, live, sl, s);
    case 4: return launch_t<KIND, KC, 4>(Xr, Xc, Vt, part, n1_pad, n2_pad, nsplit, live, sl, s);
  }
  return set_error(GP_ERR_ARG, "internal: unsupported column block count %d", rb);
}

template <int KIND>
static gp_status launch_kc(int kc, int rb, const _Float16* Xr, const _Float16* Xc,
                           const _Float16* Vt, float* part, int64_t n1_pad, int64_t n2_pad,
                           int nsplit, const int* live, const StageLists* sl, hipStream_t s) {
  switch (kc) {
    case 1: return launch_rb<KIND, 1>(rb, Xr, Xc, Vt, part, n1_pad, n2_pad, nsplit, live, sl, s);
    case 2: return launch_rb<KIND, 2>(rb, Xr, Xc, Vt, part, n1_pad, n2_pad, nsplit, live, sl, s);
    case 3: return launch_rb<KIND, 3>(rb, Xr, Xc, Vt, part, n1_pad, n2_pad, nsplit, live, sl, s);
    case 4: return launch_rb<KIND, 4>(rb, Xr, Xc, Vt, part, n1_pad, n2_pad, nsplit, live, sl, s);
    case 5: return launch_rb<KIND, 5>(rb, Xr, Xc, Vt, part, n1_pad, n2_pad, nsplit, live, sl, s);
  }
  return set_error(GP_ERR_ARG, "internal: unsupported operand width %d", kc * 32);
}

gp_status launch_main(int kind, int kc, int rb, const _Float16* Xr, const _Float16* Xc,
                      const _Float16* Vt, float* part, int64_t n1_pad, int64_t n2_pad, int nsplit,
                      const int* live, double entries, hipStream_t s, const StageLists* sl) {
  if (n1_pad == 0) return GP_OK;
  void* tok = prof::begin(s);
  gp_status st;
  switch (kind) {
    case GP_KERNEL_RBF:
      st = launch_kc<GP_KERNEL_RBF>(kc, rb, Xr, Xc, Vt, part, n1_pad, n2_pad, nsplit, live, sl, s);
      break;
    case GP_KERNEL_MATERN52:
      st = launch_kc<GP_KERNEL_MATERN52>(kc, rb, Xr, Xc, Vt, part, n1_pad, n2_pad, nsplit, live, sl, s);
      break;
    case GP_KERNEL_MATERN12:
      st = launch_kc<GP_KERNEL_MATERN12>(kc, rb, Xr, Xc, Vt, part, n1_pad, n2_pad, nsplit, live, sl, s);
      break;
    case GP_KERNEL_MATERN32:
      st = launch_kc<GP_KERNEL_MATERN32>(kc, rb, Xr, Xc, Vt, part, n1_pad, n2_pad, nsplit, live, sl, s);
      break;
    default:
      return set_error(GP_ERR_ARG, "unknown kernel kind %d", kind);
  }
  prof::end(tok, s, entries, kind);
  return st;
}

// One thread per output, the split sums in split order with 16 loads in flight
// (the sum of many splits is otherwise as many dependent trips to memory: 56 of
// 10,000 x 8, 37 MB with the padding, 16.1 -> 7.5 us).
__global__ __launch_bounds__(256) void reduce_kernel(
    const float* __restrict__ part, int nsplit, int64_t n1, int64_t n1_pad, int r, int rp,
    const float* __restrict__ inv_scale, float a2, float s2, const float* __restrict__ V,
    int64_t ldv, float* __restrict__ out, int64_t ldo, const int* __restrict__ live) {
  if (live && *live == 0) return;
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= n1 * r) return;
  const int64_t i = e / r;
  const int c = (int)(e % r);
  const float vi = V ? V[i * ldv + c] : 0.0f, inv = inv_scale[c];
  const float* p = part + i * rp + c;
  const int64_t step = n1_pad * rp;
  float acc = 0.0f;
  for (int x = 0; x < nsplit; x += 16) {
    float t[16];
#pragma unroll
    for (int u = 0; u < 16; ++u) t[u] = x + u < nsplit ? p[(x + u) * step] : 0.0f;
#pragma unroll
    for (int u = 0; u < 16; ++u)
      if (x + u < nsplit) acc += t[u];
  }
  float o = (a2 * inv) * acc;
  if (V) o = fmaf(s2, vi, o);
  out[i * ldo + c] = o;
}

gp_status launch_reduce(const float* part, int nsplit, int64_t n1, int64_t n1_pad, int r, int rp,
                        const float* inv_scale, float a2, float s2, const float* V, int64_t ldv,
                        float* out, int64_t ldo, const int* live, hipStream_t s) {
  const int64_t total = n1 * r;
  if (total == 0) return GP_OK;
  reduce_kernel<<<(unsigned)ceil_div(total, 256), 256, 0, s>>>(part, nsplit, n1, n1_pad, r, rp,
                                                               inv_scale, a2, s2, V, ldv, out,
                                                               ldo, live);
  GP_HIP(hipGetLastError());
  return GP_OK;
}

int choose_splits(int64_t n1_pad, int64_t n2_pad, bool lists) {
  const int64_t rblocks = n1_pad / kRowsPerBlock;
  const int64_t nstage = n2_pad / JT;
  // enough work groups for ~8 per CU on 256 CUs, in multiples of the 8 XCDs
  int64_t want = ceil_div(2048, std::max<int64_t>(rblocks, 1));
  want = round_up(std::max<int64_t>(want, 8), 8);
  want = std::min<int64_t>(want, 64);
  // but no shorter than 8 stages while 512 groups remain: a group's start (row
  // operands, first stage) takes as long as two stages, and its sums are written
  // and read once per split.  n = 8000, R = 16: 63 splits 33.5 us, 16 27.6; n = 10000,
  // R = 8: 56 splits 38.8, 16 34.7 (256 groups: 8 splits 36.8); at 50,000 points 16
  // splits 608 us, 8 645.
  if (!lists)
    want = std::min(want, std::max(round_up(ceil_div(512, std::max<int64_t>(rblocks, 1)), 8),
                                   nstage / 64 * 8));
  const int rule = (int)std::max<int64_t>(1, std::min<int64_t>(want, nstage));
  return tune::f16_splits(n1_pad, n2_pad, rule);
}

}  // namespace f16
}  // namespace gpmi
