// Internal declarations shared by the gpmi host code and kernels (gfx950).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <string>

#include "gpmi.h"

namespace gpmi {

constexpr int kMaxDim = 64;

// Kernel hyperparameters as passed by value to device code.
struct KParams {
  int kind;
  int d;
  float a2;      // outputscale
  float s2;      // noise
  float ls[kMaxDim];
};

// ---- error state (per host thread) ----
gp_status set_error(gp_status st, const char* fmt, ...);
void clear_error();

#define GP_HIP(expr)                                                              \
  do {                                                                            \
    hipError_t e_ = (expr);                                                       \
    if (e_ != hipSuccess)                                                         \
      return ::gpmi::set_error(GP_ERR_HIP, "%s failed: %s (%s:%d)", #expr,        \
                               hipGetErrorString(e_), __FILE__, __LINE__);        \
  } while (0)

#define GP_TRY(expr)                 \
  do {                               \
    gp_status s_ = (expr);           \
    if (s_ != GP_OK) return s_;      \
  } while (0)

__host__ __device__ inline int64_t round_up(int64_t x, int64_t m) { return (x + m - 1) / m * m; }
__host__ __device__ inline int64_t ceil_div(int64_t x, int64_t m) { return (x + m - 1) / m; }

// Bump allocator over one device block; every sub-buffer is 256-byte aligned.
struct Arena {
  char* base = nullptr;
  size_t cap = 0;
  size_t off = 0;
  template <class T>
  T* take(size_t count) {
    size_t bytes = (count * sizeof(T) + 255) & ~size_t(255);
    if (off + bytes > cap) return nullptr;
    T* p = reinterpret_cast<T*>(base + off);
    off += bytes;
    return p;
  }
};

// Library-owned device workspace cached per (device, stream).  Growing it
// synchronises the stream first so no queued kernel still uses the old block.
gp_status workspace_get(hipStream_t s, size_t bytes, Arena* out);
// Free every per-stream workspace (waits for each device first); bytes freed.
size_t workspace_release();
// Free every cached preconditioner block; bytes freed.
size_t block_cache_release();

// Device blocks returned by long-lived handles, kept per (device, size) for
// the next handle of the same size (at most kBlockCacheBytes in total, beyond
// which blocks are freed), so a handle built and destroyed repeatedly does not
// pay hipMalloc and the device synchronisation of hipFree each time.
// block_cache_put expects no queued work to use the block any more.
constexpr size_t kBlockCacheBytes = size_t(4) << 30;
gp_status block_cache_get(size_t bytes, void** out);
void block_cache_put(int device, void* p, size_t bytes);

// Autotuned launch-shape decisions (tune.cpp); built-in rules until gp_autotune.
namespace tune {
constexpr int kBuckets = GP_TUNE_BUCKETS;
int64_t bucket_rows(int b);
int bucket_of(int64_t n1_pad);
// column splits of the single-problem binary16 product (fallback: built-in rule)
int f16_splits(int64_t n1_pad, int64_t n2_pad, int fallback);
int bt_split_div();      // batched: splits = clamp(stages / div, 1, 8)
bool bt_persistent();    // batched: persistent product launch
}  // namespace tune

// Opt-in launch timing of the fused product (gp_profile_*).
namespace prof {
void* begin(hipStream_t s);                       // nullptr when disabled
void end(void* token, hipStream_t s, double entries, int kind);
}  // namespace prof

// Device fill (usable under stream capture, unlike a memset node).
gp_status fill_f32(float* p, int64_t n, float v, hipStream_t s);

// Validation helpers.
gp_status check_kernel(const gp_kernel* k, int32_t d, bool need_noise, KParams* kp);
bool overlaps(const void* a, size_t abytes, const void* b, size_t bbytes);

// ---------------------------------------------------------------------------
// Kernel-matrix product, float16 matrix-core path (a1, a2 of the hot path).
// ---------------------------------------------------------------------------
namespace f16 {
constexpr int kRowsPerBlock = 256;   // 4 waves x 4 subtiles x 16 rows
constexpr int kStageCols = 128;      // columns per LDS stage

// Width (halfs) of the augmented operand rows for dimension d: binary16
// operands carry the column-side factors as hi + lo pairs, bfloat16 operands
// (8-bit significands) as three parts.
inline int aug_width(int d) { return (int)round_up(2 * d + 4, 32); }
inline int aug_width_bf16(int d) { return (int)round_up(3 * d + 6, 32); }

// Right-hand sides V (n x r, row stride ld) and their scaled, transposed 16-bit
// copy Vt (rp x n_pad, rp <= 64) with the per-column scales.  scale_mode 0: power
// of two from the column maxima; 1: fixed_scale for every column.  pmax: scratch
// for the maxima, kMaxGroups x r uint32.
constexpr int kMaxGroups = 256;
template <typename T>
struct Rhs {
  const float* V;
  int64_t n;
  int r;
  int64_t ld;
  int rp;
  int64_t n_pad;
  int scale_mode;
  float fixed_scale, fixed_inv;
  uint32_t* pmax;
  T* Vt;
  float* scale;
  float* inv_scale;
};

// The operands of a product (T = _Float16 or __bf16): the augmented rows of
// either side (null: left out) and, if given, the right-hand sides.  bfloat16
// operands: inputs divided by the lengthscale rounded to bfloat16, column-side
// factors in three bfloat16 parts (width aug_width_bf16(d)).
template <typename T>
gp_status operands(const float* X1, int64_t n1, int64_t n1_pad, T* Xr, const float* X2, int64_t n2,
                   int64_t n2_pad, T* Xc, const KParams& kp, const Rhs<T>* rhs, hipStream_t s);
// The right-hand sides alone, from `groups` rows of maxima in pmax.  A launch
// with *live == 0 does nothing.
template <typename T>
gp_status quant(const Rhs<T>& q, int groups, const int* live, hipStream_t s);

// The fused product with bfloat16 operands (no stage lists).
gp_status launch_main_bf16(int kind, int kc, int rb, const __bf16* Xr, const __bf16* Xc,
                           const __bf16* Vt, float* part, int64_t n1_pad, int64_t n2_pad,
                           int nsplit, const int* live, double entries, hipStream_t s);

// Per-row-block lists of the column stages a truncated product visits.
struct StageLists {
  const int* lists;    // row block b: stage ids lists[b * ld + p], p < counts[b], increasing
  const int* counts;
  int64_t ld;
};

// Main fused product over prepared operands: part[nsplit][n1_pad][rp].
// If live is non-null and *live == 0 the launch does nothing (used by the
// solver once every column is frozen).
// `entries` (n1 x n2 of the unpadded sets) is recorded by the launch timer.
// With stage lists, each row block visits only its listed stages (column
// splits keep their stage-id ranges, so skipping zero tiles leaves every sum
// unchanged).
gp_status launch_main(int kind, int kc, int rb, const _Float16* Xr, const _Float16* Xc,
                      const _Float16* Vt, float* part, int64_t n1_pad, int64_t n2_pad,
                      int nsplit, const int* live, double entries, hipStream_t s,
                      const StageLists* sl = nullptr);

// out[i][c] = a2 * inv_scale[c] * sum_x part[x][i][c] + s2 * V[i][c] (V may be
// null); V and out have row strides ldv and ldo.
gp_status launch_reduce(const float* part, int nsplit, int64_t n1, int64_t n1_pad, int r, int rp,
                        const float* inv_scale, float a2, float s2, const float* V, int64_t ldv,
                        float* out, int64_t ldo, const int* live, hipStream_t s);

// lists: a product over stage lists, whose groups keep only part of their stages
int choose_splits(int64_t n1_pad, int64_t n2_pad, bool lists = false);

// Symmetric product of one point set (kmvm_sym.hip): panels of 1536 points,
// each kernel value of two distinct panels evaluated once for both sides.
// Operands, right-hand sides (rp = 16) and the output use n_pad = sym_pad(n).
struct SymPlan {
  int64_t n_pad;
  int panels;
  int64_t stages;
  int64_t chunk;            // stages per work item
  int64_t items;
  int64_t rowpart_floats;
  int64_t colpart_floats;
  char* items_dev;          // carved by sym_carve
  int* first;
  int64_t* colbase;
  float* rowpart;
  float* colpart;
};
bool sym_supported(int d, int r);   // one 32-wide operand chunk, r <= 16
// smallest point count the solver and gp_kmvm give to the symmetric product
constexpr int64_t kSymMinN = 16384;
int64_t sym_pad(int64_t n);
SymPlan sym_plan(int64_t n_pad);
size_t sym_bytes(const SymPlan& pl);
gp_status sym_carve(SymPlan& pl, Arena& ar);
// writes the item table (once per plan, before the first launch)
gp_status sym_prepare(const SymPlan& pl, hipStream_t s);
gp_status sym_launch(int kind, const SymPlan& pl, const _Float16* Xr, const _Float16* Xc,
                     const _Float16* Vt, const int* live, double entries, hipStream_t s);
gp_status sym_reduce(const SymPlan& pl, int64_t n, int r, const float* inv_scale, float a2,
                     float s2, const float* V, int64_t ldv, float* out, int64_t ldo,
                     const int* live, hipStream_t s);
}  // namespace f16

// ---------------------------------------------------------------------------
// Kernel-matrix product on the vector ALUs: float32 entries, float32 or
// float64 accumulation.
// ---------------------------------------------------------------------------
namespace valu {
constexpr int kRowsPerBlock = 256;
constexpr int kStageCols = 64;
// part is float (acc32) or double (acc64): [nsplit][n1][r]
// skip: the launch does nothing when *skip != 0
gp_status launch_partial(const KParams& kp, const float* X1, int64_t n1, const float* X2,
                         int64_t n2, const float* V, int r, void* part, bool acc64, int nsplit,
                         const int* live, hipStream_t s, const int* skip = nullptr);
gp_status launch_reduce32(const float* part, int nsplit, int64_t n1, int r, float a2, float s2,
                          const float* V, float* out, const int* live, hipStream_t s);
int choose_splits(int64_t n1, int64_t n2, int d);
// column splits of the float64-accumulated product (true residual)
int choose_splits64(int64_t n1, int64_t n2, int d);
}  // namespace valu

// ---------------------------------------------------------------------------
// Float32 product on the matrix cores (kmvm_split.hip): exact integer products
// for the distances, entries and right-hand sides in three bfloat16 parts.
// ---------------------------------------------------------------------------
namespace split {
constexpr int kStageCols = 64;         // columns per LDS stage
constexpr int kSplitMaxDim = 28;       // d + 4 slots of the first 32-wide chunk
// the widest boxes (half diagonal in lengthscales): the gradient, whose other form
// has larger errors throughout, and the true residual on fine operands ...
constexpr float kSplitMaxRadius = 32.0f;
// ... and the float32 product.  Its error against float64 is half the vector form's
// where far entries weigh, the same where little but the diagonal is left, and within
// 3% above it on clusters of sd 0.1 up to here (Matern, d >= 12: 5 to 15% at 31)
constexpr float kSplitProductRadius = 20.0f;
// smallest sets and smallest vector-form work n1 n2 (2 d + r + 12) (operations)
// that take this form: its four extra launches cost about 20 us, which the
// vector form's time passes near there.  Vector form and this one: N = 3000, d = 8,
// R = 16 (work 4e8): 36 us and 44; N = 4000 (7e8): 47 and 44; N = 5000 (1.1e9): 95 and
// 52; N = 6000, d = 3, R = 1 (7e8): 48 and 38; N = 9000 (1.5e9): 90 and 48; 500 x
// 20,000, d = 8, R = 16 (4e8): 56 and 65; 60,000 x 400, d = 5, R = 8 (7e8): 62 and 67
constexpr int64_t kSplitMinRows = 256;
constexpr double kSplitMinWork = 1073741824.0;
// Scale data of a prepared point set, written on the device.
struct Info {
  float cs;                            // exponent scale times u^2: a signed power of two
  int ok;                              // 1: this form runs; 0: the vector form does
  double inv_u;
  double centre[kMaxDim];
};
__host__ __device__ constexpr int operand_chunks(int d) { return 1 + (5 * d + 6 + 31) / 32; }
// fine operands: chunks of the exact second sum, and all of them
__host__ __device__ constexpr int f_chunks(int d) { return (2 * d + 31) / 32; }
__host__ __device__ constexpr int fine_chunks(int d) { return f_chunks(d) + operand_chunks(d); }
// f_chunks from the width: d <= 16 have five chunks at most
__host__ __device__ constexpr int f_chunks_of(int kc) { return kc <= 5 ? 1 : 2; }
static_assert(fine_chunks(16) == 5 && fine_chunks(17) == 6, "f_chunks_of");
// 16-row subtiles per wave (their operands stay in registers)
__host__ __device__ constexpr int subtiles(int kc, bool fine = false) {
  return kc <= (fine ? 4 : 3) ? 4 : 2;
}
struct Plan {
  int kc, rp, nsplit, groups1, groups2;
  bool same;                           // X1 and X2 are one set
  bool fine;                           // fine operands (split_tile.h)
  float radius;                        // of the widest box
  int64_t n1_pad, n2_pad;
  _Float16 *Xr, *Xc;
  Info* info;
  float* box;
};
// whether a float32 product of these sizes takes this form (the inputs' range
// is checked on the device)
bool use(int kind, int64_t n1, int64_t n2, int d, int r);
Plan plan(int64_t n1, int64_t n2, int d, int r, bool same, int most_splits, float radius,
          bool fine = false);
size_t operand_bytes(const Plan& p, int d);
size_t part_bytes(const Plan& p);
gp_status carve(Plan& p, int d, Arena& ar);
// box, unit and Info of both sets (box: of the same sets, from another plan's
// measure); then their operands too (once per point set)
gp_status measure(const Plan& p, const KParams& kp, const float* X1, int64_t n1, const float* X2,
                  int64_t n2, hipStream_t s, const float* box = nullptr);
gp_status prepare(const Plan& p, const KParams& kp, const float* X1, int64_t n1, const float* X2,
                  int64_t n2, hipStream_t s, bool measured = false);
// out = a2 K V (+ s2 V); vpart (vsplit x n1 x r) takes the vector form's sums
// when the inputs' range rules this form out (null: it is known not to).
gp_status product(const Plan& p, const KParams& kp, const float* X1, int64_t n1, const float* X2,
                  int64_t n2, const float* V, int r, float* part, float* vpart, int vsplit,
                  bool add_noise, float* out, const int* live, hipStream_t s);
// Float64-accumulated sums of one point set (kmvm_split64.hip): part[split][i][c]
// = sum over the split's columns of k(x_i, x_j) V_jc, the vector form's layout;
// the inputs' range is known to allow it.
// from this many points, where one right-hand side pays for the operands' 20 us.  One
// residual on float64 distances against one on the operands: N = 8200: 85 us and 79
// (d = 3, R = 1), 98 and 114 (d = 8, R = 5), 104 and 123 (d = 8, R = 16); N = 10,000:
// 117 and 82, 132 and 127, 138 and 141; N = 20,000: 374 and 158, 428 and 299, 443 and
// 396; N = 40,000: 1344 and 453, 1536 and 947, 1546 and 1307
constexpr int64_t kSplit64MinPoints = 8192;
bool use64(int kind, int64_t n, int d);
int choose_splits64(const Plan& p, int r);
gp_status partial64(const Plan& p, const KParams& kp, int64_t n, const float* V, int r,
                    double* part, int nsplit, hipStream_t s);
}  // namespace split

// ---------------------------------------------------------------------------
// Conjugate-gradient step kernels (a3-a8 of the hot path).
// ---------------------------------------------------------------------------
namespace cg {
constexpr int kMaxR = 64;
constexpr int kMaxBlocks = 512;
constexpr int kReorthChunks = 256;

// Per-solve scalars, resident in device memory.
struct State {
  double lg[kMaxR];          // log gamma_k (logsumexp mode) or gamma_k
  double alpha[kMaxR];
  double beta[kMaxR];
  double bnorm2[kMaxR];
  double true_rel[kMaxR];
  float inv_sqrt_g[kMaxR];   // 1/sqrt(gamma_k), scale of the appended basis pair
  float rel[kMaxR];          // recursive relative residual
  int active[kMaxR];
  int converged[kMaxR];
  int breakdown[kMaxR];
  int iters[kMaxR];
  int k;                     // iterations done
  int nactive;
  int nbasis;                // basis pairs stored
  int append_slot;           // slot the next direction kernel writes
};

struct Dims {
  int64_t n;
  int r;
  int rp2;                   // power of two >= r
  int grid;                  // blocks of the reductions
};
Dims make_dims(int64_t n, int r);

gp_status init_state(State* st, const float* B, int64_t n, int r, double* pd, hipStream_t s,
                     const Dims& dm);
gp_status init_residual(const float* B, const float* q, float* x, float* rr, bool x0_given,
                        const State* st, const Dims& dm, hipStream_t s);
gp_status dq_step(const float* d, const float* q, State* st, bool lse, float* pm, float* ps,
                  double* pd, const Dims& dm, hipStream_t s);
gp_status update_step(float* x, float* rr, const float* d, const float* q, const State* st,
                      const Dims& dm, hipStream_t s);
// pcoef holds max_basis * reorth_chunks(n) * kMaxR floats.
int reorth_chunks(int64_t n);
// jmax: an upper bound on the stored pairs (<= max_basis); only that many
// coefficient blocks per row chunk are launched.
gp_status reorth_pass(const float* U, const float* W, float* rr, State* st, float* pcoef,
                      float* coef, int max_basis, int jmax, const Dims& dm, hipStream_t s);
// Both CGS2 passes in one coefficient sweep and one update sweep through the
// basis Gram matrix; pgram is sized as pcoef, c1 and coef hold max_basis * kMaxR
// floats, gram max_basis^2 * r floats (written one column per call).
gp_status reorth_gram(const float* U, const float* W, float* rr, State* st, float* pcoef,
                      float* pgram, float* c1, float* gram, float* coef, int max_basis, int jmax,
                      const Dims& dm, hipStream_t s);
gp_status rz_step(const float* rr, const float* z, State* st, bool lse, bool init, double tol,
                  int min_iter, float* pm, float* ps, double* pd, float* history,
                  uint32_t* colmax, int rp, const Dims& dm, hipStream_t s);
gp_status direction_step(const float* z, float* d, const float* rr, float* U, float* W,
                         State* st, bool init, bool reorth, uint32_t* colmax, const Dims& dm,
                         hipStream_t s);
// The step between two float32 products of a small unpreconditioned solve in
// one launch: from the product's split sums part[nsplit][n][r] of d to the next
// direction (dq_step .. direction_step with z = r).  `pairs`: an upper bound on
// the stored pairs.
bool fused_step_fits(const Dims& dm, bool reorth, int pairs);
gp_status fused_step(const float* part, int nsplit, float a2, float s2, float* x, float* rr,
                     float* d, float* U, State* st, float* gram, int max_basis, bool reorth,
                     bool lse, double tol, int min_iter, float* history, const Dims& dm,
                     hipStream_t s);
// true residual: res = b - (a2 * sum + s2 * x) from float64 partials; sets st->true_rel
gp_status true_residual_finish(const double* part, int nsplit, const float* B, const float* x,
                               float a2, float s2, State* st, double* pd, const Dims& dm,
                               hipStream_t s);
}  // namespace cg

// ---------------------------------------------------------------------------
// Pivoted-Cholesky preconditioner (a6, a9).
// ---------------------------------------------------------------------------
namespace pc {
constexpr int kMaxRank = 128;
}  // namespace pc

// ---------------------------------------------------------------------------
// Pseudo-loss gradient (Sec. 5.3, Eq. approx) and training step kernels.
// ---------------------------------------------------------------------------
namespace grad {
// The stream's workspace for launch() over `rows` rows, r columns, and `extra`
// bytes: with the split form's operands where the rule takes that form
// (*split_form), without them when they do not fit.
gp_status workspace(hipStream_t s, int64_t rows, int64_t n, int kind, int d, bool ard, int r,
                    size_t extra, Arena* ar, bool* split_form);
// out (device, L + 3 doubles): dL/dl.., dL/da^2, dL/ds^2, 1/2 y^T u_0 over
// rows [i0, i1); partial sums are carved from ar.
gp_status launch(const KParams& kp, bool ard, const float* X, int64_t n, const float* U,
                 const float* B, int r, int64_t i0, int64_t i1, bool split_form, double* out, Arena& ar,
                 hipStream_t s);
}  // namespace grad

namespace train {
constexpr int kMaxP = GP_TRAIN_MAX_PARAMS;
// Optimiser state, device resident.
struct DevState {
  double raw[kMaxP];
  double m[kMaxP];
  double v[kMaxP];
  double theta[kMaxP];
  double grad[kMaxP + 1];    // gradient estimate, then 1/2 y^T u_0
  double rgrad[kMaxP];       // objective gradient in raw values
  int step;
};
struct AdamOpts {
  double lr, beta1, beta2, eps;
  bool priors;
};
gp_status launch_rademacher(uint64_t seed, uint64_t first, int64_t rows, int cols, float* out,
                            int64_t ld, hipStream_t s);
// Adam on raw values from st->grad (nl lengthscales, then a^2 and s^2).
gp_status launch_adam(DevState* st, int nl, int64_t n, const AdamOpts& o, hipStream_t s);
// theta = constrained(raw).
gp_status launch_theta(DevState* st, int nl, hipStream_t s);
}  // namespace train

}  // namespace gpmi

// Opaque preconditioner handle of the C ABI.
struct gp_precond {
  int device;
  int64_t n;
  int d;
  int rank;              // rank actually built
  gpmi::KParams kp;
  double* L64;           // rank x n, column-major (each pivot column contiguous)
  float* L32;            // float32 copy for the apply
  double* Cinv;          // rank x rank, inverse of I + s^-2 L^T L
  int64_t* piv_dev;
  int64_t* piv_host;
  double trace_residual;
  double* scratch;       // apply partials
  float* Y32;            // rank x 64
  void* block;           // one device block holding the buffers above
  size_t block_bytes;
};

namespace gpmi {
namespace pc {
// z = P^{-1} r for an n x r block (r <= 64), on stream s; live as for the MVM.
gp_status apply(const gp_precond* P, const float* rr, float* z, const cg::Dims& dm,
                const int* live, hipStream_t s);
}  // namespace pc
}  // namespace gpmi
