// Internal declarations shared by the HIP translation units of libprac.
// Nothing here is part of the C ABI (see include/prac.h).
#pragma once

#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>
#include <stddef.h>
#include <stdint.h>

#include <utility>
#include <vector>

#include "prac.h"

typedef unsigned short bf16_t;  // raw bf16 bit pattern
#define PRAC_MAX_DEVICES 64      // per-device tables (kernel attributes, the static scratch block's address)

struct prac_ctx {
  int device;
  hipStream_t stream;
  char* ws;           // device scratch, grown on demand
  size_t ws_bytes;
  char* static_scratch;  // this device's copy of the library's static scratch block (prac_weight_grad_static)
  int* d_flag;        // device-side numeric failure flag (0 = fine)
  int last_hip;       // last hipError_t that made a call fail
  int n_cu;
  int tune_splits;    // > 0: override the token-split count of C^T dY (tuning hook)
  int tune_one_launch;  // 1: the bf16 weight gradient as one launch instead of three (slabs, reduction, P T)
  int tune_tail;        // after the slabs of C^T dY: 0 built-in choice, 1 slab sum and P T as two launches, 2 as one
  int* d_sync;        // PRAC_SYNC_TILES x 3 counters of the one-launch weight gradient (zero between launches)
  float* part32;        // PRAC_PART32_BYTES for the token-split partial sums of the fp32 weight gradient (part of the ctx,
                        // not of the scratch block that grows: the split, and with it the bits of dW, never depends on
                        // what the ctx ran before)
  float* tails;         // n_cu * PRAC_TAIL_BYTES for the partial sums of CtdyTails' helpers and of launch_compress_ws (part of the ctx;
                        // only for calls that work in the scratch block too, see prac_workspace_bytes)
  int prof_kind;      // kernel kind bracketed by events (0: none), see prac_profile_select
  int prof_stride;    // every prof_stride-th launch of that kind carries the event pair
  int64_t prof_seen;  // launches of that kind since the selection
  hipEvent_t ev_start, ev_stop;  // set by ProfScope: the next PRAC_LAUNCH attaches them to its kernel
  std::vector<std::pair<hipEvent_t, hipEvent_t>> prof_pairs;  // recorded, not yet read
  std::vector<hipEvent_t> prof_pool;                          // idle events
};

#define PRAC_PART32_BYTES ((size_t)8 << 20)
#define PRAC_TAIL_BYTES ((size_t)256 * 128 * 4)  // a 256 x 128 tile of fp32 partial sums, one per compute unit

// Brackets the launches issued during its lifetime with a HIP event pair on the ctx
// stream when the ctx is profiling this kernel kind.
struct ProfScope {
  prac_ctx* ctx;
  ProfScope(prac_ctx* c, int kind);
  ~ProfScope();
};

// Bump allocator over the ctx scratch for one API call.
struct WsPlan {
  size_t off = 0;
  size_t take(size_t bytes) {
    size_t o = off;
    off += (bytes + 255) & ~size_t(255);
    return o;
  }
};
int prac_ws_reserve(prac_ctx* ctx, size_t bytes);  // PRAC_OK / PRAC_ENOMEM / PRAC_EHIP

static inline int64_t round_up64(int64_t x, int64_t m) { return (x + m - 1) / m * m; }
// The streaming kernels address a row of a tile as a 32-bit byte offset from the tile's first row (at most 128
// rows of `pitch` 2-byte elements): row pitches up to this many elements keep it below 2^32.
constexpr int64_t PRAC_MAX_STREAM_PITCH = (int64_t)1 << 23;

// ---- bf16 MFMA GEMM ---------------------------------------------------------
// Out(M x N) = sum_k A(m,k) * B(k,n) over bf16 operands with fp32 accumulation.
// a_kc: A is stored M x K (K contiguous, lda) else K x M (M contiguous, lda).
// b_kc: B is stored N x K (K contiguous, ldb) else K x N (N contiguous, ldb).
struct GemmOperandB {
  const bf16_t* B;
  int64_t ldb;
  int N;
  void* out;  // out_bf16 ? bf16 : fp32, row-major M x N
  int64_t ldo;
};
struct GemmBf16Args {
  const bf16_t* A;
  int64_t lda;
  int M, K;
  bool a_kc, b_kc;
  GemmOperandB b0;     // columns of the first output
  GemmOperandB b1;     // optional second output sharing A (b1.B == nullptr: none)
  bool out_bf16;       // output element type (ignored when splits > 1)
  float beta;          // out = acc + beta * out (fp32 / bf16 out, splits == 1)
  int splits;          // > 1: split the K range, write fp32 slabs to `partial`
  float* partial;      // splits x M x N (b0 only), slab stride M*N
  int tile_hint;       // 0 auto
};
int launch_gemm_bf16(prac_ctx* ctx, const GemmBf16Args& a);

// ---- generic strided GEMM (fp32 / bf16 in, fp32 out) ----------------------------
// Out(m,n) = alpha * sum_k A(m,k) B(k,n) + beta * Out(m,n); element (m,k) of A at
// A[m*a_rs + k*a_cs], (k,n) of B at B[k*b_rs + n*b_cs]; accumulation in fp32 or
// fp64 (acc64).  k_stride > 1 visits k = 0, k_stride, 2 k_stride, ... (< K).
struct GemmGenArgs {
  const void* A;
  const void* B;
  prac_dtype adt, bdt;
  int64_t a_rs, a_cs, b_rs, b_cs;
  int M, N;
  int64_t K, k_stride;
  float* out;
  int64_t ldo;
  float alpha, beta;
  bool acc64;
  double* out64;  // when non-null the fp64 result is written here instead (ldo applies)
  int splits;     // > 1 with slabs != nullptr: split the reduction, then sum the slabs
  void* slabs;    // splits * M * N accumulators (fp64 if acc64 else fp32)
  size_t slab_bytes;  // size of `slabs`; a launch whose slabs would not fit is refused (PRAC_EINVAL)
};
int launch_gemm_generic(prac_ctx* ctx, const GemmGenArgs& a);
// ---- fp32 products on the matrix cores (gemm_f32.hip) ----------------------------
// Products launch_gemm_generic hands to gemm_f32.hip; with splits > 1 that leaves the partial sums in a.slabs.
bool gemm_f32_takes(const GemmGenArgs& a);
int launch_gemm_f32(prac_ctx* ctx, const GemmGenArgs& a, int splits);
// T32x64_ONE_ROUND: 32 x 64 in the form for a single round of workgroups
enum class F32Tile { T128x128 = 128128, T128x64 = 128064, T64x64 = 64064, T32x64 = 32064, T32x64_ONE_ROUND = 1032064, T32x32 = 32032 };
// tile of a workgroup for an M x N product over K in `splits` ranges; a_k_fast: A's k runs along memory
F32Tile f32_tile(int n_cu, int M, int N, int64_t K, int splits, bool a_k_fast);
// dW (d x m, fp32 or bf16) = P (sum of the slabs [splits][c][m], rows >= k_lo times scale_hi) (+ beta dW), all in fp32;
// the slabs may be overwritten
int launch_f32_sum_pt(prac_ctx* ctx, const float* P, int64_t ldp, float* slabs, int splits, int c, int k_lo,
                      float scale_hi, int d, int m, void* dW, int64_t lddw, bool out_bf16, float beta);

// ---- small helpers -------------------------------------------------------------
// out[i] = alpha * sum_s part[s*stride + i] + beta * out[i], i < n (fp32)
int launch_reduce_slabs(prac_ctx* ctx, const float* part, int splits, int64_t stride, float* out,
                        int64_t n, float alpha, float beta);
// out (n x n, ldo) = sum of the symmetric partial sums part[splits][n][n], of which only 64 x 64 blocks on and above the diagonal
// are read; with one of them out may be part (ldo = n)
int launch_reduce_symmetric(prac_ctx* ctx, const float* part, int splits, int n, float* out, int64_t ldo);
// out (N x M fp32, ld = ldo) = transpose of sum_s part[s][j][n], j < M
int launch_reduce_transpose_f32(prac_ctx* ctx, const float* part, int splits, int M, int N, float* out, int64_t ldo);
int launch_philox(prac_ctx* ctx, uint64_t seed, uint32_t draw, uint32_t stream, void* out, int64_t n,
                  bool normal);
// The packed basis, bf16 copies of P (d x c) with zeros behind its ends: Pt (c x ldpt) = P^T, Pn (d x ldpn) = P, Pf [nkb][ncb][64][8], a B operand
// in fragment order, and Pa [nrb][nckb][64][8], P as an A operand: block (rb, kb), lane 32 h + i, element e is P[32 rb + i][16 kb + 8 h + e].
// ldpt, ldpn multiples of 64; Pf's blocks cover all of the others.
struct PackedBasis {
  bf16_t *Pt, *Pn, *Pf, *Pa;
  int64_t ldpt, ldpn;
  int nkb, ncb, nrb, nckb;
};
int launch_pack_basis(prac_ctx* ctx, const float* P, int64_t d, int64_t ldp, int c, const PackedBasis& o);
int launch_cast_out(prac_ctx* ctx, const float* src, int64_t lds, void* dst, prac_dtype odt,
                    int64_t ldd, int rows, int cols, float beta);

// ---- kernels of the per-step path (ws_kernels.hip, hot_kernels.hip) -----------------
// Wfrag != nullptr: also Y (N x m, ldy) = X W, W in the fragment order of Pfrag with ncb_w column blocks
// any_element: rows of X start on any element and own nothing past their last column (d >= 8); Pfrag then holds the fp32 P
// as launch_pack_pfrag_split leaves it.  part: n_cu * PRAC_TAIL_BYTES of partial sums, for a product with few tiles (nullptr: one launch,
// which writes nothing but its outputs)
int launch_compress_ws(prac_ctx* ctx, const bf16_t* X, int64_t ldx, int N, int d, const bf16_t* Pfrag, int ncb,
                       int c, bf16_t* C, int64_t ldc, bool packed, const bf16_t* Wfrag, int ncb_w, int m,
                       bf16_t* Y, int64_t ldy, bool any_element = false, float* part = nullptr);
// C = X P by small tiles whose sum over d is split over a workgroup's waves (tile_kernels.hip); aligned rows only
enum class CompressTile { NONE, T32x32, T32x64, T32x128 };
CompressTile compress_tile(int n_cu, int N, int c);  // NONE: enough rows for compress_ws_kernel
int launch_compress_tile(prac_ctx* ctx, CompressTile tile, const bf16_t* X, int64_t ldx, int N, int d, const bf16_t* Pfrag, int ncb, int c,
                         bf16_t* C, int64_t ldc, bool packed);
// out_h (N x n[h], bf16) = A (N x c bf16, row-major with lda or packed; c <= 256) B_h for up to PRAC_CTDY_MAX_OUT outputs,
// B_h in fragment order [nkb][ncb[h]][64][8], zero past row c and column n[h]: nkb = wide_kblocks(c), ncb[h] a multiple
// of 8 covering n[h]; recon: the reconstruction (one output).  Rows of out_h may start on any element.
inline int wide_kblocks(int c) { return c <= 128 ? 8 : (c <= 256 ? 16 : 0); }
int launch_wide_ws(prac_ctx* ctx, bool recon, const bf16_t* A, int64_t lda, bool packed, int N, int c, int nkb, int n_out,
                   const bf16_t* const* B, const int* ncb, const int* n, bf16_t* const* out, const int64_t* ldo);
// 256-column groups per workgroup: the fewest rounds of workgroups, each as long as two groups (its start) and its own
inline int wide_groups_per_wg(int n_cu, int tiles_m, int groups) {
  int best = 1;
  int64_t best_cost = INT64_MAX;
  for (int gper = 1; gper <= groups; ++gper) {
    const int64_t wgs = (int64_t)tiles_m * ((groups + gper - 1) / gper), cost = (wgs + n_cu - 1) / n_cu * (2 + gper);
    if (cost <= best_cost) {
      best = gper;
      best_cost = cost;
    }
  }
  return best;
}
// W (bf16; w_layout 0: d x m, 1: m x d; ldw) -> [nkb][ncb_w][64][8] fragment order, zero padded
int launch_pack_wfrag(prac_ctx* ctx, const bf16_t* W, int64_t ldw, int w_layout, int64_t d, int m, int nkb,
                      int ncb_w, bf16_t* out);
// Token ranges of unequal length, for one round of workgroups where the tiles of T (256 x 128) do not divide the compute units.
// Every tile gets `main` workgroups of `len` units of 128 tokens each; what is left at the end of its tokens, `tail` units, goes
// to `helpers` workgroups, which share the tails of all tiles in equal runs of `run` units (tile after tile).  main == 0: equal
// ranges.  Partial sums are blocks of block_rows x 128, a tile each: `blocks` holds [main][t1 - t0], `tail_blocks` the pieces
// of the tails in order (tile t's piece by helper q is number t + q, less that of the first).  Only tiles t0 .. t1 - 1 (row groups of
// T after each other) are formed.
struct CtdyTails {
  int main = 0, len = 0, tail = 0, helpers = 0, run = 0;
  int block_rows = 0, t0 = 0, t1 = 0;
  float* blocks = nullptr;
  float* tail_blocks = nullptr;
};
// first helper that works on tile t's tail, and how many do
static inline __host__ __device__ int ctdy_tail_first(const CtdyTails& p, int t) { return (int)((int64_t)t * p.tail / p.run); }
static inline __host__ __device__ int ctdy_tail_parts(const CtdyTails& p, int t) {
  return (int)(((int64_t)(t + 1) * p.tail - 1) / p.run) - ctdy_tail_first(p, t) + 1;
}
static inline __host__ __device__ int ctdy_tail_block(const CtdyTails& p, int t, int q) {
  return t + q - p.t0 - ctdy_tail_first(p, p.t0);
}
// blocks that the tails of tiles t0 .. t1 - 1 take at most; no more than compute units for all of them
static inline int ctdy_tail_blocks(const CtdyTails& p, int t0, int t1) {
  return t1 - 1 + (int)(((int64_t)t1 * p.tail - 1) / p.run) - t0 - ctdy_tail_first(p, t0) + 1;
}
// token-split partial sums of C^T dY_h for n_out outputs that share C; slabs[h] is splits x c x sld[h] (sld: row pitch, m[h]
// where nullptr).  any_element: rows of
// dY_h may start on any element, and a row owns nothing past its last column (then m[h] >= 8); otherwise they are 16-byte
// aligned and own whole 16-byte chunks (the caller says which: where the rows are a sample of a matrix, their pitch does not).
// tails with main > 0: unequal ranges instead (slabs, splits and sld are not looked at).
// upper (one output, m = c, the same matrix as C and dY): the slabs hold only the tiles on and above the diagonal.
#define PRAC_CTDY_MAX_OUT 4
int launch_ctdy_ws(prac_ctx* ctx, const bf16_t* Cpk, int c, int N, int n_out, const bf16_t* const* dY,
                   const int64_t* lddy, const int* m, float* const* slabs, int splits, bool any_element,
                   int range_tokens = 0, const int* sld = nullptr, const CtdyTails* tails = nullptr, bool upper = false);
// tiles (256 rows x 128 columns) of a square matrix that hold an element on or above its diagonal
static inline __host__ __device__ int ctdy_upper_tiles(int tiles_n, int row_groups) {
  return row_groups * tiles_n - row_groups * (row_groups - 1);
}
// tokens of a range (whole 128-token tiles; the last ranges may be short or empty); launch_ctdy_ws takes another value for a
// part of the ranges of a longer product
inline int64_t ctdy_range_tokens(int64_t N, int splits) { return ((N + 127) / 128 + splits - 1) / splits * 128; }
// The whole weight gradient in one launch: partial slabs, their sum as T (bf16, fragment order, rows >= k_lo
// scaled) and dW_h = P T_h, the workgroups of a column tile meeting through `cnt` (PRAC_SYNC_INTS_PER_TILE
// ints per 128-column tile over all outputs, zero before and after the launch).  For shapes that
// wgrad_fused_takes says can.
#define PRAC_SYNC_TILES 4096
#define PRAC_SYNC_INTS_PER_TILE 8
#define PRAC_SYNC_BYTES ((size_t)PRAC_SYNC_TILES * PRAC_SYNC_INTS_PER_TILE * sizeof(int))
bool wgrad_fused_takes(int n_cu, int c, int n_out, const int64_t* m, int splits);
int launch_wgrad_fused(prac_ctx* ctx, const bf16_t* Cpk, int c, int N, int n_out, const bf16_t* const* dY,
                       const int64_t* lddy, const int* m, float* const* slabs, int splits, int k_lo, float scale_hi,
                       int nckb, const int* nmb, bf16_t* const* Tf, const bf16_t* Pa, int d, void* const* dW,
                       const int64_t* lddw, bool out_bf16, float beta, int* cnt);
int launch_pack_pfrag(prac_ctx* ctx, const float* P, int64_t d, int64_t ldp, int c, int nkb, int ncb, bf16_t* out);
// the fp32 P exactly, as three bf16 parts: [nkb / 16][3][16][ncb][64][8]
int launch_pack_pfrag_split(prac_ctx* ctx, const float* P, int64_t d, int64_t ldp, int c, int nkb, int ncb, bf16_t* out);
int launch_unpack_c(prac_ctx* ctx, const bf16_t* Cpk, int N, int c, bf16_t* C, int64_t ldc);
int launch_pack_c(prac_ctx* ctx, const bf16_t* C, int64_t ldc, int N, int c, bf16_t* Cpk);

// (sld and tails as for launch_ctdy_ws; with tails only the part of T_h in tiles t0 .. t1 - 1, and the padding behind a row group's
// last tile with that)
int launch_reduce_to_tfrag(prac_ctx* ctx, int n_out, const float* const* slabs, int splits, int c, const int* m, int k_lo,
                           float scale_hi, int nkb, const int* nmb, bf16_t* const* Tf, const int* sld, const CtdyTails& tails);
// dW_h (d x m_h) = P T_h (+ beta dW_h) for n_out <= PRAC_CTDY_MAX_OUT outputs in one launch
int launch_pt(prac_ctx* ctx, const bf16_t* Pa, int n_out, const bf16_t* const* Tf, int d, const int* m, int nkb,
              const int* nmb, void* const* dW, const int64_t* lddw, bool out_bf16, float beta);

// The whole weight gradient of a small layer in one launch (bf16; dY rows and, unless packed, C rows on 16-byte
// boundaries); Pa as for launch_pt, nkb = ceil(c / 16)
bool small_wgrad_takes(int n_cu, int64_t N, int64_t d, int c, int n_out, const int64_t* m);
int launch_small_wgrad(prac_ctx* ctx, const bf16_t* C, int64_t ldc, bool packed, int N, int c, int k_lo, float scale_hi, int n_out,
                       const bf16_t* const* dY, const int64_t* lddy, const int* m, const bf16_t* Pa, int nkb, int d,
                       void* const* dW, const int64_t* lddw, bool out_bf16, float beta);
// dW_h (d x m_h) = P (scaled sum of the slabs of C^T dY_h) (+ beta dW_h) in one launch: the slab reduction and
// launch_pt without T passing through memory; same arithmetic in the same order, bit-identical results
bool sum_pt_eligible(int n_out, const int* m, int splits);  // shapes the one-launch form covers
int launch_sum_pt(prac_ctx* ctx, const bf16_t* Pa, int n_out, const float* const* slabs, int splits, int c, int k_lo,
                  float scale_hi, int nkb, int d, const int* m, void* const* dW, const int64_t* lddw, bool out_bf16,
                  float beta);

// P (d x c fp32, ldp) -> B operand of Xh = C Ps^T in fragment order [nkb][ncb][64][8] (bf16, zero padded):
// element (k = column of P, n = row of P) = P[n][k] * (k >= k_lo ? scale_hi : 1)
int launch_pack_ptfrag(prac_ctx* ctx, const float* P, int64_t d, int64_t ldp, int c, int k_lo, float scale_hi,
                       int nkb, int ncb, bf16_t* out);

// ---- eigenvectors of a small symmetric matrix (sym_eig.hip) ----------------------
// Z (n x k fp32, row-major): the k eigenvectors of the symmetric part of H (n x n fp64) with the largest eigenvalues, in descending
// order; n <= SYM_EIG_MAX.  scratch: sym_eig_doubles(n), 32-byte aligned.
#define SYM_EIG_MAX 256
size_t sym_eig_doubles(int n);
int launch_sym_eig(prac_ctx* ctx, const double* H, int n, int k, double* scratch, float* Z);

// ---- basis fit -----------------------------------------------------------------
int fit_basis_device(prac_ctx* ctx, const void* X, prac_dtype xdt, int64_t N, int64_t d, int64_t ldx,
                     int k, int r, uint64_t seed, uint32_t draw, int refresh, const prac_fit_opts& o,
                     float* P, int64_t ldp);
size_t gram_scratch_bytes(int n_cu, const void* X, prac_dtype xdt, int64_t N, int64_t d,
                          int64_t ldx, int64_t row_stride, int64_t ldg);
// scratch of one prac_fit_basis call (X is only looked at for its alignment)
size_t fit_scratch_bytes(int n_cu, const void* X, prac_dtype xdt, int64_t N, int64_t d, int64_t ldx, int k, int r,
                         int refresh, const prac_fit_opts& o);
int64_t fit_slab_margin(int n_cu, prac_dtype xdt, int64_t N, int64_t d, int k, int r, int refresh,
                        const prac_fit_opts& o);
int gram_device(prac_ctx* ctx, const void* X, prac_dtype xdt, int64_t N, int64_t d, int64_t ldx,
                int64_t row_stride, float* G, int64_t ldg, char* scratch);

// Launch on the ctx stream; when a ProfScope is open, the kernel's own begin / end time
// stamps go into its event pair (so the measured time excludes launch gaps; a launcher with two kernels in a scope hands one
// event to each).
#define PRAC_LAUNCH(ctx, kern, grid, block, smem, ...)                                              \
  do {                                                                                             \
    if ((ctx)->ev_start || (ctx)->ev_stop) {                                                       \
      hipExtLaunchKernelGGL(kern, grid, block, smem, (ctx)->stream, (ctx)->ev_start, (ctx)->ev_stop, 0, \
                            __VA_ARGS__);                                                          \
      (ctx)->ev_start = nullptr;                                                                   \
      (ctx)->ev_stop = nullptr;                                                                    \
    } else {                                                                                       \
      hipLaunchKernelGGL(kern, grid, block, smem, (ctx)->stream, __VA_ARGS__);                     \
    }                                                                                              \
  } while (0)

#define PRAC_HIP_TRY(ctx, expr)                 \
  do {                                          \
    hipError_t e__ = (expr);                    \
    if (e__ != hipSuccess) {                    \
      (ctx)->last_hip = (int)e__;               \
      return PRAC_EHIP;                         \
    }                                           \
  } while (0)
