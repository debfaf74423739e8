// Basis fit: P = [Q1 | Q2] (Section 4.3 construction; Alg. 1, both refresh branches).
//
// Q1: the paper takes the top-r_1 right singular vectors of X "via SVD".  They are
// the dominant eigenvectors of G = X^T X, found here by block power iteration
// V <- orth(G V) on a block of b = k + oversample columns, followed by a
// Rayleigh-Ritz step (eigenvectors of the small matrix V^T G V: sym_eig.hip up to 256 columns, one-sided Jacobi above).
// Q2: S is drawn from the counter-based Gaussian generator, projected twice onto the
// complement of Q1 and orthonormalised.  orth() is Cholesky-QR with an fp64 Gram
// matrix, which yields the thin-QR factor with a positive-diagonal R, i.e. the
// same Q2 that Householder QR with sign normalisation gives.
#include <algorithm>

#include "frag_utils.h"

namespace {

// ---------------------------------------------------------------- Cholesky (upper)
template <int N, typename F>
__device__ __forceinline__ void chol_static_for(F&& f) {
  if constexpr (N > 0) {
    chol_static_for<N - 1>(f);
    f(std::integral_constant<int, N - 1>{});
  }
}

__device__ __forceinline__ double readlane_f64(double x, int l) {
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(x), l),
                          __builtin_amdgcn_readlane(__double2loint(x), l));
}

// Largest diagonal entry of W, in every thread of a workgroup of 1024 (s_red: 16 doubles of LDS).
__device__ __forceinline__ double chol_diag_max(const double* W, int b, double* s_red) {
  double mx = 0.0;
  for (int i = threadIdx.x; i < b; i += 1024) mx = fmax(mx, W[(int64_t)i * b + i]);
  for (int o = 32; o > 0; o >>= 1) mx = fmax(mx, __shfl_xor(mx, o));
  if ((threadIdx.x & 63) == 0) s_red[threadIdx.x >> 6] = mx;
  __syncthreads();
  mx = 0.0;
  for (int w = 0; w < 16; ++w) mx = fmax(mx, s_red[w]);
  return mx;
}

// Elimination of a panel of 16 rows in one wave.  Every row of 16 lanes holds the diagonal block (lane l & 15: its column, rows
// u <= l & 15 of it; what is below is never read) in `diag` and 16 other columns of the panel in `col`, which become R^-T times
// themselves (R = R_jj).  It divides by the pivots (L D L^T) and takes their square roots at the end, a pivot per lane.
// The time is the chain from one pivot to the next and the issue of the updates, so: a multiplier is broadcast to the row of
// lanes by the multiply-add that uses it (DPP row_newbcast; two lane reads into scalar registers and a multiply-add take three
// times as long: 14 to 21 cycles against 5), the reciprocal is one third-order step on the hardware's estimate (2^-23, cubed), and
// the order is fixed by hand: next pivot first, the other updates behind it (the empty statements pin it).  A pivot that is not
// above `tiny`, or not finite, is replaced; returns whether there was one.  after_six() runs behind the sixth pivot.
// (the instructions below read lanes of a register that may have been written just before: two wait states)
template <int L>
__device__ __forceinline__ double row_bcast_f64(double x) {
  double r;
  asm volatile("s_nop 1\nv_mov_b64_dpp %0, %1 row_newbcast:%2 row_mask:0xf bank_mask:0xf\n" : "=v"(r) : "v"(x), "n"(L));
  return r;
}
template <int L, bool FRESH>  // acc += (x of lane L) * y; FRESH: x may have been written just before
__device__ __forceinline__ void row_fma_f64(double& acc, const double& x, const double& y) {
  if constexpr (FRESH)
    asm volatile("s_nop 1\nv_fmac_f64_dpp %0, %1, %2 row_newbcast:%3 row_mask:0xf bank_mask:0xf\n"
                 : "+v"(acc) : "v"(x), "v"(y), "n"(L));
  else
    asm volatile("v_fmac_f64_dpp %0, %1, %2 row_newbcast:%3 row_mask:0xf bank_mask:0xf\n" : "+v"(acc) : "v"(x), "v"(y), "n"(L));
}
template <typename Mid>
__device__ __forceinline__ bool chol_eliminate(double (&diag)[16], double (&col)[16], double tiny, Mid&& after_six) {
  const double big = 1.7e308;
  auto clamp = [&](double x) __attribute__((always_inline)) {  // (a NaN becomes tiny)
    asm volatile("v_max_f64 %0, %0, %1\nv_min_f64 %0, %0, %2\n" : "+v"(x) : "v"(tiny), "v"(big));
    return x;
  };
  auto pin = [](double& x) __attribute__((always_inline)) { asm volatile("" : "+v"(x)); };
  double p = clamp(row_bcast_f64<0>(diag[0]));
  double inv = __builtin_amdgcn_rcp(p);
  {
    const double e = fma(-p, inv, 1.0);
    inv = fma(inv, fma(e, e, e), inv);
  }
  chol_static_for<15>([&](auto tc) __attribute__((always_inline)) {
    constexpr int T = decltype(tc)::value;
    double s = -(diag[T] * inv);
    pin(s);
    row_fma_f64<T + 1, true>(diag[T + 1], s, diag[T]);
    p = clamp(row_bcast_f64<T + 1>(diag[T + 1]));
    double x = __builtin_amdgcn_rcp(p);
    pin(x);
    row_fma_f64<T + 1, false>(col[T + 1], s, col[T]);
    if constexpr (T + 2 < 16) {
      row_fma_f64<T + 2, false>(diag[T + 2], s, diag[T]);
      row_fma_f64<T + 2, false>(col[T + 2], s, col[T]);
    }
    double e = fma(-p, x, 1.0);
    pin(e);
    double e2 = fma(e, e, e);
    pin(e2);
    inv = fma(x, e2, x);
    pin(inv);
    if constexpr (T + 3 < 16)
      chol_static_for<13 - T>([&](auto ic) __attribute__((always_inline)) {
        constexpr int U = T + 3 + decltype(ic)::value;
        row_fma_f64<U, false>(diag[U], s, diag[T]);
        row_fma_f64<U, false>(col[U], s, col[T]);
      });
    if constexpr (T == 5) after_six();
  });
  const int l = threadIdx.x & 15;
  double piv = 1.0;
#pragma unroll
  for (int u = 0; u < 16; ++u) piv = l == u ? diag[u] : piv;
  const bool bad = __any(!(piv > tiny) || !isfinite(piv));
  piv = clamp(piv);
  double rs = __builtin_amdgcn_rsq(piv);
  rs = rs * (1.5 - 0.5 * piv * rs * rs);
  rs = rs * (1.5 - 0.5 * piv * rs * rs);
  chol_static_for<16>([&](auto uc) __attribute__((always_inline)) {
    constexpr int U = decltype(uc)::value;
    col[U] *= row_bcast_f64<U>(rs);
  });
  return bad;
}

// The same for a panel in LDS (`panel`, ldp doubles apart; column c is column j0 + c of W, wpad of them, the first 16 the
// diagonal block), 64 of its columns per wave (every wave repeats the diagonal block, bit for bit): group g holds the columns
// 16 + 64 g .., and they go to W and back to the panel.  Group -1 takes the identity instead and writes the diagonal block's place
// in W: R_jj^-1 (what the triangular solve multiplies with).  Non-finite or non-positive pivots raise *flag.
constexpr int CH_GRP = 64;
__device__ __forceinline__ void chol_panel_group(double* panel, int ldp, int wpad, int g, double tiny, double* W, int b,
                                                 int j0, int* flag) {
  const int lane = threadIdx.x & 63, i = lane & 15;
  const int c = g < 0 ? 0 : 16 + CH_GRP * g + lane;
  const bool in = c < wpad;
  double diag[16], col[16];
#pragma unroll
  for (int u = 0; u < 16; ++u) {
    diag[u] = panel[u * ldp + i];
    col[u] = g < 0 ? (i == u ? 1.0 : 0.0) : (in ? panel[u * ldp + c] : 0.0);
  }
  const bool bad = chol_eliminate(diag, col, tiny, [] {});
  if (g < 0) {
    if (lane < 16 && j0 + i < b) {
#pragma unroll
      for (int u = 0; u < 16; ++u)
        if (j0 + u < b) W[(int64_t)(j0 + i) * b + j0 + u] = col[u];  // (below the diagonal: zeros)
    }
    if (bad && lane == 0) atomicOr(flag, 1);
  } else if (in) {
#pragma unroll
    for (int u = 0; u < 16; ++u) {
      panel[u * ldp + c] = col[u];
      if (j0 + u < b && j0 + c < b) W[(int64_t)(j0 + u) * b + j0 + c] = col[u];
    }
  }
}

// Both kernels below: in place on the row-major b x b fp64 matrix W, the upper triangle of W = R^T R (after `shift_rel` of
// its entry, of the largest entry in the second kernel, is added to each diagonal entry) becomes R, with the inverse of every 16 x 16 diagonal block of R in that block's place.
// One workgroup of 1024 threads, the columns padded to a multiple of 16 with the identity; products and updates are 16 x 16 tiles
// on v_mfma_f64_16x16x4_f64.
typedef double f64x4_t __attribute__((ext_vector_type(4)));
constexpr int CH_NB = 16;  // panel height = block size of the fp64 matrix instruction
constexpr int CH_TB = 4;   // trailing tiles a wave has in flight
constexpr int CH_MAX = 1024;
// What is added to a diagonal entry: a pivot's rounding is a few 1e-16 of its own column's square, so a share of that keeps it positive, and
// a short column (a direction that the batch has only as rounding noise) comes out as long as the others.  A share of the largest entry leaves
// such columns short by 1e9 and more after three passes, past what the rest of the fit mends (fp32 batches of rank 1 to 5, 8 to 100
// columns asked for: 170 of 288 fits refused, now none).  Blocks wider than 256 columns keep that share: the rotations that follow there do not wait for
// columns below 1e-13 to settle, and full-length noise does not settle in their sixteen sweeps.  `least`: a column of zeros stays one.
struct CholShift {
  double rel, least;
  __device__ __forceinline__ CholShift(double rel_, double mx) : rel(rel_), least(1e-13 * rel_ * mx) {}
  __device__ __forceinline__ double of(double x) const { return fmax(rel * x, least); }
};

// b <= 256: the whole matrix stays in registers as 16 x 16 upper-triangular tiles.  Wave 0 eliminates the diagonal blocks, with
// the identity beside them, which leaves R_jj^-T; the other 15 waves hold the tiles (round robin, nine at most: both fit the 128
// registers of a wave), multiply their tiles of row j by R_jj^-T and update their trailing tiles with the result.  A tile's
// accumulators are, register by register, also its operand layout in both products (element (4 v + fk, fi) is register v
// of lane (fi, fk) as a result, and k = 4 v + fk, m or n = fi as an operand), so tiles pass through LDS in lane order, untransposed.
// What bounds it is the chain of 256 pivots, so wave 0 waits for nothing else: tiles (j, j + 1) and (j + 1, j + 1), updated up to
// panel j - 1, are handed to it while it eliminates block j, and it forms the next diagonal block from them itself; the
// trailing update of panel j - 1 runs beside that elimination.  Two barriers per panel.
// 53 us per launch at b = 256 in a cold fit of 2048 features, 59 in a refit of 4096 (84 / 98 us before: the elimination's multipliers
// through scalar registers, five waves eliminating and everything else waiting for them, no update beside it): 16 panels of 5600
// cycles (elimination 3600), the first nine up to 13000, where the update is bound by the fp64 matrix cores' rate.
constexpr int CHR_MAX = 256, CHR_NBK = CHR_MAX / CH_NB, CHR_W = 15, CHR_UT = 9;
constexpr int CHR_SPARE = 9;  // block rows that leave three tiles to the waves beside wave 0, if the others cannot hold all
static_assert(12 * CHR_UT + 3 * CHR_SPARE >= CHR_NBK * (CHR_NBK + 1) / 2 - 1, "every tile but the first has an owner");
constexpr int CHR_ML = CH_NB + 2;  // pitch of the 16 x 16 blocks that change layout in LDS

struct __align__(16) CholRegLds {
  double diag[CH_NB * CHR_ML];     // wave 0's next diagonal block on its way from tile layout to a column per lane
  double m[CH_NB * CHR_ML];        // R_jj^-T, element (u, c) at c * CHR_ML + u
  double hand[2][256];             // the tiles handed to wave 0, in lane order: (j, j + 1), (j + 1, j + 1)
  double panel[CHR_NBK][256];      // row j of R, a tile per block column, in lane order
  double red[16];
};

// a + f^T x for 16 x 16 tiles, as two chains of matrix instructions (one depends on the other's result for about 100 cycles)
__device__ __forceinline__ f64x4_t chol_mul(const f64x4_t& f, const f64x4_t& x, f64x4_t a) {
  f64x4_t b = {0.0, 0.0, 0.0, 0.0};
  a = __builtin_amdgcn_mfma_f64_16x16x4f64(f[0], x[0], a, 0, 0, 0);
  b = __builtin_amdgcn_mfma_f64_16x16x4f64(f[1], x[1], b, 0, 0, 0);
  a = __builtin_amdgcn_mfma_f64_16x16x4f64(f[2], x[2], a, 0, 0, 0);
  b = __builtin_amdgcn_mfma_f64_16x16x4f64(f[3], x[3], b, 0, 0, 0);
  return a + b;
}

// tile (I, J) of W (element (4 v + fk, fi) in register v), and the shift of its diagonal, with the identity outside b x b
__device__ __forceinline__ f64x4_t chol_load_tile(const double* W, int b, int I, int J) {
  const int fi = threadIdx.x & 15, fk = (threadIdx.x & 63) >> 4;
  const char* const base = reinterpret_cast<const char*>(W);
  const unsigned c = min(CH_NB * J + fi, b - 1);
  f64x4_t t;
#pragma unroll
  for (int v = 0; v < 4; ++v)  // (32-bit offsets: one register per address)
    t[v] = *reinterpret_cast<const double*>(base + 8u * (unsigned)(min(CH_NB * I + 4 * v + fk, b - 1) * b + c));
  return t;
}
__device__ __forceinline__ void chol_border(f64x4_t& t, int b, CholShift shift, int I, int J) {
  const int fi = threadIdx.x & 15, fk = (threadIdx.x & 63) >> 4, c = CH_NB * J + fi;
  if (I == J) {  // uniform
#pragma unroll
    for (int v = 0; v < 4; ++v) t[v] += 4 * v + fk == fi ? shift.of(t[v]) : 0.0;
  }
  if (CH_NB * (J + 1) > b) {  // uniform
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int row = CH_NB * I + 4 * v + fk;
      if (row >= b || c >= b) t[v] = row == c ? 1.0 : 0.0;
    }
  }
}

__device__ __forceinline__ void chol_wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ __forceinline__ void chol_pivot_wave(CholRegLds& s, const double* W, int b, CholShift shift, double tiny, int* flag) {
  const int lane = threadIdx.x & 63, fi = lane & 15, fk = lane >> 4;
  const int nb = (b + CH_NB - 1) / CH_NB;
  bool bad = false;
  __builtin_amdgcn_s_setprio(3);
  f64x4_t t = chol_load_tile(W, b, 0, 0);
  chol_border(t, b, shift, 0, 0);
  for (int j = 0; j < nb; ++j) {
#pragma unroll
    for (int v = 0; v < 4; ++v) s.diag[fi * CHR_ML + 4 * v + fk] = t[v];
    chol_wave_sync();
    double diag[16], col[16];
#pragma unroll
    for (int u = 0; u < 16; ++u) {
      diag[u] = s.diag[fi * CHR_ML + u];
      col[u] = fi == u ? 1.0 : 0.0;
    }
    bad = chol_eliminate(diag, col, tiny, [&] {
            if (j > 0) __syncthreads();  // B of panel j - 1, which this wave does not need: the others are there by now
          }) || bad;
    if (lane < 16) {
#pragma unroll
      for (int u = 0; u < 16; ++u) s.m[fi * CHR_ML + u] = col[u];
    }
    __syncthreads();  // A: R_jj^-T and the handed tiles are in LDS
    if (j + 1 < nb) {
      f64x4_t m, h;
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        m[v] = s.m[(4 * v + fk) * CHR_ML + fi];
        h[v] = s.hand[0][64 * v + lane];
        t[v] = s.hand[1][64 * v + lane];
      }
      const f64x4_t x = chol_mul(m, h, f64x4_t{0.0, 0.0, 0.0, 0.0});
      t = chol_mul(-x, x, t);
    }
  }
  __syncthreads();  // B of the last panel
  if (bad && lane == 0) atomicOr(flag, 1);
}

__device__ __forceinline__ void chol_tile_wave(CholRegLds& s, double* W, int b, CholShift shift, int wave) {
  const int lane = threadIdx.x & 63, fi = lane & 15, fk = lane >> 4;
  const int nb = (b + CH_NB - 1) / CH_NB, ntiles = nb * (nb + 1) / 2;
  f64x4_t acc[CHR_UT];
  int tile[CHR_UT];  // 16 I + J, -1: none
  // Waves 4, 8 and 12 share a SIMD with wave 0, whose chain every fp64 instruction of theirs delays (64 cycles each): they get only
  // what the other twelve cannot hold, the last three tiles of block rows 1 - 9.
  const bool spare = (wave & 3) == 0;
  const int n_rows = ntiles - 1 > 12 * CHR_UT ? CHR_SPARE : 0;  // b > 224
  const int others = wave - (wave >> 2);                        // 1 .. 12
#pragma unroll
  for (int e = 0; e < CHR_UT; ++e) {
    // tile number q, row by row: row I starts at I nb - I (I - 1) / 2
    int q = others + 12 * e, I = 0;
    bool live;
    if (spare) {
      live = e < n_rows;
      q = (e + 2) * nb - (e + 2) * (e + 1) / 2 - (wave >> 2);
    } else {
      for (int t = 1; t <= n_rows; ++t)  // step over the tiles of the spare waves
        if (q >= (t + 1) * nb - t * (t + 1) / 2 - 3) q += 3;
      live = q < ntiles;
    }
    if (!live) q = 0;
    while (q >= nb - I) {  // block row I holds nb - I tiles
      q -= nb - I;
      ++I;
    }
    tile[e] = live ? 16 * I + I + q : -1;
    acc[e] = chol_load_tile(W, b, I, I + q);
  }
  auto hand = [&](int t, int j, const f64x4_t& x) {  // tiles (j, j + 1) and (j + 1, j + 1) go to wave 0
    if (t == 17 * j + 1 || t == 17 * j + 17) {       // uniform
      double* h = s.hand[t == 17 * j + 17];
#pragma unroll
      for (int v = 0; v < 4; ++v) h[64 * v + lane] = x[v];
    }
  };
#pragma unroll
  for (int e = 0; e < CHR_UT; ++e)
    if (tile[e] >= 0) {  // uniform
      chol_border(acc[e], b, shift, tile[e] >> 4, tile[e] & 15);
      hand(tile[e], 0, acc[e]);
    }
  for (int j = 0; j < nb; ++j) {
    __syncthreads();  // A
    f64x4_t m;
#pragma unroll
    for (int v = 0; v < 4; ++v) m[v] = s.m[(4 * v + fk) * CHR_ML + fi];
#pragma unroll
    for (int e = 0; e < CHR_UT; ++e) {
      int t = tile[e];
      asm("" : "+s"(t));
      if (t >> 4 != j || t == 17 * j) continue;  // uniform
      const f64x4_t x = chol_mul(m, acc[e], f64x4_t{0.0, 0.0, 0.0, 0.0});
#pragma unroll
      for (int v = 0; v < 4; ++v) s.panel[t & 15][64 * v + lane] = x[v];
      const int c = CH_NB * (t & 15) + fi;
      double* const w = W + (CH_NB * j + fk) * b + c;
      if (c < b) {  // (a row block with another one behind it is whole)
#pragma unroll
        for (int v = 0; v < 4; ++v) w[4 * v * b] = x[v];
      }
    }
    if (wave == CHR_W && CH_NB * j + fi < b) {  // element (4 v + fk, fi) of R_jj^-1
      double* const w = W + CH_NB * j * b + CH_NB * j + fi;
#pragma unroll
      for (int v = 0; v < 4; ++v)
        if (CH_NB * j + 4 * v + fk < b) w[(4 * v + fk) * b] = m[v];
    }
    __syncthreads();  // B: row j of R is in LDS
#pragma unroll
    for (int e = 0; e < CHR_UT; ++e) {
      int t = tile[e];
      asm("" : "+s"(t));  // (LDS addresses are formed here, not kept in registers across panels)
      if (t < 16 * (j + 1) || t == 17 * (j + 1)) continue;  // uniform; (j + 1, j + 1): wave 0 has it
      const double* const pi = s.panel[t >> 4] + lane;
      const double* const pj = s.panel[t & 15] + lane;
#pragma unroll
      for (int v = 0; v < 4; ++v)
        acc[e] = __builtin_amdgcn_mfma_f64_16x16x4f64(-pi[64 * v], pj[64 * v], acc[e], 0, 0, 0);
      hand(t, j + 1, acc[e]);
    }
  }
}

// far != nullptr and zero: W is so close to the identity that the solve behind does without a factor (see there)
__global__ __launch_bounds__(1024) void chol_upper_reg_kernel(double* W, int b, double shift_rel, int* flag, const int* far) {
  __shared__ CholRegLds s;
  if (far && *far == 0) return;  // uniform
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const double mx = chol_diag_max(W, b, s.red);
  const CholShift shift{shift_rel, mx};
  const double tiny = 1e-300 + 1e-30 * mx;
  if (wave == 0) chol_pivot_wave(s, W, b, shift, tiny, flag);
  else chol_tile_wave(s, W, b, shift, wave);
}

// 256 < b <= 1024: the trailing matrix stays in memory; its tiles are dealt to the 16 waves four at a time so that their
// loads overlap.
__global__ __launch_bounds__(1024) void chol_upper_kernel(double* W, int b, double shift_rel, int* flag) {
  extern __shared__ __align__(16) unsigned char chol_smem[];
  const int bpad = (b + CH_NB - 1) / CH_NB * CH_NB, ldp = bpad + 2;
  double* panel = reinterpret_cast<double*>(chol_smem);  // [CH_NB][ldp]
  __shared__ double s_red[16];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const double mx = chol_diag_max(W, b, s_red);
  const double shift = shift_rel * mx;
  const double tiny = 1e-300 + 1e-30 * mx;
  const int fi = lane & 15, fk = lane >> 4;

  for (int j0 = 0; j0 < bpad; j0 += CH_NB) {
    const int wpad = bpad - j0;  // panel width, padded columns included
    // panel rows j0 .. j0+15, columns j0 .. bpad-1 (relative index c)
    for (int u = wave; u < CH_NB; u += 16)
      for (int c = lane; c < wpad; c += 64) {
        const bool real = j0 + u < b && j0 + c < b;
        double v = real ? (c >= u ? W[(int64_t)(j0 + u) * b + j0 + c] : 0.0) : (c == u ? 1.0 : 0.0);
        if (real && c == u) v += shift;
        panel[u * ldp + c] = v;
      }
    __syncthreads();
    for (int g = wave - 1; g < 0 || 16 + CH_GRP * g < wpad; g += 16) chol_panel_group(panel, ldp, wpad, g, tiny, W, b, j0, flag);
    __syncthreads();
    // trailing update, tile (I, J), I <= J, of the 16 x 16 blocks behind the panel:
    // W[i][c] -= sum_t R[t][i] R[t][c].  Lane (fi, fk) holds A(m = fi, k = fk), B(k = fk, n = fi);
    // its register v is D(m = 4 v + fk, n = fi).
    const int nb = wpad / CH_NB - 1;
    const int ntiles = nb * (nb + 1) / 2;
    for (int q0 = wave * CH_TB; q0 < ntiles; q0 += 16 * CH_TB) {
      f64x4_t acc[CH_TB];
      int ti[CH_TB], tj[CH_TB];
#pragma unroll
      for (int e = 0; e < CH_TB; ++e) {
        // tile number q -> (I, J): block row I holds nb - I tiles
        int q = q0 + e, I = 0;
        const bool live = q < ntiles;
        if (!live) q = 0;
        while (q >= nb - I) {
          q -= nb - I;
          ++I;
        }
        ti[e] = live ? I : -1;
        tj[e] = I + q;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int row = j0 + CH_NB * (I + 1) + 4 * v + fk, colg = j0 + CH_NB * (tj[e] + 1) + fi;
          acc[e][v] = (live && row < b && colg < b) ? W[(int64_t)row * b + colg] : 0.0;
        }
      }
#pragma unroll
      for (int e = 0; e < CH_TB; ++e) {
        if (ti[e] < 0) continue;  // uniform
#pragma unroll
        for (int s = 0; s < 4; ++s) {
          const double a = -panel[(4 * s + fk) * ldp + CH_NB * (ti[e] + 1) + fi];
          const double bb = panel[(4 * s + fk) * ldp + CH_NB * (tj[e] + 1) + fi];
          acc[e] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, bb, acc[e], 0, 0, 0);
        }
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int row = j0 + CH_NB * (ti[e] + 1) + 4 * v + fk, colg = j0 + CH_NB * (tj[e] + 1) + fi;
          if (row < b && colg < b) W[(int64_t)row * b + colg] = acc[e][v];
        }
      }
    }
    __syncthreads();
  }
}

// eight numbers as three bf16 parts each
__device__ __forceinline__ void split3(const float (&x)[8], u32x4 (&part)[3]) {
  float r[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) r[e] = x[e];
#pragma unroll
  for (int p = 0; p < 3; ++p) {
#pragma unroll
    for (int e = 0; e < 8; e += 2) {
      const uint32_t w = pack2_hw(r[e], r[e + 1]);
      part[p][e / 2] = w;
      r[e] -= __uint_as_float(w << 16);
      r[e + 1] -= __uint_as_float(w & 0xFFFF0000u);
    }
  }
}

// dst (rows x n fp32, pitch ldd) = src * R^-1 (src pitch lds; dst may be src: a workgroup reads its rows before it writes them)
// for the upper-triangular R (row-major n x n fp64, its 16 x 16 diagonal blocks inverted),
// in fp64 on the matrix cores.  A workgroup of eight waves solves 16 rows, as the transpose R^-T src^T: wave w holds the column
// tiles w, w + 8, ... of its rows as 16 x 16 accumulators Z_J (a result's registers are its operand layout, see above).  Step j:
// X_j = R_jj^-T Z_j, then Z_J -= R_jJ^T X_j for every J > j.  The wave that holds tile j + 1 updates it first, solves it and
// puts X_{j+1} into LDS before it updates its other tiles, so the chain of a step is eight matrix instructions and one trip through
// LDS; the parts of R for step j + 1 are requested a step ahead.  Within a tile, hardware index 4 a + b stands for
// column 4 b + a: a lane then holds four neighbouring columns of its row.
// 18.5 us at 2048 x 256, 9 us at 2048 x 128 (42 / 16.5 us in fp32 on the vector units, columns of R staged through LDS); R's lines not
// requested ahead 64 us.
// far != nullptr and zero (n <= 256): R holds src^T src instead, both triangles, which is within PANEL_ONCE of the identity, and dst is
// src (1.5 I - 0.5 src^T src), a Newton-Schulz step, also in fp64: no factorisation (57 us at n = 256).
// gate != nullptr and zero: nothing to do.
// PARTS (n <= 256): also the result as three bf16 parts for gram_times_block_kernel (its 16 rows are one k-block).
constexpr int TR_ROWS = 16, TR_W = 8;
template <int NT, bool PARTS>
__global__ __launch_bounds__(64 * TR_W) void trsm_right_upper_kernel(const float* src, int64_t lds, const double* __restrict__ R,
                                                                     float* dst, int64_t ldd, int64_t rows, int n, u32x4* parts, int ncb,
                                                                     const int* far, const int* gate) {
  if (gate && *gate == 0) return;  // uniform
  __shared__ double s_x[NT <= 2 ? TR_W * NT : 2][256];
  const bool near = NT <= 2 && far && *far == 0;  // uniform
  const int lane = threadIdx.x & 63, fi = lane & 15, fk = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int nb = (n + 15) / 16;
  const int64_t row = (int64_t)blockIdx.x * TR_ROWS + fi;
  const float* const srow = src + (row < rows ? row : rows - 1) * lds;
  // R was written by one compute unit a moment ago and is in no L2 but perhaps its own: ask for every line of its upper half at once,
  // instead of meeting a trip to memory at every step
  double touched = 0.0;
  for (int i = 4 * wave + fk; i < n; i += 4 * TR_W)
    for (int c = 16 * fi; c < n; c += 256)
      if (c + 15 >= i) touched += R[i * n + c];
  const int pfi = 4 * (fi & 3) + (fi >> 2);  // the column that hardware index fi stands for
  f64x4_t z[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    const int c = 16 * (wave + TR_W * t) + 4 * fk;
    if (c + 4 <= n) {
      const f32x4_el v = *reinterpret_cast<const f32x4_el*>(srow + c);
#pragma unroll
      for (int q = 0; q < 4; ++q) z[t][q] = (double)v[q];
    } else {
#pragma unroll
      for (int q = 0; q < 4; ++q) z[t][q] = c + q < n ? (double)srow[c + q] : 0.0;
    }
  }
  // block (I, J) of R as the operand of Z_J: element k = 4 v + fk, m = fi, i.e. row 16 I + 4 fk + v, column 16 J + pfi
  auto load_r = [&](int I, int J) __attribute__((always_inline)) {
    const int c = 16 * J + pfi, r0 = 16 * I + 4 * fk;
    // (past n: other elements of R, whose products end in columns that are not stored and are zeroed before the last block is
    // solved; no selects here, the loaded registers are not to be touched before their step)
    const int cc = min(c, n - 1);
    auto at = [&](int r) { return R[min(r, n - 1) * n + cc]; };
    return f64x4_t{at(r0), at(r0 + 1), at(r0 + 2), at(r0 + 3)};
  };
  auto put = [&](int j, const f64x4_t& x) __attribute__((always_inline)) {
#pragma unroll
    for (int v = 0; v < 4; ++v) s_x[j & 1][64 * v + lane] = -x[v];
  };
  const f64x4_t zero = {0.0, 0.0, 0.0, 0.0};
  if (near) {
    if constexpr (NT <= 2) {
#pragma unroll
      for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int v = 0; v < 4; ++v) s_x[wave + TR_W * t][64 * v + lane] = z[t][v];
      __syncthreads();
      // four blocks at a time, the next four requested before these are multiplied (past the last one: others again, times zeros)
      constexpr int BATCHES = 2 * NT * NT;
      f64x4_t m[2][4], a = zero;
      auto request = [&](auto bc) __attribute__((always_inline)) {
        constexpr int B = decltype(bc)::value;
#pragma unroll
        for (int u = 0; u < 4; ++u) m[B & 1][u] = load_r(4 * (B % (2 * NT)) + u, wave + TR_W * (B / (2 * NT)));
      };
      request(std::integral_constant<int, 0>{});
      chol_static_for<BATCHES>([&](auto bc) __attribute__((always_inline)) {
        constexpr int B = decltype(bc)::value, t = B / (2 * NT), I0 = 4 * (B % (2 * NT));
        if constexpr (B + 1 < BATCHES) request(std::integral_constant<int, B + 1>{});
        __builtin_amdgcn_sched_barrier(0);
        const int c = 16 * (wave + TR_W * t) + pfi;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          f64x4_t x;
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            x[v] = s_x[I0 + u][64 * v + lane];
            m[B & 1][u][v] = (16 * (I0 + u) + 4 * fk + v == c ? 1.5 : 0.0) - 0.5 * m[B & 1][u][v];
          }
          a = chol_mul(m[B & 1][u], x, a);
        }
        if constexpr (I0 + 4 == 8 * NT) {
          z[t] = a;
          a = zero;
        }
      });
    }
  } else {
  if (wave == 0) {
    z[0] = chol_mul(load_r(0, 0), z[0], zero);
    put(0, z[0]);
  }
  f64x4_t r[NT], d;  // blocks (j, J) of this wave's tiles, and its next diagonal block
#pragma unroll
  for (int t = 0; t < NT; ++t)
    if (wave + TR_W * t < nb) r[t] = load_r(0, wave + TR_W * t);
  const int first = min(wave == 0 ? TR_W : wave, nb - 1);
  d = load_r(first, first);
  chol_static_for<NT>([&](auto tc) {
    constexpr int T = decltype(tc)::value;
#pragma unroll 1
    for (int q = 0; q < TR_W; ++q) {
      const int j = TR_W * T + q;
      if (j + 1 >= nb) break;  // uniform
      __syncthreads();  // X_j is in LDS
      f64x4_t x;
#pragma unroll
      for (int v = 0; v < 4; ++v) x[v] = s_x[j & 1][64 * v + lane];
      auto step = [&](auto uc) {
        constexpr int U = decltype(uc)::value;
        const int J = wave + TR_W * U;
        if (J <= j || J >= nb) return;  // uniform
        z[U] = chol_mul(r[U], x, z[U]);
        r[U] = load_r(j + 1, J);  // (not needed again if the tile is solved now)
        if (J == j + 1) {
          if (16 * (J + 1) > n) {  // uniform
#pragma unroll
            for (int v = 0; v < 4; ++v) z[U][v] = 16 * J + 4 * fk + v < n ? z[U][v] : 0.0;
          }
          z[U] = chol_mul(d, z[U], zero);
          put(j + 1, z[U]);
          const int D = min(J + TR_W, nb - 1);
          d = load_r(D, D);
        }
      };
      chol_static_for<NT - T>([&](auto uc) { step(std::integral_constant<int, T + decltype(uc)::value>{}); });
    }
  });
  }
  asm volatile("" : : "v"(touched));
  if constexpr (PARTS) {
    __shared__ float tile[TR_ROWS][260];
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int c = 16 * (wave + TR_W * t) + 4 * fk + q;
        tile[fi][c] = row < rows && c < n ? (float)z[t][q] : 0.f;
      }
    __syncthreads();
    const int c = threadIdx.x & 255, h = threadIdx.x >> 8;
    if (c < 32 * ncb) {
      float x[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) x[e] = c < 128 * NT ? tile[8 * h + e][c] : 0.f;
      u32x4 part[3];
      split3(x, part);
#pragma unroll
      for (int p = 0; p < 3; ++p) parts[(((int64_t)blockIdx.x * ncb + (c >> 5)) * 3 + p) * 64 + 32 * h + (c & 31)] = part[p];
    }
  }
  if (row < rows) {
    float* const drow = dst + row * ldd;
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      const int c = 16 * (wave + TR_W * t) + 4 * fk;
      if (c + 4 <= n) {
        f32x4_el v;
#pragma unroll
        for (int q = 0; q < 4; ++q) v[q] = (float)z[t][q];
        *reinterpret_cast<f32x4_el*>(drow + c) = v;
      } else {
#pragma unroll
        for (int q = 0; q < 4; ++q)
          if (c + q < n) drow[c + q] = (float)z[t][q];
      }
    }
  }
}

// ------------------------------------------------------- symmetric eigen (Jacobi; more than 256 columns)
// One-sided (Hestenes) Jacobi on the columns of the symmetric PSD matrix H, held
// row-major so that "column" p is the contiguous row p (H is symmetric).  Rotating
// column pairs until all are mutually orthogonal gives H J = B with B's columns
// lambda_i v_i, so the eigenvectors are the normalised columns and the eigenvalues
// their norms.
//
// Block version: the b columns are cut into blocks of 16; a round-robin tournament over the blocks pairs them up, one
// workgroup per pair and one launch per tournament step.  A workgroup forms the 32 x 32 Gram matrix of its columns on the
// fp64 matrix cores, diagonalises it approximately with an inner tournament of two-sided rotations (which touch the
// Gram matrix and the accumulated rotation J, 32 x 32 each, instead of the columns), and multiplies its columns by J,
// again on the matrix cores.  The Gram matrix is fresh in every launch, so the rounding of the rotations applied to it
// never accumulates, and convergence is judged on fresh inner products.  `counts[sweep]` collects the block pairs of a
// sweep that had to be rotated, and the launches of sweep s+1 return at once when sweep s rotated nothing.

__device__ __forceinline__ void tournament_pair(int step, int i, int players_even, int& p, int& q) {
  const int n1 = players_even - 1;
  if (i == 0) {
    p = step % n1;
    q = players_even - 1;
  } else {
    p = (step + i) % n1;
    q = (step - i + n1) % n1;
  }
}

// H <- (H + H^T) / 2; block 0 also leaves the largest diagonal entry in *hmax (the scale against
// which the eigen-iteration decides that a column is numerically zero)
__global__ __launch_bounds__(1024) void symmetrize64_kernel(double* H, int b, double* hmax) {
  if (blockIdx.x == 0) {
    __shared__ double s_mx[16];
    double mx = 0.0;
    for (int i = threadIdx.x; i < b; i += 1024) mx = fmax(mx, fabs(H[(int64_t)i * b + i]));
    for (int o = 32; o > 0; o >>= 1) mx = fmax(mx, __shfl_xor(mx, o));
    if ((threadIdx.x & 63) == 0) s_mx[threadIdx.x >> 6] = mx;
    __syncthreads();
    if (threadIdx.x == 0) {
      for (int w = 1; w < 16; ++w) mx = fmax(mx, s_mx[w]);
      *hmax = mx;
    }
  }
  for (int e = blockIdx.x * 1024 + threadIdx.x; e < b * b; e += gridDim.x * 1024) {
    const int i = e / b, j = e % b;
    if (i < j) {
      const double m = 0.5 * (H[(int64_t)i * b + j] + H[(int64_t)j * b + i]);
      H[(int64_t)i * b + j] = m;
      H[(int64_t)j * b + i] = m;
    }
  }
}

// The rotation that makes columns p and q orthogonal, from their squared norms al, be and inner product ga:
// p' = cs p - sn q, q' = sn p + cs q.  True if the pair needs one (|ga| > tol sqrt(al be), compared as squares).  The angle may
// be approximate (the iteration corrects it), so tan comes from the hardware reciprocal / square root estimates; (cs, sn)
// must be a rotation to full precision, so cs = (1 + tan^2)^-1/2 gets a third-order step on top of its estimate (2^-23, cubed).
__device__ __forceinline__ bool needs_rotation(double al, double be, double ga, double tol) {
  return ga * ga > tol * tol * al * be && fabs(ga) > 1e-300;
}
__device__ __forceinline__ void rotation(double al, double be, double ga, double tol, double& cs, double& sn) {
  const double zeta = (be - al) * 0.5 * __builtin_amdgcn_rcp(ga);
  const double az = fabs(zeta);
  const double tt = copysign(__builtin_amdgcn_rcp(az + __builtin_amdgcn_sqrt(1.0 + az * az)), zeta);
  const double w = 1.0 + tt * tt;
  double c = __builtin_amdgcn_rsq(w);
  const double e = fma(-w * c, c, 1.0);
  c = fma(c * e, fma(e, 0.375, 0.5), c);
  const bool rot = needs_rotation(al, be, ga, tol);
  cs = rot ? c : 1.0;
  sn = rot ? c * tt : 0.0;
}

// x of lane g of lane row g, in every lane of that row
__device__ __forceinline__ double row_diag_f64(double x) {
  double r;
  asm volatile(
      "s_nop 1\n"
      "v_mov_b64_dpp %0, %1 row_newbcast:0 row_mask:0x1 bank_mask:0xf\n"
      "v_mov_b64_dpp %0, %1 row_newbcast:1 row_mask:0x2 bank_mask:0xf\n"
      "v_mov_b64_dpp %0, %1 row_newbcast:2 row_mask:0x4 bank_mask:0xf\n"
      "v_mov_b64_dpp %0, %1 row_newbcast:3 row_mask:0x8 bank_mask:0xf\n"
      : "=&v"(r) : "v"(x));
  return r;
}
// x of a neighbouring lane of the row of 16 (CTRL 0x101: the next one, 0x111: the one before; `edge` where there is none;
// 0x12f: the next one, lane 0 for the last)
template <int CTRL>
__device__ __forceinline__ double row_shift_f64(double x, double edge) {
  return __hiloint2double(
      __builtin_amdgcn_update_dpp(__double2hiint(edge), __double2hiint(x), CTRL, 0xf, 0xf, false),
      __builtin_amdgcn_update_dpp(__double2loint(edge), __double2loint(x), CTRL, 0xf, 0xf, false));
}

// 8 waves: 0 - 3 rotate the Gram matrix in LDS (a step reads one buffer and writes the other: one barrier), 4 - 7 the
// accumulated rotation in registers.  What bounds it is the issue of a step's instructions (two waves per SIMD) and one round trip
// through LDS, so no address is computed in it, and a row of 16 lanes passes its rotations on by DPP.
// At b = 320: 29 us per launch with all pairs, 25 us across the blocks, 12 us where no pair needs a rotation, 3.4 ms for a cold fit's seven
// sweeps; at b = 512 31, 27, 12 us and 6.5 ms.  (With every address and every thread's rotations computed in the step 29 us instead of 21 at b = 256.)
constexpr int JB_NB = 16, JB_M = 2 * JB_NB;   // columns per block and per workgroup
constexpr int JB_CW = 256, JB_CS = JB_CW + 4; // elements of each column in LDS at a time, their pitch
constexpr int JB_GS = JB_M + 1;               // pitch of the Gram matrices and of J
// Every fifth launch of a sweep rotates all pairs of its 32 columns, the others those across the two blocks: half the inner steps.
// (Chosen by a simulation of three spectra at b = 256, launches weighted by their times there: every launch full 1.67 - 1.81 ms in six to
// seven sweeps, every third 1.38 - 1.52, every fifth 1.32 - 1.47, the first of a sweep only 1.61 in eight.)  Steep spectra with few power
// iterations take up to four sweeps more that way (simulated at b = 80, singular values ~ i^-2.5, some channels 100 times the others, one
// iteration: 12 with every launch full, 14 to 16; with all pairs from the ninth sweep on 14), so the ninth sweep and later ones rotate all
// pairs and the limit lies four sweeps above the twelve that all-pair launches had.
constexpr int JB_FULL = 5, JB_FULL_FROM = 8;
constexpr int JB_SWEEPS = 16;  // before the iteration gives up
constexpr size_t JB_SMEM = (size_t)(JB_M * JB_CS + 4 * JB_M * JB_GS) * sizeof(double);
// counts[sweep] goes up by one for every pair of blocks that has a pair of columns that needed a rotation
__global__ __launch_bounds__(512) void jacobi_block_kernel(double* H, int b, int nblk_even, int step, int sweep, double tol,
                                                           unsigned* counts, const double* hmax) {
  if (sweep > 0 && counts[sweep - 1] == 0) return;  // converged in the previous sweep
  int bp, bq;
  tournament_pair(step, blockIdx.x, nblk_even, bp, bq);
  const bool full = step % JB_FULL == 0 || sweep >= JB_FULL_FROM;
  extern __shared__ __align__(16) unsigned char jac_smem[];
  double* cols = reinterpret_cast<double*>(jac_smem);  // [JB_M][JB_CS]: one chunk of the columns
  double* gram = cols + JB_M * JB_CS;                  // [3][JB_M][JB_GS]
  double* J = gram + 3 * JB_M * JB_GS;                 // [JB_M][JB_GS]: new column c = sum_l J[l][c] column l
  __shared__ double2 cs_lds[32];                       // cosines and sines of this step and the one before
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int fi = lane & 15, fk = lane >> 4;
  // local column l is column grow(l) of H; blocks past the end are byes, columns past the end are zero
  auto grow = [&](int l) { return (l < JB_NB ? bp : bq) * JB_NB + (l & (JB_NB - 1)); };
  const int nch = (b + JB_CW - 1) / JB_CW;
  auto load_chunk = [&](int ch) {
    double v[JB_M * JB_CW / 512];
#pragma unroll
    for (int e = 0; e < JB_M * JB_CW / 512; ++e) {
      const int row = grow(2 * e + (tid >> 8)), c = ch * JB_CW + (tid & 255);
      v[e] = row < b && c < b ? H[(int64_t)row * b + c] : 0.0;
    }
#pragma unroll
    for (int e = 0; e < JB_M * JB_CW / 512; ++e) cols[(2 * e + (tid >> 8)) * JB_CS + (tid & 255)] = v[e];
  };
  {  // Gram matrix: four 16 x 16 tiles, the sum over a chunk in two halves; gram[half] = partial sum
    const int half = wave >> 2, I = (wave >> 1) & 1, Jt = wave & 1;
    f64x4_t acc = {0.0, 0.0, 0.0, 0.0};
    for (int ch = 0; ch < nch; ++ch) {
      if (ch > 0) __syncthreads();
      load_chunk(ch);
      __syncthreads();
      const double* pa = cols + (16 * I + fi) * JB_CS + half * (JB_CW / 2) + fk;
      const double* pb = cols + (16 * Jt + fi) * JB_CS + half * (JB_CW / 2) + fk;
#pragma unroll 8
      for (int s = 0; s < JB_CW / 8; ++s) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(pa[4 * s], pb[4 * s], acc, 0, 0, 0);
    }
    double* g = gram + half * JB_M * JB_GS + (16 * I + fk) * JB_GS + 16 * Jt + fi;
#pragma unroll
    for (int v = 0; v < 4; ++v) g[4 * v * JB_GS] = acc[v];
  }
  __syncthreads();
  // a pair with a numerically zero column (an eigenvalue below 1e-13 of the largest: rank-deficient input) is
  // rotated but does not count towards convergence: such a column is rounding noise and its cosines never settle
  const double floor2 = 1e-26 * *hmax * *hmax;
  bool rot = false, counted = false;
  auto place = [&](int l) { return l < 16 || !full ? l : 16 + (JB_M - 1 - l); };  // of column l when the inner tournament starts
#pragma unroll
  for (int e = 0; e < 2; ++e) {
    const int r = (tid >> 5) + 16 * e, c = tid & 31;
    auto g = [&](int i, int j) { return gram[i * JB_GS + j] + gram[(JB_M + i) * JB_GS + j]; };
    const double ga = g(r, c), al = g(r, r), be = g(c, c);
    gram[(2 * JB_M + place(r)) * JB_GS + place(c)] = ga;
    if (r < c && needs_rotation(al, be, ga, tol)) {
      rot = true;
      counted = counted || fmin(al, be) > floor2;
    }
  }
  const bool any_counted = __syncthreads_or(counted);
  if (!__syncthreads_or(rot)) return;
  if (any_counted && tid == 0) atomicAdd(&counts[sweep], 1u);
  // Inner tournament.  The 32 players sit in places, pair j in places j and 16 + j, and move on after a step.  All pairs (`full`):
  // place j -> j - 1 (0 -> 17) and 16 + j -> 16 + j + 1 (31 -> 15; 16 stays), 31 steps.  Pairs across the two blocks only: the
  // lower places stay, 16 + j -> 16 + j - 1 (16 -> 31), 16 steps.  Then everybody is home.  The matrix is kept by place, so a
  // thread's addresses never change.
  const int steps = full ? JB_M - 1 : JB_NB;
  if (wave < 4) {
    // thread (i, j): the 2 x 2 block of row pair i and column pair j.  Lane l of a row holds j = l + 4 wave (mod 16), so that the
    // rotation of row pair i = 4 wave + g is in lane g of lane row g.
    const int i = 4 * wave + (lane >> 4), j = ((lane & 15) + 4 * wave) & 15;
    auto next_top = [&](int x) { return full ? (x == 0 ? 17 : x - 1) : x; };
    auto next_bottom = [&](int x) { return full ? (x == 0 ? 16 : (x == 15 ? 15 : 17 + x)) : 16 + ((x + 15) & 15); };
    const int r_al = j * JB_GS + j, r_be = (16 + j) * JB_GS + 16 + j, r_ga = j * JB_GS + 16 + j;
    const int r_a = i * JB_GS + j, r_c = (16 + i) * JB_GS + j;
    const int ti = next_top(i), tj = next_top(j), bi = next_bottom(i), bj = next_bottom(j);
    const int w_tt = ti * JB_GS + tj, w_bt = bi * JB_GS + tj, w_tb = ti * JB_GS + bj, w_bb = bi * JB_GS + bj;
    auto step = [&](const double* cur, double* nxt, double2* cs) {
      const double al = cur[r_al], be = cur[r_be], ga = cur[r_ga];
      const double a = cur[r_a], bb = cur[r_a + 16], c = cur[r_c], d = cur[r_c + 16];
      double cj, sj;
      rotation(al, be, ga, tol, cj, sj);
      if (wave == 0 && lane < 16) cs[j] = make_double2(cj, sj);
      const double ci = row_diag_f64(cj), si = row_diag_f64(sj);
      const double a1 = cj * a - sj * bb, b1 = sj * a + cj * bb, c1 = cj * c - sj * d, d1 = sj * c + cj * d;
      nxt[w_tt] = ci * a1 - si * c1;
      nxt[w_bt] = si * a1 + ci * c1;
      nxt[w_tb] = ci * b1 - si * d1;
      nxt[w_bb] = si * b1 + ci * d1;
      __syncthreads();
    };
    double* const g0 = gram + 2 * JB_M * JB_GS;
    for (int s = 0; s + 1 < steps; s += 2) {
      step(g0, gram, cs_lds);
      step(gram, g0, cs_lds + 16);
    }
    if (steps & 1) step(g0, gram, cs_lds);
  } else {
    // The accumulated rotation J stays in registers, two of its rows per lane row, lane j the columns of the players in places j and
    // 16 + j, and follows one step behind.
    const int j = lane & 15, r0 = 8 * (wave - 4) + 2 * (lane >> 4), home = full ? JB_M - 1 - j : JB_NB + j;
    double x[2], y[2];
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      x[e] = r0 + e == j ? 1.0 : 0.0;
      y[e] = r0 + e == home ? 1.0 : 0.0;
    }
    auto step = [&](const double2* cs) {
      __syncthreads();
      const double2 r = cs[j];
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        const double p = r.x * x[e] - r.y * y[e], q = r.y * x[e] + r.x * y[e];
        if (full) {
          x[e] = row_shift_f64<0x101>(p, q);
          y[e] = row_shift_f64<0x111>(j == 0 ? p : q, q);
        } else {
          x[e] = p;
          y[e] = row_shift_f64<0x12f>(q, q);
        }
      }
    };
    for (int s = 0; s + 1 < steps; s += 2) {
      step(cs_lds);
      step(cs_lds + 16);
    }
    if (steps & 1) step(cs_lds);
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      J[(r0 + e) * JB_GS + j] = x[e];
      J[(r0 + e) * JB_GS + home] = y[e];
    }
  }
  __syncthreads();
  // columns <- J^T columns, 32 elements of every column per wave and chunk
  for (int ch = 0; ch < nch; ++ch) {
    if (nch > 1) {
      if (ch > 0) __syncthreads();
      load_chunk(ch);
      __syncthreads();
    }
    f64x4_t acc[2][2] = {};
#pragma unroll
    for (int s = 0; s < JB_M / 4; ++s) {
      const double* pj = J + (4 * s + fk) * JB_GS + fi;
      const double* pc = cols + (4 * s + fk) * JB_CS + 32 * wave + fi;
#pragma unroll
      for (int mi = 0; mi < 2; ++mi)
#pragma unroll
        for (int ni = 0; ni < 2; ++ni)
          acc[mi][ni] = __builtin_amdgcn_mfma_f64_16x16x4f64(pj[16 * mi], pc[16 * ni], acc[mi][ni], 0, 0, 0);
    }
#pragma unroll
    for (int mi = 0; mi < 2; ++mi)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int row = grow(16 * mi + 4 * v + fk);
#pragma unroll
        for (int ni = 0; ni < 2; ++ni) {
          const int c = ch * JB_CW + 32 * wave + 16 * ni + fi;
          if (row < b && c < b) H[(int64_t)row * b + c] = acc[mi][ni][v];
        }
      }
  }
}

// eigenvalues = column norms; normalise the columns in place; raise flag bit 2 if the last
// sweep still rotated
__global__ __launch_bounds__(1024) void jacobi_finish_kernel(double* H, int b, double* lambda, const unsigned* counts,
                                                             int last_sweep, int* flag) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  if (blockIdx.x == 0 && tid == 0 && counts[last_sweep] != 0) atomicOr(flag, 2);
  for (int p = blockIdx.x * 16 + wave; p < b; p += gridDim.x * 16) {
    double* hp = H + (int64_t)p * b;
    double al = 0.0;
    for (int t = lane; t < b; t += 64) al += hp[t] * hp[t];
    for (int o = 32; o > 0; o >>= 1) al += __shfl_xor(al, o);
    const double nrm = sqrt(al);
    const double inv = nrm > 0.0 ? 1.0 / nrm : 0.0;
    for (int t = lane; t < b; t += 64) hp[t] *= inv;
    if (lane == 0) lambda[p] = nrm;
  }
}

__global__ void zero_u32_kernel(unsigned* p, int n) {
  for (int i = threadIdx.x; i < n; i += blockDim.x) p[i] = 0u;
}

// Z (b x k fp32, row-major) = the k eigenvectors with the largest eigenvalues, in
// descending order; eigenvector p is row p of Hn (normalised Jacobi output).
// A wave per eigenvector: its rank is the number of larger eigenvalues.
__global__ __launch_bounds__(256) void select_top_kernel(const double* __restrict__ Hn, const double* __restrict__ lambda,
                                                         int b, int k, float* Z) {
  const int lane = threadIdx.x & 63, p = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (p >= b) return;
  const double me = lambda[p];
  int rk = 0;
  for (int o = lane; o < b; o += 64) {
    const double v = lambda[o];
    rk += (v > me) || (v == me && o < p);
  }
  for (int o = 32; o > 0; o >>= 1) rk += __shfl_xor(rk, o);
  if (rk < k)
    for (int t = lane; t < b; t += 64) Z[(int64_t)t * k + rk] = (float)Hn[(int64_t)p * b + t];
}

__global__ __launch_bounds__(256) void copy_cols_kernel(const float* __restrict__ src, int64_t lds, float* dst,
                                                        int64_t ldd, int64_t rows, int cols) {
  const int64_t total = rows * cols;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += (int64_t)gridDim.x * blockDim.x)
    dst[(i / cols) * ldd + i % cols] = src[(i / cols) * lds + i % cols];
}

// ------------------------------------------------------- G V
// Y = G V for the iteration (G symmetric d x d, V d x b, both fp32), on the bf16 matrix instructions: every number as three bf16 parts
// that add up to it exactly (8 significant bits each, rounded to nearest), and of the nine products the six down to
// 2^-17 of the largest; the other three come to less than 2^-24 of a product.  The sums are fp32 as before, a sixteenth as many.
// Parts lie in fragment order, a 32 x 16 piece of an operand as 3 x [64 lanes][8]: G as [row blocks][k-blocks], split once per fit, V as
// [k-blocks][column blocks], written by the triangular solve that makes it.
// A workgroup has 32 rows and 64 columns, its eight waves every eighth k-block; their sums meet in LDS, in wave order.  Bound by L2
// (9 KB per twelve matrix instructions of a wave, 302 MB per launch at d = 2048, b = 256); a larger tile would leave compute units idle or
// need ranges of k and their sum.  16.8 us there, where fp32 instructions took 27 and the sum of two ranges 5.  |Y - G V| against 64 bits: 0.4 to
// 0.9 of theirs in six shapes of d 256 to 2048, b 2 to 256 (1.3e-7 of |Y| against 3.0e-7 at d = 2048, b = 256).
// Blocks of more than GV_MAX columns keep the fp32 instructions: their factorisation is shifted by a share of the largest diagonal entry
// (see CholShift), and of batches of lower rank than the block the noise that rounding leaves in the surplus columns has to be above that.
// With less of it 4 of 92 such fits of 240 drawn ones that were accepted were refused.
constexpr int GV_MAX = 256;
// Narrower blocks and fewer features keep the fp32 instructions too: a launch costs more than their product (fixed 5 us against 3), cutting G into parts 3 to 120 us
// more, and G in parts is half as many bytes again, read once per 64 columns.  Fits on fp32 instructions less fits on parts, us (2048 rows, d x b):
// 1024 x 65 -8, x 128 -1, x 130 24; 768 x 130 -2, x 256 8; 1536 x 64 -2, x 66 16, x 128 54; 2048 x 64 -28, x 66 9; 2502 x 32 -20, x 64 31; 4096 x 32 -54, x 64 10,
// x 256 264; 6007 x 64 212; 7001 x 32 -202, x 64 54; 8192 x 64 -158 (parts past the last cache), x 66 84, x 128 66.
inline bool gv_parts(int64_t d, int b) {
  if (b > GV_MAX) return false;
  return b > 128 ? d >= 1024 : b > 64 ? d >= 1536 : b > 32 && d >= 2500 && d <= 7000;
}
constexpr int GV_W = 8, GV_D = 4;  // waves, k-blocks in flight
static inline int gv_kblocks(int64_t d) { return (int)(round_up64(d, 16 * GV_W) / 16); }
static inline size_t gv_g_bytes(int64_t d) { return (size_t)((d + 31) / 32) * gv_kblocks(d) * 3072; }
static inline int gv_col_blocks(int b) { return (b + 63) / 64 * 2; }
static inline size_t gv_v_bytes(int64_t d, int b) { return (size_t)gv_kblocks(d) * gv_col_blocks(b) * 3072; }

// The matrix instructions take a subnormal bf16 part as zero, so a row of G whose diagonal entry is below 2^-40 (then no entry of it is above 2^44) goes in
// times 2^48 and its Y comes back by as much: without that a batch of elements around 2^-64, whose third and then second parts are subnormal, lost its
// weaker directions (1.9e-3 off instead of 1.6e-5; at 2^-68 0.3).
__device__ __forceinline__ bool gv_tiny_row(float diag) { return diag < 0x1p-40f; }

// KF (G): line i, element k at src[i ld + k], pieces [line blocks][k-blocks]; otherwise at src[k ld + i], pieces [k-blocks][line blocks].
// Zeros outside lines x K.
template <bool KF>
__global__ __launch_bounds__(256) void split_parts_kernel(const float* __restrict__ src, int64_t ld, int lines, int64_t K, int nlb,
                                                          int nkb, u32x4* __restrict__ out) {
  const int64_t piece = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (piece >= (int64_t)nlb * nkb) return;
  const int lane = threadIdx.x & 63;
  const int64_t lb = KF ? piece / nkb : piece % nlb, kb = KF ? piece % nkb : piece / nlb;
  const int64_t line = 32 * lb + (lane & 31), k = 16 * kb + 8 * (lane >> 5);
  float x[8];
  if (line < lines && k + 8 <= K) {
#pragma unroll
    for (int e = 0; e < 8; ++e) x[e] = KF ? src[line * ld + k + e] : src[(k + e) * ld + line];
  } else {
#pragma unroll
    for (int e = 0; e < 8; ++e) x[e] = line < lines && k + e < K ? (KF ? src[line * ld + k + e] : src[(k + e) * ld + line]) : 0.f;
  }
  if constexpr (KF) {
    const float up = line < lines && gv_tiny_row(src[line * ld + line]) ? 0x1p48f : 1.f;
#pragma unroll
    for (int e = 0; e < 8; ++e) x[e] *= up;
  }
  u32x4 part[3];
  split3(x, part);
#pragma unroll
  for (int p = 0; p < 3; ++p) out[(piece * 3 + p) * 64 + lane] = part[p];
}

__global__ __launch_bounds__(64 * GV_W, 2) void gram_times_block_kernel(const u32x4* __restrict__ Gf, const u32x4* __restrict__ Vf,
                                                                        const float* __restrict__ G, int d, int b, int nkb, int ncb,
                                                                        float* __restrict__ Y) {
  extern __shared__ float gv_red[];  // [GV_W][32][64]
  // the column tiles of a few row blocks sit next to each other on one XCD
  const int tiles_n = ncb / 2, total = (d + 31) / 32 * tiles_n, per_xcd = (total + 7) / 8;
  const int slot = blockIdx.x >> 3, logical = (blockIdx.x & 7) * per_xcd + slot;
  if (slot >= per_xcd || logical >= total) return;
  const int tm = logical / tiles_n, tn = logical % tiles_n;
  const int lane = threadIdx.x & 63, li = lane & 31, lh = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const u32x4* const pg = Gf + (int64_t)tm * nkb * 192 + lane;
  const u32x4* const pv = Vf + (int64_t)tn * 384 + lane;
  const int64_t vrow = (int64_t)ncb * 192;
  struct Step {
    u32x4 g[3], v[2][3];
  };
  auto load = [&](Step& s, int kb) __attribute__((always_inline)) {
#pragma unroll
    for (int p = 0; p < 3; ++p) s.g[p] = pg[(int64_t)kb * 192 + p * 64];
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
      for (int p = 0; p < 3; ++p) s.v[c][p] = pv[kb * vrow + (c * 3 + p) * 64];
  };
  // the products of the high parts and the other five, which are 2^-8 of them at most, have sums of their own: six roundings per
  // k-block at the size of the sum would put Y further off than the fp32 instructions do
  f32x16 acc[2], low[2];
#pragma unroll
  for (int c = 0; c < 2; ++c)
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[c][v] = low[c][v] = 0.f;
  auto mul = [&](const Step& s) __attribute__((always_inline)) {
    constexpr int PG[5] = {2, 0, 1, 1, 0}, PV[5] = {0, 2, 1, 0, 1};
#pragma unroll
    for (int c = 0; c < 2; ++c)
      acc[c] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_frag(s.g[0]), as_frag(s.v[c][0]), acc[c], 0, 0, 0);
#pragma unroll
    for (int t = 0; t < 5; ++t)
#pragma unroll
      for (int c = 0; c < 2; ++c)
        low[c] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_frag(s.g[PG[t]]), as_frag(s.v[c][PV[t]]), low[c], 0, 0, 0);
  };
  // row of register v in the result's layout
  auto row_of = [&](int v) { return 32 * tm + 8 * (v / 4) + 4 * lh + v % 4; };
  float diag[4];  // of the four rows that this thread stores
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int row = min(row_of((wave * 4 + u) & 15), d - 1);
    diag[u] = G[(int64_t)row * d + row];
  }
  const int n = nkb / GV_W;  // (a multiple)
  Step st[GV_D];
#pragma unroll
  for (int u = 0; u < GV_D; ++u)
    load(st[u], wave + GV_W * min(u, n - 1));
  int t = 0;
  for (; t + 2 * GV_D <= n; t += GV_D) {  // (no test per request here: behind one the compiler waits for all of them)
#pragma unroll
    for (int u = 0; u < GV_D; ++u) {
      mul(st[u]);
      load(st[u], wave + GV_W * (t + GV_D + u));
      __builtin_amdgcn_sched_barrier(0);  // (requests stay where they are, or all of them end up behind the products)
    }
  }
#pragma unroll
  for (int u = 0; u < GV_D; ++u) {
    if (t + u < n) mul(st[u]);
    if (t + GV_D + u < n) load(st[u], wave + GV_W * (t + GV_D + u));
  }
#pragma unroll
  for (int u = 0; u < GV_D - 1; ++u)
    if (t + GV_D + u < n) mul(st[u]);
#pragma unroll
  for (int c = 0; c < 2; ++c)
#pragma unroll
    for (int v = 0; v < 16; ++v) gv_red[(wave * 32 + c * 16 + v) * 64 + lane] = acc[c][v] + low[c][v];
  __syncthreads();
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    const int r = wave * 4 + u;
    float x = 0.f;
#pragma unroll
    for (int w = 0; w < GV_W; ++w) x += gv_red[(w * 32 + r) * 64 + lane];
    const int row = row_of(r & 15), col = 64 * tn + 32 * (r >> 4) + li;
    if (row < d && col < b) Y[(int64_t)row * b + col] = gv_tiny_row(diag[u]) ? x * 0x1p-48f : x;
  }
}

// ------------------------------------------------------- Gram matrices of the panels
// src^T src for a d x n fp32 block (pitch n) with fp64 sums on the matrix cores: the 64 x 64 tiles of the upper triangle (all that the
// factorisation reads) times ranges of rows, as many as fill the chip; 32 x 32 per wave, 32 rows per step, the next step's
// operands requested before this one's are multiplied.  Partial sums go to `slabs` as the 16 x 16 blocks of the upper triangle, in
// register order.
// 8.8 us at 2048 x 256, 13 us at 4096 x 256 (21 and 38 us with all tiles, four times the partial sums and each step's operands
// requested when the step before was done); the sum 4.7 us.
constexpr int PG_K = 32;
static inline int pg_tiles(int n) { return ((n + 63) / 64) * ((n + 63) / 64 + 1) / 2; }
static inline size_t pg_bytes(int n) { return (size_t)(((n + 15) / 16) * ((n + 15) / 16 + 1) / 2) * 256 * 8; }  // of one range
// (*far and, without a gate, the word behind it are zeroed for the kernels that follow; gate != nullptr and zero: nothing to do)
__global__ __launch_bounds__(256) void panel_gram64_kernel(const float* __restrict__ src, int64_t lds, int64_t d, int n,
                                                           int64_t rows_per_split, double* __restrict__ slabs, int* far, const int* gate) {
  if (gate && *gate == 0) return;  // uniform
  if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x < (gate ? 1 : 2)) far[threadIdx.x] = 0;
  const int lane = threadIdx.x & 63, fi = lane & 15, fk = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int nb = (n + 63) / 64;
  int J = blockIdx.x, I = 0;  // tile number -> (I, J), I <= J
  while (J >= nb - I) {
    J -= nb - I;
    ++I;
  }
  J += I;
  const int64_t kbeg = (int64_t)blockIdx.y * rows_per_split, kend = min(d, kbeg + rows_per_split);
  const float* pa[2];
  const float* pb[2];
#pragma unroll
  for (int t = 0; t < 2; ++t) {  // columns past n repeat the last one: their products are not used
    pa[t] = src + min(64 * I + 32 * (wave >> 1) + 16 * t + fi, n - 1);
    pb[t] = src + min(64 * J + 32 * (wave & 1) + 16 * t + fi, n - 1);
  }
  f64x4_t acc[2][2] = {};
  struct Step {
    float a[PG_K / 4][2], b[PG_K / 4][2];
  };
  auto load = [&](Step& s, int64_t k0, int64_t last) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < PG_K / 4; ++u) {
      const int64_t o = min(k0 + 4 * u + fk, last) * lds;
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        s.a[u][t] = pa[t][o];
        s.b[u][t] = pb[t][o];
      }
    }
  };
  auto mul = [&](const Step& s) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < PG_K / 4; ++u)
#pragma unroll
      for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int y = 0; y < 2; ++y)
          acc[x][y] = __builtin_amdgcn_mfma_f64_16x16x4f64((double)s.a[u][x], (double)s.b[u][y], acc[x][y], 0, 0, 0);
  };
  const int64_t full = (kend - kbeg) / PG_K, last = kend - 1;
  Step s0, s1;
  load(s0, kbeg, last);
  int64_t i = 0;
  for (; i + 2 <= full; i += 2) {
    load(s1, kbeg + (i + 1) * PG_K, last);
    mul(s0);
    load(s0, kbeg + (i + 2) * PG_K, last);  // (past the range: its last row again, not used)
    mul(s1);
  }
  if (i < full) {
    load(s1, kbeg + (i + 1) * PG_K, last);
    mul(s0);
    s0 = s1;
  }
  if (kbeg + full * PG_K < kend) {  // fewer than 32 rows: the others are zero
#pragma unroll
    for (int u = 0; u < PG_K / 4; ++u)
#pragma unroll
      for (int t = 0; t < 2; ++t)
        if (kbeg + full * PG_K + 4 * u + fk > last) s0.a[u][t] = s0.b[u][t] = 0.f;
    mul(s0);
  }
  const int nb16 = (n + 15) / 16;
  double* const o = slabs + (int64_t)blockIdx.y * (nb16 * (nb16 + 1) / 2) * 256 + lane;
#pragma unroll
  for (int x = 0; x < 2; ++x)
#pragma unroll
    for (int y = 0; y < 2; ++y) {
      const int bi = 4 * I + 2 * (wave >> 1) + x, bj = 4 * J + 2 * (wave & 1) + y;
      if (bi > bj || bj >= nb16) continue;  // uniform
#pragma unroll
      for (int v = 0; v < 4; ++v) o[(bi * nb16 - bi * (bi + 1) / 2 + bj) * 256 + v * 64] = acc[x][y][v];
    }
}

// A Newton-Schulz step leaves 0.75 e^2 of W = I + E, e the norm of E: 4.7e-8 of this, below fp32 rounding.  (A norm, not the largest entry: of
// n columns with every entry at x it is n x.)
constexpr double PANEL_ONCE = 2.5e-4;

// W (n x n) = sum over the ranges, a workgroup per block of the upper triangle (with far or gate both triangles).  far (zero before; not with a
// gate): set where W may be further than PANEL_ONCE from the identity, or is not finite: a block's share of that is PANEL_ONCE over the blocks of a row, in
// Frobenius norm, so that no sum has to meet another workgroup's.
// gate: nullptr, or nothing to do where it is zero; then an entry further than `limit` from the identity's raises bit 1 of *flag.
__global__ __launch_bounds__(256) void panel_gram64_sum_kernel(const double* __restrict__ slabs, int splits, int n,
                                                               double* __restrict__ W, int* far, const int* gate, double limit, int* flag) {
  if (gate && *gate == 0) return;  // uniform
  const int nb16 = (n + 15) / 16, lane = threadIdx.x & 63;
  int J = blockIdx.x, I = 0;
  while (J >= nb16 - I) {
    J -= nb16 - I;
    ++I;
  }
  J += I;
  const int row = 16 * I + 4 * (threadIdx.x >> 6) + (lane >> 4), c = 16 * J + (lane & 15);
  double s = 0.0;
  const double* p = slabs + (int64_t)blockIdx.x * 256 + threadIdx.x;
#pragma unroll 8
  for (int z = 0; z < splits; ++z) s += p[(int64_t)z * gridDim.x * 256];
  if (row < n && c < n) {
    W[(int64_t)row * n + c] = s;
    if (row < c && (far || gate)) W[(int64_t)c * n + row] = s;
  }
  if (far || gate) {  // uniform
    const double off = row < n && c < n ? fabs(s - (row == c ? 1.0 : 0.0)) : 0.0;
    if (far) {  // uniform
      __shared__ double part[4];
      double sq = off * off;
#pragma unroll
      for (int m = 1; m < 64; m *= 2) sq += __shfl_xor(sq, m);
      if (lane == 0) part[threadIdx.x >> 6] = sq;
      __syncthreads();
      const double share = PANEL_ONCE / nb16;
      if (threadIdx.x == 0 && !(part[0] + part[1] + part[2] + part[3] <= share * share)) atomicOr(far, 1);
    }
    if (gate && __any(!(off <= limit)) && lane == 0) atomicOr(flag, 1);
  }
}

// The sum of the fp32 partial Gram matrices of a block, as fp64 (W64 != nullptr) or as the factor 1.5 I - 0.5 W of a Newton-Schulz step.
// For the latter W is the Gram matrix of a block that should be close to orthonormal: an entry further than `limit` from the
// identity (or not finite) raises bit 1 of *flag - the step that follows squares the distance, so a block that far off
// does not come out orthonormal to fp32 rounding.  again (or nullptr; then a workgroup per row): set where a row sum of |W - I|, a bound of its norm, is above PANEL_ONCE.
// (slabs may be M32 itself)
// PANEL_LAST: a last step leaves 0.75 (3e-3)^2 < 1e-5 of an entry that is alone in its row and column, and 0.75 n (3e-3)^2 at the very worst, of n equal ones.
constexpr float PANEL_LAST = 3e-3f;
__global__ __launch_bounds__(256) void panel_gram32_sum_kernel(const float* slabs, int splits, int n, double* W64, float* M32,
                                                               float limit, int* flag, int* again) {
  bool off = false;
  float sum = 0.f;
  const int total = n * n;
  const int first = again ? blockIdx.x * n + threadIdx.x : blockIdx.x * blockDim.x + threadIdx.x;
  const int end = again ? (blockIdx.x + 1) * n : total, step = again ? blockDim.x : gridDim.x * blockDim.x;
  for (int i = first; i < end; i += step) {
    float w = 0.f;
#pragma unroll 8
    for (int z = 0; z < splits; ++z) w += slabs[(int64_t)z * total + i];
    if (W64) {
      W64[i] = (double)w;
    } else {
      const float id = i / n == i % n ? 1.f : 0.f;
      off = off || !(fabsf(w - id) <= limit);
      sum += fabsf(w - id);
      M32[i] = 1.5f * id - 0.5f * w;
    }
  }
  if (off) atomicOr(flag, 1);
  if (again) {  // uniform
    __shared__ float part[4];
#pragma unroll
    for (int m = 1; m < 64; m *= 2) sum += __shfl_xor(sum, m);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = sum;
    __syncthreads();
    if (threadIdx.x == 0 && !(part[0] + part[1] + part[2] + part[3] <= (float)PANEL_ONCE)) atomicOr(again, 1);
  }
}

// row ranges of a split panel product of width n
int panel_splits(int n_cu, int64_t d, int n) {
  const int tiles = ((n + 63) / 64) * ((n + 63) / 64);
  return (int)std::max<int64_t>(1, std::min<int64_t>({(2 * n_cu + tiles - 1) / tiles, d / 64, 64}));
}
// row ranges of panel_gram64_kernel: whole steps, one workgroup per compute unit, as many as fit `bytes` of partial sums; a
// plan holds the sums of up to 64 (room for 256, and whole 64 x 64 tiles, gained nothing: 38 us per random block of 2048 x 19, 36 of
// 8192 x 16 either way)
int pg_splits(int n_cu, int64_t d, int n, size_t bytes) {
  return (int)std::max<int64_t>(1, std::min<int64_t>({n_cu / pg_tiles(n), (d + PG_K - 1) / PG_K, (int64_t)(bytes / pg_bytes(n))}));
}
size_t pg_need(int n_cu, int64_t d, int n) { return n > 0 ? pg_splits(n_cu, d, n, 64 * pg_bytes(n)) * pg_bytes(n) : 0; }

struct FitWs {
  size_t G, V, Y, W64, eig, Rinv, lam, Z, S, T, slabs, slab_bytes, gram, total;
  size_t gv_g, gv_v;  // parts of G and of the iteration's block
  size_t far;         // two words: whether a panel's Gram matrix is not near the identity, whether a second Newton-Schulz step is needed
  size_t trk_pf, trk_c, trk_slabs;  // tracking refit: V in fragment order, packed X V, slabs of (X V)^T X
  int trk_nkb, trk_ncb, trk_splits;
  int b;
  int kq;         // principal columns the iteration computes (see principal_rank); the other k - kq are drawn
  int splits_bb;  // split count of the b x b fp64 Gram products
  bool gv_parts;  // G V as bf16 parts
  int splits_gv;  // split count of G V on fp32 instructions
};

int block_width(int64_t d, int k, const prac_fit_opts& o) {
  int p = o.oversample < 0 ? 0 : (o.oversample == 0 ? k : o.oversample);
  int64_t b = (int64_t)k + p;
  if (b > d) b = d;
  if (b > 1024) b = 1024;
  if (b < k) b = k;
  return (int)b;
}

// Tracking refit (warm start, block width k, bf16 X the streaming kernels accept): no Gram
// matrix is formed.  One step is V <- orth(X^T (X V)): the compress kernel forms X V, the C^T dY
// kernel with X in the place of dY forms (X V)^T X.
bool can_track(const void* X, prac_dtype xdt, int64_t rows, int64_t d, int64_t ldx, int k, const prac_fit_opts& o) {
  // ldx itself a multiple of 8 (not only the pitch ldx * row_stride of the sampled rows): the streaming kernels
  // read a row in whole 16-byte chunks, and the last chunk of the last row must lie inside that row's ldx elements
  return o.warm_start && o.oversample < 0 && o.iters >= 1 && k > 0 && k <= 1024 && xdt == PRAC_BF16 &&
         (reinterpret_cast<uintptr_t>(X) & 15) == 0 && ldx % 8 == 0 &&
         ldx * (o.row_stride > 0 ? o.row_stride : 1) <= PRAC_MAX_STREAM_PITCH && rows >= 256 && rows >= k &&
         rows < ((int64_t)1 << 31) && d >= 128;
}

// Principal directions the (sub)sampled rows can define: a batch of fewer rows than k has rank below k, and
// the columns of Q1 past that rank are an arbitrary orthonormal completion (any one is a valid set of "top-k right
// singular vectors").  They are drawn like Q2 - Gaussian, projected onto the complement, orthonormalised -
// instead of being left to the iteration, whose blocks would be rank deficient.
int principal_rank(int k, int64_t rows) { return rows < k ? (int)rows : k; }

FitWs plan_fit(int64_t d, int k, int r, const prac_fit_opts& o, int n_cu, bool need_g, size_t gram_bytes, bool track,
               int64_t rows) {
  FitWs w{};
  WsPlan p;
  const int kq = (need_g || track) ? principal_rank(k, rows) : k;
  const int fill = k - kq;  // columns of Q1 drawn at random
  int b = track ? k : (need_g ? block_width(d, kq, o) : 0);
  if (need_g && b > rows) b = (int)rows;  // kq <= rows: the block keeps at least kq columns
  const int rf = r > fill ? r : fill;     // widest random block
  const int bb = b > rf ? b : rf;         // widest panel that goes through orth()
  w.b = b;
  w.kq = kq;
  w.G = p.take(need_g ? (size_t)d * d * 4 : 0);
  w.V = p.take((size_t)d * bb * 4);
  w.Y = p.take((size_t)d * bb * 4);
  w.W64 = p.take((size_t)bb * bb * 8);
  w.eig = p.take(need_g ? std::max<size_t>(sym_eig_doubles(b) * 8, 256) : 0);
  w.Rinv = p.take((size_t)bb * bb * 4);
  w.lam = p.take((size_t)bb * 8);
  w.far = p.take(2 * sizeof(int));
  w.Z = p.take((size_t)bb * (k > 0 ? k : 1) * 4);
  w.S = p.take((size_t)d * (rf > 0 ? rf : 1) * 4);
  w.T = p.take((size_t)(k > 0 ? k : 1) * (rf > 0 ? rf : 1) * 4);
  const int s = panel_splits(n_cu, d, bb);
  w.splits_bb = s;
  // G V (d x b, fp32): split the sum over k until the tiles fill the chip
  w.gv_parts = need_g && gv_parts(d, b);
  const bool gv_f32 = need_g && !w.gv_parts;
  const int tiles_gv = (int)((d + 63) / 64) * ((b + 63) / 64);
  int sg = gv_f32 ? (n_cu + tiles_gv - 1) / tiles_gv : 1;
  if (sg > d / 256) sg = (int)(d / 256);
  if (sg < 1) sg = 1;
  if (sg > 16) sg = 16;
  w.splits_gv = sg;
  // the slab block serves every split product of the fit: the bb x bb panel Gram matrices (fp64), G V
  // (d x b, fp32) and Q1^T S (k x r, fp32; wider than a panel Gram when k > 2 r and Q1 is not refreshed)
  const size_t slab_bb = (size_t)s * bb * bb * 8, slab_gv = sg > 1 ? (size_t)sg * d * b * 4 : 0;
  const size_t slab_kr = (size_t)s * k * rf * 4;  // also the completion's Q1^T S (kq x fill)
  w.slab_bytes = std::max(slab_bb, std::max(slab_gv, slab_kr));
  for (int n : {b, b > 0 ? kq : 0, fill, r})  // the panel Gram matrices with fp64 sums
    w.slab_bytes = std::max(w.slab_bytes, pg_need(n_cu, d, n));
  w.slabs = p.take(w.slab_bytes);
  w.gram = p.take(gram_bytes);
  w.gv_g = p.take(w.gv_parts ? gv_g_bytes(d) : 0);
  w.gv_v = p.take(w.gv_parts ? gv_v_bytes(d, b) : 0);
  if (track) {
    w.trk_nkb = (int)(round_up64(d, 256) / 16);
    w.trk_ncb = (int)round_up64((k + 31) / 32, 8);
    const int tiles = (int)((d + 127) / 128) * ((k + 255) / 256);  // 256 x 128 tiles of (X Q1)^T X
    int sp = n_cu / tiles;
    if (sp > rows / 256) sp = (int)(rows / 256);
    if (sp < 1) sp = 1;
    if (sp > 64) sp = 64;
    w.trk_splits = sp;
    w.trk_pf = p.take((size_t)w.trk_nkb * w.trk_ncb * 64 * 8 * sizeof(bf16_t));
    w.trk_c = p.take((size_t)((rows + 127) / 128) * 8 * ((k + 31) / 32) * 64 * 8 * sizeof(bf16_t));
    w.trk_slabs = p.take((size_t)sp * k * d * sizeof(float));
  }
  w.total = p.off;
  return w;
}

// the Cholesky of wide blocks keeps up to 128 KB in LDS (n <= 1024)
int set_dyn_smem(prac_ctx* ctx) {
  static bool done_dev[PRAC_MAX_DEVICES] = {};  // the attribute is per device
  bool& done = done_dev[ctx->device % PRAC_MAX_DEVICES];
  if (!done) {
    PRAC_HIP_TRY(ctx, hipFuncSetAttribute(reinterpret_cast<const void*>(chol_upper_kernel),
                                          hipFuncAttributeMaxDynamicSharedMemorySize, CH_NB * (CH_MAX + 2) * 8));
    done = true;
  }
  return PRAC_OK;
}

// src^T src for a d x n block with fp64 sums: the upper triangle of W64
// (pitch lds; near: whether it is near the identity goes to the plan's first word; gate: only where it is set, and then checked against `limit`)
int panel_gram64(prac_ctx* ctx, const FitWs& w, const float* src, int64_t lds, int64_t d, int n, double* W64, bool near,
                 const int* gate = nullptr, double limit = 0.0) {
  const int tiles = pg_tiles(n), splits = pg_splits(ctx->n_cu, d, n, w.slab_bytes);
  if (splits * pg_bytes(n) > w.slab_bytes) return PRAC_EINVAL;
  double* slabs = reinterpret_cast<double*>(ctx->ws + w.slabs);
  int* far = reinterpret_cast<int*>(ctx->ws + w.far);
  const int64_t per = round_up64((d + splits - 1) / splits, PG_K);
  const int used = (int)((d + per - 1) / per);
  hipLaunchKernelGGL(panel_gram64_kernel, dim3(tiles, used), dim3(256), 0, ctx->stream, src, lds, d, n, per, slabs, far, gate);
  hipLaunchKernelGGL(panel_gram64_sum_kernel, dim3((unsigned)(pg_bytes(n) / 2048)), dim3(256), 0, ctx->stream, slabs, used, n, W64,
                     near ? far : nullptr, gate, limit, ctx->d_flag);
  PRAC_HIP_TRY(ctx, hipGetLastError());
  return PRAC_OK;
}

// src^T src with fp32 sums on the matrix cores (enough for a block whose condition number is small), as fp64 or as the factor
// of a Newton-Schulz step
int panel_gram32(prac_ctx* ctx, const FitWs& w, const float* src, int64_t d, int n, double* W64, float* factor, float limit,
                 int* again = nullptr) {
  GemmGenArgs g{};
  g.A = src; g.B = src; g.adt = PRAC_F32; g.bdt = PRAC_F32;
  g.a_rs = 1; g.a_cs = n; g.b_rs = n; g.b_cs = 1;
  g.M = n; g.N = n; g.K = d; g.k_stride = 1;
  g.ldo = n; g.alpha = 1.f; g.beta = 0.f;
  float* M32 = reinterpret_cast<float*>(ctx->ws + w.Rinv);
  const float* sums = M32;
  int splits = 1, rc;
  if (gemm_f32_takes(g)) {
    splits = w.splits_bb;
    if (splits > 1 && (size_t)splits * n * n * 4 > w.slab_bytes) return PRAC_EINVAL;
    g.out = M32;
    g.slabs = ctx->ws + w.slabs;
    rc = launch_gemm_f32(ctx, g, splits);
    if (splits > 1) sums = reinterpret_cast<const float*>(g.slabs);
  } else {  // n = 1
    g.out = M32;
    g.splits = w.splits_bb;
    g.slabs = ctx->ws + w.slabs;
    g.slab_bytes = w.slab_bytes;
    rc = launch_gemm_generic(ctx, g);
  }
  if (rc) return rc;
  hipLaunchKernelGGL(panel_gram32_sum_kernel, dim3(again ? n : (n * n + 255) / 256), dim3(256), 0, ctx->stream, sums, splits, n, W64, factor,
                     limit, ctx->d_flag, again);
  PRAC_HIP_TRY(ctx, hipGetLastError());
  return PRAC_OK;
}

// V (d x n, pitch n) as parts for G V
int split_block(prac_ctx* ctx, const float* V, int64_t d, int n, u32x4* parts) {
  const int nkb = gv_kblocks(d), ncb = gv_col_blocks(n);
  hipLaunchKernelGGL(split_parts_kernel<false>, dim3((unsigned)(((int64_t)nkb * ncb + 3) / 4)), dim3(256), 0, ctx->stream, V, (int64_t)n, n,
                     d, ncb, nkb, parts);
  PRAC_HIP_TRY(ctx, hipGetLastError());
  return PRAC_OK;
}

// dst (pitch ldd; may be src) = src R^-1 with R^T R = src^T src (+ shift): one Cholesky-QR pass.  parts: the result also as parts for G V
// (their padding past d is there already).  any_basis: of src's span any orthonormal basis will do, so a block that is orthonormal but for
// PANEL_ONCE gets a Newton-Schulz step instead (decided on the device).
int cholqr_pass(prac_ctx* ctx, const FitWs& w, const float* src, float* dst, int64_t ldd, int64_t d, int n, double shift, bool gram64,
                u32x4* parts, bool any_basis) {
  double* W64 = reinterpret_cast<double*>(ctx->ws + w.W64);
  int* far = any_basis && gram64 && n <= CHR_MAX ? reinterpret_cast<int*>(ctx->ws + w.far) : nullptr;
  int rc = gram64 ? panel_gram64(ctx, w, src, n, d, n, W64, far != nullptr) : panel_gram32(ctx, w, src, d, n, W64, nullptr, 0.f);
  if (rc) return rc;
  rc = set_dyn_smem(ctx);
  if (rc) return rc;
  if (n > CH_MAX) return PRAC_EUNSUPPORTED;
  if (n <= CHR_MAX)
    hipLaunchKernelGGL(chol_upper_reg_kernel, dim3(1), dim3(1024), 0, ctx->stream, W64, n, shift, ctx->d_flag, far);
  else
    hipLaunchKernelGGL(chol_upper_kernel, dim3(1), dim3(1024),
                       (size_t)CH_NB * (round_up64(n, CH_NB) + 2) * sizeof(double), ctx->stream, W64, n, shift, ctx->d_flag);
  const dim3 tgrid((unsigned)((d + TR_ROWS - 1) / TR_ROWS)), tblock(64 * TR_W);
  const int ncb = gv_col_blocks(n);
  auto solve = [&](auto kern, u32x4* p) {
    hipLaunchKernelGGL(kern, tgrid, tblock, 0, ctx->stream, src, (int64_t)n, W64, dst, ldd, d, n, p, ncb, far, nullptr);
  };
  if (parts && n > GV_MAX) return PRAC_EINVAL;
  if (parts && n <= 128) solve(trsm_right_upper_kernel<1, true>, parts);
  else if (parts) solve(trsm_right_upper_kernel<2, true>, parts);
  else if (n <= 128) solve(trsm_right_upper_kernel<1, false>, nullptr);
  else if (n <= 256) solve(trsm_right_upper_kernel<2, false>, nullptr);
  else if (n <= 512) solve(trsm_right_upper_kernel<4, false>, nullptr);
  else solve(trsm_right_upper_kernel<8, false>, nullptr);
  PRAC_HIP_TRY(ctx, hipGetLastError());
  return PRAC_OK;
}

// dst (pitch ldd) = src (1.5 I - 0.5 src^T src): one Newton-Schulz step towards orthonormal columns.  For a block
// with ||src^T src - I|| = e the result has 0.75 e^2: the cheap second pass after a Cholesky-QR pass,
// made of two products and no factorisation.
int polish_pass(prac_ctx* ctx, const FitWs& w, const float* src, float* dst, int64_t ldd, int64_t d, int n, float limit, int* again = nullptr) {
  float* M32 = reinterpret_cast<float*>(ctx->ws + w.Rinv);
  int rc = panel_gram32(ctx, w, src, d, n, nullptr, M32, limit, again);
  if (rc) return rc;
  GemmGenArgs g{};
  g.A = src; g.B = M32; g.adt = PRAC_F32; g.bdt = PRAC_F32;
  g.a_rs = n; g.a_cs = 1; g.b_rs = n; g.b_cs = 1;
  g.M = (int)d; g.N = n; g.K = n; g.k_stride = 1;
  g.out = dst; g.ldo = ldd; g.alpha = 1.f; g.beta = 0.f; g.acc64 = false; g.out64 = nullptr;
  return launch_gemm_generic(ctx, g);
}

// Two of these steps, the second (in place, in fp64) only where the first starts further than PANEL_ONCE from orthonormal, as it does where a
// batch is steep or of low rank; decided on the device: three launches that find nothing to do take 8 us, a step 31 (4096 x 256).
// Behind a panel_gram64 without a gate; n <= 256.
int polish_once_or_twice(prac_ctx* ctx, const FitWs& w, const float* src, float* dst, int64_t ldd, int64_t d, int n) {
  double* W64 = reinterpret_cast<double*>(ctx->ws + w.W64);
  int* far = reinterpret_cast<int*>(ctx->ws + w.far);
  int rc = polish_pass(ctx, w, src, dst, ldd, d, n, 0.5f, far + 1);
  if (rc) return rc;
  rc = panel_gram64(ctx, w, dst, ldd, d, n, W64, false, far + 1, PANEL_LAST);
  if (rc) return rc;
  auto solve = [&](auto kern) {
    hipLaunchKernelGGL(kern, dim3((unsigned)((d + TR_ROWS - 1) / TR_ROWS)), dim3(64 * TR_W), 0, ctx->stream, dst, ldd, W64, dst, ldd, d, n,
                       nullptr, 0, far, far + 1);
  };
  if (n <= 128) solve(trsm_right_upper_kernel<1, false>);
  else solve(trsm_right_upper_kernel<2, false>);
  PRAC_HIP_TRY(ctx, hipGetLastError());
  return PRAC_OK;
}

// out (d x n fp32, pitch ldo) <- orth(Y): `passes` rounds of Cholesky-QR (the first one shifted), then
// `polish` Newton-Schulz steps.  Y is overwritten, and so is the work space V; out may be V or somewhere else.
// gram64_first = false: the first Gram matrix is summed in fp32 (well-conditioned blocks only).  parts (no polish, ldo = n): the result also
// as parts for G V.  Passes from any_basis_from on may give another basis of the same span.
int cholqr(prac_ctx* ctx, const FitWs& w, float* Y, float* V, int64_t d, int n, int passes, double first_shift, float* out,
           int64_t ldo, int polish = 0, bool gram64_first = true, u32x4* parts = nullptr,
           int any_basis_from = 1 << 30) {
  float* src = Y;
  for (int pass = 0; pass < passes + polish; ++pass) {
    if (pass == passes && polish == 2 && n <= CHR_MAX) return polish_once_or_twice(ctx, w, src, out, ldo, d, n);
    const bool last = pass == passes + polish - 1;
    // a solve may stay where it is, a product may not
    float* dst = last ? out : (src == Y ? V : Y);
    const int64_t ldd = last ? ldo : n;
    if (pass >= passes && dst == src) return PRAC_EINVAL;
    // Later passes work on a block that is orthonormal up to the first pass's error, except in
    // directions where the input was rank deficient: there the Gram matrix is zero up to rounding
    // (a few 1e-16), and the shift has to be safely above that for the pivot to stay positive.
    // the last Newton-Schulz step must start with every entry within PANEL_LAST of orthonormal (see there for where it ends); earlier
    // ones may start anywhere inside the step's region of convergence
    int rc = pass < passes ? cholqr_pass(ctx, w, src, dst, ldd, d, n, pass == 0 ? first_shift : 1e-13, pass > 0 || gram64_first,
                                         last ? parts : nullptr, pass >= any_basis_from)
                           : polish_pass(ctx, w, src, dst, ldd, d, n, last ? PANEL_LAST : 0.5f);
    if (rc) return rc;
    src = dst;
  }
  return PRAC_OK;
}

// The scratch plan of one fit: which path runs (tracking / Gram-based) and where everything lives.
struct FitPlan {
  bool do_q1, do_q2, track;
  int64_t rows;
  FitWs L;
};
FitPlan make_fit_plan(int n_cu, const void* X, prac_dtype xdt, int64_t N, int64_t d, int64_t ldx, int k, int r,
                      int refresh, const prac_fit_opts& o) {
  FitPlan f{};
  f.do_q1 = (refresh & PRAC_REFRESH_PRINCIPAL) && k > 0;
  f.do_q2 = (refresh & PRAC_REFRESH_RANDOM) && r > 0;
  const int64_t stride = o.row_stride > 0 ? o.row_stride : 1;
  f.rows = (N + stride - 1) / stride;
  if (!f.do_q1 && !f.do_q2) return f;  // nothing to refresh: no scratch
  f.track = f.do_q1 && can_track(X, xdt, f.rows, d, ldx, k, o);
  const size_t gram_bytes = f.do_q1 && !f.track ? gram_scratch_bytes(n_cu, X, xdt, N, d, ldx, stride, d) : 0;
  f.L = plan_fit(d, k, r, o, n_cu, f.do_q1 && !f.track, gram_bytes, f.track, f.rows);
  return f;
}

}  // namespace

size_t fit_scratch_bytes(int n_cu, const void* X, prac_dtype xdt, int64_t N, int64_t d, int64_t ldx, int k, int r,
                         int refresh, const prac_fit_opts& o) {
  const FitPlan f = make_fit_plan(n_cu, X, xdt, N, d, ldx, k, r, refresh, o);
  return (f.do_q1 || f.do_q2) ? f.L.total : 0;
}

// Bytes by which the slab block of the plan exceeds the largest split product of the fit (negative:
// a product would not fit).  The products are listed here as fit_basis_device issues them.
int64_t fit_slab_margin(int n_cu, prac_dtype xdt, int64_t N, int64_t d, int k, int r, int refresh,
                        const prac_fit_opts& o) {
  const FitPlan f = make_fit_plan(n_cu, nullptr, xdt, N, d, d, k, r, refresh, o);
  const FitWs& L = f.L;
  if (!f.do_q1 && !f.do_q2) return 0;
  size_t need = 0;
  auto product = [&](int splits, int64_t M, int64_t Nn, size_t esz) {
    if (splits > 1) need = std::max(need, (size_t)splits * M * Nn * esz);
    if (M == Nn) need = std::max(need, pg_need(n_cu, d, (int)M));
  };
  if (f.do_q1) {
    const int n = L.b;  // block width of the iteration (k when tracking)
    product(L.splits_bb, n, n, 8);                    // panel Gram matrices of orth(), Rayleigh-Ritz
    if (!f.track) product(L.splits_gv, d, n, 4);      // G V
    product(L.splits_bb, L.kq, L.kq, 8);              // tidy passes on Q1
    const int fill = k - L.kq;
    if (fill > 0) {
      product(L.splits_bb, L.kq, fill, 4);            // the completion's Q1^T S
      product(L.splits_bb, fill, fill, 8);            // and its panel Gram matrices
    }
  }
  if (f.do_q2) {
    if (k > 0) product(L.splits_bb, k, r, 4);         // Q1^T S
    product(L.splits_bb, r, r, 8);                    // panel Gram matrices of orth(S_o)
  }
  return (int64_t)L.slab_bytes - (int64_t)need;
}

int fit_basis_device(prac_ctx* ctx, const void* X, prac_dtype xdt, int64_t N, int64_t d, int64_t ldx, int k, int r,
                     uint64_t seed, uint32_t draw, int refresh, const prac_fit_opts& o, float* P, int64_t ldp) {
  const FitPlan plan = make_fit_plan(ctx->n_cu, X, xdt, N, d, ldx, k, r, refresh, o);
  const bool do_q1 = plan.do_q1, do_q2 = plan.do_q2, track = plan.track;
  if (!do_q1 && !do_q2) return PRAC_OK;
  if (k > 1024 || r > 1024) return PRAC_EUNSUPPORTED;  // single-workgroup panel kernels
  const int64_t stride = o.row_stride > 0 ? o.row_stride : 1;
  const int64_t rows = plan.rows;
  const FitWs& L = plan.L;
  int rc = prac_ws_reserve(ctx, L.total);
  if (rc) return rc;
  float* G = reinterpret_cast<float*>(ctx->ws + L.G);
  float* V = reinterpret_cast<float*>(ctx->ws + L.V);
  float* Y = reinterpret_cast<float*>(ctx->ws + L.Y);
  hipStream_t st = ctx->stream;

  if (track) {
    // V starts as the previous Q1.  The span is what matters (compression and the estimator are
    // invariant to a rotation inside Q1), so there is no Rayleigh-Ritz step: each iteration is one
    // subspace-iteration step on X^T X, orthonormalised by Cholesky-QR (two passes on the last).
    const bf16_t* Xb = reinterpret_cast<const bf16_t*>(X);
    const int64_t ld = ldx * stride;
    bf16_t* Pf = reinterpret_cast<bf16_t*>(ctx->ws + L.trk_pf);
    bf16_t* Cpk = reinterpret_cast<bf16_t*>(ctx->ws + L.trk_c);
    float* slabs = reinterpret_cast<float*>(ctx->ws + L.trk_slabs);
    const int dm = (int)d;
    for (int it = 0; it < o.iters; ++it) {
      rc = launch_pack_pfrag(ctx, it == 0 ? P : V, d, it == 0 ? ldp : (int64_t)k, k, L.trk_nkb, L.trk_ncb, Pf);
      if (rc) return rc;
      rc = launch_compress_ws(ctx, Xb, ld, (int)rows, dm, Pf, L.trk_ncb, k, Cpk, 0, true, nullptr, 0, 0, nullptr, 0, false,
                              ctx->tails);
      if (rc) return rc;
      rc = launch_ctdy_ws(ctx, Cpk, k, (int)rows, 1, &Xb, &ld, &dm, &slabs, L.trk_splits, false);
      if (rc) return rc;
      rc = launch_reduce_transpose_f32(ctx, slabs, L.trk_splits, k, dm, Y, k);
      if (rc) return rc;
      // One power step from an orthonormal block leaves a condition number of at most lambda_1 /
      // lambda_k, within reach of a Cholesky factor of the fp64 Gram matrix with a shift just above its
      // rounding (so that a rank-deficient batch still factors); the last
      // iteration then gets one or two Newton-Schulz steps in place of a second factorisation.
      const bool last = it == o.iters - 1;
      rc = cholqr(ctx, L, Y, V, d, k, 1, 1e-14, last ? P : V, last ? ldp : (int64_t)k, last ? 2 : 0);
      if (rc) return rc;
    }
  } else if (do_q1) {
    const int b = L.b;
    const int k = L.kq;  // the columns this iteration computes: all of Q1 unless the batch has fewer rows than that
    rc = gram_device(ctx, X, xdt, N, d, ldx, o.row_stride, G, d, ctx->ws + L.gram);
    if (rc) return rc;

    // start block: Gaussian (stream 0); warm start puts the previous Q1 in front
    rc = launch_philox(ctx, seed, draw, 0u, V, d * b, true);
    if (rc) return rc;
    if (o.warm_start) {
      hipLaunchKernelGGL(copy_cols_kernel, dim3(ctx->n_cu * 4), dim3(256), 0, st, P, ldp, V, (int64_t)b, d, k);
      PRAC_HIP_TRY(ctx, hipGetLastError());
    }
    u32x4* const Gf = reinterpret_cast<u32x4*>(ctx->ws + L.gv_g);
    u32x4* const Vf = L.gv_parts ? reinterpret_cast<u32x4*>(ctx->ws + L.gv_v) : nullptr;
    if (Vf) {
      const int nkb = gv_kblocks(d), nrb = (int)((d + 31) / 32);
      hipLaunchKernelGGL(split_parts_kernel<true>, dim3((unsigned)(((int64_t)nrb * nkb + 3) / 4)), dim3(256), 0, st, G, d, (int)d, d, nrb,
                         nkb, Gf);
      PRAC_HIP_TRY(ctx, hipGetLastError());
      rc = split_block(ctx, V, d, b, Vf);
      if (rc) return rc;
    }
    // The start block goes into the first product as it is: a Gaussian block and the previous
    // (orthonormal) Q1 are both well conditioned, and every product is orthonormalised anyway.
    for (int it = 0; it <= o.iters; ++it) {
      // Y = G V
      if (!Vf) {
        GemmGenArgs g{};
        g.A = G; g.B = V; g.adt = PRAC_F32; g.bdt = PRAC_F32;
        g.a_rs = 1; g.a_cs = d; g.b_rs = b; g.b_cs = 1;  // G(m, k) read as G[k][m]: G is symmetric
        g.M = (int)d; g.N = b; g.K = d; g.k_stride = 1;
        g.splits = L.splits_gv; g.slabs = ctx->ws + L.slabs; g.slab_bytes = L.slab_bytes;
        g.out = Y; g.ldo = b; g.alpha = 1.f; g.beta = 0.f; g.acc64 = false; g.out64 = nullptr;
        rc = launch_gemm_generic(ctx, g);
        if (rc) return rc;
      } else {
        hipLaunchKernelGGL(gram_times_block_kernel, dim3(((d + 31) / 32 * (gv_col_blocks(b) / 2) + 7) / 8 * 8), dim3(64 * GV_W),
                           GV_W * 32 * 64 * sizeof(float), st, Gf, Vf, G, (int)d, b, gv_kblocks(d), gv_col_blocks(b), Y);
      }
      PRAC_HIP_TRY(ctx, hipGetLastError());
      if (it == o.iters) break;  // the last product feeds Rayleigh-Ritz
      // one shifted pass keeps the block well conditioned; the last iteration orthonormalises fully
      // (two passes: the second starts from a block whose condition number is already near one)
      rc = cholqr(ctx, L, Y, V, d, b, it == o.iters - 1 ? 2 : 1, 1e-11, V, b, 0, true, Vf, 1);
      if (rc) return rc;
    }
    // Rayleigh-Ritz: H = V^T (G V), eigenvectors of H, Q1 = V Z[:, :k]
    double* H = reinterpret_cast<double*>(ctx->ws + L.W64);
    double* lam = reinterpret_cast<double*>(ctx->ws + L.lam);
    float* Z = reinterpret_cast<float*>(ctx->ws + L.Z);
    {
      GemmGenArgs g{};
      g.A = V; g.B = Y; g.adt = PRAC_F32; g.bdt = PRAC_F32;
      g.a_rs = 1; g.a_cs = b; g.b_rs = b; g.b_cs = 1;
      g.M = b; g.N = b; g.K = d; g.k_stride = 1;
      g.out = nullptr; g.out64 = H; g.ldo = b; g.alpha = 1.f; g.beta = 0.f; g.acc64 = true;
      g.splits = L.splits_bb; g.slabs = ctx->ws + L.slabs; g.slab_bytes = L.slab_bytes;
      rc = launch_gemm_generic(ctx, g);
      if (rc) return rc;
    }
    if (b <= SYM_EIG_MAX) {
      rc = launch_sym_eig(ctx, H, b, k, reinterpret_cast<double*>(ctx->ws + L.eig), Z);
      if (rc) return rc;
    } else {
      const int nblk = (b + JB_NB - 1) / JB_NB, nblk_even = nblk + (nblk & 1);
      // columns count as orthogonal below this cosine: the Ritz vectors are re-orthonormalised in
      // fp32 afterwards, so anything far below fp32 rounding is spent effort
      constexpr double JACOBI_TOL = 1e-10;
      unsigned* counts = reinterpret_cast<unsigned*>(ctx->ws + L.eig);
      static bool smem_dev[PRAC_MAX_DEVICES] = {};
      bool& smem_set = smem_dev[ctx->device % PRAC_MAX_DEVICES];
      if (!smem_set) {
        PRAC_HIP_TRY(ctx, hipFuncSetAttribute(reinterpret_cast<const void*>(jacobi_block_kernel),
                                              hipFuncAttributeMaxDynamicSharedMemorySize, (int)JB_SMEM));
        smem_set = true;
      }
      hipLaunchKernelGGL(zero_u32_kernel, dim3(1), dim3(64), 0, st, counts, JB_SWEEPS);
      double* hmax = reinterpret_cast<double*>(counts + JB_SWEEPS);
      hipLaunchKernelGGL(symmetrize64_kernel, dim3(16), dim3(1024), 0, st, H, b, hmax);
      for (int sweep = 0; sweep < JB_SWEEPS; ++sweep)
        for (int step = 0; step < nblk_even - 1; ++step)
          hipLaunchKernelGGL(jacobi_block_kernel, dim3(nblk_even / 2), dim3(512), JB_SMEM, st, H, b, nblk_even, step, sweep, JACOBI_TOL,
                             counts, hmax);
      hipLaunchKernelGGL(jacobi_finish_kernel, dim3(16), dim3(1024), 0, st, H, b, lam, counts, JB_SWEEPS - 1, ctx->d_flag);
      hipLaunchKernelGGL(select_top_kernel, dim3((b + 3) / 4), dim3(256), 0, st, H, lam, b, k, Z);
    }
    PRAC_HIP_TRY(ctx, hipGetLastError());
    {
      GemmGenArgs g{};
      g.A = V; g.B = Z; g.adt = PRAC_F32; g.bdt = PRAC_F32;
      g.a_rs = b; g.a_cs = 1; g.b_rs = k; g.b_cs = 1;
      g.M = (int)d; g.N = k; g.K = b; g.k_stride = 1;
      g.out = Y; g.ldo = k; g.alpha = 1.f; g.beta = 0.f; g.acc64 = false; g.out64 = nullptr;
      rc = launch_gemm_generic(ctx, g);
      if (rc) return rc;
    }
    // tidy the rounding of the last product (two Cholesky-QR passes and a Newton-Schulz step: with more
    // Ritz vectors asked for than the data has rank, the surplus ones are rounding noise, far from
    // orthogonal to each other, and one pass leaves 1e-4 or more), then store Q1 into P[:, :k]
    rc = cholqr(ctx, L, Y, V, d, k, 2, 1e-13, P, ldp, 1, true, nullptr, 0);
    if (rc) return rc;
  }

  // P[:, kk : kk + rr] = orth((I - Q Q^T)^2 S) for Q = P[:, :kk] and the Gaussian d x rr block S of Philox
  // stream `stream`
  auto random_block = [&](int k, int r, uint32_t stream) -> int {
    float* S = reinterpret_cast<float*>(ctx->ws + L.S);
    float* T = reinterpret_cast<float*>(ctx->ws + L.T);
    int rc = launch_philox(ctx, seed, draw, stream, S, d * r, true);
    if (rc) return rc;
    if (k > 0) {
      for (int rep = 0; rep < 2; ++rep) {
        // T = Q^T S  (k x r), S -= Q T
        GemmGenArgs g{};
        g.A = P; g.B = S; g.adt = PRAC_F32; g.bdt = PRAC_F32;
        g.a_rs = 1; g.a_cs = ldp; g.b_rs = r; g.b_cs = 1;
        g.M = k; g.N = r; g.K = d; g.k_stride = 1;
        // fp32 sums on the matrix cores: the second projection removes what rounding left of the first
        g.out = T; g.ldo = r; g.alpha = 1.f; g.beta = 0.f; g.acc64 = false; g.out64 = nullptr;
        g.splits = L.splits_bb; g.slabs = ctx->ws + L.slabs; g.slab_bytes = L.slab_bytes;
        rc = launch_gemm_generic(ctx, g);
        if (rc) return rc;
        GemmGenArgs h{};
        h.A = P; h.B = T; h.adt = PRAC_F32; h.bdt = PRAC_F32;
        h.a_rs = ldp; h.a_cs = 1; h.b_rs = r; h.b_cs = 1;
        h.M = (int)d; h.N = r; h.K = k; h.k_stride = 1;
        h.out = S; h.ldo = r; h.alpha = -1.f; h.beta = 1.f; h.acc64 = false; h.out64 = nullptr;
        rc = launch_gemm_generic(ctx, h);
        if (rc) return rc;
      }
    }
    // a narrow projected Gaussian block is well conditioned (singular values within 1 +- sqrt(r/d) of
    // each other): fp32 sums are enough for its Gram matrix, and one Newton-Schulz step finishes it
    // (up to r = d/4, where the ratio of the extreme singular values reaches 3; wider blocks keep two
    // Cholesky-QR passes over fp64 Gram matrices)
    if ((int64_t)4 * r <= d - k) return cholqr(ctx, L, S, V, d, r, 1, 1e-13, P + k, ldp, 1, false);
    return cholqr(ctx, L, S, V, d, r, 2, 1e-13, P + k, ldp);
  };
  // the columns of Q1 that the batch's rows do not define (stream 2), then Q2 (stream 1) against all of Q1
  if (do_q1 && L.kq < k) {
    rc = random_block(L.kq, k - L.kq, 2u);
    if (rc) return rc;
  }
  if (do_q2) return random_block(k, r, 1u);
  return PRAC_OK;
}
