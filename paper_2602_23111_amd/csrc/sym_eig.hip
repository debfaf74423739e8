// The leading eigenvectors of the small symmetric matrix of the basis fit's Rayleigh-Ritz step (n <= 256, fp64): Householder
// reduction to a tridiagonal T (one workgroup), bisection on Sturm counts for the eigenvalues (a workgroup each), inverse iteration on T
// and the reflectors applied to its vectors (eight vectors per workgroup).
// Why not rotations: a sweep of one-sided Jacobi is a chain of n - 1 dependent steps and takes seven sweeps, the reduction is one
// such chain.  At n = 256, k = 128 the rotations took 1.72 ms.
// Accuracy: columns are reduced from the front, where the power iteration has put the large directions, so that a step's rounding is
// relative to what is left of a graded matrix.
// Equal eigenvalues: inverse iteration tells eigenvectors apart by their eigenvalues, and eigenvalues equal to fp64 rounding gave the same vector
// twice (batches of low rank, whose Ritz values are zero up to rounding; an exactly diagonal H).  So T's diagonal is moved by up to 2^-33 of each
// entry, by another fraction in every row: the eigenvalues come apart by some 1e-13, and their vectors come out orthogonal to 1e-3 or, now and
// then, two or three of them to a few tenths, which the caller's orthonormalisation mends.  2^-33 is below what fp32 rounding of V and G V does to
// H, and as much as the cosine at which the rotations of wider blocks stop.  775 matrices of 1 to 256 rows with equal, zero, nearly equal
// and graded eigenvalues in random directions and along the axes: the smallest singular value of the k vectors (fp32) was below 0.3 for 262 of
// them and below 1e-7, a lost vector, for many; now it is below 0.3 for 9 and 0.03 at least.
#include <algorithm>
#include <type_traits>

#include "frag_utils.h"
#include "philox.h"

namespace {

typedef double f64x2_t __attribute__((ext_vector_type(2)));
typedef double f64x4_t __attribute__((ext_vector_type(4)));
typedef f64x4_t f64x4_el __attribute__((aligned(8)));

// x of another lane: CTRL 0xB1 lane ^ 1, 0x4E lane ^ 2, 0x141 the mirror image in eight lanes, 0x140 in sixteen, 0x104 lane + 4, 0x128 lane ^ 8
template <int CTRL>
__device__ __forceinline__ double dpp_f64(double x) {
  return __hiloint2double(__builtin_amdgcn_update_dpp(0, __double2hiint(x), CTRL, 0xf, 0xf, true),
                          __builtin_amdgcn_update_dpp(0, __double2loint(x), CTRL, 0xf, 0xf, true));
}
// a + b where lanes 32 - 63 (SWAP 32; odd rows of sixteen: SWAP 16) of a and the other lanes of b have changed places: lane l of the lower half has
// a[l] + a[l + 32], of the upper half b[l - 32] + b[l]
template <int SWAP>
__device__ __forceinline__ double swap_add_f64(double a, double b) {
  const auto lo = SWAP == 32 ? __builtin_amdgcn_permlane32_swap(__double2loint(a), __double2loint(b), false, false)
                             : __builtin_amdgcn_permlane16_swap(__double2loint(a), __double2loint(b), false, false);
  const auto hi = SWAP == 32 ? __builtin_amdgcn_permlane32_swap(__double2hiint(a), __double2hiint(b), false, false)
                             : __builtin_amdgcn_permlane16_swap(__double2hiint(a), __double2hiint(b), false, false);
  return __hiloint2double(hi[0], lo[0]) + __hiloint2double(hi[1], lo[1]);
}
// the sum over the wave, in every lane
__device__ __forceinline__ double wave_sum_f64(double x) {
  x += dpp_f64<0xB1>(x);
  x += dpp_f64<0x4E>(x);
  x += dpp_f64<0x141>(x);
  x += dpp_f64<0x140>(x);
  x = swap_add_f64<16>(x, x);
  return swap_add_f64<32>(x, x);
}
__device__ __forceinline__ double lane_f64(double x, int l) {
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(x), l), __builtin_amdgcn_readlane(__double2loint(x), l));
}
__device__ __forceinline__ double pick(const f64x4_t& x, int q) {  // q uniform
  const double a = q & 1 ? x[1] : x[0], b = q & 1 ? x[3] : x[2];
  return q & 2 ? b : a;
}
// 1 / x and x^-1/2: the hardware's estimate (2^-23) and one third-order step
__device__ __forceinline__ double recip_f64(double x) {
  const double r = __builtin_amdgcn_rcp(x), e = fma(-x, r, 1.0);
  return fma(r, fma(e, e, e), r);
}
__device__ __forceinline__ double rsqrt_f64(double x) {
  const double r = __builtin_amdgcn_rsq(x), e = fma(-x * r, r, 1.0);
  return fma(r * e, fma(e, 0.375, 0.5), r);
}

// ---------------------------------------------------------------- reduction to tridiagonal form
// H (n x n, its symmetric part) times `scale` (1 / largest diagonal entry) = Q T Q^T, Q = H_0 H_1 ..., H_j = I - tau_j v_j v_j^T with
// v_j zero up to j.  T's diagonal a, off-diagonal e (and its square, kept off zero for the Sturm counts).
// One workgroup; the upper triangle stays in registers as 32 x 32 tiles, three per wave, 4 x 4 elements per lane (lane 8 r + c: rows
// 4 r .., columns 4 c ..; diagonal tiles whole).  Two halves of a step j: the last wave ends reflector j - 1 (w from the tiles' shares of A v) and makes
// reflector j of row j, while the other waves take A -= v w^T + w v^T for the reflector before those (j - 2); then every tile multiplies by the
// new v.  So A is one update behind in that product and in the row taken from it, and the last wave, which has little to do there, works
// out what is missing (products of the last two reflectors' vectors).
// What bounds it is the issue of instructions, four to five clocks each, so: tiles are dealt out one by one from the last row up, and
// what is left of the matrix is spread over the SIMDs at every step; a lane's four rows are in the order in which the lanes of a row give
// them away when their sums are added up (no selects); the last wave leaves out the 64-element parts of its vectors that are done.
constexpr int TD_T = 32, TD_NT = 8, TD_MAX = TD_T * TD_NT, TD_W = 12, TD_PER = 3;
static_assert(TD_W * TD_PER >= TD_NT * (TD_NT + 1) / 2, "every tile has an owner");
struct __align__(16) TriLds {
  double v[3][TD_MAX];             // reflectors j, j - 1, j - 2 in places j mod 3
  double w[2][TD_MAX];             // w of reflectors j - 1 and j - 2
  double row[TD_MAX];              // row j + 1 of the tiles
  double miss[2][TD_MAX];          // last wave: what the product and the row miss
  double mask[TD_MAX];             // last wave: one past row j, zero up to it
  double part[TD_NT + 3][TD_MAX];  // shares of A v: rows of tile (I, J) in place J, its columns (rows by symmetry) in place I; three zeros
  double a[TD_MAX], e[TD_MAX], tau[TD_MAX], vv[TD_MAX];
};
struct TriOut {
  double *a, *e, *e2, *tau;
  double *vv;  // v_{j-1}^T v_j
  double *V;   // row j, of TD_MAX, holds v_j
};

__global__ __launch_bounds__(64 * TD_W) void tridiag_kernel(const double* __restrict__ H, int n, TriOut out) {
  __shared__ TriLds s;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // (lane numbers and addresses are formed where they are used: kept in registers across the steps, they would push tiles out)
#define TD_LANE                                \
  int lane = threadIdx.x & 63;                 \
  asm("" : "+v"(lane));                        \
  const int lr = lane >> 3, lc = lane & 7;     \
  const int perm = (lc & 1) << 1 | (lc >> 1 & 1) /* register q of a lane holds row 4 lr + (q ^ perm) of its tile */
  const int nt = (n + TD_T - 1) / TD_T;
  double acc[TD_PER][4][4];
  int ti[TD_PER], tj[TD_PER];
  {
    TD_LANE;
    double hmax = 0.0;
    for (int i = lane; i < n; i += 64) hmax = fmax(hmax, fabs(H[(int64_t)i * n + i]));
    for (int o = 32; o > 0; o >>= 1) hmax = fmax(hmax, __shfl_xor(hmax, o));
    const double half = hmax > 1e-280 && hmax < 1e280 ? 0.5 / hmax : 0.5;
#pragma unroll
    for (int t = 0; t < TD_PER; ++t) {
      int q = wave < TD_W - 1 ? (TD_W - 1) * t + wave : (TD_W - 1) * TD_PER + t, len = 1;
      while (q >= len && len <= nt) q -= len++;
      ti[t] = nt - len;  // negative: none
      tj[t] = ti[t] + q;
      const int r0 = TD_T * max(ti[t], 0) + 4 * lr, c0 = TD_T * max(tj[t], 0) + 4 * lc;
#pragma unroll
      for (int q = 0; q < 4; ++q) {
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          const int r = r0 + (q ^ perm), rr = min(r, n - 1), cc = min(c0 + c, n - 1);
          const double x = half * (H[rr * n + cc] + H[cc * n + rr]);
          acc[t][q][c] = ti[t] >= 0 && r < n && c0 + c < n ? x : 0.0;
        }
#pragma unroll
        for (int c = 0; c < 4; ++c) asm volatile("" : "+v"(acc[t][q][c]));  // (a row at a time: more would push tiles out of the registers)
      }
    }
  }
  // row g of A, from the tiles that hold it
  auto put_row = [&](int g) __attribute__((always_inline)) {
#pragma unroll
    for (int t = 0; t < TD_PER; ++t) {
      int I = ti[t], J = tj[t];
      asm("" : "+s"(I), "+s"(J));
      if (I != g / TD_T) continue;  // uniform
      TD_LANE;
      if (lr == g % TD_T / 4) {
        const int q = (g & 3) ^ perm;
        f64x4_t x;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          const double x0 = q & 1 ? acc[t][1][c] : acc[t][0][c], x1 = q & 1 ? acc[t][3][c] : acc[t][2][c];
          x[c] = q & 2 ? x1 : x0;
        }
        *reinterpret_cast<f64x4_t*>(&s.row[TD_T * J + 4 * lc]) = x;
      }
    }
  };
  // A -= v w^T + w v^T
  auto update = [&](int phase, const double* v, const double* w) __attribute__((always_inline)) {
#pragma unroll
    for (int t = 0; t < TD_PER; ++t) {
      int I = ti[t], J = tj[t];
      asm("" : "+s"(I), "+s"(J));
      if (I < phase) continue;  // uniform
      TD_LANE;
      const int r0 = TD_T * I + 4 * lr, c0 = TD_T * J + 4 * lc;
      const f64x4_t vc = *reinterpret_cast<const f64x4_t*>(v + c0), wc = *reinterpret_cast<const f64x4_t*>(w + c0);
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const double vr = v[r0 + (q ^ perm)], wr = w[r0 + (q ^ perm)];
#pragma unroll
        for (int c = 0; c < 4; ++c) acc[t][q][c] = fma(-vr, wc[c], fma(-wr, vc[c], acc[t][q][c]));
      }
    }
  };
  // this wave's shares of A v
  auto multiply = [&](int phase, const double* v) __attribute__((always_inline)) {
#pragma unroll
    for (int t = 0; t < TD_PER; ++t) {
      int I = ti[t], J = tj[t];
      asm("" : "+s"(I), "+s"(J));
      if (I < phase) continue;  // uniform
      TD_LANE;
      const int r0 = TD_T * I + 4 * lr, c0 = TD_T * J + 4 * lc;
      const f64x4_t nc = *reinterpret_cast<const f64x4_t*>(v + c0);
      double nr[4], rs[4], cs[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) nr[q] = v[r0 + (q ^ perm)];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        rs[q] = acc[t][q][0] * nc[0];
        cs[q] = acc[t][0][q] * nr[0];
      }
#pragma unroll
      for (int c = 1; c < 4; ++c)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          rs[q] = fma(acc[t][q][c], nc[c], rs[q]);
          cs[q] = fma(acc[t][c][q], nr[c], cs[q]);
        }
      // rows: over the eight lanes of a lane row; lane c < 4 ends with row 4 lr + perm
      const double h0 = rs[0] + dpp_f64<0xB1>(rs[2]), h1 = rs[1] + dpp_f64<0xB1>(rs[3]);
      double hr = h0 + dpp_f64<0x4E>(h1);
      hr += dpp_f64<0x104>(hr);
      if (lc < 4) s.part[J][r0 + perm] = hr;
      // columns: over the eight lane rows; the upper half of the wave ends with columns 2 and 3, odd rows of sixteen lanes with the odd ones
      double hc = swap_add_f64<16>(swap_add_f64<32>(cs[0], cs[2]), swap_add_f64<32>(cs[1], cs[3]));
      hc += dpp_f64<0x128>(hc);
      if (I != J && !(lr & 1)) s.part[I][c0 + (lane >> 5) * 2 + (lane >> 4 & 1)] = hc;
    }
  };
  for (int i = threadIdx.x; i < TD_MAX; i += 64 * TD_W) {
    s.row[i] = s.miss[0][i] = s.miss[1][i] = 0.0;
    s.mask[i] = i > 0 && i < n ? 1.0 : 0.0;
#pragma unroll
    for (int z = 0; z < TD_NT + 3; ++z) s.part[z][i] = 0.0;
#pragma unroll
    for (int z = 0; z < 3; ++z) s.v[z][i] = 0.0;
  }
  __syncthreads();
  put_row(0);
  __syncthreads();
  const bool last = wave == TD_W - 1;
  double tau = 0.0, lead = 0.0;  // of reflector j - 1, and its element j
  double *v0 = s.v[0], *v1 = s.v[1], *v2 = s.v[2];  // reflectors j, j - 1, j - 2
  // The last wave's vectors: lane l holds elements 64 q + l in component q; those up to the one of row j are done, and nothing reads
  // their parts of v and w.  (What they hold of the rows of the component that are done is finite, and the mask or v is zero there.)
  auto reflector = [&](auto first, int j, double* w1) __attribute__((always_inline)) {
    constexpr int C = decltype(first)::value, M = 4 - C;
    TD_LANE;
    const int i0 = 64 * C + lane;
    double x[M], p[M], v[M], w[M];
#pragma unroll
    for (int q = 0; q < M; ++q) x[q] = s.row[i0 + 64 * q] - s.miss[1][i0 + 64 * q];
    if (C > 0 || j > 0) {  // uniform
#pragma unroll
      for (int q = 0; q < M; ++q) {
        p[q] = -s.miss[0][i0 + 64 * q];
        v[q] = v1[i0 + 64 * q];
      }
      for (int z0 = j / TD_T; z0 < nt; z0 += 4) {
        double y[4][M];
#pragma unroll
        for (int z = 0; z < 4; ++z)
#pragma unroll
          for (int q = 0; q < M; ++q) y[z][q] = s.part[z0 + z][i0 + 64 * q];
#pragma unroll
        for (int q = 0; q < M; ++q) p[q] += (y[0][q] + y[1][q]) + (y[2][q] + y[3][q]);
      }
      double pv = p[0] * v[0];
#pragma unroll
      for (int q = 1; q < M; ++q) pv = fma(p[q], v[q], pv);
      const double g = -0.5 * tau * tau * wave_sum_f64(pv);
#pragma unroll
      for (int q = 0; q < M; ++q) {
        w[q] = fma(g, v[q], tau * p[q]);
        w1[i0 + 64 * q] = w[q];
      }
      const double wj = lane_f64(w[0], j & 63);
#pragma unroll
      for (int q = 0; q < M; ++q) x[q] -= fma(v[q], wj, w[q] * lead);
    }
    const double aj = lane_f64(x[0], j & 63), alpha = lane_f64((j & 63) == 63 ? x[M > 1 ? 1 : 0] : x[0], (j + 1) & 63);
#pragma unroll
    for (int q = 0; q < M; ++q) {
      x[q] *= s.mask[i0 + 64 * q];
      v0[i0 + 64 * q] = x[q];
    }
    double sq = x[0] * x[0];
#pragma unroll
    for (int q = 1; q < M; ++q) sq = fma(x[q], x[q], sq);
    const double nn = wave_sum_f64(sq);
    const bool some = nn > 1e-140;  // (tau^2 is formed; a NaN: no reflector)
    const double rn = rsqrt_f64(some ? nn : 1.0), nrm = nn * rn;
    const double norm = fma(fma(-nrm, nrm, nn), 0.5 * rn, nrm);
    const double beta = some ? -copysign(norm, alpha) : 0.0, t = some ? recip_f64(fma(fabs(alpha), norm, nn)) : 0.0;
    const double l = alpha - beta;
    if (lane == 0) {
      if (j + 1 < TD_MAX) {
        v0[j + 1] = l;
        s.mask[j + 1] = 0.0;
      }
      s.a[j] = aj;
      s.e[j] = beta;
      s.tau[j] = t;
    }
    tau = lane_f64(t, 0);
    lead = lane_f64(l, 0);
  };
  // what the product of the new v and row j + 1 miss: the update by reflector j - 1
  auto missing = [&](auto first, int j, const double* w1) __attribute__((always_inline)) {
    constexpr int C = decltype(first)::value, M = 4 - C;
    TD_LANE;
    const int i0 = 64 * C + lane;
    double x[M], v[M], w[M], wx = 0.0, vx = 0.0;
    const double wj = w1[j + 1], vj = v1[j + 1];
#pragma unroll
    for (int q = 0; q < M; ++q) {
      x[q] = v0[i0 + 64 * q];
      v[q] = v1[i0 + 64 * q];
      w[q] = w1[i0 + 64 * q];
      wx = fma(w[q], x[q], wx);
      vx = fma(v[q], x[q], vx);
    }
    double both = swap_add_f64<32>(wx, vx);
    both += dpp_f64<0xB1>(both);
    both += dpp_f64<0x4E>(both);
    both += dpp_f64<0x141>(both);
    both += dpp_f64<0x140>(both);
    both = swap_add_f64<16>(both, both);
    const double sw = lane_f64(both, 0), sv = lane_f64(both, 32);
    if (lane == 0) s.vv[j] = sv;
#pragma unroll
    for (int q = 0; q < M; ++q) {
      s.miss[0][i0 + 64 * q] = fma(v[q], sw, w[q] * sv);
      s.miss[1][i0 + 64 * q] = fma(v[q], wj, w[q] * vj);
    }
  };
  auto by_part = [&](int j, auto&& f) __attribute__((always_inline)) {
    switch (j >> 6) {
      case 0: f(std::integral_constant<int, 0>{}); break;
      case 1: f(std::integral_constant<int, 1>{}); break;
      case 2: f(std::integral_constant<int, 2>{}); break;
      default: f(std::integral_constant<int, 3>{}); break;
    }
  };
  for (int j = 0; j < n; ++j) {
    double *const w1 = s.w[(j & 1) ^ 1], *const w2 = s.w[j & 1];  // of reflectors j - 1 and j - 2
    const int phase = (j + 1) / TD_T;
    if (last) by_part(j, [&](auto c) __attribute__((always_inline)) { reflector(c, j, w1); });
    if (j > 1) update(phase, v2, w2);
    __syncthreads();  // reflector j, and w of the one before
    if (wave == TD_W - 2) {
      TD_LANE;
#pragma unroll
      for (int q = 0; q < 4; ++q) out.V[j * TD_MAX + 64 * q + lane] = q < j >> 6 ? 0.0 : v0[64 * q + lane];
    }
    if (j + 1 >= n) break;  // uniform
    if (last && j > 0) by_part(j, [&](auto c) __attribute__((always_inline)) { missing(c, j, w1); });
    multiply(phase, v0);
    put_row(j + 1);
    __syncthreads();  // the shares of A v, and row j + 1
    double* const next = v2;
    v2 = v1;
    v1 = v0;
    v0 = next;
  }
  for (int i = threadIdx.x; i < n; i += 64 * TD_W) {
    const double e = s.e[i], a = s.a[i];
    // multiples of the golden section: any run of rows has its fractions spread out evenly; zero rows are moved too
    const double u = (double)i * 0.6180339887498949, spread = u - floor(u);
    out.a[i] = fma(spread, fma(0x1p-33, fabs(a), 1e-34), a);
    out.e[i] = e;
    out.e2[i] = fmax(e * e, 1e-80);
    out.tau[i] = s.tau[i];
    out.vv[i] = i > 0 && i + 1 < n ? s.vv[i] : 0.0;
  }
#undef TD_LANE
}

// ---------------------------------------------------------------- eigenvalues
// lam[t], the eigenvalue number t from the largest, of the tridiagonal (a, e): a workgroup per t narrows its interval to a 257th per pass
// (Sturm counts at 256 points, a thread each: sign changes of the leading minors, rescaled every eighth step).  The
// first pass has geometric points of both signs down to 2^-127 of the norm bound, so that small eigenvalues of a
// graded matrix get their own digits; seven passes behind it leave 2^-56 of an interval no wider than its ends.
constexpr int BI_T = 256, BI_PASSES = 8, BI_U = 8;
__global__ __launch_bounds__(BI_T) void sturm_bisect_kernel(const double* __restrict__ a, const double* __restrict__ e2, int n,
                                                            double* __restrict__ lam) {
  __shared__ double s_red[BI_T / 64];
  __shared__ f64x2_t s_ae[TD_MAX + 2 * BI_U];
  const int tid = threadIdx.x, want = n - 1 - (int)blockIdx.x;  // eigenvalues below lam[t], at most
  double g = 0.0;
  if (tid < n) g = fabs(a[tid]) + sqrt(e2[tid]) + (tid > 0 ? sqrt(e2[tid - 1]) : 0.0);
  for (int o = 32; o > 0; o >>= 1) g = fmax(g, __shfl_xor(g, o));
  if ((tid & 63) == 0) s_red[tid >> 6] = g;
  __syncthreads();
  for (int w = 0; w < BI_T / 64; ++w) g = fmax(g, s_red[w]);
  g *= 1.0001;
  auto first = [&](int i) { return i < 128 ? -ldexp(g, -i) : ldexp(g, i - 255); };
  double lo = 0.0, step = 0.0;
  // elements past the end change no sign
  for (int i = tid; i < TD_MAX + 2 * BI_U; i += BI_T) s_ae[i] = f64x2_t{i < n ? a[i] : 4.0 * g, i < n && i > 0 ? e2[i - 1] : 0.0};
  __syncthreads();
  for (int pass = 0; pass < BI_PASSES; ++pass) {
    const double x = pass == 0 ? first(tid) : fma((double)(tid + 1), step, lo);
    double p0 = 1.0, p1 = 1.0;
    int below = 0;
    f64x2_t ae[2][BI_U];
    auto fetch = [&](f64x2_t (&to)[BI_U], int i0) __attribute__((always_inline)) {
#pragma unroll
      for (int u = 0; u < BI_U; ++u) to[u] = s_ae[i0 + u];
    };
    auto minors = [&](const f64x2_t (&m)[BI_U]) __attribute__((always_inline)) {
      unsigned signs = (unsigned)__double2hiint(p1) >> 31;
#pragma unroll
      for (int u = 0; u < BI_U; ++u) {
        const double p2 = fma(m[u][0] - x, p1, -(m[u][1] * p0));
        p0 = p1;
        p1 = p2;
        signs = __builtin_amdgcn_alignbit(signs, __double2hiint(p2), 31);  // one more bit
      }
      below += __popc((signs ^ signs >> 1) & ((1u << BI_U) - 1));
      const int ex = -__builtin_amdgcn_frexp_exp(fmax(fabs(p0), fabs(p1)));
      p0 = ldexp(p0, ex);
      p1 = ldexp(p1, ex);
    };
    fetch(ae[0], 0);
    for (int i0 = 0; i0 < n; i0 += 2 * BI_U) {
      fetch(ae[1], i0 + BI_U);
      minors(ae[0]);
      fetch(ae[0], i0 + 2 * BI_U);
      minors(ae[1]);
    }
    const int m = __syncthreads_count(below <= want);  // points at or below lam[t]
    if (pass == 0) {
      const int at = min(max(m - 1, 0), 254);
      lo = first(at);
      step = (first(at + 1) - lo) / 257.0;
    } else {
      lo = fma((double)m, step, lo);
      step /= 257.0;
    }
  }
  if (tid == 0) lam[blockIdx.x] = fma(0.5, step, lo);
}

// ---------------------------------------------------------------- eigenvectors
// Z[:, t] (n x k fp32, row-major) = Q (eigenvector of T to lam[t]).  A workgroup of eight waves takes eight of them.  Sixteen
// lanes, two for each, factor T - lam[t] from both ends towards the middle (row exchanges between neighbours) and solve twice from a random
// vector, all in LDS; what bounds that is the chain of 2 n dependent steps.  Then a wave per vector applies the reflectors from the last to
// the first, two at a time: both inner products with the vector come from one reduction, their product with each other from the reduction.
constexpr int IV_V = 8, IV_U = 8, IV_H = TD_MAX / 2;
struct IvLds {  // [row, counted from the end][lane]: lanes 0 - 7 from the front, 8 - 15 from the back
  double inv[IV_H][2 * IV_V], u1[IV_H][2 * IV_V], u2[IV_H][2 * IV_V];
  double l[IV_H][2 * IV_V];  // multiplier; its lowest bit is set where rows i and i + 1 changed places
  double x[IV_H][2 * IV_V];
  double a[TD_MAX + 2 * IV_U], e[TD_MAX + 2 * IV_U];
  double tau[TD_MAX], vv[TD_MAX];
  double f[IV_V];
};
__global__ __launch_bounds__(64 * IV_V) void tridiag_vectors_kernel(TriOut in, const double* __restrict__ lam, int n, int k, float* Z,
                                                                    int* flag) {
  extern __shared__ __align__(16) unsigned char iv_smem[];
  IvLds& s = *reinterpret_cast<IvLds*>(iv_smem);
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int h = (n + 1) / 2;  // rows of a half; one more behind the last if n is odd: no coupling, a zero in the vector
  for (int i = tid; i < TD_MAX + 2 * IV_U; i += 64 * IV_V) {
    s.a[i] = i < n ? in.a[i] : 1e3;  // (past every eigenvalue: T's are below n times its largest diagonal entry)
    s.e[i] = i + 1 < n ? in.e[i] : 0.0;
    if (i < TD_MAX) {
      s.tau[i] = i < n ? in.tau[i] : 0.0;
      s.vv[i] = i > 0 && i < n ? in.vv[i] : 0.0;
    }
  }
  {  // start vectors, in (-1, 1): four rows of a half from one counter
    constexpr int RW = 64 * IV_V / (2 * IV_V);  // rows that the workgroup fills at a time
    static_assert(IV_H == 4 * RW, "one word per row");
    const int half = tid / IV_V % 2, r0 = tid / (2 * IV_V);
    const U4 u = philox4x32_10({(uint32_t)(half * RW + r0), blockIdx.x * IV_V + tid % IV_V, 3u, 0u}, 0u, 0u);  // (streams 0 - 2 are the fit's draws)
    const uint32_t word[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int r = r0 + q * RW, g = half ? 2 * h - 1 - r : r;
      s.x[r][tid % (2 * IV_V)] = r < h && g < n ? fma((double)word[q], 0x1p-31, 0x1p-32 - 1.0) : 0.0;
    }
  }
  __syncthreads();
  if (tid < 2 * IV_V) {
    // a little off the eigenvalue: where two agree to the last bits all the same, both shifts leave both vectors in, and the start vectors tell
    // them apart
    const double lm = lam[min((int)blockIdx.x * IV_V + tid % IV_V, k - 1)] * (1.0 + 0x1p-50);
    const double tiny = 1e-60;  // (H's largest diagonal entry is one)
    auto off_zero = [&](double x) __attribute__((always_inline)) { return fabs(x) < tiny ? tiny : x; };
    auto other = [](double x) __attribute__((always_inline)) { return dpp_f64<0x128>(x); };  // the other half's
    // row r of a half: diagonal ap[r da], coupling with row r + 1 ep[r da]
    const int da = tid < IV_V ? 1 : -1;
    const double* const ap = tid < IV_V ? s.a : s.a + 2 * h - 1;
    const double* const ep = tid < IV_V ? s.e : s.e + 2 * h - 2;
    double d = ap[0] - lm, sup = ep[0], sub = sup;
    auto eliminate = [&](int r, double a1, double e1) __attribute__((always_inline)) {
      const double ai = a1 - lm;
      const bool swap = fabs(sub) > fabs(d);
      const double inv = recip_f64(off_zero(swap ? sub : d)), l = (swap ? d : sub) * inv;
      const double x = swap ? ai : sup, y = swap ? sup : ai;
      s.inv[r][tid] = inv;
      s.u1[r][tid] = x;
      s.u2[r][tid] = swap ? e1 : 0.0;
      s.l[r][tid] = __hiloint2double(__double2hiint(l), (__double2loint(l) & ~1) | (swap ? 1 : 0));
      d = fma(-l, x, y);
      sup = swap ? -l * e1 : e1;
      sub = e1;
    };
    int r0 = 0;
    for (; r0 + IV_U <= h - 1; r0 += IV_U) {
      double en[IV_U], an[IV_U];
#pragma unroll
      for (int u = 0; u < IV_U; ++u) {
        an[u] = ap[(r0 + u + 1) * da];
        en[u] = ep[(r0 + u + 1) * da];
      }
#pragma unroll
      for (int u = 0; u < IV_U; ++u) eliminate(r0 + u, an[u], en[u]);
    }
    for (; r0 < h - 1; ++r0) eliminate(r0, ap[(r0 + 1) * da], ep[(r0 + 1) * da]);
    // what is left: d x + sup x' = r, x' the other half's last element.  A pivot and the determinant are kept off zero each on its own
    // scale: without a coupling x is r / d as in every other row, however small both pivots are.
    d = off_zero(d);
    const double od = other(d), os = other(sup), size = fma(fabs(d), fabs(od), fabs(sup * os)), least = 0x1p-60 * size;
    const double dd = fma(d, od, -(sup * os)), det = recip_f64(fabs(dd) < least ? least : dd);
    double f = 1.0, big = 0.0;
    for (int solve = 0; solve < 2; ++solve) {
      double cur = s.x[0][tid] * f;
      // x <- L^-1 f x
      if (solve > 0) {
        auto forward = [&](int r, double l, double next) __attribute__((always_inline)) {
          const bool swap = __double2loint(l) & 1;
          const double y = next * f, p = swap ? y : cur, q = swap ? cur : y;
          s.x[r][tid] = p;
          cur = fma(-l, p, q);
        };
        int r = 0;
        for (; r + IV_U <= h - 1; r += IV_U) {
          double l[IV_U], next[IV_U];
#pragma unroll
          for (int u = 0; u < IV_U; ++u) {
            l[u] = s.l[r + u][tid];
            next[u] = s.x[r + u + 1][tid];
          }
#pragma unroll
          for (int u = 0; u < IV_U; ++u) forward(r + u, l[u], next[u]);
        }
        for (; r < h - 1; ++r) forward(r, s.l[r][tid], s.x[r + 1][tid]);
      } else {
        cur = s.x[h - 1][tid];
      }
      // x <- U^-1 x
      double x1 = fma(cur, od, -(sup * other(cur))) * det, x2 = other(x1);
      s.x[h - 1][tid] = x1;
      big = fabs(x1);
      auto backward = [&](int r, double y, double c0, double c1, double c2) __attribute__((always_inline)) {
        const double x = fma(-c1, x1, fma(-c2, x2, y)) * c0;
        s.x[r][tid] = x;
        big = fmax(big, fabs(x));
        x2 = x1;
        x1 = x;
      };
      int r = h - 2;
      for (; r >= IV_U - 1; r -= IV_U) {
        double y[IV_U], c0[IV_U], c1[IV_U], c2[IV_U];
#pragma unroll
        for (int u = 0; u < IV_U; ++u) {
          y[u] = s.x[r - u][tid];
          c0[u] = s.inv[r - u][tid];
          c1[u] = s.u1[r - u][tid];
          c2[u] = s.u2[r - u][tid];
        }
#pragma unroll
        for (int u = 0; u < IV_U; ++u) backward(r - u, y[u], c0[u], c1[u], c2[u]);
      }
      for (; r >= 0; --r) backward(r, s.x[r][tid], s.inv[r][tid], s.u1[r][tid], s.u2[r][tid]);
      big = fmax(big, other(big));
      f = big > 0.0 ? recip_f64(big) : 1.0;  // (all zero: flagged below)
    }
    if (tid < IV_V) s.f[tid] = f;
  }
  __syncthreads();
  const int t = blockIdx.x * IV_V + wave;
  if (t >= k) return;  // uniform
  const int i0 = 4 * lane;
  f64x4_t z = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int g = i0 + q, r = min(g < h ? g : 2 * h - 1 - g, h - 1);
    if (g < n) z[q] = s.x[r][g < h ? wave : IV_V + wave] * s.f[wave];
  }
  auto dot = [](const f64x4_t& x, const f64x4_t& y) __attribute__((always_inline)) {
    return fma(x[0], y[0], x[1] * y[1]) + fma(x[2], y[2], x[3] * y[3]);
  };
  constexpr int D = 16;  // reflectors requested ahead
  f64x4_t v[D];
  const double* const vp = in.V + i0;
  auto fetch = [&](int u, int j) __attribute__((always_inline)) { v[u] = *reinterpret_cast<const f64x4_t*>(vp + max(j, 0) * TD_MAX); };
  int j = n - 2;  // the last reflector
#pragma unroll
  for (int u = 0; u < D; ++u) fetch(u, j - u);
  for (; j >= 0; j -= D) {
#pragma unroll
    for (int u = 0; u < D; u += 2) {
      if (j - u >= 0) {  // uniform; reflectors j - u and j - u - 1
        const double t0 = s.tau[j - u], t1 = j - u > 0 ? s.tau[j - u - 1] : 0.0, c = s.vv[j - u];
        double both = swap_add_f64<32>(dot(v[u], z), dot(v[u + 1], z));
        both += dpp_f64<0xB1>(both);
        both += dpp_f64<0x4E>(both);
        both += dpp_f64<0x141>(both);
        both += dpp_f64<0x140>(both);
        both = swap_add_f64<16>(both, both);
        const double f0 = -t0 * lane_f64(both, 0), f1 = -t1 * fma(f0, c, lane_f64(both, 32));
#pragma unroll
        for (int q = 0; q < 4; ++q) z[q] = fma(f1, v[u + 1][q], fma(f0, v[u][q], z[q]));
      }
      fetch(u, j - u - D);
      fetch(u + 1, j - u - 1 - D);
    }
  }
  const double nn = wave_sum_f64(dot(z, z));
  if (!(nn > 0.0 && nn < 1e300) && lane == 0) atomicOr(flag, 2);
  const double nf = 1.0 / sqrt(nn);
#pragma unroll
  for (int q = 0; q < 4; ++q)
    if (i0 + q < n) Z[(int64_t)(i0 + q) * k + t] = (float)(z[q] * nf);
}

}  // namespace

// doubles of scratch: the reflectors, a, e, e^2, tau, vv, lambda
size_t sym_eig_doubles(int n) { return n <= SYM_EIG_MAX ? (size_t)n * (TD_MAX + 6) : 0; }

int launch_sym_eig(prac_ctx* ctx, const double* H, int n, int k, double* scratch, float* Z) {
  static_assert(SYM_EIG_MAX == TD_MAX, "");
  if (n < 1 || n > TD_MAX || k < 1 || k > n) return PRAC_EINVAL;
  static bool smem_dev[PRAC_MAX_DEVICES] = {};  // the attribute is per device
  bool& smem_set = smem_dev[ctx->device % PRAC_MAX_DEVICES];
  if (!smem_set) {
    PRAC_HIP_TRY(ctx, hipFuncSetAttribute(reinterpret_cast<const void*>(tridiag_vectors_kernel),
                                          hipFuncAttributeMaxDynamicSharedMemorySize, (int)sizeof(IvLds)));
    smem_set = true;
  }
  TriOut o;
  o.V = scratch;
  o.a = scratch + (size_t)n * TD_MAX;
  o.e = o.a + n;
  o.e2 = o.e + n;
  o.tau = o.e2 + n;
  o.vv = o.tau + n;
  double* const lam = o.vv + n;
  hipLaunchKernelGGL(tridiag_kernel, dim3(1), dim3(64 * TD_W), 0, ctx->stream, H, n, o);
  hipLaunchKernelGGL(sturm_bisect_kernel, dim3(k), dim3(BI_T), 0, ctx->stream, o.a, o.e2, n, lam);
  hipLaunchKernelGGL(tridiag_vectors_kernel, dim3((k + IV_V - 1) / IV_V), dim3(64 * IV_V), sizeof(IvLds), ctx->stream, o, lam, n, k, Z,
                     ctx->d_flag);
  PRAC_HIP_TRY(ctx, hipGetLastError());
  return PRAC_OK;
}
