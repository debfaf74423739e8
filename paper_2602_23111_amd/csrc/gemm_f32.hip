// fp32 products on the matrix cores (v_mfma_f32_32x32x2_f32): the fp32 data path of compress and the weight gradient,
// the fp32 tail of the gradients whose dY rows start on any element, and the products of the basis fit.
//
// Operands go from global memory straight into MFMA registers, no LDS and no barrier in the loop: a 64 x 64 wave tile
// needs 4 KB per 8 k for sixteen matrix instructions of 64 clocks each, far below what the vector L1 delivers, so
// the loop is bound by the matrix pipe once the loads are far enough ahead (a ring of four 8-k chunks in registers).
// What binds these products instead is how few waves a small one has, and how long each wave's chain of chunks is:
// 2048 x 64 over k = 512 has 32 tiles of 64 x 64.  The waves of a workgroup therefore also split k (their sums meet in
// LDS at the end, in wave order), and the launcher picks tile and split by the number of tiles.
//
// A chunk is 8 consecutive k.  Lane (i, h) of step s works on k = 8 q + 4 h + s, s = 0..3, so that an operand whose k runs
// along memory ("KF") is one 16-byte load per 32-row block and chunk; the other kind ("NF": its rows run along
// memory) is one 4- or 8-byte load per step, the two 32-wide blocks of a wave holding the even and the odd columns.
// Loads carry the alignment of one float: no argument needs more.
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "frag_utils.h"

namespace {

typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef f32x2 f32x2_el __attribute__((aligned(4)));

struct F32Args {
  const float* A;      // KF: A[m * lda + k], NF: A[k * lda + m]
  const float* B;      // KF: B[n * ldb + k], NF: B[k * ldb + n]
  int64_t lda, ldb;
  int M, N;
  int64_t K;
  float* out;
  int64_t ldo;
  float alpha, beta;
  int tiles_n;         // column tiles; workgroups of a row tile are consecutive
  int splits;          // gridDim.z; > 1: partial sums go to slabs [splits][M][N]
  int64_t k_per_split;  // multiple of 8
  float* slabs;
};

// One operand of a wave tile: R blocks of 32 rows (A) or columns (B).
template <bool KF, int R>
struct Operand {
  struct Chunk {
    std::conditional_t<KF, f32x4_t, std::conditional_t<R == 2, f32x2, float>> x[KF ? R : 4];
  };
  const float* p[KF ? R : 1];
  int64_t ld;
  bool odd;  // NF, R = 2: this lane's pair starts one column early (the last column of an odd count)
  // index of the lane's element i within a 32 R wide tile starting at 0
  static __device__ __forceinline__ int index(int i, int li) { return KF || R == 1 ? 32 * i + li : 2 * li + i; }
  __device__ __forceinline__ void init(const float* base, int64_t ld_, int x0, int count, int li, int lh) {
    ld = ld_;
    odd = false;
    if constexpr (KF) {
#pragma unroll
      for (int i = 0; i < R; ++i) p[i] = base + (int64_t)min(x0 + 32 * i + li, count - 1) * ld + 4 * lh;
    } else if constexpr (R == 2) {  // count >= 2
      const int x = x0 + 2 * li;
      odd = x == count - 1;
      p[0] = base + (int64_t)(4 * lh) * ld + min(x, count - 2);
    } else {
      p[0] = base + (int64_t)(4 * lh) * ld + min(x0 + li, count - 1);
    }
  }
  __device__ __forceinline__ void load(Chunk& c, int64_t k) const {
    if constexpr (KF) {
#pragma unroll
      for (int i = 0; i < R; ++i) c.x[i] = *reinterpret_cast<const f32x4_el*>(p[i] + k);
    } else {
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        const float* q = p[0] + (k + s) * ld;
        if constexpr (R == 2) c.x[s] = *reinterpret_cast<const f32x2_el*>(q);
        else c.x[s] = *q;
      }
    }
  }
  // the last, partial chunk: k values from kend on are zero and not read
  __device__ __forceinline__ void load_tail(Chunk& c, int64_t k, int64_t kend, int lh) const {
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const bool in = k + 4 * lh + s < kend;
      if constexpr (KF) {
#pragma unroll
        for (int i = 0; i < R; ++i) c.x[i][s] = in ? p[i][k + s] : 0.f;
      } else {
        const float* q = p[0] + (in ? (k + s) * ld : -(int64_t)(4 * lh) * ld);
        if constexpr (R == 2) {
          c.x[s] = *reinterpret_cast<const f32x2_el*>(q);
          if (!in) c.x[s] = f32x2{0.f, 0.f};
        } else {
          c.x[s] = in ? *q : 0.f;
        }
      }
    }
  }
  __device__ __forceinline__ float get(const Chunk& c, int s, int i) const {
    if constexpr (KF) return c.x[i][s];
    else if constexpr (R == 2) return i == 0 && odd ? c.x[s][1] : c.x[s][i];
    else return c.x[s];
  }
};

// Where k is split a wave has few chunks, and the requests past its last one would be a large part of all.  Each kernel leaves them out in the
// way that costs it less.  TEST, one per chunk: 64 x 64 tiles (us without / with it and three waves per SIMD, which keep the sums out of the
// accumulation registers: C^T dY of 4096 x 128 and 1024 in 16 ranges 17.2 / 14.7, 8192 x 256 and 2048 in four 87 / 79, X P of 8192 x 2048 -> 256 85.5 /
// 83.8), and one round of 32 x 64 tiles if A's k runs along memory (X P of 4096 x 1024 -> 128 16.2 / 14.9; in two rounds its registers cost more, 3001 x
// 1501 -> 201 34.0 / 36.6; otherwise they spill: twice the time).  SECOND_BODY for the ring's last turn: 32 x 32 tiles (C^T dY of 2048 x 64 and
// 1376 in eight ranges 11.2 / 9.7, a test 9.8; X P of 2048 x 512 -> 64 6.2 / 5.5, a test 6.4).
enum class Turn { ALL, SECOND_BODY, TEST };

// Tile (32 RM WM) x (32 RN WN) per workgroup of WM x WN x SK waves; SK waves share a wave tile and split its chunks.
template <bool AKF, bool BKF, int RM, int RN, int WM, int WN, int SK, Turn TURN>
__global__ __launch_bounds__(64 * WM * WN * SK, SK == 8 ? 4 : (SK > 1 ? 3 : 1)) void gemm_f32_kernel(F32Args a) {
  constexpr int D = 4;  // chunks in flight
  constexpr int NREG = RM * RN * 16;
  static_assert(RN <= 2, "the epilogue stores single columns or pairs");
  static_assert(SK == 1 || (WM == 1 && WN == 1 && NREG % (RN * SK) == 0), "one wave tile per workgroup when k is split");
  extern __shared__ float red[];  // SK > 1: [SK][NREG][64] (sized at the launch: a static 64 KB would make the compiler plan for two waves per SIMD)
  const int lane = threadIdx.x & 63, li = lane & 31, lh = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int sk = SK > 1 ? wave : 0, wm = SK > 1 ? 0 : wave / WN, wn = SK > 1 ? 0 : wave % WN;
  const int tn = blockIdx.x % a.tiles_n, tm = blockIdx.x / a.tiles_n;
  const int m0 = (tm * WM + wm) * 32 * RM, n0 = (tn * WN + wn) * 32 * RN;
  const int64_t kbeg = (int64_t)blockIdx.z * a.k_per_split, kend = min(a.K, kbeg + a.k_per_split);

  Operand<AKF, RM> oa;
  Operand<BKF, RN> ob;
  oa.init(a.A, a.lda, m0, a.M, li, lh);
  ob.init(a.B, a.ldb, n0, a.N, li, lh);
  f32x16 acc[RM][RN];
#pragma unroll
  for (int i = 0; i < RM; ++i)
#pragma unroll
    for (int j = 0; j < RN; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;
  typename Operand<AKF, RM>::Chunk ca[D];
  typename Operand<BKF, RN>::Chunk cb[D];
  auto mul = [&](const auto& x, const auto& y) {
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
      for (int i = 0; i < RM; ++i)
#pragma unroll
        for (int j = 0; j < RN; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(oa.get(x, s, i), ob.get(y, s, j), acc[i][j], 0, 0, 0);
  };
  const int full = kend > kbeg ? (int)((kend - kbeg) / 8) : 0;
  const int n = full > sk ? (full - sk + SK - 1) / SK : 0;  // whole chunks of this wave: sk, sk + SK, ...
  auto fetch = [&](int u, int t) {
    const int64_t k = kbeg + 8 * ((int64_t)sk + (int64_t)SK * min(t, n - 1));  // past the end: the last one again, unused
    oa.load(ca[u], k);
    ob.load(cb[u], k);
  };
  if (n > 0) {
#pragma unroll
    for (int u = 0; u < D; ++u) fetch(u, u);
    int t = 0;
    for (; t + (TURN == Turn::SECOND_BODY ? 2 : 1) * D <= n; t += D) {
#pragma unroll
      for (int u = 0; u < D; ++u) {
        mul(ca[u], cb[u]);
        if (TURN != Turn::TEST || t + D + u < n) fetch(u, t + D + u);
      }
    }
    if (TURN == Turn::SECOND_BODY && t + D <= n) {
#pragma unroll
      for (int u = 0; u < D; ++u) {
        mul(ca[u], cb[u]);
        if (t + D + u < n) fetch(u, t + D + u);
      }
      t += D;
    }
#pragma unroll
    for (int u = 0; u < D - 1; ++u)
      if (t + u < n) mul(ca[u], cb[u]);
  }
  if (kend > kbeg && kbeg + 8 * (int64_t)full < kend && full % SK == sk) {
    oa.load_tail(ca[0], kbeg + 8 * (int64_t)full, kend, lh);
    ob.load_tail(cb[0], kbeg + 8 * (int64_t)full, kend, lh);
    mul(ca[0], cb[0]);
  }

  // register r = (i * 16 + v) * RN + j of lane (li, lh) is row 8 (v / 4) + 4 lh + v % 4 of A's block i, column li of B's block j
  auto store = [&](int r, float x0, float x1) {
    const int i = r / (16 * RN), v = r / RN % 16;
    const int m = m0 + Operand<AKF, RM>::index(i, 8 * (v / 4) + 4 * lh + v % 4);
    const int na = n0 + Operand<BKF, RN>::index(0, li), nb = RN == 2 ? n0 + Operand<BKF, RN>::index(1, li) : a.N;
    if (m >= a.M) return;
    float* o;
    float al = 1.f, be = 0.f;
    if (a.splits > 1) {
      o = a.slabs + ((int64_t)blockIdx.z * a.M + m) * a.N;
    } else {
      o = a.out + (int64_t)m * a.ldo;
      al = a.alpha;
      be = a.beta;
    }
    if (!BKF && nb < a.N && be == 0.f) {
      *reinterpret_cast<f32x2_el*>(o + na) = f32x2{al * x0, al * x1};
      return;
    }
    if (na < a.N) o[na] = be == 0.f ? al * x0 : al * x0 + be * o[na];
    if (nb < a.N) o[nb] = be == 0.f ? al * x1 : al * x1 + be * o[nb];
  };
  if constexpr (SK > 1) {
#pragma unroll
    for (int i = 0; i < RM; ++i)
#pragma unroll
      for (int v = 0; v < 16; ++v)
#pragma unroll
        for (int j = 0; j < RN; ++j) red[(sk * NREG + (i * 16 + v) * RN + j) * 64 + lane] = acc[i][j][v];
    __syncthreads();
    constexpr int PER = NREG / SK;
#pragma unroll
    for (int u = 0; u < PER; u += RN) {
      const int r = sk * PER + u;
      float x[2] = {0.f, 0.f};
#pragma unroll
      for (int j = 0; j < RN; ++j)
#pragma unroll
        for (int w = 0; w < SK; ++w) x[j] += red[(w * NREG + r + j) * 64 + lane];
      store(r, x[0], x[1]);
    }
  } else {
#pragma unroll
    for (int i = 0; i < RM; ++i)
#pragma unroll
      for (int v = 0; v < 16; ++v) store((i * 16 + v) * RN, acc[i][0][v], acc[i][RN - 1][v]);
  }
}

// dW (d x m) = P T (+ beta dW), T = the sum of the slabs of C^T dY with rows >= k_lo weighted: T is summed (in slab order)
// into LDS 64 rows at a time and never goes back to memory, P's rows come straight from memory in the chunk order
// above.  128 x 64 of dW per workgroup of eight waves, 32 x 32 each.  The row tiles of a column block repeat its sum;
// the launcher sums separately where they would read the slabs too often.
constexpr int FP_K = 64;  // rows of T in LDS
struct F32SumPtArgs {
  const float* P;
  int64_t ldp;
  const float* slabs;  // [splits][c][m]
  int splits, c, k_lo;
  float scale_hi;
  int d, m;
  void* dW;
  int64_t lddw;
  float beta;
  int tiles_n;
};
template <int WC, bool OUT_BF16>
__global__ __launch_bounds__(256 * WC, WC == 2 ? 4 : 1) void f32_sum_pt_kernel(F32SumPtArgs a) {
  constexpr int TN = 32 * WC, NBUF = WC == 1 ? 2 : 1;
  __shared__ float T[NBUF][FP_K][TN];
  const int tid = threadIdx.x, lane = tid & 63, li = lane & 31, lh = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int m0 = (blockIdx.x / a.tiles_n) * 128 + wave / WC * 32, n0 = (blockIdx.x % a.tiles_n) * TN, wc = wave % WC * 32;
  const float* prow = a.P + (int64_t)min(m0 + li, a.d - 1) * a.ldp;
  f32x16 acc;
#pragma unroll
  for (int v = 0; v < 16; ++v) acc[v] = 0.f;
  const int sr = tid / (TN / 4), sc = tid % (TN / 4) * 4;  // summing: rows sr, sr + 32, columns sc .. sc + 3
  const int64_t slab = (int64_t)a.c * a.m;
  // a row's last columns are taken from its last four and moved down (m < 4: element by element)
  const int back = a.m >= 4 ? max(n0 + sc + 4 - a.m, 0) : 0;
  const float* const col = a.slabs + n0 + sc - back;
  struct P64 {
    f32x4_t x[FP_K / 8];  // P[row][k0 + 8 q + 4 lh .. + 3]
  };
  auto load_p = [&](P64& p, int k0) __attribute__((always_inline)) {
#pragma unroll
    for (int q = 0; q < FP_K / 8; ++q) {
      const int k = k0 + 8 * q + 4 * lh;
      if (k + 4 <= a.c) {
        p.x[q] = *reinterpret_cast<const f32x4_el*>(prow + k);
      } else {
#pragma unroll
        for (int s = 0; s < 4; ++s) p.x[q][s] = k + s < a.c ? prow[k + s] : 0.f;
      }
    }
  };
  // the sum of rows k0 .. + 63 as T, in `to`
  auto finish = [&](f32x4_t (&sum)[2], int k0, float (&to)[FP_K][TN]) __attribute__((always_inline)) {
    int t = threadIdx.x;  // (its indexes are formed again here: kept across the sum they cost the wide form its second workgroup per compute unit)
    asm("" : "+v"(t));
    const int sr = t / (TN / 4), sc = t % (TN / 4) * 4, back = a.m >= 4 ? max(n0 + sc + 4 - a.m, 0) : 0;
#pragma unroll
    for (int p = 0; p < 2; ++p) {
      const int k = k0 + sr + 32 * p;
      f32x4_t x = sum[p] * (k >= a.k_lo ? a.scale_hi : 1.f);
      if (back > 0) {
        const f32x4_t y = x;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          x[e] = 0.f;
#pragma unroll
          for (int f = e + 1; f < 4; ++f) x[e] = f - e == back ? y[f] : x[e];
        }
      }
      if (k >= a.c) x = f32x4_t{0.f, 0.f, 0.f, 0.f};
      *reinterpret_cast<f32x4_t*>(&to[sr + 32 * p][sc]) = x;
    }
  };
  auto multiply = [&](const P64& p, const float (&t)[FP_K][TN]) __attribute__((always_inline)) {
#pragma unroll
    for (int q = 0; q < FP_K / 8; ++q)
#pragma unroll
      for (int s = 0; s < 4; ++s)
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(p.x[q][s], t[8 * q + 4 * lh + s][wc + li], acc, 0, 0, 0);
  };
  auto by_element = [&](f32x4_t (&sum)[2], int k0) __attribute__((always_inline)) {
    for (int z = 0; z < a.splits; ++z)
#pragma unroll
      for (int p = 0; p < 2; ++p)
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (n0 + sc + e < a.m) sum[p][e] += col[z * slab + (int64_t)min(k0 + sr + 32 * p, a.c - 1) * a.m + e];
  };
  if constexpr (WC == 1) {
    // Eight slabs in flight, the last ones too (past the end: the last again, not added), and the first of the next rows of T while these
    // are multiplied.  Its registers halve the waves that fit, so where the launch fills the chip the plain loop below stays
    // ahead (23.6 us against 30.5 with 480 workgroups).
    struct Batch {
      f32x4_t x[8][2];
    };
    auto load = [&](Batch& b, int k0, int z0) __attribute__((always_inline)) {
#pragma unroll
      for (int z = 0; z < 8; ++z)
#pragma unroll
        for (int p = 0; p < 2; ++p)
          b.x[z][p] = *reinterpret_cast<const f32x4_el*>(col + min(z0 + z, a.splits - 1) * slab + (int64_t)min(k0 + sr + 32 * p, a.c - 1) * a.m);
    };
    P64 fp, fn;
    Batch b;
    load_p(fp, 0);
    if (a.m >= 4) load(b, 0, 0);
    for (int k0 = 0, it = 0; k0 < a.c; k0 += FP_K, it ^= 1) {
      f32x4_t sum[2] = {f32x4_t{0.f, 0.f, 0.f, 0.f}, f32x4_t{0.f, 0.f, 0.f, 0.f}};
      if (a.m >= 4) {  // uniform
        for (int z0 = 0; z0 < a.splits; z0 += 8) {
          if (z0 > 0) load(b, k0, z0);
#pragma unroll
          for (int z = 0; z < 8; ++z)
            if (z0 + z < a.splits) {
              sum[0] += b.x[z][0];
              sum[1] += b.x[z][1];
            }
        }
      } else {
        by_element(sum, k0);
      }
      const bool more = k0 + FP_K < a.c;  // uniform
      if (more) {
        load_p(fn, k0 + FP_K);
        if (a.m >= 4) load(b, k0 + FP_K, 0);
      }
      finish(sum, k0, T[it]);
      __syncthreads();  // (the buffer that is written next was multiplied before the barrier that everybody has passed)
      multiply(fp, T[it]);
      if (more) fp = fn;
    }
  } else {
    for (int k0 = 0; k0 < a.c; k0 += FP_K) {
      P64 fp;
      load_p(fp, k0);  // requested before the sum, which it does not depend on
      f32x4_t sum[2] = {f32x4_t{0.f, 0.f, 0.f, 0.f}, f32x4_t{0.f, 0.f, 0.f, 0.f}};
      if (a.m >= 4) {  // uniform
        const float* const q0 = col + (int64_t)min(k0 + sr, a.c - 1) * a.m;
        const float* const q1 = col + (int64_t)min(k0 + sr + 32, a.c - 1) * a.m;
#pragma unroll 8
        for (int z = 0; z < a.splits; ++z) {  // eight slabs in flight
          sum[0] += *reinterpret_cast<const f32x4_el*>(q0 + z * slab);
          sum[1] += *reinterpret_cast<const f32x4_el*>(q1 + z * slab);
        }
      } else {
        by_element(sum, k0);
      }
      if (k0 > 0) __syncthreads();  // the previous rows of T have been multiplied
      finish(sum, k0, T[0]);
      __syncthreads();
      multiply(fp, T[0]);
    }
  }
  if (OUT_BF16) {
    // neighbouring lanes hold neighbouring columns: of two registers (two rows) the even lane takes the first row's pair
    // of columns, the odd lane the second row's, so that stores are 4 bytes
    const int n = n0 + wc + (li & ~1);
#pragma unroll
    for (int v = 0; v < 16; v += 2) {
      const float give = (li & 1) ? acc[v] : acc[v + 1];
      const float got = __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(give), 0xB1, 0xf, 0xf, true));  // lane ^ 1
      float x0 = (li & 1) ? got : acc[v], x1 = (li & 1) ? acc[v + 1] : got;
      const int m = m0 + 8 * (v / 4) + 4 * lh + v % 4 + (li & 1);
      if (m >= a.d || n >= a.m) continue;
      bf16_t* o = reinterpret_cast<bf16_t*>(a.dW) + (int64_t)m * a.lddw + n;
      const bool two = n + 1 < a.m;
      if (a.beta != 0.f) {
        x0 += a.beta * __uint_as_float((uint32_t)o[0] << 16);
        if (two) x1 += a.beta * __uint_as_float((uint32_t)o[1] << 16);
      }
      const uint32_t w = pack2(x0, x1);
      if (two && (reinterpret_cast<uintptr_t>(o) & 3) == 0) {
        *reinterpret_cast<uint32_t*>(o) = w;
      } else {
        o[0] = (bf16_t)(w & 0xFFFFu);
        if (two) o[1] = (bf16_t)(w >> 16);
      }
    }
  } else {
    const int n = n0 + wc + li;
    if (n >= a.m) return;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const int m = m0 + 8 * (v / 4) + 4 * lh + v % 4;
      if (m >= a.d) continue;
      float* o = reinterpret_cast<float*>(a.dW) + (int64_t)m * a.lddw + n;
      *o = a.beta == 0.f ? acc[v] : acc[v] + a.beta * *o;
    }
  }
}

int64_t f32_k_per_split(int64_t K, int splits) { return std::max<int64_t>(round_up64((K + splits - 1) / splits, 8), 8); }

template <bool AKF, bool BKF>
void launch_gemm_f32_ops(prac_ctx* ctx, F32Args& a) {
  auto launch = [&](auto kern, int tm, int tn, int threads, int split_k = 1) {
    a.tiles_n = (a.N + tn - 1) / tn;
    const size_t smem = split_k > 1 ? (size_t)split_k * tm * tn * sizeof(float) : 0;  // at most 64 KB
    PRAC_LAUNCH(ctx, kern, dim3((unsigned)((int64_t)((a.M + tm - 1) / tm) * a.tiles_n), 1, a.splits), dim3(threads), smem, a);
  };
  switch (f32_tile(ctx->n_cu, a.M, a.N, a.K, a.splits, AKF)) {
    case F32Tile::T128x128: launch(gemm_f32_kernel<AKF, BKF, 2, 2, 2, 2, 1, Turn::ALL>, 128, 128, 256); break;
    case F32Tile::T128x64: launch(gemm_f32_kernel<AKF, BKF, 1, 2, 4, 1, 1, Turn::ALL>, 128, 64, 256); break;
    case F32Tile::T64x64: launch(gemm_f32_kernel<AKF, BKF, 2, 2, 1, 1, 4, Turn::TEST>, 64, 64, 256, 4); break;
    case F32Tile::T32x64_ONE_ROUND: launch(gemm_f32_kernel<AKF, BKF, 1, 2, 1, 1, 8, AKF ? Turn::TEST : Turn::ALL>, 32, 64, 512, 8); break;  // (AKF only)
    case F32Tile::T32x64: launch(gemm_f32_kernel<AKF, BKF, 1, 2, 1, 1, 8, Turn::ALL>, 32, 64, 512, 8); break;
    case F32Tile::T32x32: launch(gemm_f32_kernel<AKF, BKF, 1, 1, 1, 1, 8, Turn::SECOND_BODY>, 32, 32, 512, 8); break;
  }
}

}  // namespace

// Clocks a tile shape needs: the matrix instructions of a SIMD's waves (256 clocks per 32 x 32 block and 8-k chunk),
// or the chain of one wave when there are few (a ring of four chunks takes a memory latency, about 2400 clocks, to come
// round), or the bytes through L2 (about 8 KB per clock over the chip); then the stores of a wave's 16 rm rn registers,
// or the exchange of the partial tiles where k is split.  Measured at the ends of the range: 2048 x 64
// over 512 runs 9 us with 32 x 64 tiles and k split over eight waves against 17 - 23 us with 64 x 64 tiles through
// LDS; 8192 x 256 over 2048 takes 84 us (102 TFLOP/s) with 64 x 64 tiles against 143 us.
F32Tile f32_tile(int n_cu, int M, int N, int64_t K, int splits, bool a_k_fast) {
  const int64_t k = std::min(K, f32_k_per_split(K, splits));
  auto cost = [&](int tm, int tn, int rm, int rn, int waves, int sk) {
    const int64_t tiles = (int64_t)((M + tm - 1) / tm) * ((N + tn - 1) / tn) * splits;
    const double chunks = std::ceil((double)k / 8 / sk);
    const double per_simd = std::ceil((double)tiles * waves / (4.0 * n_cu));
    const double bytes = (double)tiles * (tm + tn) * 4 * k;
    return std::max({per_simd * chunks * 256 * rm * rn, std::ceil(chunks / 4) * 2400, bytes / 8192}) +
           (sk > 1 ? 1500 : per_simd * rm * rn * 700);
  };
  const double big = cost(128, 128, 2, 2, 4, 1), mid = cost(64, 64, 2, 2, 4, 4), small = cost(32, 64, 1, 2, 8, 8),
               flat = cost(128, 64, 1, 2, 4, 1);
  const double best = std::min({big, mid, small, flat});
  if (big == best) return F32Tile::T128x128;
  if (flat == best) return F32Tile::T128x64;
  // 32 x 32 tiles in place of 32 x 64 ones (same bits) or 64 x 64 ones.  A workgroup's waves share four SIMDs however many compute units idle, so
  // what counts is rounds of one workgroup per compute unit: 7 us of one per 1000 k instead of 11 (64 x 64: 20).  If A's k runs along memory,
  // more workgroups per compute unit wait for L1 (a load touches 32 lines): only without a round more.
  // us with 32 x 64 / 32 x 32: X P of 2048 x 512 -> 64, 128 small tiles, 8.7 / 5.5; 1500 x 1000 -> 100, 188, 13.7 / 10.1; 1024 x 2048 -> 256, 256, 24.4 / 15.8;
  // 8192 x 1024 -> 32, 256, 16.1 / 11.4; 5000 x 700 -> 90, 471, 17.8 / 14.9; a round more: 4096 x 1024 -> 128, 512, 14.9 / 17.4; 3001 x 1501 -> 201, 658,
  // 34.0 / 43.8.  C^T dY of 700 x 40 and 300 in two ranges, 40, 6.8 / 4.9; 2048 x 64 and 1376 in eight, 688, 11.4 / 9.7, in five, 430, 8.4 / 9.2; 1500 x 100
  // and 1000 in five, 640, 11.2 / 10.6; 8192 x 64 and 512 in 32, 1024, 11.9 / 11.6; 3001 x 201 and 1501 in five, 1645, 31.8 / 36.3.  Sixteen waves, or eight
  // chunks in flight, are 0.5 to 2 us behind.
  auto rounds = [&](int tn) { return ((int64_t)((M + 31) / 32) * ((N + tn - 1) / tn) * splits + n_cu - 1) / n_cu; };
  const bool one_more = !a_k_fast && mid != best && 7 * rounds(32) < 11 * rounds(64);
  if (rounds(32) == rounds(64) || one_more) return F32Tile::T32x32;
  if (mid == best) return F32Tile::T64x64;
  return a_k_fast && rounds(64) == 1 ? F32Tile::T32x64_ONE_ROUND : F32Tile::T32x64;
}

bool gemm_f32_takes(const GemmGenArgs& g) {
  return g.adt == PRAC_F32 && g.bdt == PRAC_F32 && !g.acc64 && !g.out64 && g.k_stride <= 1 && g.M >= 2 && g.N >= 2 &&
         (g.b_cs == 1 ? (g.a_rs == 1 || g.a_cs == 1) : (g.a_cs == 1 && g.b_rs == 1));  // (no product needs A^T B^T)
}

int launch_gemm_f32(prac_ctx* ctx, const GemmGenArgs& g, int splits) {
  F32Args a;
  const bool akf = g.a_cs == 1, bkf = g.b_cs != 1;
  a.A = reinterpret_cast<const float*>(g.A);
  a.B = reinterpret_cast<const float*>(g.B);
  a.lda = akf ? g.a_rs : g.a_cs;
  a.ldb = bkf ? g.b_cs : g.b_rs;
  a.M = g.M; a.N = g.N; a.K = g.K;
  a.out = g.out; a.ldo = g.ldo; a.alpha = g.alpha; a.beta = g.beta;
  a.splits = splits;
  a.k_per_split = f32_k_per_split(g.K, splits);
  a.slabs = reinterpret_cast<float*>(g.slabs);
  if (akf && bkf) launch_gemm_f32_ops<true, true>(ctx, a);
  else if (akf) launch_gemm_f32_ops<true, false>(ctx, a);
  else launch_gemm_f32_ops<false, false>(ctx, a);
  PRAC_HIP_TRY(ctx, hipGetLastError());
  return PRAC_OK;
}

int launch_f32_sum_pt(prac_ctx* ctx, const float* P, int64_t ldp, float* slabs, int splits, int c, int k_lo,
                      float scale_hi, int d, int m, void* dW, int64_t lddw, bool out_bf16, float beta) {
  F32SumPtArgs a;
  a.P = P; a.ldp = ldp; a.slabs = slabs; a.splits = splits; a.c = c; a.k_lo = k_lo; a.scale_hi = scale_hi;
  a.d = d; a.m = m; a.dW = dW; a.lddw = lddw; a.beta = beta;
  const int rows = (d + 127) / 128;
  // Half the columns, half the sum per workgroup, while each still has a compute unit to itself; past that the second round costs more
  // (weight gradient, 64 columns / 32: N = 2048, d = 512, m = 1376, c = 64, 172 narrow tiles, 23.4 / 19.4 us; 2048, 1024, 1024, 64, 256
  // of them, 16.1 / 15.0; 2048, 1024, 1088, 64, 272, 19.9 / 20.5; 4096, 1900, 700, 200, 330, 44.1 / 46.8; 512, 1536, 1024, 32, 384, 13.5 / 14.7).
  const bool narrow = (int64_t)((m + 31) / 32) * rows <= ctx->n_cu;
  a.tiles_n = narrow ? (m + 31) / 32 : (m + 63) / 64;
  const int64_t total = (int64_t)a.tiles_n * rows;
  if (total > INT32_MAX) return PRAC_EINVAL;
  // The sum of the slabs is repeated by every row tile; past a few dozen reads of each slab element's bytes a pass of
  // its own (into the first slab, in place) is cheaper.
  if (splits > 1 && splits * ((d + 127) / 128) > 40) {
    int rc = launch_reduce_slabs(ctx, slabs, splits, (int64_t)c * m, slabs, (int64_t)c * m, 1.f, 0.f);
    if (rc) return rc;
    a.splits = 1;
  }
  const dim3 grid((unsigned)total);
  auto launch = [&](auto kern, int threads) { PRAC_LAUNCH(ctx, kern, grid, dim3(threads), 0, a); };
  if (narrow && out_bf16) launch(f32_sum_pt_kernel<1, true>, 256);
  else if (narrow) launch(f32_sum_pt_kernel<1, false>, 256);
  else if (out_bf16) launch(f32_sum_pt_kernel<2, true>, 512);
  else launch(f32_sum_pt_kernel<2, false>, 512);
  PRAC_HIP_TRY(ctx, hipGetLastError());
  return PRAC_OK;
}
