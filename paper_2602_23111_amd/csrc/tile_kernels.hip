// C = X P for few token rows: where the 128 x 256 tiles of compress_ws_kernel leave compute units idle, smaller tiles whose
// sum over d is split over the waves of a workgroup, so that the call still is one launch that writes nothing but C.
//
// A wave multiplies every eighth 32-deep piece of k for the whole tile; operands go from memory straight to matrix registers (the rows of
// X as they lie, 32 bytes per lane and piece; P in its packed fragment order), without LDS or a barrier in the loop.  A fragment's
// k order is free as long as both operands use the same: lane half h of block b holds k = 32 g + 16 h + 8 b .. + 7, which are the
// neighbouring 16-byte halves of a lane's 32 bytes of X and half b of k-block 2 g + h of P.
// The waves' sums meet in LDS at the end and are added in wave order.
// What bounds it, with X in the caches (the same X again), is the bytes out of L2, 64 (1 + RN) d per tile (21 TB/s at 4096 x 2048 -> 256); with an X
// from memory (another one on each call, 640 MB of them) how much of it is requested at a time: 8192 x 8192 arrives at 2.4 to 3.6 TB/s.
// us per launch, compress_ws_kernel / here, X from memory and in brackets from the caches: 1024 x 256 -> 32 5.3 / 4.2 (5.3 / 4.2), 2048 x 768 -> 128
// 8.0 / 4.7 (9.1 / 4.5), 4096 x 2048 -> 64 18.9 / 11.3 (18.3 / 9.1), 4096 x 2048 -> 256 18.8 / 14.6 (18.2 / 10.7), 512 x 8192 -> 1024 59.7 / 32.2
// (59.0 / 29.7), 1018 x 5376 -> 836 41.3 / 32.3 (40.9 / 26.8), 8192 x 1024 -> 32 11.9 / 9.7 (10.6 / 6.3), 8192 x 8192 -> 128 68.7 / 54.9 (68.0 / 38.5).
#include <algorithm>
#include <type_traits>

#include "frag_utils.h"

namespace {

struct CompressTileArgs {
  const bf16_t* X;
  int64_t ldx;
  int N, d;
  const bf16_t* Pfrag;  // [nkb][ncb][64][8], zero outside d x c
  int ncb, c;
  bf16_t* C;  // row-major (ldc) or packed [ceil(N/128)*8][ccb][64][8]
  int64_t ldc;
  int ccb, packed;
  int tiles_m, tiles_n;
};

constexpr int CT_W = 8;  // waves that split k

// Tile 32 x 32 RN; D pieces of k in flight per wave.
template <int RN, int D>
__global__ __launch_bounds__(64 * CT_W) void compress_tile_kernel(CompressTileArgs a) {
  extern __shared__ __align__(16) unsigned char ct_smem[];
  f32x4_t* const red = reinterpret_cast<f32x4_t*>(ct_smem);  // [CT_W][RN][4 quads][64 lanes]
  const int bid = touch_kernel_args<sizeof(CompressTileArgs)>(blockIdx.x);
  // consecutive tiles of one row panel on one XCD
  const int total = a.tiles_m * a.tiles_n, per_xcd = (total + 7) / 8;
  const int logical = (bid & 7) * per_xcd + (bid >> 3);
  if ((bid >> 3) >= per_xcd || logical >= total) return;
  const int tm = logical / a.tiles_n, cb0 = (logical - tm * a.tiles_n) * RN, m0 = tm * 32;
  const int lane = threadIdx.x & 63, li = lane & 31, lh = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);

  // rows past N repeat the last one; they are not stored
  const char* const xbase = reinterpret_cast<const char*>(a.X + (int64_t)m0 * a.ldx);
  const uint32_t xrow = (uint32_t)min(li, a.N - 1 - m0) * (uint32_t)a.ldx * 2u, xoff = xrow + lh * 32u;
  const int64_t brow = (int64_t)a.ncb * 1024;  // bytes per k-block of fragments
  const uint32_t poff = (uint32_t)lh * (uint32_t)brow + (uint32_t)(cb0 * 64 + li) * 16u;
  const char* const pbase = reinterpret_cast<const char*>(a.Pfrag);

  f32x16 acc[RN];
#pragma unroll
  for (int j = 0; j < RN; ++j)
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[j][v] = 0.f;
  struct Piece {
    u32x4 x[2], p[RN][2];
  };
  auto load_p = [&](Piece& s, int g) __attribute__((always_inline)) {
    const char* const p = pbase + 2 * g * brow;
#pragma unroll
    for (int j = 0; j < RN; ++j)
#pragma unroll
      for (int b = 0; b < 2; ++b) s.p[j][b] = *reinterpret_cast<const u32x4*>(p + (poff + j * 1024 + b * 512));
  };
  auto load = [&](Piece& s, int g) __attribute__((always_inline)) {
    const char* const x = xbase + (int64_t)g * 64;
#pragma unroll
    for (int b = 0; b < 2; ++b) s.x[b] = *reinterpret_cast<const u32x4*>(x + (xoff + b * 16));
    load_p(s, g);
  };
  auto mul = [&](const Piece& s) __attribute__((always_inline)) {
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int j = 0; j < RN; ++j) acc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_frag(s.x[b]), as_frag(s.p[j][b]), acc[j], 0, 0, 0);
  };
  const int full = a.d / 32, n = full > wave ? (full - wave + CT_W - 1) / CT_W : 0;  // whole pieces: wave, wave + 8, ...
  Piece s[D];
  if (n > 0) {
    auto piece = [&](int t) { return wave + CT_W * min(t, n - 1); };  // past the last one: that one again, not used
#pragma unroll
    for (int u = 0; u < D; ++u) load(s[u], piece(u));
    int t = 0;
    for (; t + D <= n; t += D) {
#pragma unroll
      for (int u = 0; u < D; ++u) {
        mul(s[u]);
        load(s[u], piece(t + D + u));
      }
    }
#pragma unroll
    for (int u = 0; u < D - 1; ++u)
      if (t + u < n) mul(s[u]);
  }
  if (32 * full < a.d && full % CT_W == wave) {  // the last, partial piece: zeros past d, nothing read past the row's last chunk
    const int last = ((a.d - 1) / 8) * 8;
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      const int k = 32 * full + 16 * lh + 8 * b;
      s[0].x[b] = keep_first(*reinterpret_cast<const u32x4*>(xbase + (xrow + (uint32_t)min(k, last) * 2u)), a.d - k);
    }
    load_p(s[0], full);
    mul(s[0]);
  }

  // ---- the waves' sums: register v of lane (li, lh) is row 8 (v / 4) + 4 lh + v % 4, column li of column block j
#pragma unroll
  for (int j = 0; j < RN; ++j)
#pragma unroll
    for (int q = 0; q < 4; ++q)
      red[((wave * RN + j) * 4 + q) * 64 + lane] = f32x4_t{acc[j][4 * q], acc[j][4 * q + 1], acc[j][4 * q + 2], acc[j][4 * q + 3]};
  if (a.packed && tm == a.tiles_m - 1) {  // the padding of packed C behind the last row tile: whole 128-token tiles, zeros
    const int tb0 = m0 / 16 + 2, n_pad = (a.N + 127) / 128 * 8 - tb0;
    for (int i = wave; i < n_pad * RN; i += CT_W) {
      const int cb = cb0 + i % RN;
      if (cb < a.ccb) stream_store(reinterpret_cast<u32x4*>(a.C) + ((int64_t)(tb0 + i / RN) * a.ccb + cb) * 64 + lane, u32x4{0u, 0u, 0u, 0u});
    }
  }
  __syncthreads();
  // a wave finishes whole 16-token blocks of a column block (two quads), or single quads where there are fewer blocks than waves
  constexpr int Q = RN >= 4 ? 2 : 1, UNITS = RN * 4 / Q;
  if (wave >= UNITS) return;
  static_assert(UNITS <= CT_W, "one unit per wave");
  const int blk = wave * Q / 4, q0 = wave * Q % 4, cb = cb0 + blk;
  if (cb >= a.ccb) return;  // uniform
  f32x4_t sum[Q];
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    f32x4_t x[CT_W];
#pragma unroll
    for (int w = 0; w < CT_W; ++w) x[w] = red[((w * RN + blk) * 4 + q0 + q) * 64 + lane];
    sum[q] = x[0];
#pragma unroll
    for (int w = 1; w < CT_W; ++w) sum[q] += x[w];
  }
  const int t0 = m0 + 8 * q0 + 4 * lh;  // token of element 0
  if (a.packed) {
    u32x2 o[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (t0 + 8 * q + e >= a.N) sum[q][e] = 0.f;  // (the padding of packed C is zero)
      o[q] = u32x2{pack2_hw(sum[q][0], sum[q][1]), pack2_hw(sum[q][2], sum[q][3])};
    }
    u32x2* const dst = reinterpret_cast<u32x2*>(a.C) + (((int64_t)(m0 / 16 + q0 / 2) * a.ccb + cb) * 64 + lane) * 2 + (q0 & 1);
    if constexpr (Q == 2) stream_store(reinterpret_cast<u32x4*>(dst), u32x4{o[0].x, o[0].y, o[1].x, o[1].y});
    else stream_store(dst, o[0]);
  } else {
    const int col = cb * 32 + li;
    if (col >= a.c) return;
#pragma unroll
    for (int q = 0; q < Q; ++q)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int row = t0 + 8 * q + e;
        if (row < a.N) a.C[(int64_t)row * a.ldc + col] = (bf16_t)(pack2_hw(sum[q][e], 0.f) & 0xFFFFu);
      }
  }
}

}  // namespace

// The smallest tile whose workgroups each have a compute unit to themselves: a second round of them costs more than the larger tiles
// (X in the caches: 4096 x 2048 -> 256: 32 x 32 27.2 us, 32 x 64 18.7, 32 x 128 11.6), and past one round of the largest one compress_ws_kernel, which reads P a
// quarter as often, is ahead (8192 x 2048 -> 128 in one round 15.9, compress_ws_kernel 20.0; 8192 x 2048 -> 256 in two 27.4, 19.7).  Tiles of 64 rows
// never were the best (64 x 64 within 0.7 us of 32 x 128 at d = 768 and below, 4 us behind at 2048).
CompressTile compress_tile(int n_cu, int N, int c) {
  const int64_t rows = ((int64_t)N + 31) / 32, cols = (c + 31) / 32;
  if (rows * cols <= n_cu) return CompressTile::T32x32;
  if (rows * ((cols + 1) / 2) <= n_cu) return CompressTile::T32x64;
  if (rows * ((cols + 3) / 4) <= n_cu) return CompressTile::T32x128;
  return CompressTile::NONE;
}

int launch_compress_tile(prac_ctx* ctx, CompressTile tile, const bf16_t* X, int64_t ldx, int N, int d, const bf16_t* Pfrag, int ncb, int c,
                         bf16_t* C, int64_t ldc, bool packed) {
  if (ldx > PRAC_MAX_STREAM_PITCH || ncb % 8 != 0 || ncb * 32 < c) return PRAC_EINVAL;
  CompressTileArgs a;
  a.X = X; a.ldx = ldx; a.N = N; a.d = d; a.Pfrag = Pfrag; a.ncb = ncb; a.c = c; a.C = C; a.ldc = ldc;
  a.ccb = (c + 31) / 32; a.packed = packed ? 1 : 0;
  a.tiles_m = (int)(((int64_t)N + 31) / 32);  // as compress_tile counts them
  auto launch = [&](auto rnc, auto dc) -> int {
    constexpr int RN = decltype(rnc)::value;
    constexpr auto kern = compress_tile_kernel<RN, decltype(dc)::value>;
    constexpr size_t smem = (size_t)CT_W * RN * 4096;
    a.tiles_n = (a.ccb + RN - 1) / RN;
    const int64_t total = (int64_t)a.tiles_m * a.tiles_n;
    if (total > (1 << 28)) return PRAC_EINVAL;
    static bool done_dev[PRAC_MAX_DEVICES] = {};  // the attribute is per device
    bool& done = done_dev[ctx->device % PRAC_MAX_DEVICES];
    if (!done) {
      PRAC_HIP_TRY(ctx, hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem));
      done = true;
    }
    PRAC_LAUNCH(ctx, kern, dim3((unsigned)((total + 7) / 8 * 8)), dim3(64 * CT_W), smem, a);
    PRAC_HIP_TRY(ctx, hipGetLastError());
    return PRAC_OK;
  };
#define PRAC_IC(v) std::integral_constant<int, (v)> {}
  switch (tile) {
    case CompressTile::T32x32: return launch(PRAC_IC(1), PRAC_IC(4));
    case CompressTile::T32x64: return launch(PRAC_IC(2), PRAC_IC(4));
    case CompressTile::T32x128: return launch(PRAC_IC(4), PRAC_IC(3));
    default: return PRAC_EINVAL;
  }
#undef PRAC_IC
}
