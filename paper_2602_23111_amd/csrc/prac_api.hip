// C ABI of libprac (see include/prac.h): argument checks, scratch planning and the
// sequence of kernel launches behind each entry point.
#include <algorithm>
#include <new>

#include "prac_internal.h"

// Scratch of the entry point that allocates nothing (prac_weight_grad_static): one block per GPU,
// part of the code object, held until the process ends.  In host code the array's name is only a
// handle for hipGetSymbolAddress; prac_create asks for the block's device address once per
// device (with that device current) and everything else uses that address.
static __device__ __align__(256) unsigned char scratch[PRAC_STATIC_SCRATCH_BYTES];

namespace {

constexpr int kMaxDevices = PRAC_MAX_DEVICES;
char* g_static_scratch[kMaxDevices] = {};  // device address of `scratch` on each GPU, set by prac_create

inline bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; }
inline size_t esize(prac_dtype t) { return t == PRAC_BF16 ? 2 : 4; }
inline bool valid_dtype(int t) { return t == PRAC_F32 || t == PRAC_BF16; }
// token counts are 32-bit inside the kernels' launch arguments
inline bool bad_tokens(int64_t N) { return N < 1 || N >= ((int64_t)1 << 31); }

struct LpLayout {
  int64_t ldpt, ldpn;
  int nkb, ncb;  // fragment-order copy: 16-row blocks over round_up(d,256), 32-column blocks (multiple of 8)
  int nrb, nckb; // A-operand fragment copy: 32-row blocks over round_up(d,128), 16-column blocks over c
  size_t off_pn, off_pf, off_pa, bytes;
};
inline LpLayout lp_layout(int64_t d, int c) {
  LpLayout l;
  l.ldpt = round_up64(d, 64);
  l.ldpn = round_up64(c, 64);
  l.nkb = (int)(round_up64(d, 256) / 16);
  l.ncb = (int)round_up64((c + 31) / 32, 8);
  l.off_pn = ((size_t)c * l.ldpt * sizeof(bf16_t) + 255) & ~size_t(255);
  l.off_pf = (l.off_pn + (size_t)d * l.ldpn * sizeof(bf16_t) + 255) & ~size_t(255);
  l.nrb = (int)(round_up64(d, 128) / 32);
  l.nckb = (c + 15) / 16;
  l.off_pa = (l.off_pf + (size_t)l.nkb * l.ncb * 64 * 8 * sizeof(bf16_t) + 255) & ~size_t(255);
  l.bytes = l.off_pa + (size_t)l.nrb * l.nckb * 64 * 8 * sizeof(bf16_t);
  return l;
}
inline size_t packed_c_bytes(int64_t N, int c) {
  return (size_t)((N + 127) / 128) * 8 * ((c + 31) / 32) * 64 * 8 * sizeof(bf16_t);  // whole 128-token tiles
}

// split count for a reduction over K with `tiles` output tiles: fill the chip about
// twice over without making slabs shorter than `min_k`.
inline int pick_splits(int tiles, int64_t K, int n_cu, int min_k) {
  int s = (2 * n_cu + tiles - 1) / tiles;
  const int64_t cap = K / min_k;
  if (s > cap) s = (int)cap;
  if (s > 64) s = 64;
  return s < 1 ? 1 : s;
}

}  // namespace

int prac_ws_reserve(prac_ctx* ctx, size_t bytes) {
  if (bytes <= ctx->ws_bytes) return PRAC_OK;
  // Work already enqueued may still read the old block (on the ctx stream, or on a stream the ctx
  // was bound to earlier): wait for the device before replacing it.  Callers that must not wait
  // size the block up front (prac_workspace_bytes, prac_reserve_workspace).
  PRAC_HIP_TRY(ctx, hipDeviceSynchronize());
  if (ctx->ws) PRAC_HIP_TRY(ctx, hipFree(ctx->ws));
  ctx->ws = nullptr;
  ctx->ws_bytes = 0;
  const size_t want = bytes + bytes / 4;
  void* p = nullptr;
  hipError_t e = hipMalloc(&p, want);
  if (e != hipSuccess) {
    (void)hipGetLastError();
    e = hipMalloc(&p, bytes);
    if (e != hipSuccess) {
      (void)hipGetLastError();
      ctx->last_hip = (int)e;
      return PRAC_ENOMEM;
    }
    ctx->ws_bytes = bytes;
  } else {
    ctx->ws_bytes = want;
  }
  ctx->ws = reinterpret_cast<char*>(p);
  return PRAC_OK;
}

ProfScope::ProfScope(prac_ctx* c, int kind) : ctx(c) {
  c->ev_start = nullptr;
  c->ev_stop = nullptr;
  if (c->prof_kind != kind || kind == 0) return;
  if (c->prof_seen++ % c->prof_stride != 0) return;
  hipEvent_t ev[2] = {nullptr, nullptr};
  for (int i = 0; i < 2; ++i) {
    if (!c->prof_pool.empty()) {
      ev[i] = c->prof_pool.back();
      c->prof_pool.pop_back();
    } else if (hipEventCreate(&ev[i]) != hipSuccess) {
      (void)hipGetLastError();
      if (i == 1) c->prof_pool.push_back(ev[0]);
      return;
    }
  }
  c->prof_pairs.emplace_back(ev[0], ev[1]);
  c->ev_start = ev[0];
  c->ev_stop = ev[1];
}
ProfScope::~ProfScope() {
  // a launcher that did not take the pair leaves it unrecorded; prac_profile_read skips it
  ctx->ev_start = nullptr;
  ctx->ev_stop = nullptr;
}

namespace {
inline bool gram_fast(const void* X, prac_dtype xdt, int64_t rows, int64_t ldx, int64_t row_stride) {
  return xdt == PRAC_BF16 && aligned16(X) && ldx % 8 == 0 && rows < ((int64_t)1 << 31) &&
         ldx * (row_stride > 0 ? row_stride : 1) <= PRAC_MAX_STREAM_PITCH;
}
// bf16 rows the streaming kernels take at any alignment (a row must hold one 16-byte chunk)
inline bool stream_any(prac_dtype dt, int64_t width, int64_t pitch) {
  return dt == PRAC_BF16 && width >= 8 && pitch <= PRAC_MAX_STREAM_PITCH;
}
inline int gram_splits(int n_cu, int64_t d, int64_t rows) {
  const int tiles = (int)(((d + 127) / 128) * ((d + 127) / 128));
  return pick_splits(tiles, rows, n_cu, 512);
}
}  // namespace

namespace {
// Large Gram matrices run on the C^T dY kernel with X in both places (its streaming rate at
// d = 2048 is 2.5 times that of the tiled GEMM): X is first copied into the packed layout the
// kernel reads its C operand from.  Two forms: all tiles, whose sum of token ranges goes straight through the slabs, or only those on and above the
// diagonal (72 of 128 at d = 2048, three ranges instead of two), whose sum is written to both sides.  The latter wherever the estimate below
// says so.  Kernel and sum, all / upper, us: 32768 x 2048 233 + 10 / 155 + 15, 32768 x 768 45 + 8 / 34 + 12, 8192 x 4096 248 + 0 / 204 + 27; but
// 32768 x 256 15 + 4 / 15 + 23 (64 ranges either way, and few workgroups in the second sum), 8192 x 512 15 + 6 / 13 + 15, 2048 x 1500 22 + 7 / 18 + 16,
// 2048 x 4096 88 + 0 / 65 + 29.
inline bool gram_streaming(int64_t rows, int64_t d) { return rows >= 2048 && d >= 256; }
inline int64_t gram_stream_tiles(int64_t d, bool upper) {
  const int tiles_n = (int)((d + 127) / 128), row_groups = (int)((d + 255) / 256);
  return upper ? ctdy_upper_tiles(tiles_n, row_groups) : (int64_t)tiles_n * row_groups;
}
inline int gram_stream_splits(int n_cu, int64_t d, int64_t rows, bool upper) {
  int64_t s = n_cu / gram_stream_tiles(d, upper);
  if (s > rows / 256) s = rows / 256;
  if (s > 64) s = 64;
  return s < 1 ? 1 : (int)s;
}
// us of a form, fitted to the kernels' times in 12 shapes of d 256 to 4096: 9.5 and 1.75 per 128 tokens for a round of workgroups (0.65 of that for a last
// one that is not full), then the sum: by its bytes, in the upper form (half of the slabs read, rows that start off 128-byte lines at 2 / 3 of
// the rate) not below its trips over the slabs
inline double gram_stream_us(int n_cu, int64_t d, int64_t rows, bool upper) {
  const int splits = gram_stream_splits(n_cu, d, rows, upper);
  const int64_t wgs = gram_stream_tiles(d, upper) * splits, steps = ((rows + 127) / 128 + splits - 1) / splits;
  const double rounds = wgs <= n_cu ? 1.0 : (double)(wgs / n_cu) + (wgs % n_cu ? 0.65 : 0.0), mb = 4e-6 * (double)d * (double)d;
  const double sum = !upper ? (splits > 1 ? 1.5 + (splits + 1) * mb / 5.5 : 0.0)
                            : std::max(3.0 + 0.36 * splits, 1.0 + (0.5 * splits + 1) * mb / 3.5 * (d % 32 ? 1.5 : 1.0));
  return rounds * (9.5 + 1.75 * (double)steps) + sum;
}
struct GramPlan {
  bool streaming, upper;
  int splits;
  size_t o_part, o_g, o_pack, bytes;
};
inline GramPlan plan_gram(int n_cu, int64_t rows, int64_t d, int64_t ldg) {
  GramPlan g{};
  g.streaming = gram_streaming(rows, d);
  g.upper = g.streaming && gram_stream_us(n_cu, d, rows, true) < gram_stream_us(n_cu, d, rows, false);
  g.splits = g.streaming ? gram_stream_splits(n_cu, d, rows, g.upper) : gram_splits(n_cu, d, rows);
  WsPlan plan;
  g.o_part = plan.take(g.splits > 1 ? (size_t)g.splits * d * d * sizeof(float) : 0);
  g.o_g = plan.take(ldg == d || (g.upper && g.splits > 1) ? 0 : (size_t)d * d * sizeof(float));
  g.o_pack = plan.take(g.streaming ? packed_c_bytes(rows, (int)d) : 0);
  g.bytes = plan.off;
  return g;
}
}  // namespace

namespace {
// How a Gram matrix reads its rows: on the bf16 matrix cores in whole 16-byte chunks (aligned rows), there at the
// alignment of one element (large enough for the streaming kernel), or strided.  ldx itself decides what is aligned, not the
// pitch ldx * row_stride of the sampled rows: the chunk that holds the last row's end must lie inside that row's ldx elements.
enum class GramRows { STRIDED = 0, ALIGNED = 1, ANY = 2 };
inline GramRows gram_rows(const void* X, prac_dtype xdt, int64_t rows, int64_t d, int64_t ldx, int64_t row_stride) {
  if (gram_fast(X, xdt, rows, ldx, row_stride)) return GramRows::ALIGNED;
  return stream_any(xdt, d, ldx * row_stride) && rows < ((int64_t)1 << 31) && gram_streaming(rows, d) ? GramRows::ANY
                                                                                                      : GramRows::STRIDED;
}
}  // namespace

size_t gram_scratch_bytes(int n_cu, const void* X, prac_dtype xdt, int64_t N, int64_t d, int64_t ldx,
                          int64_t row_stride, int64_t ldg) {
  const int64_t rows = (N + row_stride - 1) / row_stride;
  if (gram_rows(X, xdt, rows, d, ldx, row_stride) == GramRows::STRIDED) return 0;
  return plan_gram(n_cu, rows, d, ldg).bytes;
}

// G = Xs^T Xs with all scratch taken from `scratch` (gram_scratch_bytes of it).
int gram_device(prac_ctx* ctx, const void* X, prac_dtype xdt, int64_t N, int64_t d, int64_t ldx, int64_t row_stride,
                float* G, int64_t ldg, char* scratch) {
  const int64_t rows = (N + row_stride - 1) / row_stride;
  const GramRows how = gram_rows(X, xdt, rows, d, ldx, row_stride);
  if (how != GramRows::STRIDED) {
    const GramPlan gp = plan_gram(ctx->n_cu, rows, d, ldg);
    const int splits = gp.splits;
    const size_t o_part = gp.o_part, o_g = gp.o_g;
    float* dense = ldg == d ? G : reinterpret_cast<float*>(scratch + o_g);
    float* partial = splits > 1 ? reinterpret_cast<float*>(scratch + o_part) : nullptr;
    int rc;
    if (gp.streaming) {
      const bf16_t* Xb = reinterpret_cast<const bf16_t*>(X);
      bf16_t* Xpk = reinterpret_cast<bf16_t*>(scratch + gp.o_pack);
      const int64_t ld = ldx * row_stride;
      rc = launch_pack_c(ctx, Xb, ld, (int)rows, (int)d, Xpk);
      if (rc) return rc;
      const int dm = (int)d;
      float* out = splits > 1 ? partial : dense;
      {
        ProfScope ps(ctx, PRAC_KERNEL_GRAM);
        rc = launch_ctdy_ws(ctx, Xpk, dm, (int)rows, 1, &Xb, &ld, &dm, &out, splits, how == GramRows::ANY, 0, nullptr, nullptr, gp.upper);
      }
      if (rc) return rc;
      if (gp.upper) return launch_reduce_symmetric(ctx, out, splits, dm, G, ldg);
    } else {
      GemmBf16Args g{};
      g.A = reinterpret_cast<const bf16_t*>(X);
      g.lda = ldx * row_stride;
      g.M = (int)d;
      g.K = (int)rows;
      g.a_kc = false;
      g.b_kc = false;
      g.b0 = GemmOperandB{reinterpret_cast<const bf16_t*>(X), ldx * row_stride, (int)d, dense, d};
      g.b1 = GemmOperandB{nullptr, 0, 0, nullptr, 0};
      g.out_bf16 = false;
      g.beta = 0.f;
      g.splits = splits;
      g.partial = partial;
      g.tile_hint = 0;
      ProfScope ps(ctx, PRAC_KERNEL_GRAM);
      rc = launch_gemm_bf16(ctx, g);
      if (rc) return rc;
    }
    if (splits > 1) {
      rc = launch_reduce_slabs(ctx, partial, splits, (int64_t)d * d, dense, (int64_t)d * d, 1.f, 0.f);
      if (rc) return rc;
    }
    if (dense != G) return launch_cast_out(ctx, dense, d, G, PRAC_F32, ldg, (int)d, (int)d, 0.f);
    return PRAC_OK;
  }
  GemmGenArgs g{};
  g.A = X; g.B = X; g.adt = xdt; g.bdt = xdt;
  g.a_rs = 1; g.a_cs = ldx; g.b_rs = ldx; g.b_cs = 1;
  g.M = (int)d; g.N = (int)d; g.K = N; g.k_stride = row_stride;
  g.out = G; g.ldo = ldg; g.alpha = 1.f; g.beta = 0.f; g.acc64 = false; g.out64 = nullptr;
  return launch_gemm_generic(ctx, g);
}

extern "C" {

const char* prac_strerror(int s) {
  switch (s) {
    case PRAC_OK: return "ok";
    case PRAC_EINVAL: return "invalid argument";
    case PRAC_ENOMEM: return "out of device memory";
    case PRAC_EHIP: return "HIP runtime error";
    case PRAC_ENUMERIC: return "numeric breakdown";
    case PRAC_EUNSUPPORTED: return "unsupported request";
    case PRAC_ENOCTX: return "null context";
    case PRAC_ETOOBIG: return "request needs more scratch than the static block holds";
    default: return "unknown status";
  }
}

int prac_create(prac_ctx** out, int device, void* hip_stream) {
  if (!out || device < 0) return PRAC_EINVAL;
  *out = nullptr;
  int ndev = 0;
  if (hipGetDeviceCount(&ndev) != hipSuccess || device >= ndev) {
    (void)hipGetLastError();
    return PRAC_EHIP;
  }
  if (hipSetDevice(device) != hipSuccess) return PRAC_EHIP;
  prac_ctx* c = new (std::nothrow) prac_ctx();
  if (!c) return PRAC_ENOMEM;
  c->device = device;
  c->stream = reinterpret_cast<hipStream_t>(hip_stream);
  c->ws = nullptr;
  c->ws_bytes = 0;
  c->d_flag = nullptr;
  c->last_hip = 0;
  c->prof_kind = 0;
  c->prof_stride = 1;
  c->prof_seen = 0;
  c->ev_start = nullptr;
  c->ev_stop = nullptr;
  c->tune_splits = 0;
  c->tune_one_launch = 0;
  c->tune_tail = 0;
  c->d_sync = nullptr;
  c->part32 = nullptr;
  c->tails = nullptr;
  hipDeviceProp_t prop;
  c->n_cu = (hipGetDeviceProperties(&prop, device) == hipSuccess) ? prop.multiProcessorCount : 256;
  // failure flag (256 bytes), the counters of the one-launch weight gradient, the fp32 partial sums, the block `tails`
  const size_t flag_bytes = 256 + PRAC_SYNC_BYTES;
  if (hipMalloc(reinterpret_cast<void**>(&c->d_flag), flag_bytes + PRAC_PART32_BYTES + (size_t)c->n_cu * PRAC_TAIL_BYTES) != hipSuccess) {
    (void)hipGetLastError();
    delete c;
    return PRAC_EHIP;
  }
  c->d_sync = c->d_flag + 64;
  c->part32 = reinterpret_cast<float*>(reinterpret_cast<char*>(c->d_flag) + flag_bytes);
  c->tails = c->part32 + PRAC_PART32_BYTES / sizeof(float);
  if (hipMemset(c->d_flag, 0, flag_bytes) != hipSuccess) {
    (void)hipGetLastError();
    (void)hipFree(c->d_flag);
    delete c;
    return PRAC_EHIP;
  }
  // address of this device's copy of the static scratch block (the device is current here)
  c->static_scratch = device < kMaxDevices ? g_static_scratch[device] : nullptr;
  if (!c->static_scratch) {
    void* p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) {
      (void)hipGetLastError();
      (void)hipFree(c->d_flag);
      delete c;
      return PRAC_EHIP;
    }
    c->static_scratch = reinterpret_cast<char*>(p);
    if (device < kMaxDevices) g_static_scratch[device] = c->static_scratch;
  }
  *out = c;
  return PRAC_OK;
}

int prac_destroy(prac_ctx* ctx) {
  if (!ctx) return PRAC_ENOCTX;
  (void)hipStreamSynchronize(ctx->stream);
  if (ctx->ws) (void)hipFree(ctx->ws);
  if (ctx->d_flag) (void)hipFree(ctx->d_flag);
  for (auto& pr : ctx->prof_pairs) {
    (void)hipEventDestroy(pr.first);
    (void)hipEventDestroy(pr.second);
  }
  for (auto& ev : ctx->prof_pool) (void)hipEventDestroy(ev);
  delete ctx;
  return PRAC_OK;
}

int prac_set_stream(prac_ctx* ctx, void* hip_stream) {
  if (!ctx) return PRAC_ENOCTX;
  ctx->stream = reinterpret_cast<hipStream_t>(hip_stream);
  return PRAC_OK;
}

int prac_sync_status(prac_ctx* ctx) {
  if (!ctx) return PRAC_ENOCTX;
  int flag = 0;
  PRAC_HIP_TRY(ctx, hipStreamSynchronize(ctx->stream));
  PRAC_HIP_TRY(ctx, hipMemcpy(&flag, ctx->d_flag, sizeof(int), hipMemcpyDeviceToHost));
  if (flag != 0) {
    PRAC_HIP_TRY(ctx, hipMemset(ctx->d_flag, 0, sizeof(int)));
    if (flag & 4) {
      // a wait between workgroups of the one-launch weight gradient gave up: its counters may be left
      // non-zero, clear them for the next launch  (bits 1 and 2 are the basis fit's: a pivot that was
      // not positive or a basis that did not come out orthonormal, an eigen-iteration that did not settle)
      PRAC_HIP_TRY(ctx, hipMemset(ctx->d_sync, 0, PRAC_SYNC_BYTES));
      return PRAC_EHIP;
    }
    return PRAC_ENUMERIC;
  }
  return PRAC_OK;
}

int prac_last_hip_error(const prac_ctx* ctx) { return ctx ? ctx->last_hip : 0; }

int prac_profile_select(prac_ctx* ctx, int kind) {
  if (kind < PRAC_KERNEL_NONE || kind > PRAC_KERNEL_SUM_P_T) return PRAC_EINVAL;
  if (!ctx) return PRAC_ENOCTX;
  ctx->prof_kind = kind;
  ctx->prof_seen = 0;
  return PRAC_OK;
}

int prac_set_tuning(prac_ctx* ctx, int key, int value) {
  if (key == PRAC_TUNE_PROFILE_STRIDE) {
    if (value < 0 || value > 1024) return PRAC_EINVAL;
    if (!ctx) return PRAC_ENOCTX;
    ctx->prof_stride = value < 1 ? 1 : value;
    return PRAC_OK;
  }
  if (key == PRAC_TUNE_WGRAD_TAIL) {
    if (value < 0 || value > 2) return PRAC_EINVAL;
    if (!ctx) return PRAC_ENOCTX;
    ctx->tune_tail = value;
    return PRAC_OK;
  }
  if (key == PRAC_TUNE_WGRAD_ONE_LAUNCH) {
    if (value != 0 && value != 1) return PRAC_EINVAL;
    if (!ctx) return PRAC_ENOCTX;
    ctx->tune_one_launch = value;
    return PRAC_OK;
  }
  if (key != PRAC_TUNE_CTDY_SPLITS || value < 0 || value > 64) return PRAC_EINVAL;
  if (!ctx) return PRAC_ENOCTX;
  ctx->tune_splits = value;
  return PRAC_OK;
}

int prac_profile_read_each(prac_ctx* ctx, float* each_ms, int64_t cap, int64_t* launches) {
  if (!launches || cap < 0 || (cap > 0 && !each_ms)) return PRAC_EINVAL;
  if (!ctx) return PRAC_ENOCTX;
  PRAC_HIP_TRY(ctx, hipStreamSynchronize(ctx->stream));
  int64_t n = 0;
  for (auto& pr : ctx->prof_pairs) {
    float ms = 0.f;
    if (hipEventElapsedTime(&ms, pr.first, pr.second) == hipSuccess) {
      if (n < cap) each_ms[n] = ms;
      ++n;
    } else {
      (void)hipGetLastError();  // a pair no launch took: its events were never recorded
    }
    ctx->prof_pool.push_back(pr.first);
    ctx->prof_pool.push_back(pr.second);
  }
  ctx->prof_pairs.clear();
  *launches = n;
  return PRAC_OK;
}

int prac_profile_read(prac_ctx* ctx, double* total_ms, int64_t* launches) {
  if (!total_ms || !launches) return PRAC_EINVAL;
  if (!ctx) return PRAC_ENOCTX;
  std::vector<float> each(ctx->prof_pairs.size());
  int rc = prac_profile_read_each(ctx, each.data(), (int64_t)each.size(), launches);
  if (rc) return rc;
  double sum = 0.0;
  for (int64_t i = 0; i < *launches; ++i) sum += each[(size_t)i];
  *total_ms = sum;
  return PRAC_OK;
}

// ---------------------------------------------------------------- Gaussian draw
int prac_philox_words(prac_ctx* ctx, uint64_t seed, uint64_t draw, uint32_t stream, uint32_t* out, int64_t n) {
  if (n < 0 || (n > 0 && !out) || draw > 0xFFFFFFFFull) return PRAC_EINVAL;
  if (!ctx) return PRAC_ENOCTX;
  return launch_philox(ctx, seed, (uint32_t)draw, stream, out, n, false);
}

int prac_philox_normal(prac_ctx* ctx, uint64_t seed, uint64_t draw, uint32_t stream, float* out, int64_t n) {
  if (n < 0 || (n > 0 && !out) || draw > 0xFFFFFFFFull) return PRAC_EINVAL;
  if (!ctx) return PRAC_ENOCTX;
  return launch_philox(ctx, seed, (uint32_t)draw, stream, out, n, true);
}

// ------------------------------------------------------------------------- Gram
int prac_gram(prac_ctx* ctx, const void* X, prac_dtype xdt, int64_t N, int64_t d, int64_t ldx, int64_t row_stride,
              float* G, int64_t ldg) {
  if (!X || !G || !valid_dtype(xdt) || bad_tokens(N) || d < 1 || d > (1 << 20) || ldx < d || ldg < d || row_stride < 1)
    return PRAC_EINVAL;
  if (!ctx) return PRAC_ENOCTX;
  const size_t need = gram_scratch_bytes(ctx->n_cu, X, xdt, N, d, ldx, row_stride, ldg);
  int rc = prac_ws_reserve(ctx, need);
  if (rc) return rc;
  return gram_device(ctx, X, xdt, N, d, ldx, row_stride, G, ldg, ctx->ws);
}

// ------------------------------------------------------------------------ basis
size_t prac_basis_lp_bytes(int64_t d, int c) {
  if (d < 1 || c < 1) return 0;
  return lp_layout(d, c).bytes;
}

int prac_pack_basis(prac_ctx* ctx, const float* P, int64_t d, int64_t ldp, int c, void* P_lp) {
  if (!P || !P_lp || d < 1 || c < 1 || c > d || ldp < c || !aligned16(P_lp)) return PRAC_EINVAL;
  if (!ctx) return PRAC_ENOCTX;
  const LpLayout l = lp_layout(d, c);
  char* base = reinterpret_cast<char*>(P_lp);
  auto at = [&](size_t off) { return reinterpret_cast<bf16_t*>(base + off); };
  return launch_pack_basis(ctx, P, d, ldp, c, {at(0), at(l.off_pn), at(l.off_pf), at(l.off_pa), l.ldpt, l.ldpn, l.nkb, l.ncb, l.nrb, l.nckb});
}

int prac_fit_basis(prac_ctx* ctx, const void* X, prac_dtype xdt, int64_t N, int64_t d, int64_t ldx, int k, int r,
                   uint64_t seed, uint64_t draw, int refresh, const prac_fit_opts* opts, float* P, int64_t ldp,
                   void* P_lp, float* scale) {
  if (!P || d < 1 || d > (1 << 20) || k < 0 || r < 0 || k + r < 1 || (int64_t)k + r > d || ldp < k + r ||
      draw > 0xFFFFFFFFull || (refresh & ~3) != 0)
    return PRAC_EINVAL;
  const bool need_x = (refresh & PRAC_REFRESH_PRINCIPAL) && k > 0;
  if (need_x && (!X || !valid_dtype(xdt) || bad_tokens(N) || ldx < d)) return PRAC_EINVAL;
  prac_fit_opts o{};
  if (opts) o = *opts;
  if (o.iters < 0 || o.row_stride < 0 || (o.warm_start != 0 && o.warm_start != 1)) return PRAC_EINVAL;
  if (o.iters == 0) o.iters = 8;
  if (o.row_stride == 0) o.row_stride = 1;
  if (P_lp && !aligned16(P_lp)) return PRAC_EINVAL;
  if (!ctx) return PRAC_ENOCTX;
  if (scale) *scale = r > 0 ? (float)((double)(d - k) / (double)r) : 0.f;
  int rc = fit_basis_device(ctx, X, xdt, N, d, ldx, k, r, seed, (uint32_t)draw, refresh, o, P, ldp);
  if (rc) return rc;
  if (P_lp) return prac_pack_basis(ctx, P, d, ldp, k + r, P_lp);
  return PRAC_OK;
}

// --------------------------------------------------------------------- compress
size_t prac_compressed_bytes(int64_t N, int c, prac_dtype dt, int c_layout, int64_t ldc) {
  if (N < 1 || c < 1 || !valid_dtype(dt)) return 0;
  if (c_layout == PRAC_C_PACKED) return dt == PRAC_BF16 ? packed_c_bytes(N, c) : 0;
  if (c_layout != PRAC_C_ROWMAJOR || ldc < c) return 0;
  return (size_t)N * ldc * esize(dt);
}

int prac_unpack_compressed(prac_ctx* ctx, const void* Cpk, int64_t N, int c, void* C, int64_t ldc) {
  if (!Cpk || !C || bad_tokens(N) || c < 1 || ldc < c || !aligned16(Cpk)) return PRAC_EINVAL;
  if (!ctx) return PRAC_ENOCTX;
  return launch_unpack_c(ctx, reinterpret_cast<const bf16_t*>(Cpk), (int)N, c, reinterpret_cast<bf16_t*>(C), ldc);
}

namespace {
// How a compress / fused-forward call runs: STREAM, the bf16 kernels on aligned rows; STREAM_ANY, the same kernels on
// rows that start on any element, with the fp32 P as three bf16 parts; STRIDED, everything else (fp32 data, rows
// of fewer than 8 elements, pitches above PRAC_MAX_STREAM_PITCH).  At N = 32768, d = 5461 (contiguous rows), c = 256
// STREAM_ANY takes 0.23 ms, packing included, where the strided kernel and its cast take 2.5 ms (and STREAM with
// padded rows 0.11 ms: a third of the matrix instructions).
enum class CompressPath { STREAM, STREAM_ANY, STRIDED };
struct CompressPlan {
  size_t o_lp, o_w, o_tmp, o_c, bytes;
  int ncb_w;
};
CompressPlan plan_compress(CompressPath path, bool fused, bool packed, bool has_lp, prac_dtype xdt, int64_t N, int64_t d,
                           int c, int64_t m) {
  CompressPlan q{};
  WsPlan plan;
  if (path != CompressPath::STRIDED) {
    const LpLayout l = lp_layout(d, c);
    if (path == CompressPath::STREAM)
      q.o_lp = plan.take(has_lp ? 0 : l.bytes);
    else
      q.o_lp = plan.take((size_t)l.nkb * 3 * l.ncb * 64 * 8 * sizeof(bf16_t));
    q.ncb_w = fused ? (int)round_up64((m + 31) / 32, 8) : 0;  // whole 256-column groups
    q.o_w = plan.take(fused ? (size_t)l.nkb * q.ncb_w * 64 * 8 * sizeof(bf16_t) : 0);
  } else {
    const bool need_tmp = xdt == PRAC_BF16;
    q.o_tmp = plan.take(need_tmp ? (size_t)N * (c > m ? c : (size_t)m) * sizeof(float) : 0);
    q.o_c = plan.take(packed ? (size_t)N * round_up64(c, 8) * sizeof(bf16_t) : 0);
  }
  q.bytes = plan.off;
  return q;
}
}  // namespace

static int compress_impl(prac_ctx* ctx, const void* X, prac_dtype xdt, int64_t N, int64_t d, int64_t ldx,
                         const void* W, int64_t m, int64_t ldw, int w_layout, const float* P, const void* P_lp,
                         int64_t ldp, int c, void* Y, int64_t ldy, void* C, int64_t ldc, int c_layout) {
  const bool fused = W != nullptr;
  const bool packed = c_layout == PRAC_C_PACKED;
  const bool fast = xdt == PRAC_BF16 && aligned16(X) && ldx % 8 == 0 && ldx <= PRAC_MAX_STREAM_PITCH &&
                    N < ((int64_t)1 << 31);
  if (packed && (xdt != PRAC_BF16 || !aligned16(C))) return PRAC_EUNSUPPORTED;
  const CompressPath path = fast ? CompressPath::STREAM
                                 : (stream_any(xdt, d, ldx) ? CompressPath::STREAM_ANY : CompressPath::STRIDED);
  const CompressPlan q = plan_compress(path, fused, packed, P_lp != nullptr, xdt, N, d, c, m);
  if (q.bytes) {
    int rc = prac_ws_reserve(ctx, q.bytes);
    if (rc) return rc;
  }
  if (fast) {
    const LpLayout l = lp_layout(d, c);
    const size_t o_lp = q.o_lp, o_w = q.o_w;
    const int ncb_w = q.ncb_w;
    int rc;
    const char* lp = reinterpret_cast<const char*>(P_lp);
    if (!lp) {
      rc = prac_pack_basis(ctx, P, d, ldp, c, ctx->ws + o_lp);
      if (rc) return rc;
      lp = ctx->ws + o_lp;
    }
    const bf16_t* Pf = reinterpret_cast<const bf16_t*>(lp + l.off_pf);
    if (!fused) {
      ProfScope ps(ctx, PRAC_KERNEL_COMPRESS);
      return launch_compress_ws(ctx, reinterpret_cast<const bf16_t*>(X), ldx, (int)N, (int)d, Pf, l.ncb, c,
                                reinterpret_cast<bf16_t*>(C), ldc, packed, nullptr, 0, 0, nullptr, 0);
    }
    // W changes every step, so it is put into fragment order on every call (a pure permutation
    // of its d x m elements), then one launch forms Y and C
    bf16_t* Wf = reinterpret_cast<bf16_t*>(ctx->ws + o_w);
    rc = launch_pack_wfrag(ctx, reinterpret_cast<const bf16_t*>(W), ldw, w_layout, d, (int)m, l.nkb, ncb_w, Wf);
    if (rc) return rc;
    ProfScope ps(ctx, PRAC_KERNEL_FUSED_FWD);
    return launch_compress_ws(ctx, reinterpret_cast<const bf16_t*>(X), ldx, (int)N, (int)d, Pf, l.ncb, c,
                              reinterpret_cast<bf16_t*>(C), ldc, packed, Wf, ncb_w, (int)m,
                              reinterpret_cast<bf16_t*>(Y), ldy, false, ctx->tails);
  }
  if (path == CompressPath::STREAM_ANY) {
    const LpLayout l = lp_layout(d, c);
    bf16_t* Ps = reinterpret_cast<bf16_t*>(ctx->ws + q.o_lp);
    int rc = launch_pack_pfrag_split(ctx, P, d, ldp, c, l.nkb, l.ncb, Ps);
    if (rc) return rc;
    bf16_t* Wf = nullptr;
    if (fused) {
      Wf = reinterpret_cast<bf16_t*>(ctx->ws + q.o_w);
      rc = launch_pack_wfrag(ctx, reinterpret_cast<const bf16_t*>(W), ldw, w_layout, d, (int)m, l.nkb, q.ncb_w, Wf);
      if (rc) return rc;
    }
    ProfScope ps(ctx, fused ? PRAC_KERNEL_FUSED_FWD : PRAC_KERNEL_COMPRESS);
    return launch_compress_ws(ctx, reinterpret_cast<const bf16_t*>(X), ldx, (int)N, (int)d, Ps, l.ncb, c,
                              reinterpret_cast<bf16_t*>(C), ldc, packed, Wf, q.ncb_w, (int)m, reinterpret_cast<bf16_t*>(Y),
                              ldy, true, ctx->tails);
  }
  // strided path: fp32 data (P used in fp32), and bf16 rows the streaming kernels do not take
  const bool need_tmp = xdt == PRAC_BF16;
  const size_t o_tmp = q.o_tmp, o_c = q.o_c;
  float* tmp = need_tmp ? reinterpret_cast<float*>(ctx->ws + o_tmp) : nullptr;
  void* Crm = packed ? static_cast<void*>(ctx->ws + o_c) : C;
  const int64_t ldcrm = packed ? round_up64(c, 8) : ldc;
  GemmGenArgs g{};
  g.A = X; g.adt = xdt; g.a_rs = ldx; g.a_cs = 1;
  g.M = (int)N; g.K = d; g.k_stride = 1; g.alpha = 1.f; g.beta = 0.f; g.acc64 = false; g.out64 = nullptr;
  // C = X P
  g.B = P; g.bdt = PRAC_F32; g.b_rs = ldp; g.b_cs = 1; g.N = c;
  g.out = need_tmp ? tmp : reinterpret_cast<float*>(C);
  g.ldo = need_tmp ? c : ldc;
  int rc = launch_gemm_generic(ctx, g);
  if (rc) return rc;
  if (need_tmp) {
    rc = launch_cast_out(ctx, tmp, c, Crm, PRAC_BF16, ldcrm, (int)N, c, 0.f);
    if (rc) return rc;
    if (packed) {
      rc = launch_pack_c(ctx, reinterpret_cast<const bf16_t*>(Crm), ldcrm, (int)N, c, reinterpret_cast<bf16_t*>(C));
      if (rc) return rc;
    }
  }
  if (fused) {
    g.B = W; g.bdt = xdt; g.N = (int)m;
    if (w_layout == 1) { g.b_rs = 1; g.b_cs = ldw; } else { g.b_rs = ldw; g.b_cs = 1; }
    g.out = need_tmp ? tmp : reinterpret_cast<float*>(Y);
    g.ldo = need_tmp ? m : ldy;
    rc = launch_gemm_generic(ctx, g);
    if (rc) return rc;
    if (need_tmp) rc = launch_cast_out(ctx, tmp, m, Y, PRAC_BF16, ldy, (int)N, (int)m, 0.f);
  }
  return rc;
}

static bool bad_c_layout(int c_layout, int64_t ldc, int c) {
  if (c_layout == PRAC_C_PACKED) return false;
  return c_layout != PRAC_C_ROWMAJOR || ldc < c;
}

int prac_compress(prac_ctx* ctx, const void* X, prac_dtype xdt, int64_t N, int64_t d, int64_t ldx, const float* P,
                  const void* P_lp, int64_t ldp, int c, void* C, int64_t ldc, int c_layout) {
  if (!X || !P || !C || !valid_dtype(xdt) || bad_tokens(N) || d < 1 || d > (1 << 20) || c < 1 || c > d || ldx < d ||
      ldp < c || bad_c_layout(c_layout, ldc, c) || (P_lp && !aligned16(P_lp)))
    return PRAC_EINVAL;
  if (!ctx) return PRAC_ENOCTX;
  return compress_impl(ctx, X, xdt, N, d, ldx, nullptr, 0, 0, 0, P, P_lp, ldp, c, nullptr, 0, C, ldc, c_layout);
}

int prac_compress_fused_fwd(prac_ctx* ctx, const void* X, prac_dtype xdt, int64_t N, int64_t d, int64_t ldx,
                            const void* W, int64_t m, int64_t ldw, int w_layout, const float* P, const void* P_lp,
                            int64_t ldp, int c, void* Y, int64_t ldy, void* C, int64_t ldc, int c_layout) {
  if (!X || !P || !C || !W || !Y || !valid_dtype(xdt) || bad_tokens(N) || d < 1 || d > (1 << 20) || c < 1 || c > d ||
      m < 1 || m > (1 << 20) || ldx < d || ldp < c || bad_c_layout(c_layout, ldc, c) || ldy < m ||
      (w_layout != 0 && w_layout != 1) || ldw < (w_layout == 1 ? d : m) || (P_lp && !aligned16(P_lp)))
    return PRAC_EINVAL;
  if (!ctx) return PRAC_ENOCTX;
  return compress_impl(ctx, X, xdt, N, d, ldx, W, m, ldw, w_layout, P, P_lp, ldp, c, Y, ldy, C, ldc, c_layout);
}

}  // extern "C"

// ------------------------------------------------------------------ weight grad
namespace {

// One gradient in fp32 (fp32 data; bf16 data the streaming kernels do not take): T = C^T dY, for fp32 data as
// token-split partial sums, then their sum, the scaling factor and dW = P T in one launch.
struct WgradGenPlan {
  size_t o_t, o_crm, bytes;
};
WgradGenPlan plan_wgrad_generic(int64_t N, int64_t m, int c, bool packed) {
  WgradGenPlan q{};
  WsPlan plan;
  q.o_t = plan.take((size_t)c * m * sizeof(float));
  q.o_crm = plan.take(packed ? (size_t)N * c * sizeof(bf16_t) : 0);
  q.bytes = plan.off;
  return q;
}
// Token ranges until 64 x 64 tiles of T give every compute unit two workgroups, each range long enough for the k split
// inside a workgroup (8 waves x 4 chunks of 8); on 256 compute units 512 tiles of 16 KB just fill PRAC_PART32_BYTES.
int wgrad_f32_splits(int n_cu, int64_t N, int64_t m, int c) {
  const int64_t tiles = (int64_t)((c + 63) / 64) * ((m + 63) / 64);
  const int64_t fit = (int64_t)(PRAC_PART32_BYTES / ((size_t)c * m * sizeof(float)));
  return (int)std::max<int64_t>(1, std::min<int64_t>({2 * n_cu / tiles, N / 256, 32, fit}));
}

int weight_grad_generic(prac_ctx* ctx, char* ws, float* part32, const void* C, const void* dY, prac_dtype dt, int64_t N, int64_t m,
                        int64_t ldc, bool packed, int64_t lddy, const float* P, int64_t d, int64_t ldp, int k, int r,
                        float scale, void* dW, prac_dtype odt, int64_t lddw, float beta) {
  const int c = k + r;
  const WgradGenPlan q = plan_wgrad_generic(N, m, c, packed);
  int splits = 1;
  int rc;
  const void* Crm = C;
  int64_t ldcrm = ldc;
  if (packed) {
    rc = launch_unpack_c(ctx, reinterpret_cast<const bf16_t*>(C), (int)N, c, reinterpret_cast<bf16_t*>(ws + q.o_crm), c);
    if (rc) return rc;
    Crm = ws + q.o_crm;
    ldcrm = c;
  }
  float* T = reinterpret_cast<float*>(ws + q.o_t);
  GemmGenArgs g{};
  g.A = Crm; g.adt = dt; g.a_rs = 1; g.a_cs = ldcrm;
  g.B = dY; g.bdt = dt; g.b_rs = lddy; g.b_cs = 1;
  g.M = c; g.N = (int)m; g.K = N; g.k_stride = 1;
  g.out = T; g.ldo = m; g.alpha = 1.f; g.beta = 0.f; g.acc64 = false; g.out64 = nullptr;
  if (gemm_f32_takes(g)) {
    splits = wgrad_f32_splits(ctx->n_cu, N, m, c);
    if (splits > 1) T = part32;
    g.slabs = T;
    rc = launch_gemm_f32(ctx, g, splits);
  } else {
    rc = launch_gemm_generic(ctx, g);
  }
  if (rc) return rc;
  return launch_f32_sum_pt(ctx, P, ldp, T, splits, c, k, scale, (int)d, (int)m, dW, lddw, odt == PRAC_BF16, beta);
}

// What prac_weight_grad_static has for scratch.  It and prac_weight_grad run the same plan, so a single gradient takes more token
// ranges than one round of workgroups, or the wide form of its last product, only where that fits.
constexpr size_t WGRAD_ROOM = PRAC_STATIC_SCRATCH_BYTES - PRAC_SYNC_BYTES;

// Token ranges of C^T dY.  As many as one round of workgroups holds (one per compute unit), or more of them (that `fits` accepts) in
// several rounds where the cost rule favours that: a round costs its start (6 us) and 15.6 ns per token of a range (a k-block of 16 takes
// 0.25 us; with the 128-row tiles of c <= 128 11.5 ns), a range a write and a read of its partial sums (3 TB/s).  Where the column tiles do not divide the compute
// units, several short rounds fill them better than one long one.  Measured, one round against the rule's choice, per
// weight gradient: 86 tiles, N = 32768, c = 256 (up and gate) 2 ranges 294 us, 5 ranges 282; 172 tiles, N = 16384, c = 512 one
// range 307, 4 ranges 295 (90 MB of partial sums, past what a single gradient may use); the rule keeps 16, 5, 4 and 6 ranges for
// 16, 48, 64 and 40 tiles (next best 3 to 30 us worse).
struct WgradWork {
  int64_t tiles = 0, slab = 0;  // 256 x 128 tiles of T, bytes of one set of partial sums
  double token_us;              // of equal ranges; unequal ones always have 256-row tiles
  WgradWork(int c, int n_out, const int64_t* m) : token_us(c <= 128 ? 0.0115 : 0.0156) {
    for (int h = 0; h < n_out; ++h) {
      tiles += (int64_t)((c + 255) / 256) * ((m[h] + 127) / 128);
      slab += (int64_t)c * m[h] * 4;
    }
  }
  double equal_us(int n_cu, int64_t N, int s) const {
    return (double)((tiles * s + n_cu - 1) / n_cu) * (6.0 + token_us * (double)((N + s - 1) / s)) + (double)(2 * slab) * s / 3e6;
  }
};
template <typename Fits>
int wgrad_splits(int n_cu, int tune_splits, int c, int n_out, const int64_t* m, int64_t N, Fits fits) {
  if (tune_splits > 0) return tune_splits;
  const WgradWork w(c, n_out, m);
  const int most = (int)std::max<int64_t>(1, std::min<int64_t>(64, N / 256));
  int best = (int)std::max<int64_t>(1, std::min<int64_t>(most, n_cu / w.tiles));
  for (int s = best + 1; s <= most; ++s)
    if (w.equal_us(n_cu, N, s) < w.equal_us(n_cu, N, best) && fits(s)) best = s;
  return best;
}

// Unequal token ranges in one round (see CtdyTails) where they are at least 3 % and 2.5 us cheaper than `splits` equal ones (96
// tiles of 33 units, c = 44: 1.9 us cheaper by the estimate, 58.4 us against 56.1 with the rest of the call).  A helper's next
// piece costs it what 3 units cost (its stores and its first tile), so main ranges are the shortest that no helper exceeds.
// Measured, equal ranges against these, C^T dY alone and the whole weight gradient: 86 tiles of
// 256 units (up and gate) 5 ranges in two rounds 237 / 320 us, unequal 217 / 292; 172 tiles of 128 units (LLaMA-7B up projection)
// one range 226 / 319, unequal 183 / 282.  Pieces priced at 0, 8 and 16 units instead: 228, 220 and 225 us on the former's
// C^T dY, 200, 193 and 203 on the latter's (190 with 3, in the same run).
// Their partial sums are whole blocks of 256 (or c) x 128, however little of a tile T fills, so scratch bounds them too: where the
// blocks of the main ranges take more than 5/4 of what the equal ranges' sums do (m far below 128, c just above 256: up to 20 times),
// ranges stay equal (whole weight gradient, unequal against equal: N = 337601, d = 6638, c = 737, m = 24 133 / 123 us with 34 against
// 5 MB; 25102, 570, 283, 3324 101.5 / 105 with 29 against 17 MB).  Then one tile's blocks at a time, the least a call with a fixed scratch can do, are always the smaller of the two.
CtdyTails wgrad_tails(int n_cu, int c, int n_out, const int64_t* m, int64_t N, int splits) {
  const WgradWork w(c, n_out, m);
  const int64_t units = (N + 127) / 128;
  CtdyTails t;
  t.main = (int)(n_cu / w.tiles);
  const int64_t idle = n_cu - t.main * w.tiles;
  t.block_rows = std::min(c, 256);
  if (t.main < 1 || idle < 1 || 4 * t.main * w.tiles * t.block_rows * 128 * (int64_t)sizeof(float) > 5 * splits * w.slab) return {};
  for (int64_t len = (w.tiles * units + n_cu - 1) / n_cu; len * t.main < units; ++len) {
    const int64_t tail = units - len * t.main, run = (w.tiles * tail + idle - 1) / idle;
    const int64_t pieces = (run + tail - 2) / tail + 1;
    if (run + 3 * (pieces - 1) > len) continue;
    t.len = (int)len;
    t.tail = (int)tail;
    t.run = (int)run;
    t.helpers = (int)((w.tiles * tail + run - 1) / run);
    t.t1 = (int)w.tiles;
    const double us = 6.0 + 0.0156 * 128.0 * (double)len +
                      (double)(2 * w.slab) * ((double)t.main + 1.0 + (double)t.helpers / (double)w.tiles) / 3e6;
    const double equal = w.equal_us(n_cu, N, splits);
    return us < 0.97 * equal && us < equal - 2.5 ? t : CtdyTails{};
  }
  return {};
}

// bf16 gradients whose rows start on any element: the token-split partial sums of C^T dY come from the streaming kernel
// (bf16 products are exact in fp32, so this is the strided kernel's sum in another order), the rest stays in fp32 as
// for all data that runs the strided kernels.
struct WgradAnyPlan {
  int splits, group;  // token ranges; ranges whose rows of a row-major C are packed at a time
  size_t o_part[PRAC_CTDY_MAX_OUT], o_cpk, bytes;
};
WgradAnyPlan layout_wgrad_any(int64_t N, int c, int n_out, const int64_t* m, int splits, int group, bool packed) {
  WgradAnyPlan q{};
  q.splits = splits;
  q.group = group;
  WsPlan plan;
  for (int h = 0; h < n_out; ++h) q.o_part[h] = plan.take((size_t)splits * c * m[h] * sizeof(float));
  q.o_cpk = plan.take(packed ? 0 : packed_c_bytes(std::min(N, group * ctdy_range_tokens(N, splits)), c));
  q.bytes = plan.off;
  return q;
}
// Within `room` bytes where it can be: the ranges, and with them the bits of dW, do not depend on it.
WgradAnyPlan plan_wgrad_any(int n_cu, int tune_splits, int64_t N, int c, int n_out, const int64_t* m, bool packed,
                            size_t room = ~(size_t)0) {
  int splits = wgrad_splits(n_cu, tune_splits, c, n_out, m, N, [&](int s) {
    return n_out > 1 || layout_wgrad_any(N, c, n_out, m, s, 1, false).bytes <= WGRAD_ROOM;
  });
  const int64_t tok = ctdy_range_tokens(N, splits);
  splits = (int)((N + tok - 1) / tok);  // no empty ranges
  int group = splits;
  while (group > 1 && layout_wgrad_any(N, c, n_out, m, splits, group, packed).bytes > room) --group;
  return layout_wgrad_any(N, c, n_out, m, splits, group, packed);
}

int weight_grad_any(prac_ctx* ctx, char* ws, const WgradAnyPlan& q, const void* C, int64_t N, int64_t ldc, bool packed,
                    int n_out, const void* const* dY, const int64_t* m, const int64_t* lddy, const float* P, int64_t d,
                    int64_t ldp, int k, int r, float scale, void* const* dW, prac_dtype odt, const int64_t* lddw,
                    float beta) {
  const int c = k + r;
  const int64_t tok = ctdy_range_tokens(N, q.splits);
  int rc;
  float* part[PRAC_CTDY_MAX_OUT];
  int mi[PRAC_CTDY_MAX_OUT];
  for (int h = 0; h < n_out; ++h) {
    part[h] = reinterpret_cast<float*>(ws + q.o_part[h]);
    mi[h] = (int)m[h];
  }
  for (int s0 = 0; s0 < q.splits; s0 += q.group) {  // (once, unless the packed copy of C has to fit the static block)
    const int ranges = std::min(q.group, q.splits - s0);
    const int64_t t0 = s0 * tok, n = std::min(N - t0, ranges * tok);
    const bf16_t* Cpk = reinterpret_cast<const bf16_t*>(C);
    if (!packed) {
      rc = launch_pack_c(ctx, Cpk + t0 * ldc, ldc, (int)n, c, reinterpret_cast<bf16_t*>(ws + q.o_cpk));
      if (rc) return rc;
      Cpk = reinterpret_cast<const bf16_t*>(ws + q.o_cpk);
    }
    const bf16_t* dYp[PRAC_CTDY_MAX_OUT];
    float* slabs[PRAC_CTDY_MAX_OUT];
    for (int h = 0; h < n_out; ++h) {
      dYp[h] = reinterpret_cast<const bf16_t*>(dY[h]) + t0 * lddy[h];
      slabs[h] = part[h] + (size_t)s0 * c * m[h];
    }
    ProfScope ps(ctx, PRAC_KERNEL_CT_DY);
    rc = launch_ctdy_ws(ctx, Cpk, c, (int)n, n_out, dYp, lddy, mi, slabs, ranges, true, (int)tok);
    if (rc) return rc;
  }
  for (int h = 0; h < n_out; ++h) {
    rc = launch_f32_sum_pt(ctx, P, ldp, part[h], q.splits, c, k, scale, (int)d, mi[h], dW[h], lddw[h], odt == PRAC_BF16,
                           beta);
    if (rc) return rc;
  }
  return PRAC_OK;
}

// n_out gradients from one C on the bf16 kernels: one launch forms the token-split slabs of every
// C^T dY_h, then each output gets its slab reduction and its dW_h = P T_h.
struct WgradPlan {
  int splits;
  bool fused;  // one launch (see launch_wgrad_fused) instead of three
  bool wide;   // dW = P T by launch_wide_ws
  CtdyTails tails;  // unequal token ranges (main > 0), else `splits` equal ones
  int tiles;   // unequal ranges: tiles of T formed at a time (all, unless the partial sums have to fit the static block)
  int sld[PRAC_CTDY_MAX_OUT];  // row pitch of the partial sums: whole quads, so that they move 16 bytes at a time at any width
  int nkb;     // 16-row k-blocks of T
  int nmb[PRAC_CTDY_MAX_OUT];
  size_t o_part[PRAC_CTDY_MAX_OUT], o_blocks, o_tails, o_t[PRAC_CTDY_MAX_OUT], o_lp, o_cpk, bytes;
  size_t equal_bytes;  // what equal ranges with tight partial sums would take: decides what the static entry point refuses
};
// dW = P T by the kernel that walks column groups (launch_wide_ws) or by the tiled ones (launch_pt): the former for bf16
// results that overwrite dW, 128 < c <= 256 and more tiles of 128 x 256 than compute units.  Measured, tiled against
// walking: d = 2048, c = 256, columns 3 x 2048 15.6 / 14.5 us, 8192 19.8 / 15.3, 2 x 5461 61.9 / 23.5 (dW rows on any element;
// the tiled kernels then stored single elements); d = 8000, m = 8000, c = 200 the whole step 147.5 / 134.7; with half a
// k-tile, d = 2048, m = 6144, c = 64, 8.7 / 10.6.
bool wgrad_wide(int n_cu, int64_t d, int c, int n_out, const int64_t* m, prac_dtype odt, float beta) {
  if (odt != PRAC_BF16 || beta != 0.f || wide_kblocks(c) != 16) return false;
  int64_t groups = 0;
  for (int h = 0; h < n_out; ++h) groups += (m[h] + 255) / 256;
  return (d + 127) / 128 * groups > n_cu;
}
// Equal ranges: partial sums in rows of m (tight) or of whole quads.  Unequal ones: the blocks of `tiles` tiles at a time; those of
// the tails are here only if `own_tails`, otherwise in the ctx's block for them (PRAC_TAIL_BYTES).
WgradPlan layout_wgrad_fast(int64_t N, int64_t d, int c, int n_out, const int64_t* m, int splits, bool packed, bool has_lp, bool wide,
                            bool tight, const CtdyTails& tails = {}, int tiles = 0, bool own_tails = false) {
  WgradPlan q{};
  const LpLayout l = lp_layout(d, c);
  q.splits = splits;
  q.tails = tails;
  q.tiles = tiles;
  q.wide = wide;
  q.nkb = wide ? wide_kblocks(c) : l.nckb;
  WsPlan plan;
  for (int h = 0; h < n_out; ++h) {
    q.nmb[h] = (int)round_up64((m[h] + 31) / 32, wide ? 8 : 4);  // 32-column blocks of T, whole 256- or 128-column tiles
    q.sld[h] = (int)(tight ? m[h] : round_up64(m[h], 4));
    q.o_part[h] = plan.take(tails.main > 0 ? 0 : (size_t)splits * c * q.sld[h] * sizeof(float));
    q.o_t[h] = plan.take((size_t)q.nkb * q.nmb[h] * 64 * 8 * sizeof(bf16_t));
  }
  if (tails.main > 0) {
    const size_t block = (size_t)tails.block_rows * 128 * sizeof(float);
    size_t tail_blocks = 0;
    for (int t = 0; t < tails.t1; t += tiles)
      tail_blocks = std::max<size_t>(tail_blocks, ctdy_tail_blocks(tails, t, std::min(tails.t1, t + tiles)));
    q.o_blocks = plan.take(tails.main * tiles * block);
    q.o_tails = plan.take(own_tails ? tail_blocks * block : 0);
  }
  q.o_lp = plan.take(has_lp ? 0 : l.bytes);
  q.o_cpk = plan.take(packed ? 0 : packed_c_bytes(N, c));
  q.bytes = plan.off;
  return q;
}
// (whether C is packed and P_lp at hand does not change the ranges, and with them the bits of dW; nor does `room`, which is what a
// call has that brings all of its scratch (0: as much as it asks for, and the ctx's block for the tails))
WgradPlan plan_wgrad_fast(int n_cu, int tune_splits, bool one_launch, int64_t N, int64_t d, int c, int n_out, const int64_t* m,
                          prac_dtype odt, float beta, bool packed, bool has_lp, size_t room = 0) {
  const int splits = wgrad_splits(n_cu, tune_splits, c, n_out, m, N, [&](int s) {
    return n_out > 1 || layout_wgrad_fast(N, d, c, n_out, m, s, false, false, wide_kblocks(c) == 16, true).bytes <= WGRAD_ROOM;
  });
  const CtdyTails tails = tune_splits > 0 ? CtdyTails{} : wgrad_tails(n_cu, c, n_out, m, N, splits);
  WgradPlan tight = layout_wgrad_fast(N, d, c, n_out, m, splits, packed, has_lp, false, true);
  tight.equal_bytes = tight.bytes;
  if (tails.main == 0 && one_launch && wgrad_fused_takes(n_cu, c, n_out, m, splits)) {
    tight.fused = true;
    return tight;
  }
  if (wgrad_wide(n_cu, d, c, n_out, m, odt, beta)) {
    WgradPlan w = layout_wgrad_fast(N, d, c, n_out, m, splits, packed, has_lp, true, true);
    w.equal_bytes = w.bytes;
    if (n_out > 1 || w.bytes <= WGRAD_ROOM || tight.bytes > WGRAD_ROOM) tight = w;
  }
  WgradPlan q;
  if (tails.main > 0) {
    int tiles = tails.t1;
    do q = layout_wgrad_fast(N, d, c, n_out, m, splits, packed, has_lp, tight.wide, false, tails, tiles, room > 0);
    while (room > 0 && q.bytes > room && --tiles > 0);
  } else {
    q = layout_wgrad_fast(N, d, c, n_out, m, splits, packed, has_lp, tight.wide, false);
    if (room > 0 && q.bytes > room) q = tight;
  }
  q.equal_bytes = tight.bytes;
  return q;
}

int weight_grad_fast(prac_ctx* ctx, char* ws, int* cnt, float* tail_blocks, const WgradPlan& q, const void* C, int64_t N, int64_t ldc, bool packed,
                     int n_out, const void* const* dY, const int64_t* m, const int64_t* lddy, const float* P,
                     const void* P_lp, int64_t d, int64_t ldp, int k, int r, float scale, void* const* dW,
                     prac_dtype odt, const int64_t* lddw, float beta) {
  const int c = k + r;
  const LpLayout l = lp_layout(d, c);
  const int splits = q.splits;
  int rc;
  const char* lp = reinterpret_cast<const char*>(P_lp);
  if (!lp) {
    rc = prac_pack_basis(ctx, P, d, ldp, c, ws + q.o_lp);
    if (rc) return rc;
    lp = ws + q.o_lp;
  }
  if (small_wgrad_takes(ctx->n_cu, N, d, c, n_out, m) && (packed || (aligned16(C) && ldc % 8 == 0)) && ctx->tune_splits == 0) {
    // (whatever the other tuning keys say: this form sums in another order than the kernels that they choose among)
    const bf16_t* y[PRAC_CTDY_MAX_OUT];
    int cols[PRAC_CTDY_MAX_OUT];
    for (int h = 0; h < n_out; ++h) {
      y[h] = reinterpret_cast<const bf16_t*>(dY[h]);
      cols[h] = (int)m[h];
    }
    ProfScope ps(ctx, PRAC_KERNEL_WEIGHT_GRAD);
    return launch_small_wgrad(ctx, reinterpret_cast<const bf16_t*>(C), ldc, packed, (int)N, c, k, scale, n_out, y, lddy, cols,
                              reinterpret_cast<const bf16_t*>(lp + l.off_pa), l.nckb, (int)d, dW, lddw, odt == PRAC_BF16, beta);
  }
  const bf16_t* Cpk = reinterpret_cast<const bf16_t*>(C);
  if (!packed) {
    rc = launch_pack_c(ctx, reinterpret_cast<const bf16_t*>(C), ldc, (int)N, c, reinterpret_cast<bf16_t*>(ws + q.o_cpk));
    if (rc) return rc;
    Cpk = reinterpret_cast<const bf16_t*>(ws + q.o_cpk);
  }
  const bf16_t* dYp[PRAC_CTDY_MAX_OUT];
  float* part[PRAC_CTDY_MAX_OUT];
  int mi[PRAC_CTDY_MAX_OUT];
  for (int h = 0; h < n_out; ++h) {
    dYp[h] = reinterpret_cast<const bf16_t*>(dY[h]);
    part[h] = reinterpret_cast<float*>(ws + q.o_part[h]);
    mi[h] = (int)m[h];
  }
  bf16_t* Tf[PRAC_CTDY_MAX_OUT];
  for (int h = 0; h < n_out; ++h) Tf[h] = reinterpret_cast<bf16_t*>(ws + q.o_t[h]);
  if (q.fused) {
    // one launch: slabs, their sum T (bf16, fragment order, random rows scaled) and dW_h = P T_h
    ProfScope ps(ctx, PRAC_KERNEL_WEIGHT_GRAD);
    return launch_wgrad_fused(ctx, Cpk, c, (int)N, n_out, dYp, lddy, mi, part, splits, k, scale, l.nckb, q.nmb, Tf,
                              reinterpret_cast<const bf16_t*>(lp + l.off_pa), (int)d, dW, lddw, odt == PRAC_BF16, beta,
                              cnt);
  }
  CtdyTails tails = q.tails;
  if (tails.main > 0) {
    tails.blocks = reinterpret_cast<float*>(ws + q.o_blocks);
    tails.tail_blocks = tail_blocks ? tail_blocks : reinterpret_cast<float*>(ws + q.o_tails);
  }
  auto ct_dy = [&] {  // T_h = C^T dY_h as partial sums over token ranges
    ProfScope ps(ctx, PRAC_KERNEL_CT_DY);
    return launch_ctdy_ws(ctx, Cpk, c, (int)N, n_out, dYp, lddy, mi, part, splits, false, 0, q.sld, &tails);
  };
  auto reduce = [&] {  // T_h in fragment order (bf16): partial sums added up, random rows weighted by the scaling factor
    ProfScope ps(ctx, PRAC_KERNEL_T_REDUCE);
    return launch_reduce_to_tfrag(ctx, n_out, part, splits, c, mi, k, scale, q.nkb, q.nmb, Tf, q.sld, tails);
  };
  // Slab sum, scaling factor and dW_h = P T_h in one launch where that is the faster form: measured on an
  // MI355X it is for c > 256 (rank 512 + 512 at d = m = 2048: 159 against 179 us per weight gradient), where
  // the two launches move a large T through memory and run the LDS-staged product; at c <= 256 the two
  // small launches overlap each other's start and end and win (61.6 against 66.8 us at the same d, m).
  // (every 512 rows of dW are one more workgroup per column block that repeats the slab sum: at d = 11008,
  // 22 of them, the one launch takes 180 us against 98 us for the two, so it is limited to d <= 2048)
  const bool tail_one = ctx->tune_tail == 2 || (ctx->tune_tail == 0 && l.nckb > 16 && d <= 2048);  // (never with q.wide: c > 256)
  if (tail_one && tails.main == 0 && sum_pt_eligible(n_out, mi, splits)) {
    rc = ct_dy();
    if (rc) return rc;
    ProfScope ps(ctx, PRAC_KERNEL_SUM_P_T);
    return launch_sum_pt(ctx, reinterpret_cast<const bf16_t*>(lp + l.off_pa), n_out, part, splits, c, k, scale, l.nckb,
                         (int)d, mi, dW, lddw, odt == PRAC_BF16, beta);
  }
  const int all = q.tails.t1;  // (equal ranges: 0)
  for (int t = 0; t == 0 || t < all; t += q.tiles) {
    tails.t0 = t;
    tails.t1 = std::min(all, t + q.tiles);
    rc = ct_dy();
    if (rc) return rc;
    rc = reduce();
    if (rc) return rc;
    if (tails.main == 0) break;
  }
  {
    ProfScope ps(ctx, PRAC_KERNEL_P_T);  // dW_h = P T_h, all outputs in one launch
    if (q.wide) {
      bf16_t* out[PRAC_CTDY_MAX_OUT];
      for (int h = 0; h < n_out; ++h) out[h] = reinterpret_cast<bf16_t*>(dW[h]);
      return launch_wide_ws(ctx, false, reinterpret_cast<const bf16_t*>(lp + l.off_pn), l.ldpn, false, (int)d, c, q.nkb, n_out,
                            Tf, q.nmb, mi, out, lddw);
    }
    rc = launch_pt(ctx, reinterpret_cast<const bf16_t*>(lp + l.off_pa), n_out, Tf, (int)d, mi, l.nckb, q.nmb, dW, lddw,
                   odt == PRAC_BF16, beta);
  }
  if (rc) return rc;
  return PRAC_OK;
}

// Argument checks of the weight-gradient entry points (no ctx needed).
int wgrad_check(const void* C, prac_dtype dt, int64_t N, int64_t ldc, int c_layout, int n_out, const void* const* dY,
                const int64_t* m, const int64_t* lddy, const float* P, const void* P_lp, int64_t d, int64_t ldp, int k,
                int r, void* const* dW, prac_dtype odt, const int64_t* lddw) {
  if (!C || !dY || !m || !lddy || !dW || !lddw || !P || n_out < 1 || n_out > PRAC_MAX_SHARED || !valid_dtype(dt) ||
      !valid_dtype(odt) || bad_tokens(N) || d < 1 || d > (1 << 20) || k < 0 || r < 0 || k + r < 1 || (int64_t)k + r > d ||
      (c_layout != PRAC_C_PACKED && (c_layout != PRAC_C_ROWMAJOR || ldc < k + r)) || ldp < k + r ||
      (P_lp && !aligned16(P_lp)))
    return PRAC_EINVAL;
  for (int h = 0; h < n_out; ++h)
    if (!dY[h] || !dW[h] || m[h] < 1 || m[h] > (1 << 20) || lddy[h] < m[h] || lddw[h] < m[h]) return PRAC_EINVAL;
  return PRAC_OK;
}
bool wgrad_is_any(prac_dtype dt, int n_out, const int64_t* m, const int64_t* lddy) {
  bool any = true;
  for (int h = 0; h < n_out; ++h) any = any && stream_any(dt, m[h], lddy[h]);
  return any;
}
bool wgrad_is_fast(prac_dtype dt, int64_t N, int n_out, const void* const* dY, const int64_t* lddy) {
  bool fast = dt == PRAC_BF16 && N < ((int64_t)1 << 31);
  for (int h = 0; h < n_out; ++h)
    fast = fast && aligned16(dY[h]) && lddy[h] % 8 == 0 && lddy[h] <= PRAC_MAX_STREAM_PITCH;
  return fast;
}

}  // namespace

extern "C" {

int prac_weight_grad(prac_ctx* ctx, const void* C, const void* dY, prac_dtype dt, int64_t N, int64_t m, int64_t ldc,
                     int c_layout, int64_t lddy, const float* P, const void* P_lp, int64_t d, int64_t ldp, int k,
                     int r, float scale, void* dW, prac_dtype odt, int64_t lddw, float beta) {
  return prac_weight_grad_shared(ctx, C, dt, N, ldc, c_layout, 1, &dY, &m, &lddy, P, P_lp, d, ldp, k, r, scale, &dW, odt,
                                 &lddw, beta);
}

int prac_weight_grad_static(prac_ctx* ctx, const void* C, const void* dY, prac_dtype dt, int64_t N, int64_t m,
                            int64_t ldc, int c_layout, int64_t lddy, const float* P, const void* P_lp, int64_t d,
                            int64_t ldp, int k, int r, float scale, void* dW, prac_dtype odt, int64_t lddw, float beta) {
  int rc = wgrad_check(C, dt, N, ldc, c_layout, 1, &dY, &m, &lddy, P, P_lp, d, ldp, k, r, &dW, odt, &lddw);
  if (rc) return rc;
  if (!ctx) return PRAC_ENOCTX;
  const bool packed = c_layout == PRAC_C_PACKED;
  if (packed && (dt != PRAC_BF16 || !aligned16(C))) return PRAC_EUNSUPPORTED;
  const bool fast = wgrad_is_fast(dt, N, 1, &dY, &lddy);
  WgradPlan q{};
  WgradAnyPlan qa{};
  bool any = !fast && wgrad_is_any(dt, 1, &m, &lddy);
  size_t need, o_part32 = 0;
  if (any) {
    qa = plan_wgrad_any(ctx->n_cu, ctx->tune_splits, N, k + r, 1, &m, packed, WGRAD_ROOM);
    any = qa.bytes <= WGRAD_ROOM;  // else the strided kernels, which need less scratch
  }
  if (any) {
    need = qa.bytes;
  } else if (fast) {
    q = plan_wgrad_fast(ctx->n_cu, ctx->tune_splits, ctx->tune_one_launch != 0, N, d, k + r, 1, &m, odt, beta, packed,
                        P_lp != nullptr, WGRAD_ROOM);
    need = std::max(q.bytes, q.equal_bytes);
  } else {
    need = o_part32 = plan_wgrad_generic(N, m, k + r, packed).bytes;
    if (dt == PRAC_F32 && wgrad_f32_splits(ctx->n_cu, N, m, k + r) > 1) need += PRAC_PART32_BYTES;
  }
  // the first 128 KB of the block are the counters of the one-launch weight gradient (zero when the code
  // object is loaded, and every launch leaves them zero)
  constexpr size_t kSync = PRAC_SYNC_BYTES;
  if (need > WGRAD_ROOM) return PRAC_ETOOBIG;
  // no event pairs here (creating one allocates): this call is not profiled
  const int prof = ctx->prof_kind;
  ctx->prof_kind = PRAC_KERNEL_NONE;
  char* ws = ctx->static_scratch + kSync;
  if (fast)
    rc = weight_grad_fast(ctx, ws, reinterpret_cast<int*>(ctx->static_scratch), nullptr, q, C, N, ldc, packed, 1, &dY, &m, &lddy, P, P_lp, d, ldp, k, r, scale, &dW, odt, &lddw,
                          beta);
  else if (any)
    rc = weight_grad_any(ctx, ws, qa, C, N, ldc, packed, 1, &dY, &m, &lddy, P, d, ldp, k, r, scale, &dW, odt, &lddw, beta);
  else
    rc = weight_grad_generic(ctx, ws, reinterpret_cast<float*>(ws + o_part32), C, dY, dt, N, m, ldc, packed, lddy, P, d, ldp,
                             k, r, scale, dW, odt, lddw, beta);
  ctx->prof_kind = prof;
  return rc;
}

int prac_weight_grad_shared(prac_ctx* ctx, const void* C, prac_dtype dt, int64_t N, int64_t ldc, int c_layout, int n_out,
                            const void* const* dY, const int64_t* m, const int64_t* lddy, const float* P,
                            const void* P_lp, int64_t d, int64_t ldp, int k, int r, float scale, void* const* dW,
                            prac_dtype odt, const int64_t* lddw, float beta) {
  int rc = wgrad_check(C, dt, N, ldc, c_layout, n_out, dY, m, lddy, P, P_lp, d, ldp, k, r, dW, odt, lddw);
  if (rc) return rc;
  if (!ctx) return PRAC_ENOCTX;
  const bool packed = c_layout == PRAC_C_PACKED;
  if (packed && (dt != PRAC_BF16 || !aligned16(C))) return PRAC_EUNSUPPORTED;
  if (wgrad_is_fast(dt, N, n_out, dY, lddy)) {
    const WgradPlan q = plan_wgrad_fast(ctx->n_cu, ctx->tune_splits, ctx->tune_one_launch != 0, N, d, k + r, n_out, m, odt, beta,
                                        packed, P_lp != nullptr);
    rc = prac_ws_reserve(ctx, q.bytes);
    if (rc) return rc;
    return weight_grad_fast(ctx, ctx->ws, ctx->d_sync, ctx->tails, q, C, N, ldc, packed, n_out, dY, m, lddy, P, P_lp, d, ldp, k, r, scale, dW, odt,
                            lddw, beta);
  }
  if (wgrad_is_any(dt, n_out, m, lddy)) {
    const WgradAnyPlan q = plan_wgrad_any(ctx->n_cu, ctx->tune_splits, N, k + r, n_out, m, packed);
    rc = prac_ws_reserve(ctx, q.bytes);
    if (rc) return rc;
    return weight_grad_any(ctx, ctx->ws, q, C, N, ldc, packed, n_out, dY, m, lddy, P, d, ldp, k, r, scale, dW, odt, lddw,
                           beta);
  }
  size_t need = 0;
  for (int h = 0; h < n_out; ++h) need = std::max(need, plan_wgrad_generic(N, m[h], k + r, packed).bytes);
  rc = prac_ws_reserve(ctx, need);
  if (rc) return rc;
  for (int h = 0; h < n_out; ++h) {
    rc = weight_grad_generic(ctx, ctx->ws, ctx->part32, C, dY[h], dt, N, m[h], ldc, packed, lddy[h], P, d, ldp, k, r, scale,
                             dW[h], odt, lddw[h], beta);
    if (rc) return rc;
  }
  return PRAC_OK;
}

}  // extern "C"

// ------------------------------------------------------------------ reconstruction
namespace {
struct ReconPlan {
  bool fast, direct;
  int nkb, ncb;
  int64_t ldcrm;
  size_t o_pt, o_c, o_tmp, o_crm, bytes;
};
ReconPlan plan_reconstruct(bool fast, prac_dtype dt, int64_t N, int64_t d, int c, bool packed, int64_t ldc) {
  ReconPlan q{};
  q.fast = fast;
  WsPlan plan;
  if (fast) {
    q.direct = wide_kblocks(c) > 0;  // the dedicated kernel reads packed C itself
    q.nkb = q.direct ? wide_kblocks(c) : (int)(round_up64(c, 256) / 16);
    q.ncb = (int)round_up64((d + 31) / 32, 8);
    q.ldcrm = packed ? round_up64(c, 8) : ldc;
    q.o_pt = plan.take((size_t)q.nkb * q.ncb * 64 * 8 * sizeof(bf16_t));
    q.o_c = plan.take(packed && !q.direct ? (size_t)N * q.ldcrm * sizeof(bf16_t) : 0);
  } else {
    q.o_tmp = plan.take(dt == PRAC_BF16 ? (size_t)N * d * sizeof(float) : 0);
    q.o_crm = plan.take(packed ? (size_t)N * c * sizeof(bf16_t) : 0);
  }
  q.bytes = plan.off;
  return q;
}
}  // namespace

int prac_reconstruct(prac_ctx* ctx, const void* C, prac_dtype dt, int64_t N, int64_t ldc, int c_layout, const float* P,
                     int64_t d, int64_t ldp, int k, int r, float scale, void* Xh, int64_t ldxh) {
  if (!C || !P || !Xh || !valid_dtype(dt) || bad_tokens(N) || d < 1 || d > (1 << 20) || k < 0 || r < 0 || k + r < 1 ||
      (int64_t)k + r > d || bad_c_layout(c_layout, ldc, k + r) || ldp < k + r || ldxh < d)
    return PRAC_EINVAL;
  if (!ctx) return PRAC_ENOCTX;
  const int c = k + r;
  const bool packed = c_layout == PRAC_C_PACKED;
  if (packed && (dt != PRAC_BF16 || !aligned16(C))) return PRAC_EUNSUPPORTED;
  const bool rm_ok = !packed && aligned16(C) && ldc % 8 == 0 && ldc <= PRAC_MAX_STREAM_PITCH;
  const bool fast = dt == PRAC_BF16 && (packed || rm_ok) && N < ((int64_t)1 << 31);
  const ReconPlan q = plan_reconstruct(fast, dt, N, d, c, packed, ldc);
  if (q.bytes) {
    int rc = prac_ws_reserve(ctx, q.bytes);
    if (rc) return rc;
  }
  if (fast) {
    // Xh = C Ps^T is the forward-output launch of the compress kernel with C in the role of X
    // (its "feature" dimension is c) and Ps^T in the role of W.
    const int nkb = q.nkb, ncb = q.ncb;
    const int64_t ldcrm = q.ldcrm;
    bf16_t* Pt = reinterpret_cast<bf16_t*>(ctx->ws + q.o_pt);
    int rc = launch_pack_ptfrag(ctx, P, d, ldp, c, k, scale, nkb, ncb, Pt);
    if (rc) return rc;
    if (q.direct) {
      ProfScope ps(ctx, PRAC_KERNEL_RECONSTRUCT);
      const int cols = (int)d;
      bf16_t* const out = reinterpret_cast<bf16_t*>(Xh);
      return launch_wide_ws(ctx, true, reinterpret_cast<const bf16_t*>(C), ldc, packed, (int)N, c, nkb, 1, &Pt, &ncb, &cols,
                            &out, &ldxh);
    }
    const bf16_t* Crm = reinterpret_cast<const bf16_t*>(C);
    if (packed) {
      rc = launch_unpack_c(ctx, reinterpret_cast<const bf16_t*>(C), (int)N, c, reinterpret_cast<bf16_t*>(ctx->ws + q.o_c),
                           ldcrm);
      if (rc) return rc;
      Crm = reinterpret_cast<const bf16_t*>(ctx->ws + q.o_c);
    }
    ProfScope ps(ctx, PRAC_KERNEL_RECONSTRUCT);
    return launch_compress_ws(ctx, Crm, ldcrm, (int)N, c, nullptr, 0, 0, nullptr, 0, false, Pt, ncb, (int)d,
                              reinterpret_cast<bf16_t*>(Xh), ldxh, false, ctx->tails);
  }
  // fp32 path: Xh = C1 Q1^T, then Xh += scale C2 Q2^T (a scaled copy of P would make it one product, but fp32 data needs no
  // scratch here)
  const bool need_tmp = dt == PRAC_BF16;
  const void* Crm = C;
  int64_t ldcrm = ldc;
  if (packed) {
    int rc = launch_unpack_c(ctx, reinterpret_cast<const bf16_t*>(C), (int)N, c,
                             reinterpret_cast<bf16_t*>(ctx->ws + q.o_crm), c);
    if (rc) return rc;
    Crm = ctx->ws + q.o_crm;
    ldcrm = c;
  }
  float* out = need_tmp ? reinterpret_cast<float*>(ctx->ws + q.o_tmp) : reinterpret_cast<float*>(Xh);
  bool first = true;
  for (int part = 0; part < 2; ++part) {
    const int k0 = part == 0 ? 0 : k, kn = part == 0 ? k : r;
    if (kn == 0) continue;
    GemmGenArgs g{};
    g.A = reinterpret_cast<const char*>(Crm) + (size_t)k0 * esize(dt); g.adt = dt; g.a_rs = ldcrm; g.a_cs = 1;
    g.B = P + k0; g.bdt = PRAC_F32; g.b_rs = 1; g.b_cs = ldp;  // B(kk, n) = P[n][k0 + kk]
    g.M = (int)N; g.N = (int)d; g.K = kn; g.k_stride = 1;
    g.out = out; g.ldo = need_tmp ? d : ldxh; g.acc64 = false; g.out64 = nullptr;
    g.alpha = part == 0 ? 1.f : scale;
    g.beta = first ? 0.f : 1.f;
    first = false;
    int rc = launch_gemm_generic(ctx, g);
    if (rc) return rc;
  }
  if (need_tmp) return launch_cast_out(ctx, out, d, Xh, PRAC_BF16, ldxh, (int)N, (int)d, 0.f);
  return PRAC_OK;
}

// ------------------------------------------------------------------ scratch sizing
extern "C" {

size_t prac_workspace_bytes(const prac_ctx* ctx, const prac_call_shape* sh) {
  const size_t bad = ~(size_t)0;
  if (!sh || !valid_dtype(sh->dt) || sh->N < 1 || sh->N >= ((int64_t)1 << 31) || sh->d < 1 || sh->d > (1 << 20) ||
      sh->k < 0 || sh->r < 0 || (int64_t)sh->k + sh->r > sh->d)
    return bad;
  const int n_cu = ctx ? ctx->n_cu : 256;
  const int tune = ctx ? ctx->tune_splits : 0;
  const prac_dtype dt = (prac_dtype)sh->dt;
  const int c = sh->k + sh->r;
  const bool fast = dt == PRAC_BF16 && !sh->generic;
  const bool packed = sh->c_layout == PRAC_C_PACKED;
  // where a plan looks at alignment, an unaligned pointer stands for rows that start on any element
  const void* xptr = sh->generic ? reinterpret_cast<const void*>(uintptr_t(2)) : nullptr;
  const int64_t ldq = sh->generic ? sh->d : round_up64(sh->d, 8);  // row pitch the plan assumes for X
  switch (sh->op) {
    case PRAC_OP_GRAM:
      return gram_scratch_bytes(n_cu, xptr, dt, sh->N, sh->d, ldq, sh->fit.row_stride > 0 ? sh->fit.row_stride : 1, sh->d);
    case PRAC_OP_FIT_BASIS: {
      if (c < 1) return bad;
      prac_fit_opts o = sh->fit;
      if (o.iters == 0) o.iters = 8;
      if (o.row_stride == 0) o.row_stride = 1;
      size_t b = fit_scratch_bytes(n_cu, xptr, dt, sh->N, sh->d, ldq, sh->k, sh->r, sh->refresh, o);
      return b;  // the packed copy goes to the caller's P_lp, not to scratch
    }
    case PRAC_OP_COMPRESS:
    case PRAC_OP_FUSED_FWD: {
      if (c < 1) return bad;
      const bool fused = sh->op == PRAC_OP_FUSED_FWD;
      if (fused && (sh->n_out != 1 || sh->m[0] < 1)) return bad;
      const int64_t m = fused ? sh->m[0] : 0;
      size_t need = plan_compress(fast ? CompressPath::STREAM : CompressPath::STRIDED, fused, packed, sh->have_p_lp != 0, dt,
                                  sh->N, sh->d, c, m).bytes;
      if (!fast && stream_any(dt, sh->d, sh->d))  // the shape does not say the pitch: enough for either path
        need = std::max(need, plan_compress(CompressPath::STREAM_ANY, fused, packed, sh->have_p_lp != 0, dt, sh->N, sh->d, c,
                                            m).bytes);
      return need;
    }
    case PRAC_OP_WEIGHT_GRAD: {
      if (c < 1 || sh->n_out < 1 || sh->n_out > PRAC_MAX_SHARED) return bad;
      for (int h = 0; h < sh->n_out; ++h)
        if (sh->m[h] < 1 || sh->m[h] > (1 << 20)) return bad;
      if (fast) {  // beta is not part of the shape: enough for either form of the last product
        size_t need = 0;
        for (float beta : {0.f, 1.f})
        {
          const WgradPlan q = plan_wgrad_fast(n_cu, tune, ctx && ctx->tune_one_launch, sh->N, sh->d, c, sh->n_out, sh->m,
                                              (prac_dtype)sh->odt, beta, packed, sh->have_p_lp != 0);
          need = std::max(need, std::max(q.bytes, q.tails.main > 0 ? q.equal_bytes : 0));
        }
        return need;
      }
      size_t need = 0;
      if (wgrad_is_any(dt, sh->n_out, sh->m, sh->m))
        need = plan_wgrad_any(n_cu, tune, sh->N, c, sh->n_out, sh->m, packed).bytes;
      for (int h = 0; h < sh->n_out; ++h)
        need = std::max(need, plan_wgrad_generic(sh->N, sh->m[h], c, packed).bytes);
      return need;
    }
    case PRAC_OP_RECONSTRUCT:
      if (c < 1) return bad;
      return plan_reconstruct(fast, dt, sh->N, sh->d, c, packed, c).bytes;
    default:
      return bad;
  }
}

int prac_reserve_workspace(prac_ctx* ctx, size_t bytes) {
  if (bytes == ~(size_t)0) return PRAC_EINVAL;
  if (!ctx) return PRAC_ENOCTX;
  return prac_ws_reserve(ctx, bytes);
}

int prac_debug_gram_rows(const void* X, int dt, int64_t N, int64_t d, int64_t ldx, int64_t row_stride) {
  if (!X || !valid_dtype(dt) || bad_tokens(N) || d < 1 || ldx < d || row_stride < 1) return -1;
  return (int)gram_rows(X, (prac_dtype)dt, (N + row_stride - 1) / row_stride, d, ldx, row_stride);
}

int prac_debug_f32_tile(int M, int N, int64_t K, int splits, int a_k_fast) {
  if (M < 2 || N < 2 || K < 1 || splits < 1 || a_k_fast < 0 || a_k_fast > 1) return -1;
  return (int)f32_tile(256, M, N, K, splits, a_k_fast != 0);
}

int64_t prac_debug_fit_slab_margin(const prac_call_shape* sh) {
  if (!sh) return -1;
  prac_fit_opts o = sh->fit;
  if (o.iters == 0) o.iters = 8;
  if (o.row_stride == 0) o.row_stride = 1;
  return fit_slab_margin(256, (prac_dtype)sh->dt, sh->N, sh->d, sh->k, sh->r, sh->refresh, o);
}

}  // extern "C"
