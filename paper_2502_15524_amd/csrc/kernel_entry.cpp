// Single-kernel entry points (include/hs_kernel.h).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <mutex>
#include <string>
#include <utility>
#include <vector>

#include "../../include/hs_kernel.h"
#include "hs_host.h"
#include "hs_kernels.h"
#include "kernel_entry.h"

using namespace hs;

namespace {
// Workspaces of hs_k_gemm's split tiles, allocated per device on first use and
// kept until the process ends. Calls of more than 64 rows on one device must not
// overlap. Calls of 17 to 64 rows have a workspace of their own (an 128 x 64
// partial tile per workgroup), whose launches are put one after the other by an
// event: calls of that size may come from several streams and threads.
struct GemmWs {
  float* part = nullptr;
  uint32_t* flags = nullptr;
  hipEvent_t done = nullptr;  // small: after the last launch that used it
  bool used = false;
};
constexpr int64_t kWsPartFloats = 256ll * 256 * 128;  // a 256 x 128 partial tile per workgroup
constexpr int64_t kWsSmallFloats = 256ll * 128 * 64;
constexpr int64_t kWsFlags = 256;
std::mutex g_gemm_mu;  // both workspaces, and a small call's wait, launch and record

// (with g_gemm_mu held)
hs_status gemm_ws(bool small, GemmWs** out) {
  static GemmWs ws[2][64];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64)
    return fail(HS_EHIP, "hipGetDevice failed");
  GemmWs& w = ws[small][dev];
  if (!w.part) {
    float* p = nullptr;
    uint32_t* f = nullptr;
    hipEvent_t ev = nullptr;
    const int64_t floats = small ? kWsSmallFloats : kWsPartFloats;
    if (hipMalloc(&p, floats * sizeof(float)) != hipSuccess) return fail(HS_ENOMEM, "gemm workspace");
    if (hipMalloc(&f, kWsFlags * sizeof(uint32_t)) != hipSuccess ||
        hipMemset(f, 0, kWsFlags * sizeof(uint32_t)) != hipSuccess ||
        hipDeviceSynchronize() != hipSuccess ||
        (small && hipEventCreateWithFlags(&ev, hipEventDisableTiming) != hipSuccess)) {
      (void)hipFree(p);
      if (f) (void)hipFree(f);
      return fail(HS_ENOMEM, "gemm workspace");
    }
    w.part = p;
    w.flags = f;
    w.done = ev;
  }
  *out = &w;
  return HS_OK;
}

hs_status launched(hipError_t e, const char* what) {
  if (e == hipErrorInvalidValue) return fail(HS_EINVAL, std::string(what) + ": unsupported shape");
  if (e != hipSuccess) return fail(HS_EHIP, std::string(what) + ": " + hipGetErrorString(e));
  return HS_OK;
}
}  // namespace

hs_status gemm_call(GemmArgs a, int32_t epi, void* stream) {
  hipStream_t s = static_cast<hipStream_t>(stream);
  if (a.M <= 16) return launched(gemm(a, epi, s, nullptr), "gemm");  // no workspace
  const bool small = a.M <= 64;
  std::unique_lock<std::mutex> lock(g_gemm_mu);
  GemmWs* ws = nullptr;
  const hs_status r = gemm_ws(small, &ws);
  if (r != HS_OK) return r;
  a.part = ws->part;
  a.part_floats = small ? kWsSmallFloats : kWsPartFloats;
  a.flags = ws->flags;
  a.flags_n = kWsFlags;
  if (!small) {
    lock.unlock();
    return launched(gemm(a, epi, s, nullptr), "gemm");
  }
  // (a captured launch cannot wait for work outside its graph: the caller
  // orders the graph's replays)
  hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
  hipError_t e = hipStreamIsCapturing(s, &cap);
  const bool ordered = cap == hipStreamCaptureStatusNone;
  if (e == hipSuccess && ordered && ws->used) e = hipStreamWaitEvent(s, ws->done, 0);
  LaunchInfo info{"", 0, 0};
  if (e == hipSuccess) e = gemm(a, epi, s, &info);
  if (e == hipSuccess && ordered && info.split) {
    ws->used = true;
    e = hipEventRecord(ws->done, s);
  }
  return launched(e, "gemm");
}

extern "C" hs_status hs_k_gemm(const void* X, int64_t ldx, const void* Wt, void* Y, int64_t ldy,
                               const void* R, int64_t ldr, int32_t M, int32_t N, int32_t K,
                               int32_t epi, void* stream) {
  try {
    if (!X || !Wt || !Y) return fail(HS_EINVAL, "null operand");
    GemmArgs a{static_cast<const bf16_t*>(X), ldx, static_cast<const bf16_t*>(Wt), Y, ldy,
               static_cast<const bf16_t*>(R), ldr, M, N, K};
    return gemm_call(a, epi, stream);
  } catch (...) {
    return fail(HS_EINVAL, "unexpected internal error");
  }
}

extern "C" hs_status hs_k_gemm_rmsnorm(const void* X, int64_t ldx, const void* g, float eps,
                                       const void* Wt, void* Y, int64_t ldy, const void* R,
                                       int64_t ldr, int32_t M, int32_t N, int32_t K, int32_t epi,
                                       void* stream) {
  try {
    if (!X || !g || !Wt || !Y) return fail(HS_EINVAL, "null operand");
    if (M < 1 || M > 16 || K % 64) return fail(HS_EINVAL, "needs 1 <= M <= 16 and K % 64 == 0");
    GemmArgs a{static_cast<const bf16_t*>(X), ldx, static_cast<const bf16_t*>(Wt), Y, ldy,
               static_cast<const bf16_t*>(R), ldr, M, N, K};
    a.norm_gain = static_cast<const bf16_t*>(g);
    a.norm_eps = eps;
    return gemm_call(a, epi, stream);
  } catch (...) {
    return fail(HS_EINVAL, "unexpected internal error");
  }
}

namespace {
// Sequence offsets and tiles of hs_k_attn_prefill: pinned memory the host
// writes and its device copy, pulled by a kernel. A call takes a pair for its
// duration: it gives the pair back only after a successful wait for its work.
// Up to four idle pairs per device, of at most 256 KiB each, are kept for later
// calls, in place of an allocation, two copies and a free in every call.
struct MetaBuf {
  int32_t *h = nullptr, *d = nullptr;
  size_t cap = 0;
  int dev = -1;
};
constexpr size_t kMetaMin = 1 << 12, kMetaKeep = 1 << 16, kMetaIdle = 4;
std::mutex g_meta_mu;
std::vector<MetaBuf> g_meta_idle[64];

void meta_free(const MetaBuf& m) {
  if (m.h) (void)hipHostFree(m.h);
  if (m.d) (void)hipFree(m.d);
}

bool meta_take(size_t n, MetaBuf* out) {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return false;
  {
    std::lock_guard<std::mutex> lock(g_meta_mu);
    auto& idle = g_meta_idle[dev];
    for (size_t i = 0; i < idle.size(); ++i)
      if (idle[i].cap >= n) {
        *out = idle[i];
        idle.erase(idle.begin() + i);
        return true;
      }
  }
  MetaBuf m;
  m.cap = std::max(n, kMetaMin);
  m.dev = dev;
  if (hipHostMalloc(reinterpret_cast<void**>(&m.h), m.cap * 4, hipHostMallocCoherent) != hipSuccess ||
      hipMalloc(reinterpret_cast<void**>(&m.d), m.cap * 4) != hipSuccess) {
    meta_free(m);
    return false;
  }
  *out = m;
  return true;
}

void meta_give(MetaBuf m) {
  if (m.cap <= kMetaKeep) {
    std::lock_guard<std::mutex> lock(g_meta_mu);
    auto& idle = g_meta_idle[m.dev];
    if (idle.size() < kMetaIdle) {
      idle.push_back(m);
      return;
    }
    for (auto& o : idle)
      if (o.cap < m.cap) {  // a smaller one makes room
        std::swap(o, m);
        break;
      }
  }
  meta_free(m);  // waits for the device: not with the mutex held
}
}  // namespace

extern "C" hs_status hs_k_attn_prefill(const void* qkv, void* out, const int32_t* cu, int32_t n,
                                       int32_t n_heads, int32_t n_kv_heads, int32_t head_dim,
                                       void* stream) {
  try {
    if (!qkv || !out || !cu || n < 1) return fail(HS_EINVAL, "bad arguments");
    if (n_kv_heads < 1 || n_heads % n_kv_heads) return fail(HS_EINVAL, "bad head counts");
    if (cu[0] != 0) return fail(HS_EINVAL, "cu_seqlens[0] must be 0");
    std::vector<int32_t> tiles;
    int64_t tiles64 = 0;
    int longest = 0;
    for (int i = 0; i < n; ++i) {
      const int len = cu[i + 1] - cu[i];
      if (len < 1) return fail(HS_EINVAL, "sequence lengths must be >= 1");
      tiles64 += (len + 63) / 64;
      longest = std::max(longest, len);
    }
    const int q_tile = attn_prefill_q_tile(tiles64, longest, n_heads);
    // longest rows first, as the stage orders them
    std::vector<std::pair<int32_t, int32_t>> order;
    for (int i = 0; i < n; ++i)
      for (int q = 0; q < cu[i + 1] - cu[i]; q += q_tile) order.emplace_back(-q, i);
    std::sort(order.begin(), order.end());
    for (const auto& t : order) {
      tiles.push_back(t.second);
      tiles.push_back(-t.first);
    }
    hipStream_t s = static_cast<hipStream_t>(stream);
    const size_t cu_n = ((size_t)n + 1 + 3) / 4 * 4, need = (cu_n + tiles.size() + 3) / 4 * 4;
    MetaBuf m;
    if (!meta_take(need, &m)) return fail(HS_ENOMEM, "metadata allocation failed");
    std::copy(cu, cu + n + 1, m.h);
    std::copy(tiles.begin(), tiles.end(), m.h + cu_n);
    const int ld = (n_heads + 2 * n_kv_heads) * head_dim;
    AttnPrefillArgs a{static_cast<const bf16_t*>(qkv), ld, static_cast<bf16_t*>(out),
                      n_heads * head_dim, m.d, m.d + cu_n, (int)(tiles.size() / 2), n_heads,
                      n_kv_heads, head_dim, q_tile, 0.0};
    hipError_t e = meta_pull(m.h, m.d, (int64_t)need, s);
    if (e == hipSuccess) e = attn_prefill(a, s, nullptr);
    const hipError_t es = hipStreamSynchronize(s);
    if (e == hipSuccess) e = es;
    // after a failed wait the queued work may still read the pair: it is left
    // allocated, to no other call
    if (es == hipSuccess) meta_give(m);
    return launched(e, "attn_prefill");
  } catch (...) {
    return fail(HS_EINVAL, "unexpected internal error");
  }
}

namespace {
// Split partials of hs_k_attn_decode, one buffer per device, grown on demand.
struct DecodeWs {
  float* buf = nullptr;
  int64_t floats = 0;
};
}  // namespace

int64_t hs::attn_decode_ws_floats(int32_t B, int32_t n_heads, int32_t head_dim, int32_t max_ctx) {
  if (B < 1 || n_heads < 1 || head_dim < 1 || max_ctx < 1) return 0;
  const int64_t max_splits = (max_ctx + kDecodeSplit - 1) / kDecodeSplit;
  return (int64_t)B * n_heads * max_splits * (head_dim + 2);
}

hs_status hs::attn_decode_check(const void* q, const void* pool, const int32_t* block_table,
                            const int32_t* ctx, const void* out, bool rope, const float* cos_t,
                            const float* sin_t, int32_t max_pos, int32_t B, int32_t n_heads,
                            int32_t n_kv_heads, int32_t max_blocks, int32_t max_ctx) {
  if (!q || !pool || !block_table || !ctx || !out || B < 1 || max_ctx < 1)
    return fail(HS_EINVAL, "bad arguments");
  if (n_kv_heads < 1 || n_heads < 1 || n_heads % n_kv_heads)
    return fail(HS_EINVAL, "bad head counts");
  if (max_blocks < (max_ctx + 15) / 16) return fail(HS_EINVAL, "block table too narrow");
  if (rope && (!cos_t || !sin_t || max_pos < max_ctx))
    return fail(HS_EINVAL, "RoPE tables missing or shorter than max_ctx");
  return HS_OK;
}

hs_status hs::attn_decode_run(const void* q, int64_t ldq, const void* pool, bf16_t* pool_w,
                          const int32_t* block_table, const int32_t* ctx, const float* cos_t,
                          const float* sin_t, int32_t max_pos, void* out, int64_t ldo, int32_t B,
                          int32_t n_heads, int32_t n_kv_heads, int32_t head_dim,
                          int32_t max_blocks, int32_t max_ctx, float* ws, void* stream) {
  const int max_splits = (max_ctx + kDecodeSplit - 1) / kDecodeSplit;
  AttnDecodeArgs a{static_cast<const bf16_t*>(q), ldq, static_cast<const bf16_t*>(pool),
                   block_table, ctx, ws, ws + (int64_t)B * n_heads * max_splits * head_dim,
                   static_cast<bf16_t*>(out), ldo, B, n_heads, n_kv_heads, head_dim, max_blocks,
                   max_splits, max_splits, 0.0};
  a.pool_w = pool_w;
  a.cos_t = cos_t;
  a.sin_t = sin_t;
  a.max_pos = max_pos;
  return launched(attn_decode(a, static_cast<hipStream_t>(stream), nullptr), "attn_decode");
}

namespace {
hs_status attn_decode_entry(const void* q, int64_t ldq, const void* pool, bf16_t* pool_w,
                            const int32_t* block_table, const int32_t* ctx, const float* cos_t,
                            const float* sin_t, int32_t max_pos, void* out, int64_t ldo,
                            int32_t B, int32_t n_heads, int32_t n_kv_heads, int32_t head_dim,
                            int32_t max_blocks, int32_t max_ctx, void* stream) {
  const hs_status chk = attn_decode_check(q, pool, block_table, ctx, out, pool_w != nullptr,
                                          cos_t, sin_t, max_pos, B, n_heads, n_kv_heads,
                                          max_blocks, max_ctx);
  if (chk != HS_OK) return chk;
  static DecodeWs ws[64];
  int dev = 0;
  const hipError_t ge = hipGetDevice(&dev);
  if (ge != hipSuccess || dev < 0 || dev >= 64)
    return fail(HS_EHIP, std::string("hipGetDevice: ") + hipGetErrorString(ge));
  const int64_t need = attn_decode_ws_floats(B, n_heads, head_dim, max_ctx);
  DecodeWs& w = ws[dev];
  if (w.floats < need) {
    if (w.buf) {
      (void)hipDeviceSynchronize();
      (void)hipFree(w.buf);
      w.buf = nullptr;
      w.floats = 0;
    }
    if (hipMalloc(reinterpret_cast<void**>(&w.buf), need * sizeof(float)) != hipSuccess)
      return fail(HS_ENOMEM, "attention workspace");
    w.floats = need;
  }
  return attn_decode_run(q, ldq, pool, pool_w, block_table, ctx, cos_t, sin_t, max_pos, out, ldo,
                         B, n_heads, n_kv_heads, head_dim, max_blocks, max_ctx, w.buf, stream);
}
}  // namespace

extern "C" hs_status hs_k_attn_decode(const void* q, int64_t ldq, const void* pool,
                                      const int32_t* block_table, const int32_t* ctx, void* out,
                                      int64_t ldo, int32_t B, int32_t n_heads, int32_t n_kv_heads,
                                      int32_t head_dim, int32_t max_blocks, int32_t max_ctx,
                                      void* stream) {
  try {
    return attn_decode_entry(q, ldq, pool, nullptr, block_table, ctx, nullptr, nullptr, 0, out,
                             ldo, B, n_heads, n_kv_heads, head_dim, max_blocks, max_ctx, stream);
  } catch (...) {
    return fail(HS_EINVAL, "unexpected internal error");
  }
}

extern "C" hs_status hs_k_attn_decode_rope(const void* qkv, int64_t ldqkv, void* pool,
                                           const int32_t* block_table, const int32_t* ctx,
                                           const float* cos_t, const float* sin_t,
                                           int32_t max_pos, void* out, int64_t ldo, int32_t B,
                                           int32_t n_heads, int32_t n_kv_heads, int32_t head_dim,
                                           int32_t max_blocks, int32_t max_ctx, void* stream) {
  try {
    if (!pool) return fail(HS_EINVAL, "bad arguments");
    if (ldqkv < (int64_t)(n_heads + 2 * n_kv_heads) * head_dim)
      return fail(HS_EINVAL, "qkv rows narrower than the query, key and value heads");
    return attn_decode_entry(qkv, ldqkv, pool, static_cast<bf16_t*>(pool), block_table, ctx,
                             cos_t, sin_t, max_pos, out, ldo, B, n_heads, n_kv_heads, head_dim,
                             max_blocks, max_ctx, stream);
  } catch (...) {
    return fail(HS_EINVAL, "unexpected internal error");
  }
}

extern "C" hs_status hs_k_argmax(const float* logits, int32_t n_rows, int32_t n_cols,
                                 int32_t* out, void* stream) {
  try {
    if (!logits || !out || n_rows < 1 || n_cols < 1 || n_cols % 4)
      return fail(HS_EINVAL, "needs logits, out, n_rows >= 1 and n_cols % 4 == 0");
    hipStream_t s = static_cast<hipStream_t>(stream);
    int32_t* part = nullptr;
    const size_t nb = (size_t)n_rows * argmax_chunks(n_cols) * 2 * sizeof(int32_t);
    if (hipMalloc(reinterpret_cast<void**>(&part), nb) != hipSuccess)
      return fail(HS_ENOMEM, "device allocation failed");
    hipError_t e = argmax_rows(logits, n_rows, n_cols, part, out, s, nullptr);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    (void)hipFree(part);
    return launched(e, "argmax");
  } catch (...) {
    return fail(HS_EINVAL, "unexpected internal error");
  }
}

extern "C" hs_status hs_k_rmsnorm(const void* x, const void* g, void* out, int32_t rows,
                                  int32_t hidden, float eps, void* stream) {
  try {
    if (!x || !g || !out || rows < 1) return fail(HS_EINVAL, "bad arguments");
    return launched(rmsnorm(static_cast<const bf16_t*>(x), hidden, nullptr, rows, hidden,
                            static_cast<const bf16_t*>(g), eps, static_cast<bf16_t*>(out), hidden,
                            static_cast<hipStream_t>(stream), nullptr),
                    "rmsnorm");
  } catch (...) {
    return fail(HS_EINVAL, "unexpected internal error");
  }
}
