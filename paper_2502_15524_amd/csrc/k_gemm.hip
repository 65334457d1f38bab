// bf16 GEMMs Y[m][n] = sum_k X[m][k] * W[n][k] on gfx950 MFMA with fused
// epilogues (residual add, SwiGLU, fp32 logits).
//
// Both operands are K-contiguous ([out][in] weights, token-major
// activations), so every MFMA operand fragment is one 16-byte load. The MFMA
// "A" operand is the weight tile (output features on MFMA rows) and "B" the
// activation tile (tokens on MFMA columns); each lane therefore ends up with
// 4 consecutive output features of one token and stores them as one 8-byte
// write.
//
// The weight matrix W [N][K] is stored in the tiled matrix format (1 KiB
// blocks of 8 rows x 64 k, chunk c of row r at position c ^ r, 64-column slabs
// contiguous), so both kernels read weights in long contiguous runs.
//
// Two kernels:
//  * gemm_ring   - prefill: BN x BM x 64 tiles copied straight into an LDS ring
//                  of NS stages, 8 waves, 16x16x32 bf16 MFMA, XCD-aware order;
//                  256-token tiles run a ping-pong main loop.
//  * gemm_skinny - decode (M <= 16 tokens; up to 64 of a small matrix, 16 to a
//                  workgroup): HBM-bound weight streaming, 2 to
//                  16 waves split K inside a workgroup, reduced through LDS in
//                  a fixed order (deterministic).
#include "hs_device.h"
#include "hs_kernels.h"

#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <algorithm>

#include <string>
#include <type_traits>

namespace hs {

// ---------------------------------------------------------------- epilogue

// Output column (head order) of column n of a QKV projection whose q and k
// rows are stored head-interleaved: inside a head, the 32-row group p holds
// rows 16p .. 16p + 15 of the first half, then the same rows of the second.
__device__ __forceinline__ int qk_col(const GemmArgs& a, int n) {
  if (n >= a.rope_q_cols + a.rope_kv_cols) return n;
  const int d = n & (a.rope_d - 1);
  return (n - d) + ((d >> 4) & 1) * (a.rope_d >> 1) + (d >> 5) * 16 + (d & 15);
}

// bytes from X to the end of its last row's k range, whatever the row stride
// (rows may overlap or repeat: ldx below K)
__device__ __forceinline__ uint64_t x_bytes(const GemmArgs& a, int kp) {
  return ((uint64_t)(a.M - 1) * a.ldx + kp) * 2;
}

template <int EPI>
__device__ __forceinline__ void store4(const GemmArgs& a, int m, int f, const f32x4_v& v) {
  if (m >= a.M || f >= a.N) return;
  if constexpr (EPI == EPI_STORE) f = qk_col(a, f);
  if constexpr (EPI == EPI_F32) {
    float4 o = make_float4(v[0], v[1], v[2], v[3]);
    *reinterpret_cast<float4*>(static_cast<float*>(a.Y) + (int64_t)m * a.ldy + f) = o;
  } else {
    float r0 = v[0], r1 = v[1], r2 = v[2], r3 = v[3];
    if constexpr (EPI == EPI_RESID) {
      const uint2 rr = *reinterpret_cast<const uint2*>(a.R + (int64_t)m * a.ldr + f);
      r0 += lo_bf(rr.x); r1 += hi_bf(rr.x); r2 += lo_bf(rr.y); r3 += hi_bf(rr.y);
    }
    uint2 o;
    o.x = pack2bf(r0, r1);
    o.y = pack2bf(r2, r3);
    *reinterpret_cast<uint2*>(static_cast<bf16_t*>(a.Y) + (int64_t)m * a.ldy + f) = o;
  }
}

// gate tile g and up tile u hold the same 16 FFN columns; f is the output
// column (FFN index) of the lane's first value.
__device__ __forceinline__ void store_swiglu(const GemmArgs& a, int m, int f, const f32x4_v& g,
                                             const f32x4_v& u) {
  if (m >= a.M || f >= (a.N >> 1)) return;
  uint2 o;
  o.x = pack2bf(silu_f(g[0]) * u[0], silu_f(g[1]) * u[1]);
  o.y = pack2bf(silu_f(g[2]) * u[2], silu_f(g[3]) * u[3]);
  *reinterpret_cast<uint2*>(static_cast<bf16_t*>(a.Y) + (int64_t)m * a.ldy + f) = o;
}

// QKV projection with RoPE and KV append. n is the (stored-order) column of
// x1's first value, a multiple of 4 inside the first 16 rows of a 32-row
// pair; x2 holds the pair's other 16 rows. In the q and k heads these are
// RoPE partners (rotation index i and i + D/2); in the v heads two adjacent
// 16-column groups. Values are rounded to bf16 before the rotation, as a
// separate rotation pass reading the stored projection would see them.

// rotation index of column n (< rope_q_cols + rope_kv_cols) and its table offset
__device__ __forceinline__ int64_t rope_tab_off(const GemmArgs& a, int pos, int n) {
  const int d = n & (a.rope_d - 1);
  return (int64_t)pos * (a.rope_d >> 1) + (d >> 5) * 16 + (d & 15);
}

// cv, sv: cos and sin at rope_tab_off(a, pos, n) (unused for v columns)
__device__ __forceinline__ void store_qkv_rope(const GemmArgs& a, int m, int slot, int n,
                                               const f32x4_v& x1, const f32x4_v& x2,
                                               const float4& cv, const float4& sv) {
  if (m >= a.M || n >= a.N) return;
  const int D = a.rope_d, half = D >> 1;
  uint2 o1, o2;
  o1.x = pack2bf(x1[0], x1[1]);
  o1.y = pack2bf(x1[2], x1[3]);
  o2.x = pack2bf(x2[0], x2[1]);
  o2.y = pack2bf(x2[2], x2[3]);
  int c1, c2;  // output columns of x1 and x2
  if (n < a.rope_q_cols + a.rope_kv_cols) {
    const int d = n & (D - 1);
    c1 = (n - d) + (d >> 5) * 16 + (d & 15);
    c2 = c1 + half;
    const float cc[4] = {cv.x, cv.y, cv.z, cv.w}, ss[4] = {sv.x, sv.y, sv.z, sv.w};
    const float p1[4] = {lo_bf(o1.x), hi_bf(o1.x), lo_bf(o1.y), hi_bf(o1.y)};
    const float p2[4] = {lo_bf(o2.x), hi_bf(o2.x), lo_bf(o2.y), hi_bf(o2.y)};
    float y1[4], y2[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      y1[e] = rope_first(p1[e], p2[e], cc[e], ss[e]);
      y2[e] = rope_second(p1[e], p2[e], cc[e], ss[e]);
    }
    o1 = make_uint2(pack2bf(y1[0], y1[1]), pack2bf(y1[2], y1[3]));
    o2 = make_uint2(pack2bf(y2[0], y2[1]), pack2bf(y2[2], y2[3]));
  } else {
    c1 = n;
    c2 = n + 16;
  }
  bf16_t* row = static_cast<bf16_t*>(a.Y) + (int64_t)m * a.ldy;
  *reinterpret_cast<uint2*>(row + c1) = o1;
  *reinterpret_cast<uint2*>(row + c2) = o2;
  if (slot >= 0 && n >= a.rope_q_cols) {
    // k head kh -> pool part 0, v head kh -> part 1 of the token's block
    const int n_kv = a.rope_kv_cols / D;
    const int kv = c1 - a.rope_q_cols;  // column inside the k (then v) heads
    const int kh = kv / D;              // 0 .. 2 n_kv - 1: k heads, then v heads
    bf16_t* dst = a.rope_pool + (int64_t)(slot >> 4) * 2 * n_kv * 16 * D +
                  ((int64_t)kh * 16 + (slot & 15)) * D + (kv - kh * D);
    *reinterpret_cast<uint2*>(dst) = o1;
    *reinterpret_cast<uint2*>(dst + (c2 - c1)) = o2;
  }
}

// ------------------------------------ tiled, buffer loads into an LDS ring
//
// Operand tiles go global -> LDS with buffer_load_dwordx4 ... lds (no register
// staging): one instruction moves 64 lanes x 16 B of one operand into 1 KiB of
// LDS, lane L landing at byte 16 L (8 rows x 64 k). A weight block of the
// tiled format is exactly one such instruction (its chunks are already in the
// LDS order), and consecutive row blocks of one 64-k slab are adjacent in
// memory. Activations are row-major. A lane's address is one 32-bit offset, the
// per-instruction and per-k-step parts are scalar. LDS rows are unpadded; the
// 16-byte chunks of a row are XOR-swizzled by the row index so the 16 rows of
// an MFMA fragment read hit different banks. NS stages form a ring: the
// loads for tile k + NS - 1 are in flight while tile k is multiplied, and a
// wave waits only for tile k + 1 before the workgroup barrier. The copies are
// issued from inline assembly so that the compiler neither tracks them nor
// inserts waits for them; this code waits explicitly (vmcnt) before each
// barrier. K is processed in 64-column slabs; when K % 64 != 0 the activation
// columns up to the next multiple of 64 must be zero (the weights are).

template <int N>
__device__ __forceinline__ void wait_vm() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  asm volatile("s_waitcnt vmcnt(%0)" :: "n"(N) : "memory");
}

// the same, and every LDS read of this wave is complete
template <int N>
__device__ __forceinline__ void wait_vm_lds() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" :: "n"(N) : "memory");
}

__device__ __forceinline__ void wg_barrier() { asm volatile("s_barrier" ::: "memory"); }

// Eight waves per workgroup, two per SIMD, as 2 x 4: two wave columns over the
// BN weight rows, four wave rows over the BM tokens.
constexpr int kRingWaves = 8;
template <int BN, int BM, int BK, int NS>
struct RTile {
  static constexpr int NW = kRingWaves;
  static constexpr int CPR = BK / 8;           // 16-byte chunks per row
  static constexpr int RPI = 64 / CPR;         // rows per load instruction
  static constexpr int WN = BN / 2, WM = BM / (NW / 2), TN = WN / 16, TM = WM / 16;
  static constexpr int WI = BN / NW / RPI, XI = BM / NW / RPI;  // instructions per wave
  static constexpr int LPS = WI + XI;          // loads per stage per wave
  static constexpr int W_BYTES = BN * BK * 2;
  static_assert(BK == 64, "weights come in 64-column slabs");
  static_assert(WI >= 1 && XI >= 1 && TM >= 1, "tile too small for the waves");
};

// position of chunk c of row r inside its row of eight
__device__ __forceinline__ int chunk_pos(int r, int c) { return c ^ (r & 7); }

// Multiply one stage (BK/32 steps of 32 k). Fragment reads are software
// pipelined against the MFMAs and the order is pinned with scheduling group
// barriers: the A fragment of row tile i + PD is read while the TM MFMAs of
// row tile i run, and the B fragments of the next 32-k step are read with the
// first A fragment that needs them. The last row tile of a stage is deferred
// past the workgroup barrier: it runs while the next stage's first fragments
// come from LDS. Its operands have to be in registers by that barrier, after
// which any wave may refill the stage: the wave waits for its reads (lgkmcnt)
// together with its copies.
__device__ __forceinline__ bf16x8_v lds_frag(const bf16_t* s, int r, int c) {
  return as_bf16x8(ld16(s + (r * 8 + chunk_pos(r, c)) * 8));
}

// How many row tiles ahead of its MFMAs a wave reads the A fragments: three
// for the 4- and 6-row-tile wave tiles (128 x 128 and 192 x 128 tiles;
// 512-token 7B shapes, MI355X: QKV 55.8 -> 53.8 us, o 29.3 -> 28.2), one for
// the 8-row-tile ones of 256-row tiles. The fragments and MFMAs are the same
// either way.
template <int TN>
constexpr int ring_pd() {
  return (TN == 4 || TN == 6) ? 3 : 1;
}

template <int BN, int BM, int BK, int NS, int TN, int TM, int PD, typename Dma>
__device__ __forceinline__ void ring_stage(f32x4_v (&acc)[TN][TM], bf16x8_v (&a)[PD + 1],
                                           bf16x8_v (&b)[2][TM], const bf16_t* sw,
                                           const bf16_t* sx, int wn, int wm, int fr, int g,
                                           bool pending, Dma&& dma) {
  using T = RTile<BN, BM, BK, NS>;
  constexpr int KS = BK / 32, NT = TN * KS;
  constexpr int MASK_MFMA = 0x008, MASK_DS_READ = 0x100;
  // row tile t of the stage (t = ks TN + i) uses A slot t mod (PD + 1); the
  // deferred last one must not share a slot with the next stage's first PD
  static_assert(KS == 2 && NT % (PD + 1) == 0, "A fragment slots");
  constexpr int LAST = (NT - 1) % (PD + 1);
  auto read_a = [&](int t) {
    a[t % (PD + 1)] = lds_frag(sw, wn * T::WN + (t % TN) * 16 + fr, (t / TN) * 4 + g);
  };
#pragma unroll
  for (int j = 0; j < TM; ++j) b[0][j] = lds_frag(sx, wm * T::WM + j * 16 + fr, g);
#pragma unroll
  for (int t = 0; t < PD; ++t) read_a(t);
  __builtin_amdgcn_sched_group_barrier(MASK_DS_READ, TM + PD, 0);
  // the previous stage's last row tile (operands in registers) runs while
  // this stage's first fragments are on their way from LDS
  if (pending) {
#pragma unroll
    for (int j = 0; j < TM; ++j)
      acc[TN - 1][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[LAST], b[1][j], acc[TN - 1][j], 0, 0, 0);
    __builtin_amdgcn_sched_group_barrier(MASK_MFMA, TM, 0);
  }
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    const int ks = t / TN, i = t % TN;
    dma(t);
    // A of row tile t + PD; the B fragments of the next 32-k step together
    // with the A fragment that first needs them
    const bool ra = t + PD < NT, rb = ks + 1 < KS && i == TN - PD;
    if (ra) read_a(t + PD);
    if (rb) {
#pragma unroll
      for (int j = 0; j < TM; ++j)
        b[(ks + 1) & 1][j] = lds_frag(sx, wm * T::WM + j * 16 + fr, (ks + 1) * 4 + g);
    }
    if (t == NT - 1) break;  // deferred to the next stage (or the end)
#pragma unroll
    for (int j = 0; j < TM; ++j)
      acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[t % (PD + 1)], b[ks & 1][j], acc[i][j], 0, 0, 0);
    if (ra && rb) __builtin_amdgcn_sched_group_barrier(MASK_DS_READ, TM + 1, 0);
    else if (ra) __builtin_amdgcn_sched_group_barrier(MASK_DS_READ, 1, 0);
    else if (rb) __builtin_amdgcn_sched_group_barrier(MASK_DS_READ, TM, 0);
    __builtin_amdgcn_sched_group_barrier(MASK_MFMA, TM, 0);
  }
}

// Tile schedule. Output tiles are numbered in groups of `group_n` column
// tiles (weight rows) by all row tiles (tokens), column tile fastest, so the
// workgroups that run together on one XCD share weight and activation slabs
// in its L2. A data-parallel launch (split = 1) runs one whole tile per
// workgroup. A split launch gives every tile `split` consecutive workgroups,
// each an equal contiguous share of its 64-k slabs; the one that arrives last
// finishes the tile: every contributor stores its fp32 partial tile, then
// bumps the tile's arrival counter, and the one that completes the count adds
// the partials in k order (so the result does not depend on the arrival
// order), applies the epilogue and sets the counter back to zero. No
// workgroup waits for another. (Equal shares of the whole (tile, slab) space
// instead, with two segments and two partial tiles for most workgroups, were
// 5-25 % slower wherever the chip holds two or more workgroups a tile: 40
// tokens x 15360 x 5120 38.5 against 31.3 us, x 5120 x 13824 36.9 against 32.0.)
struct GemmSched {
  int tiles_m, tiles_n, nk, group_n;
  int split;  // workgroups per tile
};

__device__ __forceinline__ void tile_coords(const GemmSched& s, int t, int& nt, int& mt) {
  const int per = s.group_n * s.tiles_m;
  const int gi = t / per, r = t - gi * per;
  const int first = gi * s.group_n;
  const int gsz = min(s.tiles_n - first, s.group_n);
  nt = first + r % gsz;
  mt = r / gsz;
}

// Ping-pong main loop (eight waves, two stages of both operands): acc = sum
// over 64-k slabs [k0, k1) of tile (n0, m0), every output summed by one wave in
// k order.
//
// A slab is multiplied in four phases of TNH x TMH x 2 MFMAs (a quarter of the
// wave's tile), each preceded by the LDS reads it adds. Waves 4 .. 7 run one
// barrier behind waves 0 .. 3, and wave w shares a SIMD with wave w + 4, so one
// of a SIMD's two waves always multiplies (at raised priority) while the
// other reads LDS and issues loads. Wave slab s, phase p reads: 0: rows' first
// half A0 and tokens' first half B0, 1: B1, 2: A1 (over A0), 3: nothing; and
// multiplies A0 B0, A0 B1, A1 B1, A1 B0.
//
// Between two barriers ("slots"), waves 0 .. 3 read in slot 2p and multiply in
// slot 2p + 1, waves 4 .. 7 one slot later. A region read in phase p is
// consumed by that phase's MFMAs, so every wave is done with it by the end of
// slot 2p + 2, and loads into it may be issued from phase p + 2 (slot 2p + 4
// or 2p + 5): slab s + 2's A0 and B0 in phase 2 of slab s, its B1 in phase 3,
// its A1 in phase 0 of slab s + 1. Whatever phase p reads has been waited for by
// the wave that loaded it at the end of its phase p - 1, before the barrier
// that opens slot 2p. A load has five to six phases (1300 cycles or more at
// 256 x 256) to land and up to 14 KiB per wave are in flight.
template <int BN, int BM, int TN, int TM, typename F>
__device__ __forceinline__ void pp_mainloop(f32x4_v (&acc)[TN][TM], const GemmArgs& a,
                                            const v4i_t& rw, const v4i_t& rx, const char* smem,
                                            uint32_t lds0, int n0, int m0, int k0, int k1,
                                            int lane, int wave, F&& after_issue) {
  constexpr int TNH = TN / 2, TMH = TM / 2, WN = BN / 2, WM = BM / 4;
  constexpr int W_BYTES = BN * 128, X_BYTES = BM * 128;
  static_assert(TN * 16 == WN && TM * 16 == WM && TN % 2 == 0 && TM % 2 == 0, "2 x 4 waves");
  static_assert(TNH == 3 || TNH == 4, "blocks of a half over eight waves");
  const int wn = wave & 1, wm = wave >> 1, fr = lane & 15, g = lane >> 4;
  const bool late = wave >= 4;
  // 8-row blocks of a half of the weight tile: 4 TNH over eight waves, two
  // each (TNH = 4); with 12, waves 0 .. 3 take two of the first half and one
  // of the second, waves 4 .. 7 the other way round
  constexpr int A0 = TNH == 4 ? 2 : 1, AS = TNH == 4 ? 4 : 3;  // fewest of a half; of both halves
  int blk[2][2];
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      int b;
      if constexpr (TNH == 4) b = 2 * wave + q;
      else b = (h == 1) == late ? 2 * (wave & 3) + q : 8 + (wave & 3);
      blk[h][q] = (b / (2 * TNH)) * (4 * TNH) + h * 2 * TNH + b % (2 * TNH);
    }
  const int sw_slab = (a.N / 8) * 1024, nb = a.N / 8 - 1;
  auto issue_a = [&](int h, int buf, int kt) {
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      if (TNH == 3 && q == 1 && (h == 1) != late) continue;  // uniform: one block of this half
      dma16(rw, lane * 16, min(n0 / 8 + blk[h][q], nb) * 1024 + kt * sw_slab,
            lds0 + buf * W_BYTES + blk[h][q] * 1024);
    }
  };
  // activations: 8 TMH blocks of 8 tokens per half, TMH per wave (rows past
  // the last re-read it; their outputs are not stored)
  int vx[2][TMH];
  uint32_t lx[2][TMH];
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int q = 0; q < TMH; ++q) {
      const int b = TMH * wave + q;
      const int row = (b / (2 * TMH)) * WM + h * 16 * TMH + (b % (2 * TMH)) * 8;
      const int r = lane >> 3;
      vx[h][q] = (min(m0 + row + r, a.M - 1) * (int)a.ldx + ((lane & 7) ^ r) * 8) * 2;
      lx[h][q] = lds0 + 2 * W_BYTES + row * 128;
    }
  auto issue_x = [&](int h, int buf, int kt) {
#pragma unroll
    for (int q = 0; q < TMH; ++q) dma16(rx, vx[h][q], kt * 128, lx[h][q] + buf * X_BYTES);
  };
  // fragment addresses: row fr of a 16-row tile, chunk 4 ks + g at (4 ks + g) ^ (row & 7)
  const int swz = (g ^ (fr & 7)) * 16;
  const int fw = (wn * WN + fr) * 128 + swz, fx = 2 * W_BYTES + (wm * WM + fr) * 128 + swz;
  bf16x8_v fa[TNH][2], fb[2][TMH][2];
  auto read_a = [&](int h, int buf) {
    const char* p0 = smem + (fw + buf * W_BYTES);
    const char* p1 = smem + ((fw ^ 64) + buf * W_BYTES);
#pragma unroll
    for (int i = 0; i < TNH; ++i) {
      fa[i][0] = as_bf16x8(ld16(p0 + (h * TNH + i) * 2048));
      fa[i][1] = as_bf16x8(ld16(p1 + (h * TNH + i) * 2048));
    }
  };
  auto read_b = [&](int h, int buf) {
    const char* p0 = smem + (fx + buf * X_BYTES);
    const char* p1 = smem + ((fx ^ 64) + buf * X_BYTES);
#pragma unroll
    for (int i = 0; i < TMH; ++i) {
      fb[h][i][0] = as_bf16x8(ld16(p0 + (h * TMH + i) * 2048));
      fb[h][i][1] = as_bf16x8(ld16(p1 + (h * TMH + i) * 2048));
    }
  };
  auto slot = [] {
    __builtin_amdgcn_sched_barrier(0);
    wg_barrier();
    __builtin_amdgcn_sched_barrier(0);
  };
  auto multiply = [&](int ha, int hb) {
    slot();
    __builtin_amdgcn_s_setprio(1);
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int i = 0; i < TNH; ++i)
#pragma unroll
        for (int j = 0; j < TMH; ++j)
          acc[ha * TNH + i][hb * TMH + j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
              fa[i][ks], fb[hb][j][ks], acc[ha * TNH + i][hb * TMH + j], 0, 0, 0);
    __builtin_amdgcn_s_setprio(0);
    slot();
  };
  const int n = k1 - k0;
  // one slab; LEFT = slabs after it (2 = two or more): which loads are still
  // to be issued and how many of this wave's may be outstanding at each wait
  auto slab = [&](int j, auto left) {
    constexpr int LEFT = decltype(left)::value;
    const int buf = j & 1;
    read_b(0, buf);
    read_a(0, buf);
    if constexpr (LEFT >= 1) issue_a(1, buf ^ 1, k0 + j + 1);
    // B1 of this slab: later are its A1 and the next slab's four parts
    wait_vm<(LEFT >= 1 ? A0 + AS + 2 * TMH : A0)>();
    multiply(0, 0);
    read_b(1, buf);
    wait_vm<(LEFT >= 1 ? AS + 2 * TMH : 0)>();  // A1 of this slab
    multiply(0, 1);
    read_a(1, buf);
    if constexpr (LEFT >= 2) {
      issue_a(0, buf, k0 + j + 2);
      issue_x(0, buf, k0 + j + 2);
    }
    multiply(1, 1);
    if constexpr (LEFT >= 2) issue_x(1, buf, k0 + j + 2);
    // A0 and B0 of the next slab
    if constexpr (LEFT >= 1) wait_vm<(LEFT >= 2 ? AS + 3 * TMH : A0 + TMH)>();
    multiply(1, 0);
  };
  issue_a(0, 0, k0);
  issue_x(0, 0, k0);
  issue_x(1, 0, k0);
  issue_a(1, 0, k0);
  if (n > 1) {
    issue_a(0, 1, k0 + 1);
    issue_x(0, 1, k0 + 1);
    issue_x(1, 1, k0 + 1);
  }
  after_issue();
  if (n > 1) wait_vm<AS + 3 * TMH>();
  else wait_vm<A0 + TMH>();
  wg_barrier();
  if (late) wg_barrier();
  for (int j = 0; j < n - 2; ++j) slab(j, std::integral_constant<int, 2>{});
  if (n > 1) slab(n - 2, std::integral_constant<int, 1>{});
  slab(n - 1, std::integral_constant<int, 0>{});
  if (!late) wg_barrier();
}

// NS stages of both operands: the loads of slab j + NS - 1 are in flight while
// slab j is multiplied. PP: the ping-pong main loop instead.
template <int BN, int BM, int NS, bool SK, int EPI, bool PP>
__global__ __launch_bounds__(64 * kRingWaves) __attribute__((amdgpu_waves_per_eu(2, 2)))
void gemm_ring(GemmArgs a, GemmSched sc) {
  constexpr int BK = 64, NW = kRingWaves;
  using T = RTile<BN, BM, BK, NS>;
  static_assert(!PP || NS == 2, "the ping-pong loop has two stages");
  constexpr int CPR = T::CPR, RPI = T::RPI, WN = T::WN, WM = T::WM, TN = T::TN, TM = T::TM;
  constexpr int LPS = T::LPS;
  static_assert((EPI != EPI_SWIGLU && EPI != EPI_QKV_ROPE) || (WN % 32) == 0,
                "SwiGLU and RoPE need 32-row pairs");
  constexpr int X_BYTES = BM * BK * 2;
  __shared__ __attribute__((aligned(1024))) char smem[NS * (T::W_BYTES + X_BYTES)];

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wn = wave & 1, wm = wave >> 1;
  const int G = gridDim.x;
  int l = blockIdx.x;  // consecutive logical workgroups on one XCD
  if ((G & 7) == 0) l = (l & 7) * (G >> 3) + (l >> 3);

  const int kp = (a.K + 63) & ~63;
  const v4i_t rw = buf_rsrc(a.W, (uint64_t)a.N * kp * 2);
  const v4i_t rx = buf_rsrc(a.X, x_bytes(a, kp));
  const int lrow = lane / CPR;
  const int lchunk = chunk_pos(lrow, lane % CPR);  // row base is a multiple of RPI
  const int wave_u = __builtin_amdgcn_readfirstlane(wave);
  const int vw = lane * 16;
  const int sw_slab = (a.N / 8) * 1024;
  const uint32_t lds0 = (uint32_t)(size_t)(__attribute__((address_space(3))) char*)smem;
  // weight stages first, then the activation stages
  const uint32_t lds_w = lds0 + wave_u * (BN / NW) * BK * 2;
  const uint32_t lds_x = lds0 + NS * T::W_BYTES + wave_u * (BM / NW) * BK * 2;
  const int fr = lane & 15, g = lane >> 4;

  f32x4_v acc[TN][TM];

  // acc = sum over k steps [k0, k1) of tile (n0, m0)
  // QKV projection with RoPE, data-parallel tiles: the tile's token
  // positions and slots, and its cos/sin rows when they fit in registers, are
  // requested right after the main loop's first operand loads, so their round
  // trips overlap the pipeline start instead of delaying the epilogue. (Extra
  // loads only make the vmcnt waits of the ring stricter: loads complete in
  // order.)
  constexpr bool ROPE_PRE = EPI == EPI_QKV_ROPE && !SK;
  // (the cos/sin rows take 4 TN TM registers: only the small tiles have room;
  // 256 x 256 spilled 100 registers)
  constexpr bool ROPE_TAB = ROPE_PRE && TN * TM <= 16;
  constexpr int RJ = ROPE_PRE ? TM : 1, RJT = ROPE_TAB ? TM : 1, RI = ROPE_TAB ? TN / 2 : 1;
  int r_pos[RJ], r_slot[RJ];
  float4 r_cos[RJT][RI], r_sin[RJT][RI];
  auto rope_fetch = [&](int n0, int m0) {
    if constexpr (ROPE_PRE) {
#pragma unroll
      for (int j = 0; j < TM; ++j) {
        const int m = m0 + wm * WM + j * 16 + fr;
        const bool in = m < a.M;
        r_pos[j] = in ? a.rope_pos[m] : 0;
        r_slot[j] = in ? a.rope_slot[m] : -1;
      }
      if constexpr (ROPE_TAB) {
        const int qk = a.rope_q_cols + a.rope_kv_cols;
#pragma unroll
        for (int j = 0; j < TM; ++j)
#pragma unroll
          for (int ip = 0; ip < TN / 2; ++ip) {
            const int n = n0 + wn * WN + ip * 32 + g * 4;
            const int64_t o = rope_tab_off(a, r_pos[j], n < qk ? n : 0);
            r_cos[j][ip] = *reinterpret_cast<const float4*>(a.rope_cos + o);
            r_sin[j][ip] = *reinterpret_cast<const float4*>(a.rope_sin + o);
          }
      }
    }
  };

  auto mainloop = [&](int n0, int m0, int k0, int k1, auto&& after_issue) {
#pragma unroll
    for (int i = 0; i < TN; ++i)
#pragma unroll
      for (int j = 0; j < TM; ++j) acc[i][j] = f32x4_v{0.f, 0.f, 0.f, 0.f};
    if constexpr (PP) {
      pp_mainloop<BN, BM>(acc, a, rw, rx, smem, lds0, n0, m0, k0, k1, lane, wave_u, after_issue);
      return;
    } else {
    // weights: block (kt, n0/8 + wave * BN/(8 NW) + q) of the tiled format;
    // rows past the last one (of either operand) re-read it, their outputs
    // are not stored
    int sw[T::WI], vx[T::XI];
#pragma unroll
    for (int q = 0; q < T::WI; ++q)
      sw[q] = min(n0 / 8 + wave_u * (BN / NW / 8) + q, a.N / 8 - 1) * 1024;
#pragma unroll
    for (int q = 0; q < T::XI; ++q)
      vx[q] = (min(m0 + wave * (BM / NW) + q * RPI + lrow, a.M - 1) * (int)a.ldx + lchunk * 8) * 2;
    // load q of a step (0 <= q < LPS): weights first
    constexpr int AHEAD = NS - 1;  // look-ahead in steps
    auto issue = [&](int j, int q) {
      const int stage = j % NS, kt = k0 + j;
      if (q < T::WI)
        dma16(rw, vw, sw[q] + kt * sw_slab, lds_w + stage * T::W_BYTES + q * 1024);
      else
        dma16(rx, vx[q - T::WI], kt * BK * 2, lds_x + stage * X_BYTES + (q - T::WI) * 1024);
    };
    // the loads of a step are spread over the row-tile steps of the current
    // slab's multiplication
    constexpr int STEPS = TN * (BK / 32);
    // Step j issues the loads of slab j + NS - 1 while it multiplies slab j.
    // The issue is behind a (uniform) branch on purpose: it splits the step
    // into scheduling regions, without which the register allocator shuffles
    // the accumulators between MFMAs. Loads complete in issue order, so before
    // slab j + 1 the wave waits until only the loads of the NS - 2 later slabs
    // are outstanding.
    const int n = k1 - k0;
#pragma unroll
    for (int t = 0; t < AHEAD; ++t)
      if (t < n)
#pragma unroll
        for (int q = 0; q < LPS; ++q) issue(t, q);
    after_issue();
    if (n >= AHEAD) wait_vm<(NS - 2) * LPS>();
    else wait_vm<0>();
    wg_barrier();
    constexpr int PD = ring_pd<TN>();
    bf16x8_v fa[PD + 1], fb[2][TM];
    for (int j = 0; j < n; ++j) {
      const bool more = j + AHEAD < n;
      const bf16_t* sws = reinterpret_cast<const bf16_t*>(smem + (j % NS) * T::W_BYTES);
      const bf16_t* sxs =
          reinterpret_cast<const bf16_t*>(smem + NS * T::W_BYTES + (j % NS) * X_BYTES);
      ring_stage<BN, BM, BK, NS, TN, TM, PD>(acc, fa, fb, sws, sxs, wn, wm, fr, g, j > 0, [&](int step) {
        if (more) {
#pragma unroll
          for (int q = step * LPS / STEPS; q < (step + 1) * LPS / STEPS; ++q) issue(j + AHEAD, q);
        }
      });
      // slab j's stage is refilled, by any wave, right after the barrier: the
      // deferred row tile's operands have to be in registers by then
      if (more) wait_vm_lds<(NS - 2) * LPS>();
      else wait_vm_lds<0>();
      wg_barrier();
    }
    // the last stage's deferred row tile
#pragma unroll
    for (int jj = 0; jj < TM; ++jj)
      acc[TN - 1][jj] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[(2 * TN - 1) % (PD + 1)], fb[1][jj], acc[TN - 1][jj], 0, 0, 0);
    }
  };

  auto epilogue = [&](int n0, int m0) {
    const int fq = g * 4;
#pragma unroll
    for (int j = 0; j < TM; ++j) {
      const int m = m0 + wm * WM + j * 16 + fr;
      if constexpr (EPI == EPI_SWIGLU) {
#pragma unroll
        for (int i = 0; i < TN; i += 2)
          store_swiglu(a, m, (n0 + wn * WN + i * 16) / 2 + fq, acc[i][j], acc[i + 1][j]);
      } else if constexpr (EPI == EPI_QKV_ROPE) {
        int pos, slot;
        if constexpr (ROPE_PRE) {
          pos = r_pos[j];
          slot = r_slot[j];
        } else {
          const bool in = m < a.M;
          pos = in ? a.rope_pos[m] : 0;
          slot = in ? a.rope_slot[m] : -1;
        }
        const int qk = a.rope_q_cols + a.rope_kv_cols;
#pragma unroll
        for (int i = 0; i < TN; i += 2) {
          const int n = n0 + wn * WN + i * 16 + fq;
          float4 cv, sv;
          if constexpr (ROPE_TAB) {
            cv = r_cos[j][i / 2];
            sv = r_sin[j][i / 2];
          } else {
            const int64_t o = rope_tab_off(a, pos, n < qk ? n : 0);
            cv = *reinterpret_cast<const float4*>(a.rope_cos + o);
            sv = *reinterpret_cast<const float4*>(a.rope_sin + o);
          }
          store_qkv_rope(a, m, slot, n, acc[i][j], acc[i + 1][j], cv, sv);
        }
      } else {
#pragma unroll
        for (int i = 0; i < TN; ++i) store4<EPI>(a, m, n0 + wn * WN + i * 16 + fq, acc[i][j]);
      }
    }
  };

  int nt, mt;
  if constexpr (!SK) {
    tile_coords(sc, l, nt, mt);
    mainloop(nt * BN, mt * BM, 0, sc.nk, [&] { rope_fetch(nt * BN, mt * BM); });
    epilogue(nt * BN, mt * BM);
  } else {
  // split: workgroup l's partial tile lives at part[l * BN * BM], in the lane
  // order of the accumulators (coalesced 1 KiB per fragment). It is written
  // and read with device-scope (sc1) accesses, which are coherent across the
  // XCDs' L2 caches on their own; a writer waits for its stores to complete
  // before its arrival is counted, so the last arrival sees every partial
  // without any cache-wide write-back or invalidation.
  constexpr int TILE_F = BN * BM;
  constexpr int kSc1 = 16;  // cache-policy bit: device scope
  typedef unsigned u32x4_v __attribute__((ext_vector_type(4)));
  const __amdgpu_buffer_rsrc_t rp =
      __builtin_amdgcn_make_buffer_rsrc(a.part, 0, 0x7FFFFFFF, kRsrcWord3);
  auto frag_off = [&](int f) { return ((f * NW + wave) * 64 + lane) * 16; };
  const int t = l / sc.split, c_me = l - t * sc.split;
  tile_coords(sc, t, nt, mt);
  mainloop(nt * BN, mt * BM, c_me * sc.nk / sc.split, (c_me + 1) * sc.nk / sc.split, [] {});
#pragma unroll
  for (int f = 0; f < TN * TM; ++f)
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4_v, acc[f / TM][f % TM]), rp,
                                           frag_off(f), l * TILE_F * 4, kSc1);
  wait_vm<0>();
  __syncthreads();
  // (every wave is past its last fragment read: the ring's first word is free)
  int& s_last = *reinterpret_cast<int*>(smem);
  if (tid == 0) {
    const uint32_t prev =
        __hip_atomic_fetch_add(a.flags + t, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    s_last = prev + 1 == (uint32_t)sc.split;
  }
  __syncthreads();
  if (!s_last) return;
  // The partials of CG contributors (8 fragments of each) are requested
  // together, so a tile of six contributors pays two round trips to memory
  // and not five (40 tokens, 5120 x 5120: 20.9 -> 19.9 us).
  constexpr int FR = TN * TM, FB = FR == 8 ? 8 : FR % 4 == 0 ? 4 : FR;
  constexpr int CG = FR <= 4 ? 8 : 4;
  static_assert(FR % FB == 0, "whole batches of fragments");
#pragma unroll
  for (int f0 = 0; f0 < FR; f0 += FB) {
    f32x4_v sum[FB];
    for (int c0 = 0; c0 < sc.split; c0 += CG) {
      f32x4_v v[CG][FB];
#pragma unroll
      for (int u = 0; u < CG; ++u) {
        const int c = c0 + u;
        if (c >= sc.split || c == c_me) continue;
#pragma unroll
        for (int f = 0; f < FB; ++f)
          v[u][f] = __builtin_bit_cast(
              f32x4_v, __builtin_amdgcn_raw_buffer_load_b128(
                           rp, frag_off(f0 + f), (t * sc.split + c) * TILE_F * 4, kSc1));
      }
#pragma unroll
      for (int u = 0; u < CG; ++u) {
        const int c = c0 + u;
        if (c >= sc.split) break;
#pragma unroll
        for (int f = 0; f < FB; ++f) {
          const f32x4_v p = c == c_me ? acc[(f0 + f) / TM][(f0 + f) % TM] : v[u][f];
          sum[f] = c == 0 ? p : sum[f] + p;
        }
      }
    }
#pragma unroll
    for (int f = 0; f < FB; ++f) acc[(f0 + f) / TM][(f0 + f) % TM] = sum[f];
  }
  if (tid == 0) __hip_atomic_store(a.flags + t, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  epilogue(nt * BN, mt * BM);
  }
}

// ------------------------------------------------------------ skinny (decode)
//
// A workgroup owns 16 * NF weight rows and 16 tokens (all, up to 16); its WV waves
// split the 64-column slabs of K. For one slab, the 2 NF row blocks of the
// workgroup are adjacent 1 KiB blocks. Each is read by one wave-wide 16-byte
// load with lane L taking bytes [16 L, 16 L + 16) (a whole block per
// instruction, non-temporal: the weights are streamed once per call), then
// stored unchanged into the wave's own LDS buffer and read back in the MFMA
// fragment order: lane (row fr, group g) takes chunk 4 ks + g of its row for
// the ks-th 32-k MFMA. The buffer keeps the block's XOR-swizzled chunk order,
// so the fragment reads are free of bank conflicts. (Loading the fragments
// straight from global memory makes every instruction touch half of each of
// 16 rows; the whole-block loads stream 10-30% faster on MI355X.) The
// activations (the B operand, tokens on the MFMA columns) are loaded in
// fragment order, lane (fr, g) taking chunk 4 ks + g of token fr: 64 bytes of
// each of 16 rows per instruction. With XS they take the weights' route
// instead: instruction h reads whole 128-byte rows of tokens 8h .. 8h + 7 into
// an image laid out and read like a weight tile's. The MFMA operands are the
// same; whole rows pay off from 8 tokens on, where the activations the previous
// kernel wrote come from beyond the XCD's L2 (8B layer at 16 tokens, in the
// decode step: o and down 36.6 -> 31.6 us together). XS = 1 requests them one slab
// ahead, as below; XS = 2 after the next slab's weights: from 13 tokens on the
// one-row-tile form is faster so (16 tokens x 4096 x 11008 17.87 -> 17.61 us, x
// 14336 22.44 -> 22.05; 8 tokens 15.50 against 15.89 and 19.24 against 19.57).
//
// A slab's loads are issued as its registers come free, weights before
// activations, so no wait for one slab covers a later one's loads. (Loads
// complete in order: with the activations of slab s requested after the weights
// of slab s + 1, the wait for them drained those as well. 7B, 8B and 13B shapes
// at 1 to 16 tokens, MI355X, before -> after: QKV 19.8 -> 18.2, 12.9 -> 11.0 and
// 27.1 -> 25.5 us, gate/up 29.9 -> 29.4, 39.2 -> 36.3 and 45.4 -> 42.3, LM head with
// its norm 178 -> 153, 13B down 26.2 -> 23.8.)

// With NORM, X is the un-normalised residual stream and the GEMM applies the
// RMSNorm of its rows itself: each loaded activation chunk is multiplied by
// the norm gain (and rounded to bf16 like a stored activation), the squares
// of the raw values are summed along the way, and the epilogue scales each
// token's outputs by 1 / sqrt(mean square + eps). Used for decode, where the
// separate norm kernel would cost a launch per projection.
template <int NF, int EPI, bool NORM, int WV, int XS>
__global__ __launch_bounds__(64 * WV) void gemm_skinny(GemmArgs a) {
  static_assert(EPI != EPI_SWIGLU || (NF % 2) == 0, "SwiGLU needs gate/up tile pairs");
  // the norm's sums of squares follow the fragment-order loads; keeping one
  // order for every batch size keeps a token's result independent of M
  static_assert(!(NORM && XS), "staged activations are built without the fused norm");
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // a call's first kernel also pulls its metadata, in its first workgroups (it
  // applies a norm: gemm() refuses a pull without one)
  int pb = 0;
  if constexpr (NORM) {
    pb = a.pull.blocks(64 * WV);
    if ((int)blockIdx.x < pb)
      return pull16(a.pull.host, a.pull.dev, a.pull.n16, blockIdx.x * 64 * WV + threadIdx.x);
  }
  const int n0 = ((int)blockIdx.x - pb) * 16 * NF;
  const int mb = blockIdx.y * 16;  // first token
  const int kp = (a.K + 63) & ~63;
  const int nslab = kp / 64;
  const int sq = (nslab + WV - 1) / WV;  // slabs per wave
  const int sb = wave * sq, se = min(nslab, sb + sq);
  const int fr = lane & 15, g = lane >> 4;
  const int slab_bytes = (a.N / 8) * 1024;
  // Loads past a wave's last slab, of row tiles past N and of tokens past M
  // get an offset past the end of their buffer: they read zeros and touch no
  // memory, and no load is behind a branch (the waits stay exact). With one row
  // tile a workgroup there is little to wait for in order, and the loads past
  // the last slab cost more than a uniform branch around them (4096 rows of
  // weights, MI355X, past -> branch: K = 4096 7.66 -> 7.30 us at 1 token and 8.20 ->
  // 7.70 at 8, K = 14336 18.73 -> 18.42 and, at 16, 22.66 -> 22.31; with two row
  // tiles, 5120 x 13824, 23.5 -> 23.9).
  constexpr bool kBranch = NF == 1;
  constexpr int kPast = (int)0x80000000u;
  const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<bf16_t*>(a.W), 0, (int)((int64_t)a.N * kp * 2), kRsrcWord3);
  const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<bf16_t*>(a.X), 0, (int)x_bytes(a, kp), kRsrcWord3);
  const __amdgpu_buffer_rsrc_t rg = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<bf16_t*>(NORM ? a.norm_gain : a.X), 0, a.K * 2, kRsrcWord3);
  // instruction (f, h) of a slab reads row block n0 / 8 + 2 f + h (N % 16 == 0,
  // so a 16-row tile is either wholly inside the matrix or wholly outside)
  const int wbase = (n0 / 8) * 1024 + lane * 16;
  int wpast[NF];
#pragma unroll
  for (int f = 0; f < NF; ++f) wpast[f] = n0 + 16 * f < a.N ? 0 : kPast;
  const int r8 = fr % 8;
  // 16-byte position of lane (fr, g)'s row inside the 2 KiB image of a 16-row tile
  const int fpos = (fr / 8) * 64 + r8 * 8;
  // activations. XS: instruction h reads token 8 h + L / 8, at 16-byte chunk
  // (L % 8) ^ (L / 8) of each slab; otherwise instruction ks reads chunk
  // 4 ks + g of token fr
  int xoff[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int m = mb + (XS ? 8 * i + (lane >> 3) : fr);
    const int chunk = XS ? (lane & 7) ^ (lane >> 3) : 4 * i + g;
    xoff[i] = m < a.M ? m * (int)a.ldx * 2 + chunk * 16 : kPast;
  }
  // per wave: the weight tiles' images of a slab, then with XS the
  // activations' (16-byte units); after the last slab, the wave's partial sums
  __shared__ pack8 wlds[WV][(NF + (XS ? 1 : 0)) * 128];

  f32x4_v acc[NF];
  float ssq = 0.f;
#pragma unroll
  for (int f = 0; f < NF; ++f) acc[f] = f32x4_v{0.f, 0.f, 0.f, 0.f};

  typedef unsigned u32x4_v __attribute__((ext_vector_type(4)));
  constexpr int kNt = 2;  // cache policy: streamed once per call
  u32x4_v wv[NF][2], xv[2], gv[2];
  auto load_x = [&](int sl) {
    // uniform, and or-ed in: a select here becomes a branch
    const int past = sl < se ? 0 : kPast;
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      xv[ks] = __builtin_amdgcn_raw_buffer_load_b128(rx, (xoff[ks] + sl * 128) | past, 0, 0);
      if constexpr (NORM)
        gv[ks] = __builtin_amdgcn_raw_buffer_load_b128(rg, (sl * 128 + (ks * 4 + g) * 16) | past, 0, 0);
    }
  };
  auto load_w = [&](int sl) {
    const int past = sl < se ? 0 : kPast;
#pragma unroll
    for (int f = 0; f < NF; ++f)
#pragma unroll
      for (int h = 0; h < 2; ++h)
        wv[f][h] = __builtin_amdgcn_raw_buffer_load_b128(
            rw, ((wbase + sl * slab_bytes) | past | wpast[f]) + (2 * f + h) * 1024, 0, kNt);
  };
  load_w(sb);
  if constexpr (XS != 2) load_x(sb);
  for (int sl = sb; sl < se; ++sl) {
    // this wave's buffer: the previous slab's fragment reads were issued
    // before these stores, and one wave's LDS operations run in order
#pragma unroll
    for (int f = 0; f < NF; ++f)
#pragma unroll
      for (int h = 0; h < 2; ++h)
        wlds[wave][(2 * f + h) * 64 + lane] = __builtin_bit_cast(pack8, wv[f][h]);
    if (!kBranch || sl + 1 < se) load_w(sl + 1);
    if constexpr (XS == 2) load_x(sl);
    pack8 xc[2], gc[2];
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      xc[ks] = __builtin_bit_cast(pack8, xv[ks]);
      if constexpr (XS) wlds[wave][NF * 128 + ks * 64 + lane] = xc[ks];
      if constexpr (NORM) gc[ks] = __builtin_bit_cast(pack8, gv[ks]);
    }
    if constexpr (XS != 2) {
      if (!kBranch || sl + 1 < se) load_x(sl + 1);
    }
    if constexpr (NORM) {
#pragma unroll
      for (int ks = 0; ks < 2; ++ks)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float x0 = lo_bf(xc[ks].w[e]), x1 = hi_bf(xc[ks].w[e]);
          ssq += x0 * x0 + x1 * x1;
          xc[ks].w[e] = pack2bf(x0 * lo_bf(gc[ks].w[e]), x1 * hi_bf(gc[ks].w[e]));
        }
    }
    asm volatile("" ::: "memory");  // keep the fragment reads after the stores
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      if constexpr (XS)  // the fragments from the staged image (read like a weight tile's)
        xc[ks] = wlds[wave][NF * 128 + fpos + ((ks * 4 + g) ^ r8)];
#pragma unroll
      for (int f = 0; f < NF; ++f) {
        const pack8 w = wlds[wave][f * 128 + fpos + ((ks * 4 + g) ^ r8)];
        acc[f] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(w), as_bf16x8(xc[ks]), acc[f],
                                                         0, 0, 0);
      }
    }
    asm volatile("" ::: "memory");  // and the next stores after these reads
  }

  // partial sums added in wave order; with SwiGLU wave p finishes the gate/up
  // pair p of the workgroup, else row tile p (by one wave alone the reads of
  // 15 partials of three tiles spilled 76 registers)
  constexpr int PAIR = EPI == EPI_SWIGLU ? 2 : 1;
  // (each wave's partials over its own, consumed, tile images: the LDS of a
  // 128256-wide LM head's workgroup stays 32 KiB and its 1002 workgroups fit
  // the chip in one round; with 48 KiB it took 175 us instead of 155)
  const auto red = [&](int w, int f) { return reinterpret_cast<f32x4_v*>(wlds[w]) + f * 64 + lane; };
  __shared__ float red_ss[WV][16];
  if constexpr (NORM) {
    // the 4 k-groups of a token (lanes fr, fr+16, fr+32, fr+48), then waves
    ssq += __shfl_xor(ssq, 16, 64);
    ssq += __shfl_xor(ssq, 32, 64);
    if (g == 0) red_ss[wave][fr] = ssq;
  }
#pragma unroll
  for (int f = 0; f < NF; ++f) *red(wave, f) = acc[f];
  __syncthreads();
  const int fq = g * 4;
  for (int p = wave; p < NF / PAIR; p += WV) {
    f32x4_v o[PAIR];
#pragma unroll
    for (int i = 0; i < PAIR; ++i) {
      o[i] = *red(0, p * PAIR + i);
#pragma unroll
      for (int w = 1; w < WV; ++w) o[i] += *red(w, p * PAIR + i);
    }
    if constexpr (NORM) {
      float tot = red_ss[0][fr];
#pragma unroll
      for (int w = 1; w < WV; ++w) tot += red_ss[w][fr];
      const float inv = 1.0f / sqrtf(tot / (float)a.K + a.norm_eps);
#pragma unroll
      for (int i = 0; i < PAIR; ++i) o[i] *= inv;
    }
    if constexpr (EPI == EPI_SWIGLU) store_swiglu(a, mb + fr, n0 / 2 + 16 * p + fq, o[0], o[1]);
    else store4<EPI>(a, mb + fr, n0 + 16 * p + fq, o[0]);
  }
}

// ------------------------------------------------------------------ launch

namespace {

// The skinny builds, as (epilogue, rows per workgroup / 16, waves per
// workgroup, staged activations): the ones the selection in gemm() takes. Those
// without staging are built with and without the norm.
#define HS_SKINNY_BUILDS(X)                                                  \
  X(EPI_F32, 2, 2, 0) X(EPI_F32, 4, 2, 0) X(EPI_F32, 8, 2, 0)               \
  X(EPI_SWIGLU, 2, 2, 0) X(EPI_SWIGLU, 4, 2, 0) X(EPI_SWIGLU, 2, 4, 0)      \
  X(EPI_SWIGLU, 4, 4, 0) X(EPI_STORE, 2, 8, 0) X(EPI_STORE, 2, 4, 0)        \
  X(EPI_STORE, 4, 4, 0) X(EPI_STORE, 3, 16, 0) X(EPI_RESID, 2, 8, 0)        \
  X(EPI_RESID, 2, 8, 1) X(EPI_RESID, 1, 16, 0) X(EPI_RESID, 1, 16, 1)       \
  X(EPI_RESID, 1, 16, 2)

template <int EPI, int NF, int WV, int XS>
hipError_t launch_skinny(const GemmArgs& a, hipStream_t s) {
  const dim3 grid((a.N + 16 * NF - 1) / (16 * NF) + a.pull.blocks(64 * WV), (a.M + 15) / 16);
  const dim3 blk(64 * WV);
  if (a.norm_gain) {
    if constexpr (XS) return hipErrorInvalidValue;
    else hipLaunchKernelGGL((gemm_skinny<NF, EPI, true, WV, 0>), grid, blk, 0, s, a);
  } else {
    hipLaunchKernelGGL((gemm_skinny<NF, EPI, false, WV, XS>), grid, blk, 0, s, a);
  }
  return hipGetLastError();
}

hipError_t dispatch_skinny(const GemmArgs& a, int epi, int nf, int wv, int xs, hipStream_t s) {
#define HS_SKINNY_CASE(EPI_, NF_, WV_, XS_) \
  if (epi == EPI_ && nf == NF_ && wv == WV_ && xs == XS_) return launch_skinny<EPI_, NF_, WV_, XS_>(a, s);
  HS_SKINNY_BUILDS(HS_SKINNY_CASE)
#undef HS_SKINNY_CASE
  return hipErrorInvalidValue;
}

template <int BN, int BM, int NS, bool SK, bool PP = false>
hipError_t dispatch_ring(const GemmArgs& a, int epi, const GemmSched& sc, int grid, hipStream_t s) {
  const dim3 blk(64 * kRingWaves);
  switch (epi) {
    case EPI_STORE: hipLaunchKernelGGL((gemm_ring<BN, BM, NS, SK, EPI_STORE, PP>), dim3(grid), blk, 0, s, a, sc); break;
    case EPI_RESID: hipLaunchKernelGGL((gemm_ring<BN, BM, NS, SK, EPI_RESID, PP>), dim3(grid), blk, 0, s, a, sc); break;
    case EPI_SWIGLU: hipLaunchKernelGGL((gemm_ring<BN, BM, NS, SK, EPI_SWIGLU, PP>), dim3(grid), blk, 0, s, a, sc); break;
    case EPI_F32: hipLaunchKernelGGL((gemm_ring<BN, BM, NS, SK, EPI_F32, PP>), dim3(grid), blk, 0, s, a, sc); break;
    case EPI_QKV_ROPE: hipLaunchKernelGGL((gemm_ring<BN, BM, NS, SK, EPI_QKV_ROPE, PP>), dim3(grid), blk, 0, s, a, sc); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

// Tile configurations and the time model gemm() chooses among them with, in us
// for nk 64-k slabs on a chip of `cus` CUs:
//   whole tiles: start + nk rounds (slab + load * fill)
//   split tiles: s_start + nk / split (s_slab + s_load * fill) + s_each * split
// with rounds = ceil(tiles / cus) and fill = the share of the chip's workgroup
// slots that hold one (a fuller chip is slower a slab: memory, caches, clock).
// Least squares over measured launches (MI355X, weights streamed from HBM) of
// nine projections of 7B, 8B and 13B shapes at 80 to 512 tokens and seven at
// 640 to 4096: each configuration's own times within 3-7 % (rms), the choice
// 0.4 % behind the best configuration of every shape on average and 8 % at
// worst. (Up to 64 rows, where it was not fitted, and some of the 64-token tiles'
// terms came out as zero, it only chooses between those two tiles: over 44 shapes
// of 17 to 64 rows 0.6 % behind the best of both on average, 11 % at worst, 33 x
// 15360 x 5120.) Against the choice by per-CU rates before it and the split launches
// before them, 16 % faster over those shapes: 160 tokens x 15360 x 5120 68.7 ->
// 42.9 us, 512 x 5120 x 13824 138.9 -> 93.8, 512 x 6144 x 4096 47.6 -> 34.6.
struct RingCfg {
  const char* name;
  int bn, bm;
  double start, slab, load;
  double s_start, s_slab, s_load, s_each;  // s_slab 0: no split build
};
const RingCfg kRing[] = {
    {"256x256", 256, 256, 8.3, 1.035, 0.461, 0, 0, 0, 0},
    {"192x256", 192, 256, 7.2, 0.888, 0.374, 0, 0, 0, 0},
    {"256x128", 256, 128, 4.9, 0.700, 0.262, 12.1, 0.097, 1.060, 1.49},
    {"192x128", 192, 128, 3.7, 0.557, 0.197, 8.9, 0.192, 0.685, 1.41},
    {"128x128", 128, 128, 2.8, 0.430, 0.141, 6.2, 0.134, 0.516, 1.26},
    {"128x64", 128, 64, 2.8, 0.339, 0.076, 0.0, 0.317, 0.145, 3.10},
    {"64x64", 64, 64, 1.6, 0.214, 0.083, 0.0, 0.283, 0.0, 2.50}};

// 256 x 256 and 192 x 256: ping-pong loop (128 and 112 KiB of LDS). Same box,
// MI355X, one-barrier loop -> ping-pong: 8192 tokens QKV 616 -> 591 us, o 219 ->
// 210, gate/up 1093 -> 1040, down 560 -> 522; 15646 tokens 8B gate/up 2822 ->
// 2688, down 1428 -> 1317; 512 tokens gate/up 87.4 -> 86.5. With operands of
// zeros, which hold the clock up, 8192-token gate/up goes 929 -> 823 us (1.80
// PFLOP/s): on real data the power limit takes half of the gain.
// 256 x 128: 3 stages, loads spread over the whole step. 192 x 128 (160 KiB)
// and 128 x 128: 4 stages, 128 x 64 (144 KiB): 6, 64 x 64: 8. The 64-token tiles
// stream weights (17 to 64 tokens: 6.1 TB/s on the 13B gate/up matrix at 40
// tokens, 84 -> 46 us; down 82 -> 28, QKV 68 -> 29, o 34 -> 15 against the decode
// kernel, whose workgroups each read all activations from L2 unpipelined).
template <int BN, int BM, int NS>
hipError_t dispatch_split(const GemmArgs& a, int epi, const GemmSched& sc, int grid, hipStream_t s) {
  return sc.split > 1 ? dispatch_ring<BN, BM, NS, true>(a, epi, sc, grid, s)
                      : dispatch_ring<BN, BM, NS, false>(a, epi, sc, grid, s);
}

hipError_t launch_ring(const RingCfg& c, const GemmArgs& a, int epi, const GemmSched& sc,
                       int grid, hipStream_t s) {
  switch (c.bn * 1000 + c.bm) {
    case 256256: return dispatch_ring<256, 256, 2, false, true>(a, epi, sc, grid, s);
    case 192256: return dispatch_ring<192, 256, 2, false, true>(a, epi, sc, grid, s);
    case 256128: return dispatch_split<256, 128, 3>(a, epi, sc, grid, s);
    case 192128: return dispatch_split<192, 128, 4>(a, epi, sc, grid, s);
    case 128128: return dispatch_split<128, 128, 4>(a, epi, sc, grid, s);
    case 128064: return dispatch_split<128, 64, 6>(a, epi, sc, grid, s);
    case 64064: return dispatch_split<64, 64, 8>(a, epi, sc, grid, s);
    default: return hipErrorInvalidValue;
  }
}

const char* kEpiName[5] = {"store", "resid", "swiglu", "f32", "qkv_rope"};

}  // namespace

int device_cus() {
  static int cus[64] = {};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
  if (!cus[dev]) {
    int n = 0;
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        n <= 0)
      n = 256;
    cus[dev] = n;
  }
  return cus[dev];
}

hipError_t gemm(const GemmArgs& a, int epi, hipStream_t s, LaunchInfo* info) {
  if (a.M <= 0 || a.N <= 0 || a.K <= 0) return hipErrorInvalidValue;
  if (epi < 0 || epi > 4) return hipErrorInvalidValue;
  // head-interleaved q/k rows: whole heads of 64 or 128, then as many v columns as k
  if (a.rope_q_cols || a.rope_kv_cols) {
    const int d = a.rope_d;
    if ((d != 64 && d != 128) || a.rope_q_cols <= 0 || a.rope_kv_cols <= 0 ||
        (a.rope_q_cols % d) || (a.rope_kv_cols % d) || a.rope_q_cols + 2 * a.rope_kv_cols != a.N)
      return hipErrorInvalidValue;
  }
  if (epi == EPI_QKV_ROPE &&
      (!a.rope_q_cols || !a.rope_pos || !a.rope_slot || !a.rope_cos || !a.rope_sin ||
       !a.rope_pool || a.rope_max_pos <= 0 || (a.ldy % 8) ||
       ((uintptr_t)a.rope_cos & 15) || ((uintptr_t)a.rope_sin & 15) ||
       ((uintptr_t)a.rope_pool & 15)))
    return hipErrorInvalidValue;
  const int64_t kp = (a.K + 63) / 64 * 64;
  if ((a.K % 8) || (a.N % 16) || (a.ldx % 8) || (a.ldy % 4)) return hipErrorInvalidValue;
  if ((a.K % 64) && a.ldx < kp) return hipErrorInvalidValue;
  if (epi == EPI_SWIGLU && (a.N % 32)) return hipErrorInvalidValue;
  if (epi == EPI_RESID && (!a.R || (a.ldr % 4))) return hipErrorInvalidValue;
  if (((uintptr_t)a.X | (uintptr_t)a.W | (uintptr_t)a.Y) & 15) return hipErrorInvalidValue;
  if (a.norm_gain && (a.M > 16 || (a.K % 64) || ((uintptr_t)a.norm_gain & 15)))
    return hipErrorInvalidValue;
  if (!pull_ok(a.pull) || (a.pull.n16 && (a.M > 16 || !a.norm_gain))) return hipErrorInvalidValue;
  // 32-bit byte offsets in the buffer loads
  if ((uint64_t)a.N * kp * 2 >= (1ull << 31) || (uint64_t)a.M * a.ldx * 2 >= (1ull << 31) ||
      ((uint64_t)(a.M - 1) * a.ldx + kp) * 2 >= (1ull << 31))
    return hipErrorInvalidValue;

  static thread_local char name[64];
  const double flops = 2.0 * a.M * (double)a.N * a.K;
  const double out_cols = epi == EPI_SWIGLU ? a.N / 2 : a.N;
  const double out_bytes = (double)a.M * out_cols * (epi == EPI_F32 ? 4 : 2) *
                           (epi == EPI_RESID ? 2 : 1);
  const double bytes = 2.0 * ((double)a.M * a.K + (double)a.N * a.K) + out_bytes;
  hipError_t e;
  bool split = false;
  // HS_GEMM_CFG="skinny" or "<tile>[,dp|,sk[<ways>]][,g<n>]" forces a choice of
  // kernel above 16 rows: tile, whole or split tiles, tile group (tuning only;
  // read on every call so that a sweep can change it between calls).
  const char* force_cfg = getenv("HS_GEMM_CFG");
  const bool forced = force_cfg && *force_cfg;
  // 17 to 64 rows of a small matrix: the decode kernel too, 16 rows to a
  // workgroup, while all its passes read at most 32 MiB of weights (from L2
  // after the first). The tiles have too few workgroups there. MI355X, decode
  // kernel / best tiles, us: 17 x 256 x 688 3.3 / 5.4, 17 x 1024 x 1024 3.7 / 6.4,
  // 64 x 1024 x 4096 7.1 / 8.8, 17 x 3072 x 2048 (24 MiB) 6.2 / 7.9, 64 x 2048 x 2048
  // (32 MiB) 7.5 / 8.1; above, 33 x 3072 x 2048 (36 MiB) 9.5 / 8.0, 17 x 4096 x 4096
  // (64 MiB) 13.2 / 11.7. SwiGLU's two waves a workgroup gain nothing (17 x 1376 x
  // 256 3.6 / 3.6, 64 x 2752 x 512 5.7 / 5.1), and a QKV projection with RoPE would
  // need a second launch.
  const bool few = a.M <= 64 && (epi == EPI_STORE || epi == EPI_RESID || epi == EPI_F32) &&
                   (uint64_t)a.N * kp * 2 * ((a.M + 15) / 16) <= (32ull << 20);
  if (a.M <= 16 || (forced ? !strcmp(force_cfg, "skinny") && a.M <= 64 : few)) {
    // a QKV projection with RoPE runs as a plain (head-order) store followed
    // by the rotation pass
    const int pe = epi == EPI_QKV_ROPE ? EPI_STORE : epi;
    // Rows per workgroup (16 NF), waves per workgroup (WV) and staged
    // activations (XS), from sweeps on MI355X over the decode projections
    // of 7B, 8B and 13B models at 1, 4, 8 and 16 tokens (us at 1 token): o and
    // down projections up to one row tile per CU run sixteen waves of one row
    // tile (7B down 15.5, eight waves 18.9), wider ones eight waves of two (13B
    // down 23.8, of one 26.2). QKV up to 8192 wide takes eight waves of two
    // (8B 11.0, four waves 14.3), wider ones three row tiles when that gives
    // one workgroup per CU (7B 18.3, two of four waves 18.6), else four waves of
    // four while that fills three quarters of the CUs (13B 25.4 and, at 16
    // tokens, 25.1 against 26.4 with two). Gate/up runs two waves of four row
    // tiles, of two where four leave fewer than 1.5 workgroups per CU (8B 35.7,
    // four waves 39.1; 7B at 16 tokens 30.2 against 32.7). Up to one workgroup of
    // four row tiles per CU it runs four waves (K = 4096, two waves / four: 8192
    // wide 24.2 / 15.2, 14336 25.9 / 21.6; above, 17408 at 8 tokens 27.8 / 28.4,
    // 18432 27.6 / 29.2), of four where that nearly fills the CUs (16384: of two
    // 25.3, of four 24.1); the LM head two waves over as many row tiles as keep about a thousand
    // workgroups. Two or four slabs requested ahead per wave instead of one were
    // 1-10 % slower nearly everywhere: the waves of a CU keep enough in flight.
    // Activations are staged from 8 tokens on in the o and down projections, which
    // take no norm. WV depends on the shape only, never on M, so that a token's
    // result (its k order) does not depend on how many tokens share the call.
    // HS_SKINNY_CFG="<NF>,1,<WV>[,<XS>]" forces a choice (tuning only; read on
    // every call so that a sweep can change it between calls).
    const char* force = getenv("HS_SKINNY_CFG");
    const int cus = device_cus();
    int nf = 2, wv = 2, xs = 0;
    if (pe == EPI_F32) {
      while (nf < 8 && a.N / (16 * nf) > 1100) nf *= 2;
    } else if (pe == EPI_SWIGLU) {
      if (a.N / 64 >= cus + cus / 2) nf = 4;
      else if (a.N / 64 <= cus) wv = 4, nf = a.N / 64 > cus * 7 / 8 ? 4 : 2;
    } else if (pe == EPI_RESID) {
      if (a.N / 16 > cus) wv = 8;
      else nf = 1, wv = 16;
      if (!a.norm_gain && a.M >= 8) xs = nf == 1 && a.M > 12 ? 2 : 1;
    } else if (pe == EPI_STORE) {
      wv = a.N <= 8192 ? 8 : 4;
      if (a.N % 48 == 0 && a.N / 48 <= cus && a.N / 48 > cus * 3 / 4) nf = 3, wv = 16;
      else if (wv == 4 && a.N / 64 > cus * 3 / 4) nf = 4;
    }
    if (force && *force) sscanf(force, "%d,%*d,%d,%d", &nf, &wv, &xs);
    if (pe == EPI_SWIGLU && (nf % 2)) nf = 2;
    e = dispatch_skinny(a, pe, nf, wv, xs, s);
    if (e == hipSuccess && epi == EPI_QKV_ROPE) {
      RopeKvArgs r{static_cast<bf16_t*>(a.Y), a.ldy, a.rope_pos, a.rope_slot, a.rope_cos,
                   a.rope_sin, a.rope_pool, a.M, a.rope_q_cols / a.rope_d,
                   a.rope_kv_cols / a.rope_d, a.rope_d, a.rope_max_pos};
      e = rope_kv(r, s, nullptr);
    }
    snprintf(name, sizeof name, "gemm_skinny_%s%s", a.norm_gain ? "norm_" : "", kEpiName[epi]);
  } else {
    // Configuration by the time model of kRing.
    const int cus = device_cus();
    const int nk = (int)(kp / 64);
    auto tiles_of = [&](const RingCfg& c) {
      return (long)((a.N + c.bn - 1) / c.bn) * ((a.M + c.bm - 1) / c.bm);
    };
    // most workgroups per tile of a split launch: as many as the chip holds, at
    // least four slabs each; 1 where a split launch is not possible
    auto split_of = [&](const RingCfg& c, long tiles) -> long {
      const long sp = std::min<long>(cus / tiles, nk / 4);
      return c.s_slab > 0 && sp >= 2 && a.part && a.flags && tiles <= a.flags_n &&
                     tiles * sp * (int64_t)c.bn * c.bm <= a.part_floats
                 ? sp
                 : 1;
    };
    const RingCfg* cfg = nullptr;
    bool sk = false;
    double best = 1e300;
    for (const RingCfg& c : kRing) {
      // up to 64 rows only the 64-token tiles, for which every workspace of
      // more than 16 rows has room: the choice does not depend on its size
      if (a.M <= 64 && c.bm != 64) continue;
      const long tiles = tiles_of(c), rounds = (tiles + cus - 1) / cus, sp = split_of(c, tiles);
      const double whole =
          c.start + (double)nk * (rounds * c.slab + c.load * tiles / cus);
      const double split =
          sp > 1 ? c.s_start + (double)nk / sp * (c.s_slab + c.s_load * (tiles * sp) / cus) + c.s_each * sp
                 : 1e300;
      if (std::min(whole, split) < best) {
        best = std::min(whole, split);
        cfg = &c;
        sk = split < whole;
      }
    }
    long ways = sk ? split_of(*cfg, tiles_of(*cfg)) : 1;
    if (a.M <= 64 && cfg->bn == 64) {
      // How many ways to split a 64 x 64 tile, by times measured up to 64 rows: the
      // model above was fitted at 80 and more, where a way costs 2.5 us, here 0.6.
      // Beyond six the merge costs more than the shorter share saves. Whole ->
      // split, 17 rows: 1024 x 4096 17.4 -> 8.5 us, 2048 x 5632 23.7 -> 10.7, 3072 x
      // 3072 14.7 -> 9.4; eight ways -> six: 2048 x 8192 13.6 -> 12.6; but a K of 1024
      // stays whole (5504 x 1024 6.7, two ways 7.7).
      const long most = std::min<long>(6, split_of(*cfg, tiles_of(*cfg)));
      double t = 0.9 * (2.8 + 0.235 * nk);
      ways = 1;
      for (long w = 2; w <= most; ++w) {
        const double tw = 3.3 + 0.26 * nk / w + 0.58 * w;
        if (tw < t) t = tw, ways = w;
      }
    }
    int group = 8;
    if (forced) {
      std::string f(force_cfg);
      for (const RingCfg& c : kRing)  // longest matching name wins
        if (f.compare(0, strlen(c.name), c.name) == 0 &&
            (f.size() == strlen(c.name) || f[strlen(c.name)] == ','))
          cfg = &c;
      ways = sk ? split_of(*cfg, tiles_of(*cfg)) : 1;
      if (f.find(",dp") != std::string::npos) ways = 1;
      const size_t sp = f.find(",sk");
      if (sp != std::string::npos) {
        ways = split_of(*cfg, tiles_of(*cfg));
        const long n = atoi(f.c_str() + sp + 3);
        if (n > 0) ways = std::min(ways, n);
      }
      const size_t gp = f.find(",g");
      if (gp != std::string::npos) group = std::max(1, atoi(f.c_str() + gp + 2));
    }
    GemmSched sc;
    sc.tiles_n = (a.N + cfg->bn - 1) / cfg->bn;
    sc.tiles_m = (a.M + cfg->bm - 1) / cfg->bm;
    sc.nk = nk;
    sc.group_n = group;
    const long tiles = (long)sc.tiles_n * sc.tiles_m;
    sc.split = (int)ways;
    const long grid = tiles * sc.split;
    if (grid > 0x7FFFFFFF) return hipErrorInvalidValue;
    e = launch_ring(*cfg, a, epi, sc, (int)grid, s);
    split = sc.split > 1;
    snprintf(name, sizeof name, "gemm_r%s%s_%s", cfg->name, sc.split > 1 ? "sk" : "", kEpiName[epi]);
  }
  if (info) {
    info->name = name;
    info->flops = flops;
    info->bytes = bytes;
    info->split = split;
  }
  return e;
}

}  // namespace hs
