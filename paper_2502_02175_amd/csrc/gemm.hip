// Recomputed-row GEMMs of the sparse prefill and of the decode passes
// (Alg. 2 of VLA-Cache: K, V, and with them Q, O and the feed-forward, are
// computed for the rows outside P_reuse only; Sec. 3.1 for the projections).
//
// y[rows, N] = x[rows, K] . W[N, K]^T with few rows (tens to a few hundred)
// against large bf16 weights: the weights are the traffic, so the kernel is
// built to stream them from HBM exactly once at full rate.
//
//  * Weights and activations are both stored in fragment order (common.h), so
//    every operand fetch is one coalesced 16-byte load per lane and feeds a
//    v_mfma_f32_32x32x16_{bf16,f16} without any shuffling.
//  * The matrix-core A operand is the WEIGHT tile (32 output features x 16 k),
//    the B operand the activation tile (16 k x 32 rows); a lane of the result
//    holds one row and 4 x 4 consecutive features, which is what the fused
//    epilogues want (rotary partners, gate/up pairs and packed 8-byte stores in
//    one lane).
//  * The kernel for one stream's prefill (gemm_rows_kernel): weight tiles go global ->
//    registers (each is used by exactly one wave, LDS would add nothing), operand rows
//    global -> LDS directly by two waves that do nothing else.  K is split over pairs of
//    waves where the feature tiles are few, and over workgroups in the projections with a
//    residual, whose partial rows the next row kernel adds up in fixed order.
//  * Row counts live in device memory (they depend on the selection), the grid
//    is sized for the worst case and surplus workgroups leave at once.
//  * Workgroup ids are dealt round-robin to the 8 XCDs; row blocks of one weight
//    tile are mapped to the same XCD so that they share its L2.
#include <algorithm>
#include <cstring>
#include "gemm_epi.h"

// Workgroup: up to 6 consumer waves and 2 producer waves.  The consumers are fb feature blocks, or 2 or 3 of
// them x 2 parts of the K range (KP); a consumer streams the weight tiles of its block and part
// into registers, UK k-tiles ahead, and multiplies them by up to 8 row tiles whose operands it
// reads from LDS.  The producers copy those operands global -> LDS directly into a ring of
// ROWS_RING chunks, for nobody else's registers and nobody else's load queue: a wave's loads
// return in issue order, so row operands (from L2) fetched by the consumers themselves would wait
// behind weights from HBM, and storing them to LDS at every 64 k cost a barrier that all waves
// reached together (with both operands and the LDS reads taken out, that kernel's 172 workgroups
// still took 36 of the 49 us of the 7B gate/up projection at 109 rows: barriers, not memory).
// Here one barrier per chunk remains, and the data it publishes is needed a chunk later.
// What is left is the rate at which a CU fetches: a copy from L2 waits in one queue with the weights
// from HBM (a probe that does nothing else: 27 us for the weights alone, 10 for the row operands
// alone, 38 for both on 172 CUs, 34 on 256, whatever is in flight), so lanes of rows past the end
// copy nothing and the tiles are cut to use most CUs.  7B shape, 109 rows, before and now: gate/up
// 49.8 -> 41.7 us (4.3 TB/s of weights), QKV 41.2 -> 33.6, O 15 -> 14.4, FFN down 29 -> 26; four
// layers with the head 742 -> 628 us, 192 rows 908 -> 764.  32 weight tiles in flight: no faster.
// fb and the row blocks follow from the row count, in the kernel where only the device knows it
// (rows_cut): with two row blocks of 288 rows gate/up runs 230 workgroups of 6 feature blocks in one round
// instead of 460 of 3 in two, and QKV 256 of 3 instead of 384 of 2, both with K in two parts.
// Four layers of 7B and the head, before and now (later steps of the other kernels included): 288 rows known
// to the host 1008 -> 865 us, 440 rows (the many-rows kernel before) 1314 -> 1176; counted by the device
// 262 rows 1064 -> 936 (1008 with 2 blocks for QKV), 478 rows 1537 -> 1310 (1419).  (K of QKV or gate/up split over workgroups instead, the last
// wave to arrive adding up: 3 us per hand-over, 288 rows -58 us where this gave -120, 109 rows +10.)
// The arguments are read together at the start: the argument buffer lies in host memory, and an argument
// that is first read later is a round trip there (decode, 32 streams of grouped queries 1545 -> 1522 us,
// the tiny shape's step 284 -> 280, for the few-rows kernel and this one).
// A wave has 256 registers (up to 8 waves on 4 SIMDs).  No instance spills: fewer weight tiles in flight
// with 5 row tiles and more, the body of every row tile count kept apart from the others (see there),
// and only as many weight tiles asked for ahead of the choice of the body as every body keeps.
// (With 17 to 26 registers of every 16-bit instance spilled, 192 rows of 7B took 795 us per four
// layers and the head, now 764; 109 rows 635, now 628.)
constexpr int ROWS_RING = 5;       // chunks of at most 32 KiB: all 160 KiB of a CU's LDS
constexpr int ROWS_FB_MIN = 2, ROWS_FB_MAX = 6;  // feature blocks per workgroup: 2 (K in two parts) or 3 to 6
constexpr int ROWS_PAIR_NA = 6;  // most row tiles per wave with 2 feature blocks where others are in the choice
// The forms of the kernel.  K in two parts: 2 feature blocks per workgroup, 2 or 3 (QKV only); K whole: up to 4 (not
// QKV), up to 6.  (Where 2 are enough the form of 2 or 3 costs 0.4 us more of 5 at the tiny shape.)
enum { ROWS_PAIRS = 2, ROWS_THREES = 3, ROWS_FOUR = 4, ROWS_SIX = 6 };
constexpr int rows_parts(int form) { return form <= ROWS_THREES ? 2 : 1; }
constexpr int rows_consumers(int form) { return form == ROWS_SIX || form == ROWS_THREES ? 6 : 4; }
constexpr int rows_threads(int form) { return 64 * (rows_consumers(form) + 2); }

template <int NA, int KP, bool W8>
struct RowsShape {
  static constexpr int CT = (NA <= 4 ? 8 : 4) / KP;   // k-tiles per chunk and part
  static constexpr int TILES = KP * CT * NA;          // operand tiles (1 KiB) per chunk
  static constexpr int UK = NA <= 4 || W8 ? 16 : NA <= 6 ? 12 : 8;  // weight tiles in flight per consumer (16 bits: 1 KiB each)
  static constexpr int XR = NA <= 4 ? 2 : 1;          // k-tiles of row operands in registers
};

// The K range of part `part` of split `s`: in 64-k steps (4 k-tiles), the longer ones first
struct RowsRange { int k0, n; };
__device__ inline RowsRange rows_range(int KS, int parts, int idx) {
  const int q = KS / parts, r = KS - q * parts;
  return {4 * (idx * q + min(idx, r)), 4 * (q + (idx < r ? 1 : 0))};
}

template <int N>
__device__ inline void rows_wait() {
#ifdef VLAC_SAFE_WAITS
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
#else
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
#endif
}
// (waits for nothing by itself: a consumer's LDS reads of the chunk it leaves have been used by
// then, a producer has waited for its copies)
__device__ inline void rows_barrier() { asm volatile("s_barrier" ::: "memory"); }

// A producer wave (half = 0, 1): with two K parts the operand tiles of part `half`, else those of
// half the k-tiles of every chunk.  At the barrier that ends chunk c the chunks c + 1 and c + 2
// have landed.
template <int NA, int KP, bool W8>
__device__ __forceinline__ void rows_produce(const GemmArgs& a, uint4* lds, int half, int s, int rt0, int row_end) {
  using Sh = RowsShape<NA, KP, W8>;
  constexpr int PER = Sh::TILES / 2;  // copies of a chunk per producer
  static_assert((ROWS_RING - 3) * PER <= 63, "the counter holds 63");
  const int KC = 4 * a.KS;
  const uint32_t lane_off = (threadIdx.x & 63) * 16u;
  const uint32_t lds0 = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)lds) + (uint32_t)half * (PER * 1024u);
  const int n_max = __builtin_amdgcn_readfirstlane(rows_range(a.KS, a.S * KP, s * KP).n);
  const int n_ch = (n_max + Sh::CT - 1) / Sh::CT, n_bar = n_max / Sh::CT;
  RowsRange rg = rows_range(a.KS, a.S * KP, s * KP + (KP == 2 ? half : 0));
  rg.k0 = __builtin_amdgcn_readfirstlane(rg.k0);  // (uniform, but divided with vector instructions)
  rg.n = __builtin_amdgcn_readfirstlane(rg.n);
  const int kt0 = KP == 2 ? 0 : half * (Sh::CT / 2);
  const char* rows[NA];
#pragma unroll
  for (int m = 0; m < NA; ++m) rows[m] = (const char*)(a.xp + (size_t)min(rt0 + m, (row_end - 1) >> 5) * KC * 64);
  // (lanes of rows past the end copy nothing: their columns of the product are dropped; row 0 of the
  // last tile always exists, so every copy is issued and the count of copies in flight stays exact)
  const bool row_on = ((row_end - 1) & ~31) + (int)(threadIdx.x & 31) < row_end;
  auto copy = [&](uint32_t d, const char* src) {
    asm volatile(
        "s_mov_b32 m0, %0\n\t"
        "s_nop 0\n\t"
        "global_load_lds_dwordx4 %1, %2"
        :
        : "s"(d), "v"(lane_off), "s"(src)
        : "memory", "m0");
  };
  auto issue = [&](int c, int slot) {
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      // (past the end of the part: a tile that nobody reads)
      const int k = min(rg.k0 + min(c * Sh::CT + kt0 + u / NA, max(rg.n - 1, 0)), KC - 1);
      const char* src = rows[u % NA] + (size_t)k * 1024;
      const uint32_t d = lds0 + (uint32_t)(slot * Sh::TILES + u) * 1024u;
      if (u % NA < NA - 2) copy(d, src);  // (only the last tile can be ragged)
      else if (rt0 + u % NA < (row_end - 1) >> 5 || row_on) copy(d, src);
    }
  };
#pragma unroll
  for (int i = 0; i < ROWS_RING - 1; ++i)
    if (i < n_ch) issue(i, i);
  if (ROWS_RING - 1 <= n_ch) rows_wait<(ROWS_RING - 3) * PER>();
  else rows_wait<0>();
  rows_barrier();
  int slot = ROWS_RING - 1;
  for (int c = 0; c < n_bar; ++c) {
    if (c + ROWS_RING - 1 < n_ch) {
      issue(c + ROWS_RING - 1, slot);
      rows_wait<(ROWS_RING - 3) * PER>();
    } else {
      rows_wait<0>();
    }
    rows_barrier();
    slot = slot + 1 == ROWS_RING ? 0 : slot + 1;
  }
}

// A consumer's weight tiles in flight; the first 8 of up to 16 are asked for before the row count is
// known (e4m3 weights: two tiles to a 16-byte slot)
template <bool W8>
struct RowsWeights {
  static constexpr int N = W8 ? 8 : 16, EARLY = N / 2;
  uint4 t[N];
};

template <int NA, int KP, int FORM, int EPI, bool F16, bool W8>
__device__ __forceinline__ void rows_body(const GemmArgs& a, uint4* lds, RowsWeights<W8>& W, int fb, int tile, int s,
                                          int rt0, int row_end) {
  using Sh = RowsShape<NA, KP, W8>;
  constexpr bool IDS_EARLY = KP == 2 || NA <= 6;
  constexpr int CT = Sh::CT, UK = Sh::UK, XR = Sh::XR, CH = Sh::TILES * 64;
  // (Opaque copies of what addresses are made from: the bodies of all row tile counts are the
  // branches of one switch, and the compiler would else compute the addresses of all of them ahead
  // of it and spill.)
  int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  asm volatile("" : "+v"(lane), "+s"(w), "+s"(tile), "+s"(s), "+s"(rt0));
  const int part = FORM == ROWS_PAIRS ? w >> 1 : KP == 2 && w >= fb ? 1 : 0;
  const int nb = FORM == ROWS_PAIRS ? tile * 2 + (w & 1) : tile * fb + w - part * fb, g = lane >> 5;
  const bool wave_on = w < fb * KP && nb < a.NB;
  f32x16 acc[NA];
#pragma unroll
  for (int m = 0; m < NA; ++m)
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[m][i] = 0.f;

  int ids[NA];
#pragma unroll
  for (int m = 0; m < NA; ++m) ids[m] = 0;
  if (w >= rows_consumers(FORM)) {
    rows_produce<NA, KP, W8>(a, lds, w - rows_consumers(FORM), s, rt0, row_end);
  } else {
    RowsRange rg = rows_range(a.KS, a.S * KP, s * KP + part);
    // (opaque: simplified by KP = 1 the last steps keep more weight tiles alive, and spill)
    if constexpr (KP == 1) asm volatile("" : "+s"(rg.n));
    const int n_max = rows_range(a.KS, a.S * KP, s * KP).n, n = rg.n;
    const int n_min = KP == 1 ? n_max : rows_range(a.KS, a.S * KP, s * KP + KP - 1).n;
    // (e4m3 weights: a 16-byte lane slot holds two k-tiles)
    const int KC = 4 * a.KS;
    const uint4* wsrc = a.wp + ((size_t)min(nb, a.NB - 1) * (W8 ? KC / 2 : KC) + (W8 ? rg.k0 / 2 : rg.k0)) * 64 + lane;
#pragma unroll
    for (int i = RowsWeights<W8>::EARLY; i < (W8 ? UK / 2 : UK); ++i)
      if (i < (W8 ? n / 2 : n)) W.t[i] = ld_stream(wsrc + (size_t)i * 64);
    uint4 X[XR][NA];
    int slot = 0;
    const uint4 *cur = lds + (size_t)part * CT * NA * 64 + lane, *nxt = cur + CH;
    auto next_chunk = [&]() {
      rows_barrier();
      slot = slot + 1 == ROWS_RING ? 0 : slot + 1;
      cur = nxt;
      nxt = slot + 1 == ROWS_RING ? nxt - (ROWS_RING - 1) * CH : nxt + CH;
    };
    // k-tile t of a run of UK: the products, and behind each the read of the operand XR k-tiles on
    auto ktile = [&](int t, bool on) {
      uint4 wt;
      if constexpr (W8) wt = e4m3_slot_half(W.t[t >> 1], t & 1);
      else wt = W.t[t];
#pragma unroll
      for (int m = 0; m < NA; ++m) {
        if (on) acc[m] = mfma32<F16>(wt, X[t % XR][m], acc[m]);
        const int c = t % CT + XR;
        X[t % XR][m] = (c < CT ? cur + (c * NA + m) * 64 : nxt + ((c - CT) * NA + m) * 64)[0];
        __builtin_amdgcn_sched_barrier(0);
      }
    };
    auto reload = [&](int t, int k) {  // W.t[t] <- k-tile k (and k + 1)
      if constexpr (W8) {
        if (t & 1) W.t[t >> 1] = ld_stream(wsrc + (size_t)(k >> 1) * 64);
      } else {
        W.t[t] = ld_stream(wsrc + (size_t)k * 64);
      }
    };
    if (IDS_EARLY && EPI != EPI_LOGITS && !(EPI == EPI_RESID && a.S > 1)) {
      // (asked for here, used by the epilogue: one round trip less at the end, where registers are left)
#pragma unroll
      for (int m = 0; m < NA; ++m) ids[m] = a.e.rows[min((rt0 + m) * 32 + (lane & 31), row_end - 1)];
    }
    rows_barrier();
#pragma unroll
    for (int x = 0; x < XR; ++x)
#pragma unroll
      for (int m = 0; m < NA; ++m) X[x][m] = cur[(x * NA + m) * 64];
    // Runs without a branch inside (the compiler then counts the loads in flight exactly); the last
    // full run and the rest step by 64 k and ask for no weights past the end.
    int base = 0;
    for (; base + 2 * UK <= n_min; base += UK) {
#pragma unroll
      for (int t = 0; t < UK; ++t) {
        ktile(t, true);
        reload(t, base + t + UK);
        if ((t + 1) % CT == 0) next_chunk();
      }
    }
    for (; base < n_max; base += UK) {
#pragma unroll
      for (int u = 0; u < UK; u += 4) {
        const int k = base + u;
        if (k < n_max) {
          const bool on = k < n;
#pragma unroll
          for (int t = u; t < u + 4; ++t) {
            if (on) ktile(t, true);
            if ((t + 1) % CT == 0) next_chunk();
          }
          if (k + UK < n) {
#pragma unroll
            for (int t = u; t < u + 4; ++t) reload(t, k + (t - u) + UK);
          }
        }
      }
    }
  }

  if constexpr (KP == 2) {
    // The parts' sums meet in LDS: part 0 finishes the first NH row tiles, part 1 the others
    // (sum = first part + second part).
    constexpr int NH = (NA + 1) / 2;
    __syncthreads();
    const int at = FORM == ROWS_PAIRS ? w & 3 : w, from = FORM == ROWS_PAIRS ? at ^ 2 : part ? w - fb : w + fb;
    float* mine = (float*)lds + (size_t)at * (NH * 16 * 64) + lane;
    const float* theirs = (const float*)lds + (size_t)from * (NH * 16 * 64) + lane;
    if (w < 2 * fb) {
#pragma unroll
      for (int m = 0; m < NA; ++m)
        if ((m >= NH) != (part == 1)) {
#pragma unroll
          for (int i = 0; i < 16; ++i) mine[((m >= NH ? m - NH : m) * 16 + i) * 64] = acc[m][i];
        }
    }
    __syncthreads();
    if (w < 2 * fb) {
#pragma unroll
      for (int m = 0; m < NA; ++m)
        if ((m >= NH) == (part == 1)) {
#pragma unroll
          for (int i = 0; i < 16; ++i) acc[m][i] += theirs[((m >= NH ? m - NH : m) * 16 + i) * 64];
        }
    }
  }
  if (!wave_on) return;
  if (!IDS_EARLY && EPI != EPI_LOGITS && !(EPI == EPI_RESID && a.S > 1)) {
#pragma unroll
    for (int m = 0; m < NA; ++m) ids[m] = a.e.rows[min((rt0 + m) * 32 + (lane & 31), row_end - 1)];
  }
  [[maybe_unused]] float gates = 0.f;
#pragma unroll
  for (int m = 0; m < NA; ++m) {
    if (KP == 2 && (m >= (NA + 1) / 2) != (part == 1)) continue;
    if constexpr (W8) scale_tile(a.wscale, nb, g, acc[m]);
    const int row = (rt0 + m) * 32 + (lane & 31);
    if (row >= row_end) continue;
    if (EPI == EPI_RESID && a.S > 1) {
      // Projection + residual with split K: every split writes its partial rows
      // [split][row][feature] and is done; the row kernel that follows (residual add +
      // RMSNorm) adds the splits up, so nothing is handed over between workgroups.
      float* dst = a.e.rpart + ((size_t)s * a.e.rpart_rows + row) * a.e.d_model + nb * 32 + 4 * g;
#pragma unroll
      for (int q4 = 0; q4 < 4; ++q4)
        *(float4*)(dst + 8 * q4) =
            make_float4(acc[m][4 * q4], acc[m][4 * q4 + 1], acc[m][4 * q4 + 2], acc[m][4 * q4 + 3]);
    } else {
      EpiIn<EPI> in;
      epilogue_load<EPI>(a.e, nb, ids[m], g, in);
      epilogue_store<EPI, F16>(a.e, nb, row, ids[m], g, acc[m], in);
      if constexpr (EPI == EPI_SWIGLU) gates = largest_gate(acc[m], gates);
    }
  }
  if constexpr (EPI == EPI_SWIGLU)
    if (__builtin_expect(__any(gates > kFarGate), 0)) {
#pragma unroll
      for (int m = 0; m < NA; ++m) {
        const int row = (rt0 + m) * 32 + (lane & 31);
        if ((KP == 2 && (m >= (NA + 1) / 2) != (part == 1)) || row >= row_end) continue;
        epilogue_store<EPI, F16, true>(a.e, nb, row, ids[m], g, acc[m], {});
      }
    }
}

// How a row count (in tiles of 32, at most 32 of them) is cut: feature blocks per workgroup and row
// blocks, 4 bits each in GemmArgs::cut, worked out by the host (rows_cut).
struct RowsCut { int fb, blocks; };
__host__ __device__ inline RowsCut rows_cut_of(uint64_t cut0, uint64_t cut1, int n_rt) {
  const int i = (n_rt - 1) & 31;
  const int code = (int)((i < 16 ? cut0 : cut1) >> (4 * (i & 15))) & 15;
  return {ROWS_FB_MIN + (code >> 1), code & 1 ? (n_rt + 7) >> 3 : (n_rt + 5) / 6};
}
__host__ __device__ inline int rows_tiles(int NB, int fb) {  // (divisions by constants)
  return fb == 2 ? (NB + 1) / 2 : fb == 3 ? (NB + 2) / 3 : fb == 4 ? (NB + 3) / 4 : fb == 5 ? (NB + 4) / 5 : (NB + 5) / 6;
}

template <int FORM, int EPI, bool F16, bool W8>
__global__ __launch_bounds__(rows_threads(FORM)) void gemm_rows_kernel(GemmArgs a) {
  extern __shared__ uint4 lds[];  // [ROWS_RING][part][k-tile][row tile][64]
  // Workgroup id -> (row block, weight tile, split); id % 8 is the XCD, and the row blocks of one
  // weight tile sit next to each other on it, so that they fetch it from HBM once.  The blocks are
  // those that the row count gives, not those that the grid has room for: its surplus workgroups
  // come last.  (With the blocks of an unknown count one behind the other the weights came from HBM
  // once per block: 211 rows of 7B, 1037 us per four layers, then 935; 408 rows 1640 and 1422.)
  // Where the count is in device memory the first weights are asked for as if there were one block
  // and the feature blocks per workgroup of few rows, which is the rule, and once more if it is not so.
  // (A loop, so that both go to the same registers: written one behind the other they are merged by
  // copies, and a copy of a register waits for the load that fills it.)
  uint64_t cut0 = a.cut[0], cut1 = a.cut[1];
  asm volatile("" : "+s"(cut0), "+s"(cut1));  // (read here; else the one that is needed is read when the count is known)
  read_args(a.xp, a.e.rows);
  RowsWeights<W8> W;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  constexpr int KP = rows_parts(FORM);
  constexpr int FB = FORM == ROWS_PAIRS ? 2 : EPI == EPI_RESID || EPI == EPI_LOGITS ? 4 : 0;  // (one for all counts)
  int n_rows = a.n_rows_val, n_rt = 0, n_blk = 1, mb = 0, fb = FB ? FB : a.fb_first, tile, s;
#pragma unroll 1
  for (;;) {
    int p = blockIdx.x;
    if (n_rows >= 0) {
      // row tiles are dealt in equal shares to as few blocks of at most 6, or of at most 8, as hold them
      n_rt = (n_rows + 31) >> 5;
      if (n_rt == 0 || n_rows >= a.rows_hi) return;  // (rows_hi and more: the many-rows kernel's share)
      const RowsCut cut = rows_cut_of(cut0, cut1, n_rt);
      const bool asked = a.n_rows_val < 0 && cut.blocks == 1 && (FB || cut.fb == fb);
      n_blk = cut.blocks;
      if (!FB) fb = cut.fb;
      if (n_blk > 1) {
        const int y = blockIdx.x >> 3;
        mb = y % n_blk;
        p = (y / n_blk) * 8 + (blockIdx.x & 7);
      }
      if (p >= rows_tiles(a.NB, fb) * a.S) return;
      if (asked) break;  // (the weights asked for are the right ones)
    }
    tile = __builtin_amdgcn_readfirstlane(p / a.S);
    s = __builtin_amdgcn_readfirstlane(p - tile * a.S);
    if (w < fb * KP && tile * fb < a.NB) {
      const int part = FORM == ROWS_PAIRS ? w >> 1 : KP == 2 && w >= fb ? 1 : 0;
      const RowsRange rg = rows_range(a.KS, a.S * KP, s * KP + part);
      const int nb = min(FORM == ROWS_PAIRS ? tile * 2 + (w & 1) : tile * fb + w - part * fb, a.NB - 1), kc = W8 ? 2 * a.KS : 4 * a.KS, k0 = W8 ? rg.k0 / 2 : rg.k0;
      const uint4* src = a.wp + (size_t)nb * kc * 64 + (threadIdx.x & 63);
      // (past the end of K the last tile is read again and not used)
#pragma unroll
      for (int i = 0; i < RowsWeights<W8>::EARLY; ++i) W.t[i] = ld_stream(src + (size_t)min(k0 + i, kc - 1) * 64);
    }
    if (n_rows >= 0) break;
    // (a scalar load, written by the kernels before this one: a vector load would wait for the weights)
    n_rows = ld_scalar(a.n_rows);
  }
  if (!FB) fb = __builtin_amdgcn_readfirstlane(fb);
  if (FORM != ROWS_PAIRS && w >= fb * KP && w < rows_consumers(FORM)) return;  // no feature block for this wave
  tile = __builtin_amdgcn_readfirstlane(tile);
  s = __builtin_amdgcn_readfirstlane(s);
  const int rt0 = __builtin_amdgcn_readfirstlane(mb * n_rt / n_blk);
  const int rt1 = __builtin_amdgcn_readfirstlane((mb + 1) * n_rt / n_blk), row_end = min(n_rows, 32 * rt1);
#define VLAC_NA(N) rows_body<N, KP, FORM, EPI, F16, W8>(a, lds, W, fb, tile, s, rt0, row_end)
  switch (rt1 - rt0) {
    case 1: VLAC_NA(1); break;
    case 2: VLAC_NA(2); break;
    case 3: VLAC_NA(3); break;
    case 4: VLAC_NA(4); break;
    case 5: VLAC_NA(5); break;
    case 6: VLAC_NA(6); break;
    case 7: VLAC_NA(7); break;
    default: VLAC_NA(8);
  }
#undef VLAC_NA
}

// ---------------------------------------------------------------------------
// At most 32 rows (the decode passes, the output head): one 32-feature block
// per workgroup, the 4 waves split its K range and add up through LDS, so the
// main loop has no barrier and no LDS traffic at all: every wave streams its
// own contiguous run of weight tiles, two batches of 8 KiB in flight, and reads
// the matching activation tiles straight from L2 (only the lanes of real rows
// load anything).  With S > 1 the K range is also split over S workgroups
// (N = d_model gives only d/32 blocks); the partial tiles are 4 KiB each.
// Where the input is the residual stream and there are at most 4 rows, its RMSNorm is
// done here as well: every workgroup normalises the rows itself (from L2, while its first
// weight tiles are in flight) and keeps the operand slices of its K range in LDS, which
// saves a launch per GEMM in the decode loop.  Split-K partial rows that the previous
// projection left behind are added to the rows on the way (in a fixed order, the same in
// every workgroup), and workgroup 0 stores the completed rows for the next projection.
// ---------------------------------------------------------------------------
// XMODE: where the row operand comes from.
//   X_GLOBAL  every lane loads its 16 bytes of the 32-row operand tile from L2 (any row count)
//   X_NORM4/8 RMSNorm of fp32 rows of at most 4096 / 8192 elements, slices [k/8][row] in LDS
enum { X_GLOBAL = 0, X_NORM4 = 1, X_NORM8 = 2 };

template <int EPI, bool F16, int XMODE, bool W8>
__global__ __launch_bounds__(256, XMODE == X_NORM8 ? 2 : 3) void gemm_few_kernel(GemmArgs a) {
  __shared__ float red[3][16][64];
  extern __shared__ uint4 xlds[];  // operand slices [k/8 - lo8][row]
  constexpr int U = 8;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  read_epilogue_args<EPI>(a);
  const int nb = blockIdx.x / a.S, s = blockIdx.x - nb * a.S;
  const int n_rows = min(a.n_rows_val >= 0 ? a.n_rows_val : *a.n_rows, 32);
  if (n_rows <= 0) return;
  const int KC = 4 * a.KS;
  // (e4m3 weights come two k-tiles to a 16-byte slot: ranges start and end on even tiles)
  const int ev = W8 ? 1 : 0;
  const int per = ((KC + a.S - 1) / a.S + ev) & ~ev, c_lo = s * per, c_hi = min(KC, c_lo + per);
  const int perw = ((max(c_hi - c_lo, 0) + 3) / 4 + ev) & ~ev, w_lo = c_lo + w * perw,
            w_hi = min(c_hi, w_lo + perw);
  const uint4* wsrc = a.wp + (size_t)nb * (W8 ? KC / 2 : KC) * 64 + lane;
  const uint4* xsrc = a.xp + lane;
  const int lo8 = 2 * c_lo, n8 = 2 * max(c_hi - c_lo, 0);  // this workgroup's k/8 range

  f32x16 acc;
#pragma unroll
  for (int i = 0; i < 16; ++i) acc[i] = 0.f;
  uint4 bw[2][U], ax[2][U];
  // Loads are unconditional and never touch the loaded data (past the end of the range
  // the weight index is clamped and the activation tile is replaced by a tile of zeros),
  // so the compiler keeps a whole batch in flight behind the MFMAs.  Lanes of rows >=
  // n_rows read the tile of zeros as well (1 KiB that stays in L1): with 8 rows a wave
  // then fetches 256 bytes of operand rows per k-tile from L2 instead of 1 KiB, as much
  // as its weight tile.
  const bool row_lane = (lane & 31) < n_rows;
  auto load = [&](int c, uint4(&b)[U], uint4(&x)[U]) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int cc = max(min(c + u, w_hi - 1), 0);
      if constexpr (!W8) b[u] = ld_stream(wsrc + (size_t)cc * 64);
      else if (u < U / 2) b[u] = ld_stream(wsrc + (size_t)max(min((c >> 1) + u, (w_hi >> 1) - 1), 0) * 64);
      if constexpr (XMODE == X_GLOBAL) {
        const uint4* xs = (c + u < w_hi && row_lane) ? xsrc + (size_t)cc * 64 : a.zero_tile + lane;
        x[u] = *xs;
      }
    }
  };
  auto compute = [&](int c, uint4(&b)[U], uint4(&x)[U]) {
    if constexpr (XMODE != X_GLOBAL) {
      const int j = lane & 31, g = lane >> 5;
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int cc = max(min(c + u, w_hi - 1), 0);
        x[u] = (j < n_rows && c + u < w_hi) ? xlds[(cc * 2 + g - lo8) * n_rows + j]
                                            : make_uint4(0, 0, 0, 0);
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if constexpr (W8) acc = mfma32<F16>(e4m3_slot_half(b[u >> 1], u & 1), x[u], acc);
      else acc = mfma32<F16>(b[u], x[u], acc);
    }
  };

  // Loads return in issue order: row 0, the gains and the first two splits of its partial
  // rows are requested BEFORE the first two batches of weight tiles, which then fly while
  // the row is normalised.
  constexpr int MAXI = XMODE == X_NORM8 ? 8 : 4;  // 4 values per thread and 1024 of the row
  [[maybe_unused]] float4 v[MAXI], gn[MAXI], t0[MAXI], t1[MAXI];
  if constexpr (XMODE != X_GLOBAL) {
    const NormIn& nm = a.norm;
    const size_t pstride = (size_t)nm.part_rows * nm.d;
#pragma unroll
    for (int i = 0; i < MAXI; ++i) {
      const int k = tid * 4 + i * 1024;
      v[i] = gn[i] = t0[i] = t1[i] = make_float4(0.f, 0.f, 0.f, 0.f);
      if (k < nm.d) {
        v[i] = *(const float4*)(nm.src + k);
        gn[i] = *(const float4*)(nm.gain + k);
        if (nm.part_S > 0) t0[i] = *(const float4*)(nm.part + k);
        if (nm.part_S > 1) t1[i] = *(const float4*)(nm.part + pstride + k);
      }
    }
  }
  __builtin_amdgcn_sched_barrier(0);
  load(w_lo, bw[0], ax[0]);
  load(w_lo + U, bw[1], ax[1]);
  __builtin_amdgcn_sched_barrier(0);

  if constexpr (XMODE != X_GLOBAL) {
    // RMSNorm of the rows: x * rsqrt(mean(x^2) + eps) * g, with x = source row + partial
    // rows in split order.  One pass over each row: every thread keeps its values in
    // registers, the sum of squares goes through LDS.
    const NormIn& nm = a.norm;
    const int d = nm.d;
    const size_t pstride = (size_t)nm.part_rows * d;
    auto add4 = [](float4& x, const float4& y) { x.x += y.x; x.y += y.y; x.z += y.z; x.w += y.w; };
    auto finish_row = [&](int j) {
#pragma unroll
      for (int i = 0; i < MAXI; ++i) {
        add4(v[i], t0[i]);
        add4(v[i], t1[i]);
      }
      for (int ss = 2; ss < nm.part_S; ++ss) {
#pragma unroll
        for (int i = 0; i < MAXI; ++i) {
          const int k = tid * 4 + i * 1024;
          if (k < d) add4(v[i], *(const float4*)(nm.part + ss * pstride + (size_t)j * d + k));
        }
      }
      if (nm.dst && blockIdx.x == 0) {
#pragma unroll
        for (int i = 0; i < MAXI; ++i) {
          const int k = tid * 4 + i * 1024;
          if (k < d) *(float4*)(nm.dst + (size_t)j * nm.dst_stride + k) = v[i];
        }
      }
      float ss = 0.f;
#pragma unroll
      for (int i = 0; i < MAXI; ++i)
        ss += v[i].x * v[i].x + v[i].y * v[i].y + v[i].z * v[i].z + v[i].w * v[i].w;
      for (int o = 32; o > 0; o >>= 1) ss += __shfl_xor(ss, o);
      __syncthreads();  // red is free again
      if (lane == 0) red[0][0][w] = ss;
      __syncthreads();
      const float r =
          rsqrtf((red[0][0][0] + red[0][0][1] + red[0][0][2] + red[0][0][3]) / (float)d + nm.eps);
#pragma unroll
      for (int i = 0; i < MAXI; ++i) {
        const int k = tid * 4 + i * 1024, k8 = k >> 3;
        if (k8 >= lo8 && k8 < lo8 + n8) {  // k >= d: zeros (K padding)
          uint2* dst = (uint2*)&xlds[(k8 - lo8) * n_rows + j];
          dst[(k >> 2) & 1] = make_uint2(pack_op2<F16>(v[i].x * r * gn[i].x, v[i].y * r * gn[i].y),
                                         pack_op2<F16>(v[i].z * r * gn[i].z, v[i].w * r * gn[i].w));
        }
      }
    };
    // row 0 apart from the loop: its loads are older than the weight tiles, and code
    // shared with the later rows would wait for those as well
    finish_row(0);
    for (int j = 1; j < n_rows; ++j) {
#pragma unroll
      for (int i = 0; i < MAXI; ++i) {
        const int k = tid * 4 + i * 1024;
        if (k < d) {
          v[i] = *(const float4*)(nm.src + (size_t)j * nm.src_stride + k);
          if (nm.part_S > 0) t0[i] = *(const float4*)(nm.part + (size_t)j * d + k);
          if (nm.part_S > 1) t1[i] = *(const float4*)(nm.part + pstride + (size_t)j * d + k);
        }
      }
      finish_row(j);
    }
    __syncthreads();
  }

  // The batch a compute phase needs must have been issued BEFORE the batch that flies
  // behind it; the fences stop the instruction scheduler from mixing the phases (which
  // would drain the queue every iteration).  The last two batches ask for nothing more: loads
  // past the end of the range (clamped to its last tile) would be real traffic.
  int c = w_lo;
  for (; c + 2 * U < w_hi; c += 2 * U) {
    compute(c, bw[0], ax[0]);
    __builtin_amdgcn_sched_barrier(0);
    load(c + 2 * U, bw[0], ax[0]);
    __builtin_amdgcn_sched_barrier(0);
    compute(c + U, bw[1], ax[1]);
    __builtin_amdgcn_sched_barrier(0);
    load(c + 3 * U, bw[1], ax[1]);
    __builtin_amdgcn_sched_barrier(0);
  }
  compute(c, bw[0], ax[0]);
  compute(c + U, bw[1], ax[1]);

  if (w > 0) {
#pragma unroll
    for (int i = 0; i < 16; ++i) red[w - 1][i][lane] = acc[i];
  }
  __syncthreads();
  if (w > 0) return;
#pragma unroll
  for (int i = 0; i < 16; ++i) acc[i] += red[0][i][lane] + red[1][i][lane] + red[2][i][lane];
  if constexpr (W8) scale_tile(a.wscale, nb, lane >> 5, acc);

  if (EPI == EPI_RESID && a.S > 1) {
    // the split's partial rows [split][row][feature] are left for the consumer (the fused
    // norm of the next projection, or the residual + norm row kernel) to add up: nothing is
    // handed over in here
    const int slot = lane & 31, g = lane >> 5;
    if (slot < n_rows) {
      float* dst = a.e.rpart + ((size_t)s * a.e.rpart_rows + slot) * a.e.d_model + nb * 32 + 4 * g;
#pragma unroll
      for (int q4 = 0; q4 < 4; ++q4)
        *(float4*)(dst + 8 * q4) =
            make_float4(acc[4 * q4], acc[4 * q4 + 1], acc[4 * q4 + 2], acc[4 * q4 + 3]);
    }
    return;
  }
  if (a.S > 1) {  // wave 0 alone hands over / collects the partial tile
    float* base = a.partial + (size_t)nb * a.S * 1024;
#pragma unroll
    for (int i = 0; i < 16; ++i) st_coherent(base + (size_t)s * 1024 + i * 64 + lane, acc[i]);
    stores_done();
    int last = 0;
    if (lane == 0) {
      const int old = atomicAdd(a.counters + nb, 1);
      last = (old == a.S - 1);
      if (last) a.counters[nb] = 0;
    }
    last = __shfl(last, 0);
    if (!last) return;
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[i] = 0.f;
    for (int ss = 0; ss < a.S; ++ss) {  // fixed order, 16 loads in flight
      float t[16];
#pragma unroll
      for (int i = 0; i < 16; ++i) t[i] = ld_coherent(base + (size_t)ss * 1024 + i * 64 + lane);
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[i] += t[i];
    }
  }
  const int slot = lane & 31;
  if (slot < n_rows) {
    const int id = (EPI == EPI_LOGITS) ? 0
                   : (a.e.decode_pos >= 0 ? ((slot << 16) | a.e.decode_pos) : a.e.rows[slot]);
    epilogue_tile<EPI, F16>(a.e, nb, slot, id, lane >> 5, acc);
  }
}

// The same for rows that do not have their norm made here (5 to 32 of them, and any number in the projections with a
// residual), with FB feature blocks per workgroup: the
// operand rows, as many bytes per k-tile as a weight tile when there are 32 of them, come from L2 once for
// all FB blocks, and FB is what gives the chip whole rounds of workgroups (few_blocks).  K is dealt to the
// workgroups and waves, and their sums added, as in gemm_few_kernel: the results are the same bits.
// Bound by the fetch rate of a CU.  32 rows of grouped queries (d_model 1536), before and now: gate/up, 560
// blocks, 16.6 -> 13.9 us; FFN down, 288 -> 144 workgroups, 12.5 -> 10.7; head 23.7 -> 19.3.  7B,
// gate/up of 8 rows 31.2 -> 29.7, of 32 rows 34.7 -> 29.7; QKV of 32 rows 26.0 -> 23.8.
template <int EPI, bool F16, bool W8, int FB>
__global__ __launch_bounds__(256, FB == 3 ? 1 : 2) void gemm_few_wide_kernel(GemmArgs a) {
  constexpr int U = FB == 4 ? 4 : 8, UW = W8 ? U / 2 : U;
  __shared__ float red[4][FB][16][64];
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  read_epilogue_args<EPI>(a);
  const int nb0 = blockIdx.x / a.S * FB, s = blockIdx.x % a.S;
  const int n_rows = min(a.n_rows_val >= 0 ? a.n_rows_val : *a.n_rows, 32);
  if (n_rows <= 0) return;
  const int KC = 4 * a.KS;
  // (as in gemm_few_kernel)
  const int ev = W8 ? 1 : 0;
  const int per = ((KC + a.S - 1) / a.S + ev) & ~ev, c_lo = s * per, c_hi = min(KC, c_lo + per);
  const int perw = ((max(c_hi - c_lo, 0) + 3) / 4 + ev) & ~ev, w_lo = c_lo + w * perw, w_hi = min(c_hi, w_lo + perw);
  const uint4* wsrc[FB];
#pragma unroll
  for (int f = 0; f < FB; ++f) wsrc[f] = a.wp + (size_t)min(nb0 + f, a.NB - 1) * (W8 ? KC / 2 : KC) * 64 + lane;
  const uint4* xsrc = a.xp + lane;
  const bool row_lane = (lane & 31) < n_rows;
  f32x16 acc[FB];
#pragma unroll
  for (int f = 0; f < FB; ++f)
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[f][i] = 0.f;
  uint4 bw[2][FB][UW], ax[2][U];
  auto load = [&](int c, uint4(&b)[FB][UW], uint4(&x)[U]) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int cc = max(min(c + u, w_hi - 1), 0), ch = max(min((c >> 1) + u, (w_hi >> 1) - 1), 0);
#pragma unroll
      for (int f = 0; f < FB; ++f)
        if (u < UW) b[f][u] = ld_stream(wsrc[f] + (size_t)(W8 ? ch : cc) * 64);
      const uint4* xs = (c + u < w_hi && row_lane) ? xsrc + (size_t)cc * 64 : a.zero_tile + lane;
      x[u] = *xs;
    }
  };
  auto compute = [&](uint4(&b)[FB][UW], uint4(&x)[U]) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int f = 0; f < FB; ++f) {
        if constexpr (W8) acc[f] = mfma32<F16>(e4m3_slot_half(b[f][u >> 1], u & 1), x[u], acc[f]);
        else acc[f] = mfma32<F16>(b[f][u], x[u], acc[f]);
      }
  };
  load(w_lo, bw[0], ax[0]);
  load(w_lo + U, bw[1], ax[1]);
  __builtin_amdgcn_sched_barrier(0);
  int c = w_lo;
  for (; c + 2 * U < w_hi; c += 2 * U) {
    compute(bw[0], ax[0]);
    __builtin_amdgcn_sched_barrier(0);
    load(c + 2 * U, bw[0], ax[0]);
    __builtin_amdgcn_sched_barrier(0);
    compute(bw[1], ax[1]);
    __builtin_amdgcn_sched_barrier(0);
    load(c + 3 * U, bw[1], ax[1]);
    __builtin_amdgcn_sched_barrier(0);
  }
  compute(bw[0], ax[0]);
  compute(bw[1], ax[1]);

  // wave f finishes block f
#pragma unroll
  for (int f = 0; f < FB; ++f)
    if (f != w) {
#pragma unroll
      for (int i = 0; i < 16; ++i) red[w][f][i][lane] = acc[f][i];
    }
  __syncthreads();
#pragma unroll
  for (int f = 0; f < FB; ++f) {
    const int nb = nb0 + f, slot = lane & 31, g = lane >> 5;
    if (f != w || nb >= a.NB) continue;
    f32x16 t;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      float p[4];
#pragma unroll
      for (int ww = 0; ww < 4; ++ww) p[ww] = ww == f ? acc[f][i] : red[ww][f][i][lane];
      t[i] = p[0] + (p[1] + p[2] + p[3]);
    }
    if constexpr (W8) scale_tile(a.wscale, nb, g, t);
    if (slot < n_rows) {
      if (EPI == EPI_RESID && a.S > 1) {
        float* dst = a.e.rpart + ((size_t)s * a.e.rpart_rows + slot) * a.e.d_model + nb * 32 + 4 * g;
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4)
          *(float4*)(dst + 8 * q4) = make_float4(t[4 * q4], t[4 * q4 + 1], t[4 * q4 + 2], t[4 * q4 + 3]);
      } else {
        const int id = (EPI == EPI_LOGITS) ? 0 : (a.e.decode_pos >= 0 ? ((slot << 16) | a.e.decode_pos) : a.e.rows[slot]);
        epilogue_tile<EPI, F16>(a.e, nb, slot, id, g, t);
      }
    }
  }
}

// Feature blocks per workgroup of the kernels for up to 32 rows (1: gemm_few_kernel).  Taken is the least estimate of
// rounds of 256 workgroups x what a workgroup fetches per k-tile, in 32nds of a KiB: a weight tile of 16-bit operands is
// 32; the operand rows, which come from L2, count a sixth of their bytes.  A last round that is not full costs half of what
// is missing (one block per workgroup, three workgroups to a CU: three quarters); 32 rounds' worth of start and end.
// An even number of blocks pays for weights whose workgroups' runs start a multiple of 256 KiB apart: all of them
// ask the same few channels, above all with a power of two between two blocks.  (The K parts of the projections with a
// residual start apart.)  A hand-over between workgroups (K split, no residual) is made by gemm_few_kernel only.
// Measured over 6400 launches of 7 to 340 us (K 256 to 17920, 32 to 4752 blocks, 1 to 32 rows, 16- and 8-bit weights): on
// average 4.8 % faster than one block each, 1.2 % of them more than 5 % slower (at most 18 %: K 512, 1344 blocks, 32 rows 18.9
// and 22.3 us).  One block against several, us: K 2048, 512 blocks, 8 rows 15.7 and 17.9 (one is taken), 4008 blocks 88
// and 105 (one); K 4096, 896 blocks, 16 rows 43.8 and 48.3 (one), 688 blocks, 8 rows 33.5 and 32.8 (three), 384 blocks, 32
// rows 26.3 and 23.7 (two); K 1536, 1000 blocks, 32 rows 25.9 and 21.1 (four); K 2560, 1000 blocks, 8-bit weights, 8 rows
// 20.8 and 19.4 (four).  The projections with a residual come here with 1 to 4 rows too: K 8960, 48 blocks in 6
// parts, 1 row 12.0 and 11.7 (two).  QKV with few k-tiles to a wave, K 512, 480 blocks, 32 rows 10.6 and 11.7 (one).
static int few_blocks(int epi, int n_blocks, int KS, int S, int rows, bool w8) {
#ifdef VLAC_SAFE_WAITS
  return 1;  // (gemm_few_wide_kernel adds in the same order: a test compares the two libraries bit for bit)
#endif
  const int KC = 4 * KS;
  if (S > 1 && epi != EPI_RESID) return 1;
  if (epi == EPI_QKV && KC < (w8 ? 64 : 48)) return 1;
  int best = 1;
  double least = 0;
  for (int fb = 1; fb <= (epi == EPI_LOGITS ? 4 : 3); ++fb) {
    const int n = (n_blocks + fb - 1) / fb * S, full = (n + 255) / 256 * 256, weight = fb * (w8 ? 16 : 32);
    const bool same = epi != EPI_RESID && fb % 2 == 0 && KC * weight % 8192 == 0, most = (KC & (KC - 1)) == 0 && n_blocks >= 512;
    const double rounds = fb == 1 ? 0.25 * n + 0.75 * full : 0.5 * (n + full);
    const double fetch = weight * (!same ? 1. : most ? 1.25 : 1.03) + rows / 6. + 0.4;
    const double cost = (rounds * fetch + 32 * 256) * (fb == 1 ? 1. : fb == 3 ? 1.035 : 1.015);  // (3: one workgroup per CU)
    if (fb == 1 || cost < least) { least = cost; best = fb; }
  }
  return best;
}

static const int kRowsLds = ROWS_RING * 32 * 1024;

template <int FORM, int EPI>
static hipError_t set_attr() {
  hipError_t e = hipFuncSetAttribute((const void*)gemm_rows_kernel<FORM, EPI, false, false>,
                                     hipFuncAttributeMaxDynamicSharedMemorySize, kRowsLds);
  if (e != hipSuccess) return e;
  e = hipFuncSetAttribute((const void*)gemm_rows_kernel<FORM, EPI, true, false>,
                          hipFuncAttributeMaxDynamicSharedMemorySize, kRowsLds);
  if (e != hipSuccess) return e;
  return hipFuncSetAttribute((const void*)gemm_rows_kernel<FORM, EPI, true, true>,
                             hipFuncAttributeMaxDynamicSharedMemorySize, kRowsLds);
}

int gemm_init() {
  hipError_t e;
#define VLAC_SET(FORM)                                                    \
  if ((e = set_attr<FORM == ROWS_FOUR ? ROWS_THREES : FORM, EPI_QKV>()) != hipSuccess) return (int)e; \
  if ((e = set_attr<FORM, EPI_SWIGLU>()) != hipSuccess) return (int)e;
  VLAC_SET(ROWS_PAIRS) VLAC_SET(ROWS_FOUR) VLAC_SET(ROWS_SIX)
  if ((e = set_attr<ROWS_PAIRS, EPI_RESID>()) != hipSuccess) return (int)e;
  if ((e = set_attr<ROWS_FOUR, EPI_RESID>()) != hipSuccess) return (int)e;
  if ((e = set_attr<ROWS_FOUR, EPI_LOGITS>()) != hipSuccess) return (int)e;
#undef VLAC_SET
  return gemm_tall_init();
}

template <int FORM, int EPI, bool F16, bool W8>
static void launch_rows_one(const GemmArgs& a, int grid, hipStream_t st) {
  hipLaunchKernelGGL((gemm_rows_kernel<FORM, EPI, F16, W8>), dim3(grid), dim3(rows_threads(FORM)), kRowsLds, st, a);
}
// (which forms a projection has: see above; the projections with a residual take 2 or 4 feature blocks, the head 4)
template <int FORM, bool F16, bool W8>
static void launch_rows(int epi, const GemmArgs& a, int grid, hipStream_t st) {
  constexpr int QKV = FORM == ROWS_FOUR ? ROWS_SIX : FORM, GATE_UP = FORM == ROWS_THREES ? ROWS_PAIRS : FORM,
                RESID = FORM == ROWS_PAIRS ? ROWS_PAIRS : ROWS_FOUR;
  switch (epi) {
    case EPI_QKV: launch_rows_one<QKV, EPI_QKV, F16, W8>(a, grid, st); break;
    case EPI_RESID: launch_rows_one<RESID, EPI_RESID, F16, W8>(a, grid, st); break;
    case EPI_SWIGLU: launch_rows_one<GATE_UP, EPI_SWIGLU, F16, W8>(a, grid, st); break;
    default: launch_rows_one<ROWS_FOUR, EPI_LOGITS, F16, W8>(a, grid, st); break;
  }
}

template <bool F16, int XMODE, bool W8>
static void launch_few(int epi, const GemmArgs& a, int grid, size_t shm, hipStream_t st) {
  switch (epi) {
    case EPI_QKV:
      hipLaunchKernelGGL((gemm_few_kernel<EPI_QKV, F16, XMODE, W8>), dim3(grid), dim3(256), shm, st, a);
      break;
    case EPI_RESID:
      hipLaunchKernelGGL((gemm_few_kernel<EPI_RESID, F16, XMODE, W8>), dim3(grid), dim3(256), shm, st, a);
      break;
    case EPI_SWIGLU:
      hipLaunchKernelGGL((gemm_few_kernel<EPI_SWIGLU, F16, XMODE, W8>), dim3(grid), dim3(256), shm, st, a);
      break;
    default:
      hipLaunchKernelGGL((gemm_few_kernel<EPI_LOGITS, F16, XMODE, W8>), dim3(grid), dim3(256), shm, st, a);
      break;
  }
}

template <bool F16, bool W8>
static void launch_few_wide(int epi, int fb, const GemmArgs& a, hipStream_t st) {
  const dim3 grid((a.NB + fb - 1) / fb * a.S), block(256);
#define VLAC_WIDE(EPI_, FB_) hipLaunchKernelGGL((gemm_few_wide_kernel<EPI_, F16, W8, FB_>), grid, block, 0, st, a)
#define VLAC_WIDE_FB(EPI_)            \
  {                                   \
    if (fb == 2) VLAC_WIDE(EPI_, 2);  \
    else VLAC_WIDE(EPI_, 3);          \
  }                                   \
  break
  switch (epi) {
    case EPI_QKV: VLAC_WIDE_FB(EPI_QKV);
    case EPI_RESID: VLAC_WIDE_FB(EPI_RESID);
    case EPI_SWIGLU: VLAC_WIDE_FB(EPI_SWIGLU);
    default:
      if (fb == 4) VLAC_WIDE(EPI_LOGITS, 4);
      else VLAC_WIDE_FB(EPI_LOGITS);
  }
#undef VLAC_WIDE_FB
#undef VLAC_WIDE
}

// LDS budget of the normalised rows (on top of 12 KiB of static LDS)
static const size_t kStageBytes = 49152;

bool gemm_can_fuse_norm(int n_rows_host, int decode_pos, int kpad) {
  return n_rows_host >= 1 && n_rows_host <= 4 && decode_pos >= 0 && kpad <= 8192 &&
         (size_t)(kpad / 8) * n_rows_host * 16 <= kStageBytes;
}

// From this many rows on (the capacity of the launch: streams x tokens; the actual row count of a
// sparse prefill is known on the device only) the GEMMs go to the kernel built for matrix-core bound
// work.  Full recomputes, four layers and the head, many-rows against one-stream kernel: 7B, 352 rows
// 1069 and 941 us, 448 rows 1211 and 1154, 500 rows 1376 and 1323; grouped queries, 380 rows 589
// and 472, 500 rows 636 and 578.  Decode passes of many streams, four layers, two tokens of 7B: 353 streams 3404 and 2960,
// 400 streams 3708 and 3427, 500 streams 4260 and 4077; three tokens of grouped queries: 353 streams
// 1918 and 1492, 500 streams 2157 and 1933.  (Weights stored as e4m3 codes: the many-rows kernel
// multiplies fp16 operands, its instances for such weights only apply the scales to the results; up to 1023 rows stay with
// the one-stream kernel, from 1024 rows on the matrix is expanded to fp16 before every launch, 3 bytes of traffic per
// weight against the 2 rows flops per weight that such a launch spends on it.)
static const int kTallRows = 512;
static bool use_tall(const vlac_ctx* c, int rows_cap) {
  return c->w8 ? rows_cap >= 1024 && c->wdeq : rows_cap >= kTallRows;
}

// Most splits the many-rows GEMM with a residual epilogue may use (they need S partial rows
// of fp32 per row in the workspace, and the row kernel that keeps a row in registers)
static int tall_resid_smax(const vlac_ctx* c, int epi, int rows_cap, int d_model) {
  if (epi != EPI_RESID || d_model > 8192) return 1;
  const size_t fit = c->rpart_floats / ((size_t)rows_cap * d_model);
  return fit >= 8 ? 8 : fit >= 3 ? (int)fit : 1;
}

// Feature blocks per workgroup of the projections with a residual, which split K besides (2 leave K
// to two pairs of waves): 4 blocks and 8 splits where K is long, which fetches a third less per
// workgroup but doubles the partial rows; 2 blocks and half the splits where it is not.
static int rows_resid_fb(int n_blocks, int KS) { return KS >= 128 && n_blocks >= 128 ? 4 : 2; }

// Row blocks of the one-stream kernel at most (see rows_cut)
static int rows_blocks_max(int rows) { return ((rows + 31) / 32 + 5) / 6; }

// Split factor of the one-stream kernel: the projections with a residual, whose partial rows the
// row kernel that follows adds up, split K.  Taken is the split with the least rounds of 256
// workgroups x (a workgroup's steps of 64 k, and 4 for its start and end); a workgroup keeps at
// least 4 steps.  The blocks that multiply the workgroups are known with the row count; where only
// its bound is known every count of blocks up to that weighs the same.  (With the split that gives
// one block a workgroup per CU, two blocks took two rounds: grouped queries with 8-bit weights, 28
// layers, 384 rows 3607 us, now 3226; at most 288 rows, 262 recomputed, 3230 and 2825.)
// The others do not split over workgroups: a hand-over between them costs more than idle CUs.
static int rows_kernel_splits(const vlac_ctx* c, int epi, int n_blocks, int KS, int rpart_rows, int d_model, int rows_most,
                              bool known) {
  if (epi != EPI_RESID) return 1;
  const int tiles = rows_tiles(n_blocks, rows_resid_fb(n_blocks, KS)), most = rows_blocks_max(rows_most);
  int best = 1, least = 0x7fffffff;
  for (int S = 1; S <= 8 && S <= std::max(KS / 4, 1) && (size_t)S * rpart_rows * d_model <= c->rpart_floats; ++S) {
    int cost = 0;
    for (int n = known ? most : 1; n <= most; ++n) cost += (tiles * S * n + 255) / 256 * ((KS + S - 1) / S + 4);
    if (cost < least) { least = cost; best = S; }
  }
  return best;
}

// Where the many-rows kernel serves a capacity at which a sparse prefill usually leaves few rows
// (the count is known on the device only), BOTH kernels are launched for a GEMM: up to
// kSmallRows - 1 rows the one-stream kernel works, from there on the other, and the idle one leaves at
// once, which costs 3 us per GEMM (456 rows, 7B: 1346 us for four layers and the head without the idle one, 1357
// with it).  So both are launched only where the reuse lists are long enough to
// leave fewer than kFewRows rows (top-k 100 of two camera views is not), and up to a capacity
// of 767 rows: at 70 % static about 0.38 of it is recomputed, more than that and the second launch would
// mostly be the idle one.  Two streams of 288 tokens with long lists used in part (rows counted on the
// device), four layers and the head, one-stream against many-rows kernel, us:
//   rows        258          320          384          448
//   7B f16      945 1110     991 1142    1085 1199    1180 1337
//   7B bf16                  (296 rows: 958 1129)    1061 1175    1149 1311
//   grouped q.  437  610     454  616     494  626     516  656
// (7B, about 142 rows 742 and 964, 218 rows 879 and 1036; one stream of 720 tokens, 270 rows 1005 and 1164, 420 rows
// 1216 and 1387.)  The K splits of the one-stream kernel are those of up to kFewRows - 1 rows, which is what
// such a call usually has (chosen over all counts up to kSmallRows - 1, grouped queries took 479 us at 258 rows, 543 at 384).
static const int kSmallRows = 449, kFewRows = 257;
// (Rows longer than 8192 elements: the row kernel that adds the partial rows up there takes a
// fixed split factor, so the choice between two kernels with different factors is not offered.)
static bool use_both(const vlac_ctx* c, int rows_cap, int n_rows_host) {
  return use_tall(c, rows_cap) && !c->w8 && n_rows_host < 0 && rows_cap < 768 && c->rows_floor < kFewRows &&
         c->cfg.d_model <= 8192;
}

SplitAdapt gemm_resid_adapt(vlac_ctx* c, int n_blocks, int kpad, int rows_cap, const int* n_rows, int n_rows_host) {
  SplitAdapt ad = {nullptr, nullptr, 0, 0, 0};
  if (!use_tall(c, rows_cap)) return ad;
  const int d_model = n_blocks * 32, S_max = tall_resid_smax(c, EPI_RESID, rows_cap, d_model);
  const bool both = use_both(c, rows_cap, n_rows_host);
  if (n_rows_host >= 0) {
    if (S_max > 1) ad.S_known = tall_plan((n_blocks + 7) >> 3, n_rows_host, S_max, kpad / 64).S;
  } else if (both || S_max > 1) {
    ad.split = c->split;
    ad.n_rows = n_rows;
    if (both) {
      ad.small_below = kSmallRows;
      ad.S_small = rows_kernel_splits(c, EPI_RESID, n_blocks, kpad / 64, rows_cap, d_model, kFewRows - 1, false);
    }
  }
  return ad;
}

// With fewer workgroups than this even two feature blocks each leave the chip half empty: then 2 it is, whatever the
// row count (grouped queries, QKV of 64 blocks, 211 and 288 rows: 3 and 4 blocks 14 and 19 us per four layers slower)
static const int kRowsPairTiles = 128;

// How the one-stream kernel cuts `rt` row tiles (at most 32: 1023 rows) and NB feature blocks: blocks of
// at most 6 or 8 row tiles, feature blocks per workgroup 2 (QKV: or 3) with K in two parts and 3 to 6 with K whole (the
// projections with a residual: as given, with their S splits).  A workgroup takes a CU's whole LDS, so
// what counts is rounds of 256 workgroups x what a workgroup fetches per k (its weight rows, a block's
// operand rows; a CU fetches about 50 GB/s with weights from HBM and row operands from L2 in one queue).
// (7 row tiles of 7B QKV are faster with 3 feature blocks in two row blocks than with 2 in one, 6 with 2)
struct RowsChoice { RowsCut cut; int code, cost; };
static RowsChoice rows_cut(int epi, int NB, int KS, int S, int rt, int k_parts) {
  RowsChoice best = {{0, 0}, 0, 0x7fffffff};
  const bool pairs_only = epi != EPI_QKV || rows_tiles(NB, 2) < kRowsPairTiles;
  const int fix = epi == EPI_LOGITS ? 4 : epi == EPI_RESID ? rows_resid_fb(NB, KS) : 0;
  const int lo = fix ? fix : k_parts == 2 ? 2 : 3, hi = fix ? fix : k_parts == 1 ? ROWS_FB_MAX : pairs_only ? 2 : 3;
  for (int fb = lo; fb <= hi; ++fb) {
    for (int eight = 0; eight < 2; ++eight) {
      const int n = eight ? (rt + 7) / 8 : (rt + 5) / 6, na = (rt + n - 1) / n;
      if (fb == 2 && hi > 2 && na > ROWS_PAIR_NA) continue;
      const int cost = (rows_tiles(NB, fb) * S * n + 255) / 256 * (fb + na) + n - 1;
      if (cost < best.cost) best = {{fb, n}, (fb - ROWS_FB_MIN) << 1 | eight, cost};
    }
  }
  return best;
}

// K in two parts where two feature blocks per workgroup fit one round of the chip.  It is so for every row count
// that the device decides, so that a row's result does not depend on how many others are recomputed; where the host
// knows the count K may stay whole if that is cheaper (8-bit weights, 600 rows of 7B: QKV in one round instead of two).
static int rows_k_parts(int epi, int NB, int KS, int rt_known) {
  if (NB > 512) return 1;
  if (!rt_known || rows_tiles(NB, 2) < kRowsPairTiles) return 2;
  return rows_cut(epi, NB, KS, 1, rt_known, 1).cost < rows_cut(epi, NB, KS, 1, rt_known, 2).cost ? 1 : 2;
}

// the one-stream kernel for up to rows_cap rows, K split as for up to rows_split of them; sets and returns a.S
static int launch_rows_kernel(vlac_ctx* c, int epi, GemmArgs& a, int rows_cap, int rows_split, const GemmEpi& e, hipStream_t st) {
  a.S = rows_kernel_splits(c, epi, a.NB, a.KS, e.rpart_rows, e.d_model, rows_split, a.n_rows_val >= 0);
  const int rt_cap = std::min((rows_cap + 31) / 32, 32), rt_known = a.n_rows_val >= 0 ? (a.n_rows_val + 31) / 32 : 0;
  const int k_parts = rows_k_parts(epi, a.NB, a.KS, rt_known);
  a.cut[0] = a.cut[1] = 0;
  int grid = 0, fb_most = 0;
  for (int rt = rt_known ? rt_known : 1; rt <= (rt_known ? rt_known : rt_cap); ++rt) {
    const RowsChoice ch = rows_cut(epi, a.NB, a.KS, a.S, rt, k_parts);
    const RowsCut cut = ch.cut;
    a.cut[(rt - 1) >> 4] |= (uint64_t)ch.code << (4 * ((rt - 1) & 15));
    if (rt <= 4) a.fb_first = cut.fb;  // (what few rows usually get)
    fb_most = std::max(fb_most, cut.fb);
    grid = std::max(grid, (rows_tiles(a.NB, cut.fb) * a.S + 7) / 8 * 8 * cut.blocks);
  }
#define VLAC_ROWS(FORM_)                                                                  \
  {                                                                                       \
    if (c->w8) launch_rows<FORM_, true, true>(epi, a, grid, st);                   \
    else if (c->f16) launch_rows<FORM_, true, false>(epi, a, grid, st);            \
    else launch_rows<FORM_, false, false>(epi, a, grid, st);                       \
  }
  if (fb_most == 2) VLAC_ROWS(ROWS_PAIRS)
  else if (epi == EPI_QKV && k_parts == 2) VLAC_ROWS(ROWS_THREES)
  else if (fb_most <= 4) VLAC_ROWS(ROWS_FOUR)
  else VLAC_ROWS(ROWS_SIX)
#undef VLAC_ROWS
  return a.S;
}

int launch_gemm(vlac_ctx* c, int epi, const bf16_t* wp, const float* wscale, int n_blocks, int kpad,
                const bf16_t* xp,
                 const int* n_rows, int n_rows_host, int rows_cap, const GemmEpi& e, hipStream_t st,
                 const NormIn* norm) {
  GemmArgs a;
  a.wp = (const uint4*)wp;
  a.wscale = c->w8 ? wscale : nullptr;
  a.xp = (const uint4*)xp;
  a.zero_tile = (const uint4*)c->zero_tile;
  a.NB = n_blocks;
  a.KS = kpad / 64;
  a.n_rows = n_rows;
  a.n_rows_val = n_rows_host;
  a.rows_lo = 0;
  a.rows_hi = 0x7fffffff;
  memset(&a.norm, 0, sizeof(a.norm));
  if (norm) a.norm = *norm;
  a.partial = c->partial;
  a.counters = c->counters;
  a.split = c->split;
  a.e = e;
  const int cls = rows_cap <= 32 ? 0 : 1;
  const bool timed = c->prof_kind == epi + 4 * cls && c->prof_n < c->prof_cap;
  if (timed) (void)hipEventRecord(c->prof_start[c->prof_n], st);
  if (cls == 0) {
    // one workgroup per 32-feature block; K is split over workgroups only when there
    // are fewer blocks than CUs, and never below 32 k-tiles (8 per wave) per workgroup
    const int KC = kpad / 16;
    int S = (256 + n_blocks - 1) / n_blocks;
    if (S > KC / 32) S = KC / 32;
    if (S > 8) S = 8;
    if (S < 1 || n_blocks > c->n_counters || (size_t)n_blocks * 8 * 1024 > c->partial_floats) S = 1;
    a.S = S;
    const int grid = n_blocks * S;
    if (norm) {  // only offered when gemm_can_fuse_norm() holds
      // LDS for the normalised rows: this workgroup's share of K, [k/8][row] 16-byte slices
      const int per = ((KC + S - 1) / S + (c->w8 ? 1 : 0)) & ~(c->w8 ? 1 : 0);  // as in the kernel
      const size_t shm = (size_t)(2 * per) * n_rows_host * 16;
      if (norm->d <= 4096) {
        if (c->w8) launch_few<true, X_NORM4, true>(epi, a, grid, shm, st);
        else if (c->f16) launch_few<true, X_NORM4, false>(epi, a, grid, shm, st);
        else launch_few<false, X_NORM4, false>(epi, a, grid, shm, st);
      } else {
        if (c->w8) launch_few<true, X_NORM8, true>(epi, a, grid, shm, st);
        else if (c->f16) launch_few<true, X_NORM8, false>(epi, a, grid, shm, st);
        else launch_few<false, X_NORM8, false>(epi, a, grid, shm, st);
      }
    } else if (const int fb = few_blocks(epi, n_blocks, a.KS, S, n_rows_host >= 0 ? n_rows_host : rows_cap, c->w8); fb > 1) {
      if (c->w8) launch_few_wide<true, true>(epi, fb, a, st);
      else if (c->f16) launch_few_wide<true, false>(epi, fb, a, st);
      else launch_few_wide<false, false>(epi, fb, a, st);
    } else {
      if (c->w8) launch_few<true, X_GLOBAL, true>(epi, a, grid, 0, st);
      else if (c->f16) launch_few<true, X_GLOBAL, false>(epi, a, grid, 0, st);
      else launch_few<false, X_GLOBAL, false>(epi, a, grid, 0, st);
    }
  } else if (use_tall(c, rows_cap)) {
    int S_small = 0;
    if (use_both(c, rows_cap, n_rows_host)) {
      GemmArgs r = a;
      r.rows_hi = kSmallRows;
      S_small = launch_rows_kernel(c, epi, r, kSmallRows - 1, kFewRows - 1, e, st);
      a.rows_lo = kSmallRows;
    }
    if (c->w8) {
      launch_expand_e4m3(a.wp, (uint4*)c->wdeq, (size_t)n_blocks * 2 * a.KS, st);
      a.wp = (const uint4*)c->wdeq;
    }
    // (the projections with a residual may split K and leave partial rows to the next row kernel)
    launch_gemm_tall(c->f16, epi, a, rows_cap, tall_resid_smax(c, epi, rows_cap, e.d_model), st);
    if (S_small > a.S) a.S = S_small;  // (the caller learns the most splits either kernel may leave)
  } else {
    launch_rows_kernel(c, epi, a, rows_cap, rows_cap, e, st);
  }
  if (timed) {
    (void)hipEventRecord(c->prof_stop[c->prof_n], st);
    (void)hipEventRecord(c->prof_mark[c->prof_n++], st);  // marker after marker: the bracket's own cost
  }
  return a.S;
}
