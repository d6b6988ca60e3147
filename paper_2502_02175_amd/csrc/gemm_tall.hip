// Recomputed-row GEMMs with MANY rows (batched streams: thousands of rows per layer;
// Alg. 2 of VLA-Cache over the rows outside P_reuse of every stream at once).
//
// With thousands of rows the weights are no longer the traffic: the GEMM is bound by the
// matrix cores, and behind them by what reaches a CU from L2 (measured here: 20 to 27 bytes
// per clock and CU), so the operand bytes fetched per MFMA are what has to be kept small.
// A work item is 256 features x 256 rows (16 KiB of operands per 64 MFMAs), and both operand
// tiles are shared through LDS:
//
//  * 4 waves, one per SIMD; a wave owns 4 feature blocks x 4 row tiles = 16 accumulator
//    tiles (256 accumulator registers), and one k-tile is 16 MFMAs for 8 operand fragments
//    read from LDS.
//  * Operands are in fragment order (common.h): a tile is 1 KiB that a wave copies global ->
//    LDS as it lies (global_load_lds_dwordx4: lane l's 16 bytes land at base + 16 l) and
//    reads back with one 16-byte LDS read per lane, conflict-free.
//  * A stage is 32 k: at 256 x 256, 16 weight tiles + 16 activation tiles = 32 KiB; a ring of 5
//    stages (all 160 KiB of a CU's LDS), copies run 4 stages ahead (lower items: stages of 28 and 24
//    KiB, 5 and 6 of them, see TallRing).  Every wave copies a quarter of a stage, 8, 7 or 6 tiles,
//    whatever the row count (tiles past the end are clamped to a valid one and never read), so
//    that the number of copies in flight is the same for every wave at every step:
//    the copies are inline assembly that the compiler does not see (it treats its own
//    LDS-direct loads as aliasing every LDS read and drains the load queue at each), and
//    their waits are placed by hand (tall_wait; a build with -DVLAC_SAFE_WAITS waits for
//    everything instead and must give the same bits).
//  * One barrier per stage, placed behind the first MFMA of its second k-tile: the fragments
//    of a k-tile are read while the MFMAs of the one before run, across the barrier as well.
//  * The grid is one workgroup per CU; a workgroup runs its work items one after the other
//    and copies the first stages of the next item during the last steps of the one before.
//  * Row blocks of 192 or 128 rows (a wave owns 4 x 3 or 4 x 2 tiles), and K split in up to 8
//    parts in the projections with a residual (whose consumer, residual add + RMSNorm, adds
//    the partial rows up), where that takes less time by the estimate of tall_plan, which the kernel
//    evaluates on the device from the actual row count; it leaves the K parts for the consumer to read.
//  * Behind its last product an item has the CU to itself (one wave per SIMD), so what it does with its sums
//    counts in full.  The sums stay in their registers until a tile's turn (copied out of them all at once
//    behind the loop, they spilled 80 to 110 registers); what an epilogue reads is asked for ahead of the stores
//    of the row tile before it; and where a lane's access would be a cache line of its own (residual rows, partial
//    rows, rotary factors) the tile goes through 4 KiB of LDS, so that 4 or 8 lanes share a line.  What is left
//    per item of 8 x 1057 tokens (7B; products 80 to 100 us): SwiGLU 4.5 us, QKV 10 (L2 requests), residual rows
//    10.5 (memory).  Whole calls before and after: 8 x 1057 tokens of 7B 4853 -> 4659 us, 32 x 304 of grouped
//    queries 2847 -> 2633, 601 tokens of 7B 1303 -> 1268.
//  * Measured against this design and not kept: a 512-feature x 128-row item with the weight
//    tiles fetched global -> registers by 8 waves (20 KiB per 64 MFMAs: 5 to 8 % slower at
//    the 7B layer shape with 2700 to 8400 rows, equal at d_model 1536); rings of 4 stages
//    (equal); all copies of a stage issued together instead of one per MFMA (7 % slower: a
//    wave's copies and LDS reads hold up its own MFMAs); hardware dispatch of one workgroup
//    per item (equal at K 4096, 5 % slower at K 1536, where an item is short).  With the
//    copies or the LDS reads taken out (wrong results, timing only) the gate/up GEMM at 2712
//    rows goes from 440 to 362 and 422 us, with both out to 346 us: the matrix cores
//    themselves, with one barrier per stage and the last of 3.7 rounds of items a partial
//    one, do not get past 0.57 of the published peak on this chip.
#include "gemm_epi.h"

namespace {

// Per item shape (FW feature blocks and RT row tiles per wave): a stage is 4 FW weight tiles and
// 4 RT activation tiles, a quarter of which each wave copies; as many stages as a CU's 160 KiB of
// LDS hold.
template <int FW, int RT>
struct TallRing {
  static constexpr int COPIES = FW + RT;           // copies (1 KiB) per stage and wave
  static constexpr int STAGE = 256 * COPIES;       // uint4 per stage: 32, 28 or 24 KiB
  static constexpr int N = 160 / (4 * COPIES);     // stages: 5, 5 or 6
  static constexpr int YOUNGER = COPIES * (N - 2); // copies behind the stage a step waits for
  static_assert(YOUNGER <= 63, "the counter holds 63");
};
typedef float f32x4 __attribute__((ext_vector_type(4)));
constexpr int kTallLds = 160 * 1024;
template <int N>
__device__ inline void tall_wait() {
#ifdef VLAC_SAFE_WAITS
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
#else
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
#endif
}
// Between a wave's stores to LDS and its reads of what other lanes stored (and between those reads and the next stores):
// the compiler, which sees one lane, may else move one past the other.  No instruction: a wave's LDS accesses are worked
// off in order.
__device__ __forceinline__ void lanes_exchange() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");
  __builtin_amdgcn_wave_barrier();
}
// Waits here for a load that not every path goes on to use.  Left open it would be waited for where its register is
// written next, in the loop of the item after: with every copy that is younger, at each of its steps.
template <class T>
__device__ __forceinline__ void arrived(const T& v) { asm volatile("" ::"v"(v)); }
constexpr int kTallGrid = 256;          // one workgroup per CU (a workgroup takes all of a CU's LDS)

// A work item: weight tile, K part, row block
struct TallItem { int tile, s, mb; };

// RT: row tiles per wave (4: blocks of 256 rows, 3: of 192, 2: of 128); NA: how many of them hold rows.
// Runs item `it`; `nx` is the item this workgroup runs next (chain: there is one, and the last
// RING - 1 steps of this item copy its first stages instead of stages past the end).
// prefilled: the copies of this item's first RING - 1 stages have been issued already (by
// the item before) into the ring from `slot` on.  Returns the ring slot after the last stage.
template <int FW, int RT, int NA, int EPI, bool F16, bool W8>
__device__ __forceinline__ int tall_body(const GemmArgs& a, uint4* lds, TallItem it, TallItem nx, bool chain,
                                          bool prefilled, int slot, int n_rows, int S) {
  constexpr int RING = TallRing<FW, RT>::N, STAGE = TallRing<FW, RT>::STAGE, C = TallRing<FW, RT>::COPIES;
  constexpr int AHEAD = RING - 1;  // stages that the copies run ahead
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wi = w & 1, wj = w >> 1;  // feature half, row interleave
  const int KC = 4 * a.KS;
  // part s of S of the 32-k steps of K
  const int sq = (2 * a.KS) / S, sr = (2 * a.KS) % S;
  const int step0 = it.s * sq + min(it.s, sr), n_steps = sq + (it.s < sr ? 1 : 0);
  const int step0n = nx.s * sq + min(nx.s, sr), n_steps_n = sq + (nx.s < sr ? 1 : 0);
  const int row0 = it.mb * (64 * RT);
  const int nb0 = it.tile * (2 * FW);
  // A stage in LDS: the 2 FW feature blocks, then the 2 RT row tiles, both k-tiles of each (2 KiB that
  // lie together in global memory as well).  Wave w copies the C = FW + RT KiB from w C on.
  // (scalar base addresses: a copy is then one scalar select, one scalar add and the load, with
  // the lane's 16-byte offset in one register for all of them; a wave has one instruction stream,
  // and what a copy costs to issue is taken from its MFMAs)
  const char *src[C], *srcn[C];
  const uint32_t dst0 = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)lds) + (uint32_t)(w * C) * 1024u;
  const uint32_t lane_off = (uint32_t)lane * 16u;
#pragma unroll
  for (int j = 0; j < C; ++j) {
    const int c = w * C + j, row = c >> 1, half = c & 1;
    auto base = [&](int tile, int mb, int step) {
      const uint4* t = row < 2 * FW ? a.wp + ((size_t)min(tile * (2 * FW) + row, a.NB - 1) * KC + 2 * step) * 64
                               : a.xp + ((size_t)min(mb * (2 * RT) + row - 2 * FW, a.x_tiles - 1) * KC + 2 * step) * 64;
      return (const char*)t + half * 1024;
    };
    src[j] = base(it.tile, it.mb, step0);
    srcn[j] = base(nx.tile, nx.mb, step0n);
  }
  // copy j of this wave's C of stage i.
  // Stages past this item's last are the next item's first (chain), else its last again
  // (never read): the number of copies per step is the same at every step.
  auto copy_one = [&](int i, int slot_, int j) {
    const bool mine = i < n_steps || !chain;
    const size_t k = (size_t)(mine ? min(i, n_steps - 1) : min(i - n_steps, n_steps_n - 1)) * 2048;  // 2 k-tiles of 1 KiB
    const char* sp = (mine ? src[j] : srcn[j]) + k;
    const uint32_t d = dst0 + (uint32_t)slot_ * (STAGE * 16) + (uint32_t)j * 1024u;
    asm volatile(
        "s_mov_b32 m0, %0\n\t"
        "s_nop 0\n\t"
        "global_load_lds_dwordx4 %1, %2"
        :
        : "s"(d), "v"(lane_off), "s"(sp)
        : "memory", "m0");
  };

  constexpr int NX = NA > 0 ? NA : 1;
  f32x16 acc[FW][NX];
#pragma unroll
  for (int f = 0; f < FW; ++f)
#pragma unroll
    for (int m = 0; m < NX; ++m)
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[f][m][i] = 0.f;

  // Fragments of a k-tile: weight blocks FW wi + f, row tiles 2 m + wj of the block (the two
  // row halves interleave, so that a ragged last block splits evenly).  A wave has one
  // instruction stream and nothing else runs on its SIMD, so whatever is not an MFMA is
  // issued BETWEEN the MFMAs of a k-tile, one piece after each: the LDS reads of the next
  // k-tile's fragments (FW + NA of them) and the copies of a stage.
  uint4 W0[FW], X0[NX], W1[FW], X1[NX];
  auto read_one = [&](const uint4* s, int q, uint4(&Wf)[FW], uint4(&Xf)[NX]) {
#pragma unroll
    for (int f = 0; f < FW; ++f)
      if (q == f) Wf[f] = s[(FW * wi + f) * 128];
#pragma unroll
    for (int m = 0; m < NA; ++m)
      if (q == FW + m) Xf[m] = s[FW * 256 + (2 * m + wj) * 128];
  };

  // Copies in flight: C per stage and wave.  When step i needs stage i + 1 (at its barrier)
  // the stages i + 2 .. i + RING - 1 have been asked for behind it: "at most C (RING - 2)
  // outstanding" means that this wave's part of stage i + 1 has landed, and the barrier makes
  // that all four parts.  The same barrier says that every wave has read all of stage i (its
  // LDS reads are waited for before it), whose slot the copies of stage i + RING may then
  // overwrite; they are issued during step i + 1.  Stages are numbered on through a chain of
  // items, so all of this holds across the item boundary as well: the barrier of an item's
  // last step is the one that waits for the next item's stage 0.  (Other vector-memory
  // operations of the wave, the epilogue's, are all younger or all older than the copies a
  // step waits for; loads return in issue order, so they can only make a wait longer.)
  if (!prefilled) {
    int sl = slot;
#pragma unroll
    for (int i = 0; i < AHEAD; ++i) {
#pragma unroll
      for (int j = 0; j < C; ++j) copy_one(i, sl, j);
      sl = sl + 1 == RING ? 0 : sl + 1;
    }
    tall_wait<TallRing<FW, RT>::YOUNGER>();
    __syncthreads();
  }
  if constexpr (NA > 0) {
#pragma unroll
    for (int q = 0; q < FW + NA; ++q) read_one(lds + slot * STAGE + lane, q, W0, X0);
  }
  int i = 0;
  do {  // (an item has at least one step; a loop that might have none would copy the sums behind it)
    const int slot_next = slot + 1 == RING ? 0 : slot + 1, slot_copy = slot == 0 ? RING - 1 : slot - 1;
    const uint4* cur = lds + slot * STAGE + lane;
    const uint4* nxt = lds + slot_next * STAGE + lane;
    // k-tile 0 of stage i (fragments W0, X0); meanwhile: read k-tile 1, copy stage i + AHEAD
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int q = 0; q < FW * NX; ++q) {
      if constexpr (NA > 0) acc[q / NX][q % NX] = mfma32<F16>(W0[q / NX], X0[q % NX], acc[q / NX][q % NX]);
      if constexpr (NA > 0) read_one(cur + 64, q, W1, X1);
      if constexpr (FW * NX >= C) {  // one copy after each of the last C MFMAs
        if (q >= FW * NX - C) copy_one(i + AHEAD, slot_copy, q - (FW * NX - C));
      } else {                      // fewer MFMAs than copies: some are followed by two
#pragma unroll
        for (int j = 0; j < C; ++j)
          if (j * FW * NX / C == q) copy_one(i + AHEAD, slot_copy, j);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    if constexpr (NA > 0) {
#pragma unroll
      for (int q = FW * NX; q < FW + NA; ++q) read_one(cur + 64, q, W1, X1);  // (NA = 1: 5 reads, 4 MFMAs)
    }
    // k-tile 1 (W1, X1): its first MFMA covers the barrier; then read k-tile 0 of stage i + 1
    // (after the last step: of a stage that is not this item's; the next item reads its own)
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int q = 0; q < FW * NX; ++q) {
      if constexpr (NA > 0) acc[q / NX][q % NX] = mfma32<F16>(W1[q / NX], X1[q % NX], acc[q / NX][q % NX]);
      if (q == 0) {
        tall_wait<TallRing<FW, RT>::YOUNGER>();
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __syncthreads();
      } else if constexpr (NA > 0) {
        read_one(nxt, q - 1, W0, X0);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    if constexpr (NA > 0) {
#pragma unroll
      for (int q = FW * NX - 1; q < FW + NA; ++q) read_one(nxt, q, W0, X0);
    }
    slot = slot_next;
  } while (++i < n_steps);
  if (!chain) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // no copy outlives the item
    __syncthreads();                                  // (the next item's copies overwrite any slot)
  }

  if constexpr (NA > 0) {
    const int g = lane >> 5;
    auto result = [&](int f, int m) __attribute__((always_inline)) {
      // (pinned: else all 16 tiles are copied to the other half of the registers behind the loop, and spill there)
      asm volatile("" : "+a"(acc[f][m]));
      f32x16 t = acc[f][m];
      if constexpr (W8) scale_tile(a.wscale, min(nb0 + FW * wi + f, a.NB - 1), g, t);
      return t;
    };
    auto block = [&](int f) { return min(nb0 + FW * wi + f, a.NB - 1); };  // (for loads: past the end the last again)
    // 4 KiB of the stage this item read last, in this wave's quarter of it: free until the wave itself copies
    // a stage of the next item there.  [row of 32][chunk of 16 bytes, 8 of them], chunks swizzled by the row.
    f32x4* tile = (f32x4*)(lds + (slot == 0 ? RING - 1 : slot - 1) * STAGE + w * (C * 64));
    auto slot_of = [&](int m, int r) { return row0 + (2 * m + wj) * 32 + r; };
    const int j = lane & 31;
    if constexpr (EPI == EPI_RESID) {
      // A lane of the products holds 4 features of a row of its own: stored like that, every lane of an access
      // is a cache line of its own.  Turned round in LDS 8 lanes hold the 32 features of a row.
      const int q = lane >> 3, c = lane & 7;  // a lane's rows are 8 r + q
      auto turned = [&](int f, int m, f32x4(&v)[4]) __attribute__((always_inline)) {
        const f32x16 t = result(f, m);
        lanes_exchange();
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4)
          tile[j * 8 + ((2 * q4 + g) ^ (j & 7))] = (f32x4){t[4 * q4], t[4 * q4 + 1], t[4 * q4 + 2], t[4 * q4 + 3]};
        lanes_exchange();
#pragma unroll
        for (int r = 0; r < 4; ++r) v[r] = tile[(8 * r + q) * 8 + (c ^ q)];
      };
      if (S > 1) {
        // split K: the partial rows [part][row][feature] are left to the row kernel that follows
        // (residual add + RMSNorm), which adds the parts up in order
#pragma unroll
        for (int m = 0; m < NA; ++m) {
          float* dp = a.e.rpart + ((size_t)it.s * a.e.rpart_rows + slot_of(m, q)) * a.e.d_model + (nb0 + FW * wi) * 32 + 4 * c;
#pragma unroll
          for (int f = 0; f < FW; ++f)
            if (nb0 + FW * wi + f < a.NB) {
              f32x4 v[4];
              turned(f, m, v);
#pragma unroll
              for (int r = 0; r < 4; ++r)
                if (slot_of(m, 8 * r + q) < n_rows) *(f32x4*)(dp + (size_t)(8 * r) * a.e.d_model + 32 * f) = v[r];
            }
        }
      } else {
        int ids[NA][4];
#pragma unroll
        for (int m = 0; m < NA; ++m)
#pragma unroll
          for (int r = 0; r < 4; ++r) ids[m][r] = a.e.rows[(uint32_t)min(slot_of(m, 8 * r + q), n_rows - 1)];
        f32x4 in[2][FW][4];  // residual rows, asked for ahead of the stores of the row tile before
        auto ask = [&](int m) __attribute__((always_inline)) {
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int id = ids[m][r];
            const float* rs = a.e.resid_src + ((size_t)(id >> 16) * a.e.resid_seq_stride + (id & 0xffff)) * a.e.d_model + 4 * c;
#pragma unroll
            for (int f = 0; f < FW; ++f)
              in[m & 1][f][r] = *(const f32x4*)(rs + 32 * block(f));
          }
        };
        ask(0);
#pragma unroll
        for (int m = 0; m < NA; ++m) {
          if (m + 1 < NA) ask(m + 1);
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int f = 0; f < FW; ++f)
#pragma unroll
            for (int r = 0; r < 4; ++r) arrived(in[m & 1][f][r]);
          float* hp[4];
#pragma unroll
          for (int r = 0; r < 4; ++r)
            hp[r] = a.e.h + ((size_t)(ids[m][r] >> 16) * a.e.h_seq_stride + (ids[m][r] & 0xffff)) * a.e.d_model +
                    (nb0 + FW * wi) * 32 + 4 * c;
#pragma unroll
          for (int f = 0; f < FW; ++f)
            if (nb0 + FW * wi + f < a.NB) {
              f32x4 v[4];
              turned(f, m, v);
#pragma unroll
              for (int r = 0; r < 4; ++r)
                if (slot_of(m, 8 * r + q) < n_rows) *(f32x4*)(hp[r] + 32 * f) = in[m & 1][f][r] + v[r];
            }
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    } else if constexpr (EPI == EPI_QKV) {
      // The rotary factors of a query or key block, 16 cosines and 16 sines per row, are asked for 4 lanes to a
      // row, ahead of the stores of the row tile before, and reach the lanes that need them through LDS.
      const int q = lane >> 2, c = lane & 3;  // a lane's rows are 16 p + q
      auto chunk = [](int row, int k) { return row * 8 + (k ^ (((row & 1) << 2) | ((row >> 1) & 3))); };
      const int bph = a.e.head_dim >> 5, nb_rot = (a.e.n_q_heads + a.e.n_kv_heads) * bph, half = a.e.head_dim >> 1;
      int ids[NA], pos[NA][2];
#pragma unroll
      for (int m = 0; m < NA; ++m) {
        ids[m] = a.e.rows[(uint32_t)min(slot_of(m, j), n_rows - 1)];
#pragma unroll
        for (int p = 0; p < 2; ++p) pos[m][p] = a.e.rows[(uint32_t)min(slot_of(m, 16 * p + q), n_rows - 1)] & 0xffff;
      }
      f32x4 in[2][FW][4];  // cosines, sines of rows 16 p + q
      auto ask = [&](int m) __attribute__((always_inline)) {
        if (nb0 + FW * wi < nb_rot) {  // (the last blocks of a wave may be value blocks: asked for all the same)
#pragma unroll
          for (int f = 0; f < FW; ++f)
#pragma unroll
            for (int p = 0; p < 2; ++p) {
              const uint32_t at = (uint32_t)(pos[m][p] * half + 16 * ((nb0 + FW * wi + f) & (bph - 1)) + 4 * c);
              in[m & 1][f][p] = *(const f32x4*)(a.e.rope_cos + at);
              in[m & 1][f][2 + p] = *(const f32x4*)(a.e.rope_sin + at);
            }
        }
      };
#pragma unroll
      for (int m = 0; m < NA; ++m) {
        arrived(ids[m]);
        arrived(pos[m][0]);
        arrived(pos[m][1]);
      }
      ask(0);
#pragma unroll
      for (int m = 0; m < NA; ++m) {
        if (m + 1 < NA) ask(m + 1);
        __builtin_amdgcn_sched_barrier(0);
        if (nb0 + FW * wi < nb_rot) {
#pragma unroll
          for (int f = 0; f < FW; ++f)
#pragma unroll
            for (int p = 0; p < 4; ++p) arrived(in[m & 1][f][p]);
        }
#pragma unroll
        for (int f = 0; f < FW; ++f) {
          const int nb = nb0 + FW * wi + f;
          EpiIn<EPI> mine = {};
          if (nb < nb_rot) {
            lanes_exchange();
#pragma unroll
            for (int p = 0; p < 2; ++p) {
              tile[chunk(16 * p + q, c)] = in[m & 1][f][p];
              tile[chunk(16 * p + q, 4 + c)] = in[m & 1][f][2 + p];
            }
            lanes_exchange();
#pragma unroll
            for (int q4 = 0; q4 < 2; ++q4) {
              const f32x4 x = tile[chunk(j, 2 * q4 + g)], y = tile[chunk(j, 4 + 2 * q4 + g)];
              mine.c[q4] = make_float4(x[0], x[1], x[2], x[3]);
              mine.s[q4] = make_float4(y[0], y[1], y[2], y[3]);
            }
          }
          if (nb < a.NB) {
            const f32x16 t = result(f, m);
            if (slot_of(m, j) < n_rows) epilogue_store<EPI, F16>(a.e, nb, slot_of(m, j), ids[m], g, t, mine);
          }
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    } else {
      [[maybe_unused]] float gates = 0.f;
      auto store = [&](auto far) __attribute__((always_inline)) {
#pragma unroll
        for (int m = 0; m < NA; ++m)
          if (slot_of(m, j) < n_rows) {
#pragma unroll
            for (int f = 0; f < FW; ++f)
              if (nb0 + FW * wi + f < a.NB) {
                const f32x16 t = result(f, m);
                if constexpr (EPI == EPI_SWIGLU && !far.value) gates = largest_gate(t, gates);
                epilogue_store<EPI, F16, far.value>(a.e, nb0 + FW * wi + f, slot_of(m, j), 0, g, t, {});
              }
          }
      };
      store(std::false_type{});
      if constexpr (EPI == EPI_SWIGLU)
        // (one branch per item: between the tiles it would part them)
        if (__builtin_expect(__any(gates > kFarGate), 0)) store(std::true_type{});
    }
  }
  return slot;
}

template <int FW, int RT, int EPI, bool F16, bool W8>
__device__ __forceinline__ int tall_dispatch(const GemmArgs& a, uint4* lds, TallItem it, TallItem nx, bool chain,
                                              bool prefilled, int slot, int n_rows, int S) {
  // row tiles of this block, dealt to the two row halves alternately
  const int nt = min(2 * RT, (n_rows - it.mb * (64 * RT) + 31) >> 5);
  const int wj = __builtin_amdgcn_readfirstlane(threadIdx.x >> 7);
  const int na = (nt - wj + 1) >> 1;  // wave-uniform, 0 .. RT
#define VLAC_TALL_CASE(N)                                                                                      \
  if constexpr (N < RT)                                                                                        \
    if (na == N) return tall_body<FW, RT, N, EPI, F16, W8>(a, lds, it, nx, chain, prefilled, slot, n_rows, S);
  VLAC_TALL_CASE(0) VLAC_TALL_CASE(1) VLAC_TALL_CASE(2) VLAC_TALL_CASE(3) VLAC_TALL_CASE(4)
#undef VLAC_TALL_CASE
  return tall_body<FW, RT, RT, EPI, F16, W8>(a, lds, it, nx, chain, prefilled, slot, n_rows, S);
}

template <int FW, int RT, int EPI, bool F16, bool W8>
__device__ __forceinline__ void tall_items(const GemmArgs& a, uint4* lds, const TallPlan& pl, int n_rows) {
  // Work items are (weight tile, K part, row block) triples, listed with the row blocks of one
  // weight tile and part next to each other, and the list is cut into eight equal runs, one
  // per XCD (workgroup id % 8), so that the row blocks of a weight tile share it in one L2 and
  // every XCD gets the same number of items.  The grid is one workgroup per CU; a workgroup
  // takes every (grid / 8)-th item of its XCD's run, one after the other, and starts the
  // copies of its next item's first stages during the last steps of the one before it, so
  // that only a workgroup's first item waits for its operands.
  const int items = pl.items(), per = (items + 7) >> 3;
  const int x = blockIdx.x & 7, stride = gridDim.x >> 3;
  auto item_of = [&](int j) {
    const int i = x * per + j;
    const int vt = i / pl.row_blocks;
    TallItem t;
    t.mb = i - vt * pl.row_blocks;
    t.tile = vt / pl.S;
    t.s = vt - t.tile * pl.S;
    if constexpr (EPI == EPI_QKV) {
      // Every eighth weight tile, from both ends in turn: each XCD gets its share of the value blocks, whose
      // results go to the cache in 2-byte pieces, and few of them at a time (a round of them at once kept an
      // L2 busy for 16 us behind the products, all of them on three XCDs 28).
      const int qt = pl.tiles >> 3, rt = pl.tiles & 7, far = t.tile - rt * (qt + 1);
      const int x = far < 0 ? t.tile / (qt + 1) : rt + far / max(qt, 1), n = far < 0 ? qt + 1 : max(qt, 1);
      const int k = far < 0 ? t.tile % (qt + 1) : far % max(qt, 1);
      t.tile = 8 * (k & 1 ? n - 1 - (k >> 1) : k >> 1) + x;
    }
    return t;
  };
  auto exists = [&](int j) { return j < per && x * per + j < items; };
  int j = blockIdx.x >> 3;
  if (!exists(j)) return;
  // (chains need every part of K to have at least as many steps as the copies run ahead)
  const bool can_chain = (2 * a.KS) / pl.S >= TallRing<FW, RT>::N - 1;
  TallItem it = item_of(j);
  bool prefilled = false;
  int slot = 0;
  for (;;) {
    const int jn = j + stride;
    const bool chain = can_chain && exists(jn);
    const TallItem nx = chain ? item_of(jn) : it;
    slot = tall_dispatch<FW, RT, EPI, F16, W8>(a, lds, it, nx, chain, prefilled, slot, n_rows, pl.S);
    if (!exists(jn)) break;
    prefilled = chain;
    it = item_of(jn);
    j = jn;
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
}

// NARROW: items of 192 features are in the choice (a kernel of its own: their code beside the other
// shapes' cost a whole prefill of thousands of rows, where it is never taken, 0.3 to 0.5 %)
// W8: weights expanded from e4m3 codes, whose scales (one per output feature) the results are multiplied by
template <int EPI, bool F16, bool NARROW, bool W8>
__global__ __launch_bounds__(256) void gemm_tall_kernel(GemmArgs a) {
  extern __shared__ uint4 lds[];  // TallRing<FW, RT>::N stages
  const int n_rows = a.n_rows_val >= 0 ? a.n_rows_val : *a.n_rows;
  if (n_rows < a.rows_lo) return;  // the one-stream kernel's share
  const TallPlan pl = tall_plan((a.NB + 7) >> 3, n_rows, EPI == EPI_RESID ? a.S : 1, a.KS);
  if (EPI == EPI_RESID && blockIdx.x == 0 && threadIdx.x == 0) *a.split = pl.S;
  if constexpr (NARROW) {
    TallPlan p3;
    if (tall_plan_192(a.NB, n_rows, pl, &p3)) {
      if (p3.rt == 5) tall_items<3, 5, EPI, F16, W8>(a, lds, p3, n_rows);
      else tall_items<3, 3, EPI, F16, W8>(a, lds, p3, n_rows);
      return;
    }
  }
  if (pl.rt == 4) tall_items<4, 4, EPI, F16, W8>(a, lds, pl, n_rows);
  else if (pl.rt == 3) tall_items<4, 3, EPI, F16, W8>(a, lds, pl, n_rows);
  else tall_items<4, 2, EPI, F16, W8>(a, lds, pl, n_rows);
}

template <int EPI, bool F16, bool NARROW, bool W8>
hipError_t set_lds() {
  return hipFuncSetAttribute((const void*)gemm_tall_kernel<EPI, F16, NARROW, W8>, hipFuncAttributeMaxDynamicSharedMemorySize,
                             kTallLds);
}
template <int EPI, bool F16, bool W8>
hipError_t set_lds_both() {
  const hipError_t e = set_lds<EPI, F16, false, W8>();
  if constexpr (EPI == EPI_QKV || EPI == EPI_SWIGLU) return e != hipSuccess ? e : set_lds<EPI, F16, true, W8>();
  return e;
}
template <bool F16, bool W8>
hipError_t set_lds_all() {
  hipError_t e = set_lds_both<EPI_QKV, F16, W8>();
  if (e == hipSuccess) e = set_lds_both<EPI_SWIGLU, F16, W8>();
  if (e == hipSuccess) e = set_lds_both<EPI_RESID, F16, W8>();
  if (e == hipSuccess) e = set_lds_both<EPI_LOGITS, F16, W8>();
  return e;
}

template <bool F16, bool W8>
void launch_tall_t(int epi, const GemmArgs& a, int grid, bool narrow, hipStream_t st) {
#define VLAC_TALL_LAUNCH(EPI_, NARROW_) \
  hipLaunchKernelGGL((gemm_tall_kernel<EPI_, F16, NARROW_, W8>), dim3(grid), dim3(256), kTallLds, st, a)
  switch (epi) {
    case EPI_QKV:
      if (narrow) VLAC_TALL_LAUNCH(EPI_QKV, true);
      else VLAC_TALL_LAUNCH(EPI_QKV, false);
      break;
    case EPI_SWIGLU:
      if (narrow) VLAC_TALL_LAUNCH(EPI_SWIGLU, true);
      else VLAC_TALL_LAUNCH(EPI_SWIGLU, false);
      break;
    case EPI_RESID: VLAC_TALL_LAUNCH(EPI_RESID, false); break;
    default: VLAC_TALL_LAUNCH(EPI_LOGITS, false); break;
  }
#undef VLAC_TALL_LAUNCH
}

__global__ __launch_bounds__(256) void expand_e4m3_kernel(const uint4* __restrict__ codes,
                                                          uint4* __restrict__ tiles, size_t n) {
  // thread = one lane's slot: the 8 codes of k-tile 2c and the 8 of k-tile 2c + 1
  const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
  const uint4 slot = codes[i];
  const size_t pair = i >> 6, lane = i & 63;
  tiles[(2 * pair) * 64 + lane] = e4m3_slot_half(slot, 0);
  tiles[(2 * pair + 1) * 64 + lane] = e4m3_slot_half(slot, 1);
}

}  // namespace

void launch_expand_e4m3(const uint4* codes, uint4* tiles, size_t n_slots, hipStream_t st) {
  const size_t n = n_slots * 64;
  hipLaunchKernelGGL(expand_e4m3_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, codes, tiles, n);
}

int gemm_tall_init() {
  hipError_t e = set_lds_all<true, false>();
  if (e == hipSuccess) e = set_lds_all<false, false>();
  if (e == hipSuccess) e = set_lds_all<true, true>();
  return (int)e;
}

void launch_gemm_tall(bool f16, int epi, GemmArgs& a, int rows_cap, int S_max, hipStream_t st) {
  a.S = (epi == EPI_RESID && S_max > 1) ? S_max : 1;
  a.x_tiles = (rows_cap + 31) / 32;
  // the grid covers the most work items any row count up to rows_cap can give (the plan
  // changes its row blocks and K parts with the row count)
  const int tiles = (a.NB + 7) >> 3;
  const bool narrow = (epi == EPI_QKV || epi == EPI_SWIGLU) && rows_cap <= kNarrowRows;
  int most = 0;
  for (int n = 64; n < rows_cap + 64; n += 64) {
    const TallPlan pl = tall_plan(tiles, std::min(n, rows_cap), a.S, a.KS);
    most = std::max(most, pl.items());
    TallPlan p3;
    if (narrow && tall_plan_192(a.NB, std::min(n, rows_cap), pl, &p3)) most = std::max(most, p3.items());
  }
  const int grid = std::min(((most + 7) / 8) * 8, kTallGrid);
  if (a.wscale) launch_tall_t<true, true>(epi, a, grid, narrow, st);
  else if (f16) launch_tall_t<true, false>(epi, a, grid, narrow, st);
  else launch_tall_t<false, false>(epi, a, grid, narrow, st);
}
