// Stage (a): Medusa-head projection, per-head top-k and tree-token assembly.
//
// SpecMemo Sec. 3.1: l parallel heads read the last hidden state, and head i's
// top-k tokens populate level i+1 of the candidate tree (Eq. 2); a node's token
// depends only on its depth and rank.
//
// z[b][i][v] = sum_c W[i][v][c] * h[b][c].  The weight stream (l * vocab * hidden
// bf16, 2.1 GB for a 70B-shaped model) is the largest read of the step and is
// HBM-bound for any batch of a verify step, so waves stream 64 vocabulary rows
// each with 16-byte loads and contract them on the 16x16x32 bf16 matrix cores
// (batch padded to 16s: the padding costs matrix-core time that is far below
// the load time).  Packed heads: head_gemm; row-major ones: head_rows.
#include <type_traits>

#include "device.h"
#include "internal.h"

namespace specmemo {

namespace {

// Weights are read once per step: nontemporal loads keep them from displacing
// the hidden states and logits in the caches.
typedef unsigned u32x4_t __attribute__((ext_vector_type(4)));
__device__ __forceinline__ uint4 ld16_stream(const uint4 *p) {
  return __builtin_bit_cast(uint4, __builtin_nontemporal_load(reinterpret_cast<const u32x4_t *>(p)));
}

// Packed weights (see specmemo_pack_heads) against up to 16 NB hidden states:
// head_logits with EPI = 0, residual blocks with EPI = 1.
//
// Bound by the weight stream (HBM) up to 128 hidden states, so the weights are
// read once for all of them: a wave keeps the accumulators of one 64-row group
// x 16 NB states in registers and streams the group's 1 KB operand tiles.
// 4 heads x 32000 x 8192, this kernel alone: 10 states 300 us (7.0 TB/s of
// weights), 120 states 332 to 341 us (6.2 TB/s; 1345 us with top-k when 32 states were
// the most that shared a stream).
//
// KS waves share a row group and split its k steps in contiguous ranges, whose
// partial sums meet in LDS: see launch_gemm_nb for when.
//
// Weights: PRE k steps (4 KB each) in flight per wave, a step's registers
// refilled right after its products; BURST (one batch tile): eight steps at a
// time, refilled together, the states read at their use.  States of one batch
// tile: each wave loads its own beside the weights.  Of more: the block's waves share them
// through LDS in chunks of KC k steps per range, two buffers; a chunk is
// fetched to registers two chunks ahead and stored one ahead, and the barrier
// between chunks is bare, because __syncthreads() would wait for the weights
// in flight.  LDS entry of (row r, 8-column part c) of a 1 KB piece is
// 4 r + (c ^ state_slot_swz(r)): a wave's 16-byte writes (four lanes a row, as they
// are coalesced) and reads (16 rows at one part) are both free of bank
// conflicts.
//
// EPI = 0, gmax non-null: each (batch row, head) row also gets the maximum of
// every 64-row group, [B][n_heads][nG], from which the top-k pass finds the
// groups that can hold a top-k value.
__device__ __forceinline__ int state_slot_swz(int r) { return ((r >> 1) ^ (r >> 2)) & 3; }

template <int NW, int NB, int KS, int KC, int EPI, bool BURST = false>
__global__ __launch_bounds__(64 * NW, 8 / NW) void head_gemm(
    const uint16_t *__restrict__ h, int64_t h_head_stride, const uint4 *__restrict__ Wp,
    const uint16_t *__restrict__ bias, float *__restrict__ z, uint16_t *__restrict__ hout, int B, int hidden, int rows,
    int n_heads, int nG, int nS, float *__restrict__ gmax) {
  constexpr int PRE = BURST ? 8 : 4;             // k steps in flight per wave
  constexpr bool kShare = NB > 1;                // states through LDS
  static_assert(PRE % KC == 0 && NW % KS == 0 && (!kShare || (NB * KS * KC) % NW == 0), "whole chunks and pieces");
  constexpr int RG = NW / KS;                    // row groups per block
  constexpr int kPer = kShare ? NB * KS * KC / NW : 1;   // 16-byte pieces of a chunk per thread
  constexpr int kBuf = kShare ? KS * KC * NB * 64 : 0;        // entries of a states buffer
  constexpr int kTile = NW * 4 * 64;             // a batch tile of every wave, for the ranges' sums
  constexpr int kRed = KS == 1 ? 0 : NB == 1 ? kTile : 2 * kTile;
  __shared__ u32x4_t hsh[2 * kBuf > kRed ? 2 * kBuf : kRed > 0 ? kRed : 1];
  // the wave's number, made uniform for the compiler: its bases then stay in scalar registers
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int head = blockIdx.y, b0 = blockIdx.z * 16 * NB;
  const int G = blockIdx.x * RG + wave / KS, sl = wave % KS;
  const bool active = G < nG;
  const int r16 = lane & 15, kq = lane >> 4;
  const int nF = hidden >> 5;                    // whole k steps; a rest of hidden % 32 columns follows the loop
  const int len = (nF + KS - 1) / KS;            // k steps of a range (the last ranges may hold fewer)
  const int s_begin = sl * len, n_mine = max(0, min(nF - s_begin, len));
  // pipelined steps: whole groups of PRE that every range has
  const int n_main = max(0, nF - (KS - 1) * len) / PRE * PRE;
  const uint4 *wp = Wp + ((int64_t)(head * (int64_t)nG + (active ? G : 0)) * nS + s_begin) * 4 * 64;
  const uint16_t *hbase = h + head * h_head_stride;

  f32x4 acc[NB][4];
#pragma unroll
  for (int n = 0; n < NB; ++n)
#pragma unroll
    for (int t = 0; t < 4; ++t) acc[n][t] = f32x4{0.f, 0.f, 0.f, 0.f};

  u32x4_t hreg[kPer];
  uint32_t hoff[kPer];                           // this thread's bytes of the pieces, from row b0
#pragma unroll
  for (int i = 0; i < kPer; ++i) {
    const int n = (i * NW + wave) % NB;        // piece NW i + wave: batch tile, then step of the chunk, then range
    hoff[i] = (uint32_t)min(16 * n + (lane >> 2), B - 1 - b0) * (uint32_t)(2 * hidden) + 16u * (lane & 3);
  }
  const uint8_t *hb0 = reinterpret_cast<const uint8_t *>(hbase + (int64_t)b0 * hidden);
  auto hfetch = [&](int c) {   // rows past B repeat the last one, chunks past the end the last step: neither is used
#pragma unroll
    for (int i = 0; i < kPer; ++i) {
      const int r = (i * NW + wave) / NB;
      const int st = min((r / KC) * len + c * KC + r % KC, nF - 1);
      hreg[i] = *reinterpret_cast<const u32x4_t *>(hb0 + 64 * (int64_t)st + hoff[i]);
    }
  };
  const int wr = (lane & ~3) + ((lane & 3) ^ state_slot_swz(lane >> 2));
  auto hstore = [&](int buf) {
#pragma unroll
    for (int i = 0; i < kPer; ++i) hsh[buf * kBuf + (i * NW + wave) * 64 + wr] = hreg[i];
  };
  const int rd = 4 * r16 + (kq ^ state_slot_swz(r16));

  auto contract = [&](const uint4 (&at)[4], const bf16x8 &bv, int n) {
#pragma unroll
    for (int t = 0; t < 4; ++t)
      acc[n][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, at[t]), bv, acc[n][t], 0, 0, 0);
  };
  if (n_main > 0) {
    // No branch between the loads in flight: one that may be skipped makes the
    // compiler wait for all of them.
    uint4 a[PRE][4];
    u32x4_t own[kShare ? 1 : PRE];               // one batch tile: the wave's own states, loaded with the weights
    const uint16_t *ho = hbase + (int64_t)min(b0 + r16, B - 1) * hidden + 32 * s_begin + 8 * kq;
    auto fetch = [&](int s, int u) {
      if constexpr (!kShare && !BURST) own[u] = *reinterpret_cast<const u32x4_t *>(ho + 32 * s);
      const uint4 *wn = wp + (int64_t)s * 4 * 64;
#pragma unroll
      for (int t = 0; t < 4; ++t) a[u][t] = ld16_stream(wn + t * 64 + lane);
    };
    auto group = [&](int t0, auto more) {        // PRE steps; `more`: each then fetches the step PRE further on
#pragma unroll
      for (int u = 0; u < PRE; ++u) {
        if constexpr (kShare) {
          const int c = (t0 + u) / KC;           // chunk of this step
          if (u % KC == 0) {
            hstore((c + 1) & 1);
            hfetch(c + 2);
          }
          const u32x4_t *hb = &hsh[(c & 1) * kBuf + ((sl * KC + u % KC) * NB) * 64 + rd];
#pragma unroll
          for (int n = 0; n < NB; ++n) contract(a[u], __builtin_bit_cast(bf16x8, hb[n * 64]), n);
        } else if constexpr (BURST) {
          contract(a[u], __builtin_bit_cast(bf16x8, ld16_or_zero(b0 + r16 < B, ho + 32 * (t0 + u))), 0);
        } else {
          contract(a[u], __builtin_bit_cast(bf16x8, own[u]), 0);
        }
        if constexpr (!BURST) {
          if constexpr (decltype(more)::value) fetch(t0 + u + PRE, u);
          __builtin_amdgcn_sched_barrier(0);     // the loads stay here: their distance is the prefetch
        }
        if (kShare && u % KC == KC - 1) asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
      }
      if constexpr (BURST && decltype(more)::value)
#pragma unroll
        for (int u = 0; u < PRE; ++u) fetch(t0 + PRE + u, u);
    };
#pragma unroll
    for (int u = 0; u < PRE; ++u) fetch(u, u);
    if constexpr (kShare) {
      hfetch(0);
      hstore(0);
      hfetch(1);
      __syncthreads();
    }
    int t0 = 0;
    for (; t0 + PRE < n_main; t0 += PRE) group(t0, std::true_type{});
    group(t0, std::false_type{});
  }
  // The range's last steps, and in the last range hidden % 32 columns more,
  // four, two or one at a time: states straight from memory, zero past hidden.
  const int n_all = n_mine + (sl == KS - 1 ? nS - nF : 0);
  auto rest = [&](int s0, auto count) {
    constexpr int C = decltype(count)::value;
    uint4 at[C][4];
#pragma unroll
    for (int u = 0; u < C; ++u) {
      const int st = s0 + u < n_mine ? s_begin + s0 + u : nF;
#pragma unroll
      for (int t = 0; t < 4; ++t) at[u][t] = ld16_stream(wp + ((int64_t)(st - s_begin) * 4 + t) * 64 + lane);
    }
#pragma unroll
    for (int u = 0; u < C; ++u) {
      const int k = 32 * (s0 + u < n_mine ? s_begin + s0 + u : nF) + 8 * kq;
#pragma unroll
      for (int n = 0; n < NB; ++n) {
        const int b = b0 + 16 * n + r16;
        const bool in = b < B && k < hidden;
        contract(at[u], __builtin_bit_cast(bf16x8, ld16_or_zero(in, hbase + (int64_t)(in ? b : 0) * hidden + (in ? k : 0))), n);
      }
    }
  };
  int s0 = n_main;
  for (; s0 + 4 <= n_all; s0 += 4) rest(s0, std::integral_constant<int, 4>{});
  if (s0 + 2 <= n_all) {
    rest(s0, std::integral_constant<int, 2>{});
    s0 += 2;
  }
  if (s0 < n_all) rest(s0, std::integral_constant<int, 1>{});
  // The ranges' sums, added in range order, one batch tile at a time (two
  // buffers in turn).  Wave n % KS of a row group finishes tile n: with one wave
  // for all, the rest waited for its stores (residual blocks of 512 columns, 2
  // heads, 128 states, 8 tiles a block: 36.5 us, of which 30 were this).
  if constexpr (KS > 1) {
    f32x4 *red = reinterpret_cast<f32x4 *>(hsh);
    __syncthreads();                             // every wave is past its reads of the states
#pragma unroll
    for (int n = 0; n < NB; ++n) {
      f32x4 *buf = red + (n & 1) * kTile;
      const bool mine = n % KS == sl;
      if (!mine)
#pragma unroll
        for (int t = 0; t < 4; ++t) buf[(wave * 4 + t) * 64 + lane] = acc[n][t];
      __syncthreads();
      if (mine)
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          const f32x4 own = acc[n][t];
          f32x4 v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int w = 0; w < KS; ++w) {
            const f32x4 part = w == sl ? own : buf[((wave - sl + w) * 4 + t) * 64 + lane];
            v = w == 0 ? part : v + part;
          }
          acc[n][t] = v;
        }
    }
  }
  if (!active) return;
  // C layout: lane holds column (batch) lane&15, rows 4*(lane>>4) + 0..3 of each tile.
#pragma unroll
  for (int n = 0; n < NB; ++n) {
    if (KS > 1 && n % KS != sl) continue;
    const int b = b0 + 16 * n + r16;
    if constexpr (EPI == 0) {
      float m = -INFINITY;
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const int row = 64 * G + t * 16 + 4 * kq;
#pragma unroll
        for (int j = 0; j < 4; ++j) m = row + j < rows ? fmaxf(m, acc[n][t][j]) : m;
      }
      if (gmax) {   // the column's four lanes: l, l ^ 16, l ^ 32, l ^ 48
        m = fmaxf(m, __shfl_xor(m, 16));
        m = fmaxf(m, __shfl_xor(m, 32));
      }
      if (b >= B) continue;
      float *zr = z + ((int64_t)b * n_heads + head) * rows;
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const int row = 64 * G + t * 16 + 4 * kq;
        if ((rows & 3) == 0) {                   // rows start 16-byte aligned: the lane's four are all in or all out
          if (row < rows) *reinterpret_cast<f32x4 *>(zr + row) = acc[n][t];
        } else {
#pragma unroll
          for (int j = 0; j < 4; ++j)
            if (row + j < rows) zr[row + j] = acc[n][t][j];
        }
      }
      if (gmax && kq == 0) gmax[((int64_t)b * n_heads + head) * nG + G] = m;
    } else {
      if (b >= B) continue;
      const uint16_t *hin = h + (int64_t)b * hidden;
      const uint16_t *bh = bias + (int64_t)head * hidden;
      uint16_t *o = hout + ((int64_t)head * B + b) * hidden;
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const int row = 64 * G + t * 16 + 4 * kq;
#pragma unroll
        for (int j = 0; j < 4; ++j)
          if (row + j < hidden) {
            const float y = acc[n][t][j] + bf16_to_f32(bh[row + j]);
            o[row + j] = f32_to_bf16(bf16_to_f32(hin[row + j]) + y / (1.f + expf(-y)));
          }
      }
    }
  }
}

// Row-major heads (nn.Linear layout), up to 16 NB states.  A matrix operand
// loaded to registers takes 64 bytes of each of 16 rows per instruction, which
// the memory system serves at 4.7 TB/s; so the weights go to LDS directly, 256
// bytes of each of 4 rows per instruction, and are read there in operand order.
// Eight waves of 16 rows share the states of a chunk of 128 columns; a ring of
// SLOTS chunks is filled by direct loads and ordered by vmcnt waits and one
// bare barrier per chunk.  A row's 16-byte part c sits at c ^ (row % 16): 16
// rows read at one part lie in distinct banks.  hidden % 128 columns follow
// from registers.  Blocks start their sweeps at different chunks: rows a power
// of two apart, read at one offset by all blocks, keep to a few memory channels
// (rows of 8192: 498 us without, 355 us with; of 5120: 215 and 217 us).
// 4 heads, 4 states, 32003 x 5120: 268 -> 217 us; 10 states, 32000 x 8192: 402 ->
// 355 us (5.9 TB/s); 16 states, 18001 x 5120: 283 -> 149 us; 40 states, 32000 x
// 4096, one weight stream instead of two: 453 -> 196 us; 65 to 128 states (two
// slots), 32003 x 5120: 937 to 1367 -> 327 to 364 us.  One block fills a unit, so a
// last round that is nearly empty costs one: 33 states, 17001 x 7800 (532 blocks)
// 275 us, 3.9 TB/s.  gmax: as in head_gemm.
template <int NB, int SLOTS>
__global__ __launch_bounds__(512, 2) void head_rows(const uint16_t *__restrict__ h, int64_t h_head_stride,
                                                    const uint8_t *__restrict__ W, float *__restrict__ z, int B,
                                                    int hidden, int rows, int n_heads, int nG,
                                                    float *__restrict__ gmax) {
  constexpr int kRow = 256;                                   // bytes of a row per chunk
  constexpr int kW = 128 * kRow, kSlot = kW + 16 * NB * kRow;
  constexpr int kLoads = 4 + NB;                              // direct loads per wave and chunk
  __shared__ __attribute__((aligned(1024))) uint8_t ring[SLOTS * kSlot];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int head = blockIdx.y, b0 = blockIdx.z * 16 * NB;
  const int r16 = lane & 15, kq = lane >> 4;
  const int row0 = blockIdx.x * 128 + wave * 16, last = rows - 1;
  const int nc = hidden < 1 << 27 ? hidden >> 7 : 0;          // whole chunks (rows past 2^27 columns: all from registers)
  const int rot = nc ? (int)((blockIdx.x + 7u * head) % (unsigned)nc) : 0;
  // Load i of a wave: LDS rows 4 i + lane / 16 of its tile, part lane % 16 of
  // the slot's row, which holds the row's part (lane % 16) ^ (row % 16).
  const uint8_t *wb = uniform_ptr(W + ((int64_t)head * rows + min(row0, last)) * hidden * 2);
  const uint16_t *hb = h + head * h_head_stride;
  const uint8_t *hb8 = uniform_ptr(reinterpret_cast<const uint8_t *>(hb + (int64_t)b0 * hidden));
  uint32_t woff[4], hoff[NB];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int r = 4 * i + kq;
    woff[i] = (uint32_t)min(r, max(last - row0, 0)) * (uint32_t)(2 * hidden) + 16u * (r16 ^ r);   // rows past the last repeat it
  }
  // states: 4 NB loads per chunk, spread over the waves (waves 4 to 7 repeat those of 0 to 3)
#pragma unroll
  for (int n = 0; n < NB; ++n) {
    const int r = 4 * (wave & 3) + kq;
    hoff[n] = (uint32_t)min(16 * n + r, B - 1 - b0) * (uint32_t)(2 * hidden) + 16u * (r16 ^ r);
  }
  const uint32_t lds0 = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(lds_void_t *)ring);
  auto issue = [&](int c, int slot) {
    const int cc = c + rot < nc ? c + rot : c + rot - nc;
    const uint32_t base = lds0 + slot * kSlot;
#pragma unroll
    for (int n = 0; n < NB; ++n) lds_load16(hb8 + (int64_t)kRow * cc, hoff[n], base + kW + (16 * n + 4 * (wave & 3)) * kRow);
#pragma unroll
    for (int i = 0; i < 4; ++i) lds_load16(wb + (int64_t)kRow * cc, woff[i], base + (16 * wave + 4 * i) * kRow);
  };
  f32x4 acc[NB][2];
#pragma unroll
  for (int n = 0; n < NB; ++n) acc[n][0] = acc[n][1] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int c = 0; c < SLOTS - 1; ++c)
    if (c < nc) issue(c, c);
  auto chunk = [&](int c, auto slot_c) {
    constexpr int slot = decltype(slot_c)::value;
    // chunks issued after this one: up to SLOTS - 2
    const int later = min(nc - 1 - c, SLOTS - 2);
    if (later >= 2) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * kLoads) : "memory");
    else if (later == 1) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(kLoads) : "memory");
    else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    ring_barrier();      // every wave's loads of this chunk are in, and its reads of the slot refilled next are done
    if (c + SLOTS - 1 < nc) issue(c + SLOTS - 1, (slot + SLOTS - 1) % SLOTS);
    const uint8_t *s = ring + slot * kSlot;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int part = 16 * ((4 * u + kq) ^ r16);
      const bf16x8 a = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4_t *>(s + (16 * wave + r16) * kRow + part));
#pragma unroll
      for (int n = 0; n < NB; ++n) {
        const bf16x8 b = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4_t *>(s + kW + (16 * n + r16) * kRow + part));
        acc[n][u & 1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, acc[n][u & 1], 0, 0, 0);
      }
    }
  };
  for (int c = 0; c < nc; c += SLOTS) {
    chunk(c, std::integral_constant<int, 0>{});
    if (c + 1 < nc) chunk(c + 1, std::integral_constant<int, 1>{});
    if constexpr (SLOTS >= 3)
      if (c + 2 < nc) chunk(c + 2, std::integral_constant<int, 2>{});
    if constexpr (SLOTS == 4)
      if (c + 3 < nc) chunk(c + 3, std::integral_constant<int, 3>{});
  }
  const uint8_t *wr = wb + (int64_t)min(r16, max(last - row0, 0)) * hidden * 2;
  for (int k = (nc << 7) + 8 * kq; k - 8 * kq < hidden; k += 32) {   // the last hidden % 128 columns
    const bf16x8 a = __builtin_bit_cast(bf16x8, ld16_or_zero(k < hidden, wr + 2 * (int64_t)k));
#pragma unroll
    for (int n = 0; n < NB; ++n) {
      const int b = b0 + 16 * n + r16;
      const bool in = b < B && k < hidden;
      const bf16x8 hv = __builtin_bit_cast(bf16x8, ld16_or_zero(in, hb + (int64_t)(in ? b : 0) * hidden + (in ? k : 0)));
      acc[n][0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, hv, acc[n][0], 0, 0, 0);
    }
  }
  float (*tops)[16 * NB] = reinterpret_cast<float (*)[16 * NB]>(ring);   // [wave][state]: maximum of the wave's 16 rows
  if (gmax) ring_barrier();                                   // every wave is past its reads of the ring
#pragma unroll
  for (int n = 0; n < NB; ++n) {
    const int b = b0 + 16 * n + r16, row = row0 + 4 * kq;
    const f32x4 v = acc[n][0] + acc[n][1];
    if (gmax) {
      float m = -INFINITY;
#pragma unroll
      for (int j = 0; j < 4; ++j) m = row + j < rows ? fmaxf(m, v[j]) : m;
      m = fmaxf(m, __shfl_xor(m, 16));
      m = fmaxf(m, __shfl_xor(m, 32));
      if (kq == 0) tops[wave][16 * n + r16] = m;
    }
    if (b >= B) continue;
    float *zr = z + ((int64_t)b * n_heads + head) * rows + row;
    if ((rows & 3) == 0) {
      if (row < rows) *reinterpret_cast<f32x4 *>(zr) = v;
    } else {
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (row + j < rows) zr[j] = v[j];
    }
  }
  if (gmax) {
    __syncthreads();
    for (int i = threadIdx.x; i < 32 * NB; i += 512) {        // the block's two 64-row groups
      const int g = i / (16 * NB), c = i % (16 * NB), G = 2 * blockIdx.x + g, b = b0 + c;
      if (G < nG && b < B)
        gmax[((int64_t)b * n_heads + head) * nG + G] =
            fmaxf(fmaxf(tops[4 * g][c], tops[4 * g + 1][c]), fmaxf(tops[4 * g + 2][c], tops[4 * g + 3][c]));
    }
  }
}

// One thread per 16-byte chunk of the packed buffer (see specmemo_pack_heads).
__global__ __launch_bounds__(256) void pack_heads_bf16(const uint16_t *__restrict__ src, uint4 *__restrict__ dst,
                                                       int vocab, int hidden, int nG, int nS, int64_t chunks) {
  const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (idx >= chunks) return;
  const int l = (int)(idx & 63);
  int64_t rest = idx >> 6;
  const int t = (int)(rest & 3);
  rest >>= 2;
  const int s = (int)(rest % nS);
  rest /= nS;
  const int G = (int)(rest % nG);
  const int head = (int)(rest / nG);
  const int row = 64 * G + 16 * t + (l & 15);
  const int col = 32 * s + 8 * (l >> 4);
  uint4 v = {0u, 0u, 0u, 0u};
  if (row < vocab && col < hidden)    // hidden % 8 == 0: the 8 columns are all inside or all outside
    v = *reinterpret_cast<const uint4 *>(src + ((int64_t)head * vocab + row) * hidden + col);
  dst[idx] = v;
}

// fp32 heads: a wave takes four vocabulary rows and J states at once, lanes
// stride the hidden dimension by 16 bytes, so that each of the 4 + J loads of a
// stride feeds several products; the 4 J sums are reduced together, each step
// halving what a lane holds (4 J shuffles, not 24 J).  hidden % 8 == 0.  3 heads,
// 32 states, 8000 x 1024: 408 us with one row per wave and 4-byte loads, 145 us.
// EPI as in head_gemm.
template <int EPI, int J>
__global__ __launch_bounds__(256) void head_logits_f32(const float *__restrict__ h, int64_t h_head_stride,
                                                       const float *__restrict__ W,
                                                       float *__restrict__ z, const float *__restrict__ bias,
                                                       float *__restrict__ hout, int B, int hidden,
                                                       int vocab, int n_heads) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int head = blockIdx.y;
  const int row0 = (blockIdx.x * 4 + wave) * 4;
  if (row0 >= vocab) return;
  const float *wr[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) wr[r] = W + ((int64_t)head * vocab + min(row0 + r, vocab - 1)) * hidden;
  h += head * h_head_stride;
  const int b0 = blockIdx.z * J;
  float v[4 * J];
#pragma unroll
  for (int i = 0; i < 4 * J; ++i) v[i] = 0.f;
  for (int c = 4 * lane; c < hidden; c += 256) {
    f32x4 w[4], x[J];
#pragma unroll
    for (int r = 0; r < 4; ++r) w[r] = *reinterpret_cast<const f32x4 *>(wr[r] + c);
#pragma unroll
    for (int j = 0; j < J; ++j) x[j] = *reinterpret_cast<const f32x4 *>(h + (int64_t)min(b0 + j, B - 1) * hidden + c);
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int j = 0; j < J; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) v[r * J + j] = fmaf(w[r][e], x[j][e], v[r * J + j]);
  }
  int off = 32, idx = 0;                       // idx: the sum this lane ends up with
#pragma unroll
  for (int cnt = 2 * J; cnt >= 1; cnt >>= 1, off >>= 1) {
    const bool up = lane & off;
    idx += up ? cnt : 0;
#pragma unroll
    for (int i = 0; i < cnt; ++i) {
      const float keep = up ? v[i + cnt] : v[i], send = up ? v[i] : v[i + cnt];
      v[i] = keep + __shfl_xor(send, off);
    }
  }
  const int rest = off;                        // lanes that differ below the last step still hold partial sums
#pragma unroll
  for (int o = 32; o > 0; o >>= 1)
    if (o <= rest) v[0] += __shfl_xor(v[0], o);
  const int row = row0 + idx / J, b = b0 + idx % J;
  if ((lane & (2 * rest - 1)) == 0 && row < vocab && b < B) {
    if constexpr (EPI == 0) {
      z[((int64_t)b * n_heads + head) * vocab + row] = v[0];
    } else {
      const float y = v[0] + bias[(int64_t)head * vocab + row];
      hout[((int64_t)head * B + b) * vocab + row] = h[(int64_t)b * hidden + row] + y / (1.f + expf(-y));
    }
  }
}

// Top-k of one (sequence, head) logit row per block, in the order larger value
// first, equal values by lower id.
//  1. Every thread takes the max of its values.
//  2. T = the k-th largest of 64 maxima, each over the threads of one lane
//     number: k of these sets hold a value >= T, so the row's k-th best value
//     is >= T and every top-k value is >= T.  (Sets of neighbouring threads
//     leave most sets empty on short rows, T is then -inf and every value is
//     gathered: 10 rows x 4 heads of 2000, hidden 256, k 10, the whole call
//     12.5 us by the row scan, 663 us from the group maxima, 8.9 us now.)
//  3. Values >= T are gathered into LDS; a gathered value's output slot is the
//     number of gathered values that beat it (values below T beat none).
//  4. If ties at T overflow the buffer, the k picks are instead made in k
//     rounds, each taking the best value worse than the previous pick.
// The block of head i also writes the tree tokens of level i+1 (head 0: the
// root token).
constexpr int kTopkThreads = 1024;
constexpr int kTopkCand = 2048;
constexpr int kTopkU = 8;            // float4 groups per thread per batch

__global__ __launch_bounds__(kTopkThreads) void topk_rows(TopkArgs a) {
  constexpr int kWavesT = kTopkThreads / 64;
  const int row = blockIdx.x;                 // b * n_heads + head
  const int b = row / a.n_heads, head = row % a.n_heads;
  const int k = a.k[head];
  const int vocab = a.vocab;
  const float *x = a.z + (int64_t)row * vocab;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  __shared__ __attribute__((aligned(16))) float cv[kTopkCand + 4];
  __shared__ __attribute__((aligned(16))) int ci[kTopkCand + 4];
  __shared__ float lmax[kWavesT][64];
  __shared__ float thr;
  __shared__ float rbv[kWavesT];
  __shared__ int rbi[kWavesT];
  __shared__ float selv[kMaxTopk];
  __shared__ int sel[kMaxTopk];
  __shared__ int ncand;
  if (tid == 0) ncand = 0;

  // This sequence's tree fields for the level this head fills (fetched now so
  // their latency overlaps the row scan).
  const int n0 = a.node_off[b], n1 = a.node_off[b + 1];
  int my_depth = 0, my_rank = 0;
  if (n0 + tid < n1) {
    my_depth = a.depth[n0 + tid];
    my_rank = a.rank[n0 + tid];
  }

  // The row is read in batches of kTopkU groups per thread, all loads of a
  // batch in flight together; a group is a float4 (ids 4 g .. 4 g + 3) when
  // rows start 16-byte aligned (vocab % 4 == 0), else one float.  A row of one
  // batch (vocab <= 4 * 1024 * kTopkU) stays in registers for the gather.
  const bool vec = (vocab & 3) == 0;
  const int ngrp = vec ? vocab >> 2 : vocab;
  const float4 *x4 = reinterpret_cast<const float4 *>(x);
  constexpr float NEG = -INFINITY;
  float4 q[kTopkU];
  auto load_batch = [&](int g0) {
#pragma unroll
    for (int u = 0; u < kTopkU; ++u) {
      const int g = g0 + u * kTopkThreads + tid;
      q[u] = g < ngrp ? (vec ? x4[g] : float4{x[g], NEG, NEG, NEG}) : float4{NEG, NEG, NEG, NEG};
    }
  };
  constexpr int kBatch = kTopkU * kTopkThreads;

  // With the projection's 64-row group maxima (a.gmax), the threshold comes
  // from those maxima and only the groups whose maximum reaches it are read.
  // Fewer than 2 k groups give a low threshold, or none: such a row (under 128 k
  // values) is scanned (2000 values, k 32: 113 us from 32 maxima, 9.4 us scanned).
  const bool pruned = a.gmax != nullptr && a.nG >= 2 * k && a.nG <= kTopkThreads * kTopkU;
  const float *gm_row = pruned ? a.gmax + (int64_t)row * a.nG : nullptr;

  // 1. thread max (of its values, or of its groups' maxima)
  float mx = NEG;
  if (pruned) {
#pragma unroll
    for (int u = 0; u < kTopkU; ++u) {
      const int g = u * kTopkThreads + tid;
      mx = fmaxf(mx, g < a.nG ? gm_row[g] : NEG);
    }
  } else {
    for (int g0 = 0; g0 < ngrp; g0 += kBatch) {
      load_batch(g0);
#pragma unroll
      for (int u = 0; u < kTopkU; ++u) mx = fmaxf(mx, fmaxf(fmaxf(q[u].x, q[u].y), fmaxf(q[u].z, q[u].w)));
    }
  }
  // 2. T = the k-th largest of the 64 maxima over the waves
  lmax[wave][lane] = mx;
  __syncthreads();
  if (wave == 0) {
    float g = mx;
#pragma unroll
    for (int w = 1; w < kWavesT; ++w) g = fmaxf(g, lmax[w][lane]);
    int above = 0;                    // sets whose max beats this one (ties by lane)
#pragma unroll
    for (int j = 0; j < 64; ++j) {
      const float o = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(g), j));
      above += (o > g || (o == g && j < lane)) ? 1 : 0;
    }
    if (above == k - 1) thr = g;
  }
  __syncthreads();
  const float T = thr;

  // 3. gather values >= T
  auto gather = [&](float xv, int v) {
    if (xv >= T) {
      const int slot = atomicAdd(&ncand, 1);
      if (slot < kTopkCand) {
        cv[slot] = xv;
        ci[slot] = v;
      }
    }
  };
  if (pruned) {
    // the groups whose maximum reaches T, then their values >= T (one thread
    // per value of 16 groups at a time)
    __shared__ int sel_g[kTopkCand];
    __shared__ int nsel;
    if (tid == 0) nsel = 0;
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kTopkU; ++u) {
      const int g = u * kTopkThreads + tid;
      if (g < a.nG && gm_row[g] >= T) {
        const int slot = atomicAdd(&nsel, 1);
        if (slot < kTopkCand) sel_g[slot] = g;
      }
    }
    __syncthreads();
    const int ns = min(nsel, kTopkCand);
    if (nsel > kTopkCand) {
      if (tid == 0) ncand = kTopkCand + 1;      // too many: the k-round selection below
    } else {
      for (int e0 = 0; e0 < ns * 64; e0 += kTopkThreads) {
        const int e = e0 + tid;
        if (e < ns * 64) {
          const int v = 64 * sel_g[e >> 6] + (e & 63);
          if (v < vocab) gather(x[v], v);
        }
      }
    }
  } else
  for (int g0 = 0; g0 < ngrp; g0 += kBatch) {
    if (ngrp > kBatch) load_batch(g0);   // one batch: still in registers
#pragma unroll
    for (int u = 0; u < kTopkU; ++u) {
      const int g = g0 + u * kTopkThreads + tid;
      if (g < ngrp && fmaxf(fmaxf(q[u].x, q[u].y), fmaxf(q[u].z, q[u].w)) >= T) {
        if (vec) {
          gather(q[u].x, 4 * g);
          gather(q[u].y, 4 * g + 1);
          gather(q[u].z, 4 * g + 2);
          gather(q[u].w, 4 * g + 3);
        } else {
          gather(q[u].x, g);
        }
      }
    }
  }
  __syncthreads();
  const int n = ncand;
  if (n <= kTopkCand) {
    // rank of candidate c = number of candidates that beat it, counted by one
    // wave (candidates c = wave, wave + 16, ...) with a ballot per 64
    for (int c = wave; c < n; c += kWavesT) {
      const float v = cv[c];
      const int id = ci[c];
      int rank = 0;
      for (int j0 = 0; j0 < n; j0 += 64) {
        const int j = j0 + lane;
        const int jr = j < n ? j : 0;
        const bool beats = j < n && better(cv[jr], ci[jr], v, id);
        rank += __builtin_popcountll(__builtin_amdgcn_ballot_w64(beats));
      }
      if (lane == 0 && rank < k) {
        sel[rank] = id;
        selv[rank] = v;
      }
    }
  } else {
    // 4. k rounds over the row: the best value worse than the previous pick
    float pv = INFINITY;
    int pi = -1;
    for (int j = 0; j < k; ++j) {
      float bv = -INFINITY;
      int bi = INT32_MAX;
      for (int v = tid; v < vocab; v += kTopkThreads) {
        const float xv = x[v];
        if (better(pv, pi, xv, v) && better(xv, v, bv, bi)) {
          bv = xv;
          bi = v;
        }
      }
      wave_argbest(bv, bi);
      if (lane == 0) {
        rbv[wave] = bv;
        rbi[wave] = bi;
      }
      __syncthreads();
      bv = rbv[0];
      bi = rbi[0];
#pragma unroll
      for (int w = 1; w < kWavesT; ++w)
        if (better(rbv[w], rbi[w], bv, bi)) {
          bv = rbv[w];
          bi = rbi[w];
        }
      if (tid == 0) {
        sel[j] = bi;
        selv[j] = bv;
      }
      pv = bv;
      pi = bi;
      __syncthreads();
    }
  }
  __syncthreads();
  int32_t *ids = a.ids + (int64_t)row * a.kmax;
  for (int j = tid; j < a.kmax; j += kTopkThreads) {
    ids[j] = j < k ? sel[j] : -1;
    if (a.vals) a.vals[(int64_t)row * a.kmax + j] = j < k ? selv[j] : -INFINITY;
  }
  if (n0 + tid < n1) {                        // trees have at most kMaxNodes <= 1024 nodes
    if (tid == 0) {
      if (head == 0) a.node_tok[n0] = a.root_tok[b];
    } else if (my_depth == head + 1) {
      a.node_tok[n0 + tid] = sel[my_rank];
    }
  }
}

}  // namespace

namespace {

// Kernel form for NB batch tiles.  One round of blocks, one per compute unit,
// streams best, so a block takes the fewest row groups (1, 2, 4 or 8) with
// which the launch still is one.  With fewer it runs in more rounds (1128
// groups x 8192 columns: 208 us at 8 groups per block, 239 us at 4), with more
// it leaves units idle (752 groups x 8192: 200 us at 8, 124 us at 4; 500 groups
// x 8192: 182, 106 and 82 us at 8, 4 and 2).  Past one round 8-wave blocks
// (each fills its unit) stay ahead while the last round is nearly full (8020
// groups x 4096, 120 states: 895 against 973 us), else 4-wave blocks, two to a
// unit, leave the shorter tail (2500 groups x 4096: 208 against 243 us).  With
// one batch tile the waves share nothing, and a nearly full round is 1 to 3%
// faster in 4-wave blocks (1940 groups x 7800: 295 against 297 us; 2000 x 4096:
// 153 against 161 us), a full one with the weights in bursts (2000 x 8192: 307
// against 317 us; 1940 groups: 299 against 295 us; columns below 1024 end before a
// second burst: 2000 groups x 256, 1 state, 11.6 us in bursts, 10.6 without, x 512
// 21.6 and 20.0, x 1024 41.0 and 43.6); 4 groups a block of residual blocks also go
// in 4-wave blocks (640 groups x 8192, 10 states: 105 us, 113 in split 8-wave ones;
// heads stay split, whose sums of two ranges lie nearer to 64 bits: 576 groups x
// 8192 4.0e-7, in one range 5.8e-7, at 109 and 102 us).
// Two tiles share states, and only a round that is full of short rows is
// faster in 4-wave blocks (2000 groups, 17 states: x 1024 44 against 54 us, x 4096
// 157 against 165, x 5120 194 against 193; 1940 x 4096 152 and 154; 1500 x 4096
// 126 and 116).
template <int EPI, int NB>
void launch_gemm_nb(const void *h, int64_t h_head_stride, const void *w, const void *bias, float *z, void *hout,
                      int B, int hidden, int rows, int n_heads, float *gmax, hipStream_t st) {
  const int nG = packed_row_groups(rows), nS = packed_k_steps(hidden);
  auto go = [&](auto kern, int waves, int groups) {
    dim3 grid((nG + groups - 1) / groups, n_heads, (B + 16 * NB - 1) / (16 * NB));
    hipLaunchKernelGGL(kern, grid, dim3(64 * waves), 0, st, static_cast<const uint16_t *>(h), h_head_stride,
                       static_cast<const uint4 *>(w), static_cast<const uint16_t *>(bias), z,
                       static_cast<uint16_t *>(hout), B, hidden, rows, n_heads, nG, nS, gmax);
  };
  const int64_t cus = device_cus();   // each holds one 8-wave block or two 4-wave blocks
  auto blocks = [&](int groups) { return (int64_t)((nG + groups - 1) / groups) * n_heads; };
  const int64_t rounds = (blocks(8) + cus - 1) / cus;
  const bool full = blocks(8) * 100 >= rounds * cus * 97;
  if (blocks(1) <= cus) {
    go(head_gemm<4, NB, 4, (NB <= 4 ? 2 : 1), EPI>, 4, 1);
  } else if (blocks(2) <= cus) {
    if constexpr (NB >= 6) go(head_gemm<8, NB, 4, (NB == 6 ? 2 : 1), EPI>, 8, 2);
    else go(head_gemm<4, NB, 2, 4, EPI>, 4, 2);
  } else if (blocks(4) <= cus) {
    if constexpr (NB == 1 && EPI == 1) go(head_gemm<4, 1, 1, 4, EPI>, 4, 4);
    else go(head_gemm<8, NB, 2, (NB >= 6 ? 2 : 4), EPI>, 8, 4);
  } else if (NB == 1                        ? blocks(8) * 8 <= cus * 7
             : NB == 2 && hidden <= 4096    ? !full && (rounds == 1 || blocks(8) * 10 >= rounds * cus * 9)
                                            : rounds == 1 || blocks(8) * 10 >= rounds * cus * 9) {
    go(head_gemm<8, NB, 1, 4, EPI>, 8, 8);
  } else if (NB == 1 && full && hidden >= 1024) {
    if constexpr (NB == 1) go(head_gemm<4, 1, 1, 4, EPI, true>, 4, 4);
  } else {
    go(head_gemm<4, NB, 1, 4, EPI>, 4, 4);
  }
}

template <int EPI>
hipError_t launch_gemm(const void *h, int64_t h_head_stride, const void *w, const void *bias, float *z, void *hout,
                         int B, int hidden, int rows, int n_heads, float *gmax, hipStream_t st) {
  // batch tiles of a block: the fewest of 1, 2, 4, 6, 8 that hold the batch (past 128 states, groups of 128);
  // the shared states are addressed with 32 bits from a group's first row, which 2^24 columns could exceed
  int nb = B <= 16 || hidden >= 1 << 24 ? 1 : B <= 32 ? 2 : B <= 64 ? 4 : B <= 96 ? 6 : 8;
  // Few row groups leave units idle, and the weights are small: the batch is spread over blocks with as few tiles
  // as still make one round (residual blocks of 512 columns, 2 heads, 128 states: 6.4 us at 1, 7.7 at 2, 9.2 at 4,
  // 15.6 at 8 tiles; of 4096: 54 us at 1, which makes 4 rounds, 26.5 at 4, 47 at 8).  Past one round short rows,
  // whose epilogue outweighs the weights, stay at 4 (2048 columns, 5 heads, 128 states: 24.5 us at 4, 29.8 at 8;
  // 4096 columns, 189 groups, 100 states: 42.8 and 39.8 us).
  const int64_t groups = (int64_t)packed_row_groups(rows) * n_heads, cus = device_cus();
  if (groups <= cus) {
    for (int n = 1; n <= 4; n *= 2)
      if (n < nb && groups * ((B + 16 * n - 1) / (16 * n)) <= cus) nb = n;
    if (nb > 4 && hidden <= 2048) nb = 4;
  }
  auto kern = nb == 1   ? launch_gemm_nb<EPI, 1>
              : nb == 2 ? launch_gemm_nb<EPI, 2>
              : nb == 4 ? launch_gemm_nb<EPI, 4>
              : nb == 6 ? launch_gemm_nb<EPI, 6>
                        : launch_gemm_nb<EPI, 8>;
  kern(h, h_head_stride, w, bias, z, hout, B, hidden, rows, n_heads, gmax, st);
  return hipGetLastError();
}

template <int EPI>
void launch_f32(const void *h, int64_t h_head_stride, const void *w, const void *bias, float *z, void *hout, int B,
                int hidden, int rows, int n_heads, hipStream_t st) {
  // short rows: few products per reduction, so fewer sums at a time (21 states, 1558 x 280: 9 us at 2, 15 us at 4;
  // 32 states, 8000 x 1024: 223 us at 2, 145 us at 4, 166 us at 8)
  const int J = B == 1 ? 1 : B == 2 || hidden <= 640 ? 2 : 4;
  auto kern = J == 1 ? head_logits_f32<EPI, 1> : J == 2 ? head_logits_f32<EPI, 2> : head_logits_f32<EPI, 4>;
  hipLaunchKernelGGL(kern, dim3((rows + 15) / 16, n_heads, (B + J - 1) / J), dim3(256), 0, st, static_cast<const float *>(h),
                     h_head_stride, static_cast<const float *>(w), z, static_cast<const float *>(bias),
                     static_cast<float *>(hout), B, hidden, rows, n_heads);
}

}  // namespace

hipError_t launch_head_logits(int dt, const void *h, int64_t h_head_stride, const void *w, bool packed, float *z,
                              int B, int hidden, int vocab, int n_heads, hipStream_t st, float *gmax) {
  if (dt == 1 && packed)
    return launch_gemm<0>(h, h_head_stride, w, nullptr, z, nullptr, B, hidden, vocab, n_heads, gmax, st);
  if (dt == 1) {
    // batch tiles of a block: the fewest of 1, 2, 4, 8 that hold the batch; a ring as deep as LDS allows.  The
    // states are addressed with 32 bits from a block's first row, which 2^24 columns could exceed.
    int nb = B <= 16 || hidden >= 1 << 24 ? 1 : B <= 32 ? 2 : B <= 64 ? 4 : 8;
    // A vocabulary that leaves units idle (one block a unit): as few tiles as still make one round (2 heads, 128
    // states, 50 x 1000: 5.8 us at 1 tile, 17.3 at 8; 4000 x 4096: 30.7 us at 1, two rounds, 19.4 at 2, 46.5 at 8).
    const int64_t blocks = (int64_t)((vocab + 127) / 128) * n_heads, cus = device_cus();
    for (int n = 1; n <= 4; n *= 2)
      if (n < nb && blocks * ((B + 16 * n - 1) / (16 * n)) <= cus) nb = n;
    const dim3 grid((vocab + 127) / 128, n_heads, (B + 16 * nb - 1) / (16 * nb));
    auto kern = nb == 1 ? head_rows<1, 4> : nb == 2 ? head_rows<2, 3> : nb == 4 ? head_rows<4, 3> : head_rows<8, 2>;
    hipLaunchKernelGGL(kern, grid, dim3(512), 0, st, static_cast<const uint16_t *>(h), h_head_stride,
                       static_cast<const uint8_t *>(w), z, B, hidden, vocab, n_heads, packed_row_groups(vocab), gmax);
  } else {
    launch_f32<0>(h, h_head_stride, w, nullptr, z, nullptr, B, hidden, vocab, n_heads, st);
  }
  return hipGetLastError();
}

hipError_t launch_resblock(int dt, const void *h, const void *w1, const void *b1, void *out, int B, int hidden,
                           int n_heads, hipStream_t st) {
  if (dt == 1) return launch_gemm<1>(h, 0, w1, b1, nullptr, out, B, hidden, hidden, n_heads, nullptr, st);
  launch_f32<1>(h, 0, w1, b1, nullptr, out, B, hidden, hidden, n_heads, st);
  return hipGetLastError();
}

hipError_t launch_pack_heads(const void *src, void *dst, int n_heads, int vocab, int hidden, hipStream_t st) {
  const int nG = packed_row_groups(vocab), nS = packed_k_steps(hidden);
  const int64_t chunks = (int64_t)n_heads * nG * nS * 4 * 64;
  hipLaunchKernelGGL(pack_heads_bf16, dim3((unsigned)((chunks + 255) / 256)), dim3(256), 0, st,
                     static_cast<const uint16_t *>(src), static_cast<uint4 *>(dst), vocab, hidden, nG, nS, chunks);
  return hipGetLastError();
}

hipError_t launch_topk(const TopkArgs &a, int B, hipStream_t st) {
  hipLaunchKernelGGL(topk_rows, dim3(B * a.n_heads), dim3(kTopkThreads), 0, st, a);
  return hipGetLastError();
}

}  // namespace specmemo
