// Stage 2 for batches whose slots hold many rows, whatever the M-tile of
// stage 1 and for all three element types: both GEMMs on items of up to 256
// rows x 256 packed weight rows, computed by eight wavefronts.
//
// * Rows are taken per slot, not per M-tile: a slot's rows are contiguous, so
//   "wide tile" u of a slot is its rows 256 u .. 256 u + 255.  The M-tile only
//   sets the padding between slots.
// * Operands in MFMA operand order: the weights from tempo_moe_pack_weights,
//   the activation rows of every wide tile from k_pack_wide, and h from the
//   gate/up epilogue.  Per 128-byte contraction step a packed tile is 4 KB per
//   live block of 32 rows; rows 32b .. 32b + 31 form piece b, four 1 KB loads j
//   in which lane l holds 16-byte chunk c(j, l) of row 32b + l % 32 (fp8
//   c = 4 (j / 2) + 2 (l / 32) + j % 2, bf16 c = 2 j + l / 32), like the packed
//   weights.  A tile starts where its first row's offset puts it (offsets are
//   multiples of the M-tile, so of 32), so that packed rows take no more room
//   than padded ones.  fp8 activation scales lie alike, 32 fp32 per live block
//   and step.
// * Eight wavefronts, two per SIMD: wavefront (wm, wn) takes the row blocks
//   2 i + wm (i = 0 .. 3) against the weight rows 64 wn .. 64 wn + 63 (two
//   pieces j), 128 accumulator registers per lane.  With fp32 block scales a
//   step's product of a row block has to be scaled in VALU before it is added
//   (acc += p * (sA * sW), 16 FMAs per 32 x 32 tile), so the accumulators have
//   to be VGPRs; the second wavefront of a SIMD keeps the matrix pipe busy
//   meanwhile.  The weights are the MFMAs' first operand: a lane owns one
//   token row, so sA is one register per row block.
// * Operands stream through LDS by DMA, 144 KB of ring in one of two forms.
//   Tiles of more than four live row blocks: two slots of weights (32 KB, one
//   step each) and five half-steps of activations (16 KB); a step has two
//   barriers, fragments are read one row block ahead of their MFMAs, and each
//   load is issued between two MFMAs.  Measured (18 slots H 4096 I 1536, 11486
//   rows, gate/up GEMM): fp8 201 us with the loads in bursts and the fragments
//   read at the start of a half-step, 181 like this (157 with neither loads
//   nor fragment reads: the matrix pipes at 2.1 GHz, the rescale, barriers and
//   the uneven last round of items are what is left); UE8M0 179 -> 163, bf16
//   312 -> 294 (242 without loads and reads).  Smaller tiles: whole
//   steps, three slots of 48 KB or, for one live row block, four of 36 KB,
//   since these wait for their weights (64 or 96 KB of them in flight; 36
//   slots H 7168 I 2048, 5024 rows, gate/up 297 -> 272, down 193 -> 155 us).
// * Items are dealt as in the other large-tile kernels: tiles sorted by live
//   row blocks, groups of 4 tiles x all weight blocks, runs per XCD, rounds
//   alternately forwards and backwards; every second XCD works through its
//   items from the small end.  Row blocks of padding only are not computed.
//   What whole rounds leave over goes by halves of items (one weight block of
//   128 rows; four wavefront rows x two, three to seven slots of whole steps),
//   but not in fp8 gate/up, whose h scale spans both blocks (halves of a tile's
//   rows would keep it whole; not built): the last round is the small tiles',
//   and a chip half filled with whole items waits for their latency.
//   Measured: 4097 tokens of 10 slots H 2048 I 1408, UE8M0 down 31.7 -> 23.4
//   us; bf16 18 slots, 1499 tokens, gate/up 129 -> 123, 4096 rows of 512
//   tokens down 61 -> 55, 11486 rows gate/up 295 -> 286.
//   Items are never split: a row's sums run over its steps in order, so its
//   result depends on its own inputs alone.
// * gate/up epilogue: SwiGLU; fp8: the amax of each row over the item's 128
//   h columns (one contraction step of the down GEMM), the scale amax / 448
//   (power of two for UE8M0) and the e4m3 codes, packed for the down GEMM.
#include <algorithm>

#include "gemm_stream.h"

namespace tempo {
namespace {

using namespace gemm;

constexpr int WT_M = 256;                    // rows of a wide tile
constexpr int WT_THREADS = 512;              // eight wavefronts
constexpr int WT_STEP = 32 * 1024;           // bytes of a step of 256 rows
constexpr int WT_UNIT = WT_STEP / 2;         // a half-step of activations: row blocks 0..3 or 4..7
constexpr int WT_NA = 5;                     // activation half-steps in the ring
constexpr int WT_SCW = 160;                  // scale bytes of one wavefront: 32 rows, then two weight blocks
constexpr int WT_SC = 8 * WT_SCW;            // scales of a step (fp8)
constexpr int WT_A = 0;                      // LDS ring: activations,
constexpr int WT_W = WT_NA * WT_UNIT;        //   weights (2 slots),
constexpr int WT_S = WT_W + 2 * WT_STEP;     //   scales (up to 4 slots)
                                             //   (4 slots, or 7 where items are halved)
constexpr int WT_MAX_SORT = 768;             // tiles the cost-ordered list covers (beyond: tile order)
constexpr int WT_GM = 4;                     // tiles per group of the item order

enum WideType : int { kWideF8 = 0, kWideMX = 1, kWideBf16 = 2 };

struct WideArgs {
  const char* A;          // packed activation tiles
  const float* A_sc;      // fp8: their scales
  const char* W;          // packed weights
  size_t w_slot_bytes;
  const float* Wsp;       // fp8: packed weight scales [slot][block][step][4]
  size_t ws_slot_floats;
  const uint64_t* wtab;
  int wfield, sfield;
  char* C;                // gate/up: packed h tiles; down: y_perm rows (bf16)
  float* C_sc;            // gate/up, fp8: their scales
  const int32_t* slot_counts;
  const int32_t* slot_offsets;
  int S, KT, NB, max_tiles;  // KT: steps per item; NB: 128-row weight blocks
  int row_cap;
  int ld_out;             // down: bytes of a row of y_perm
  uint64_t* t0;
  uint64_t* t1;
  int timing;
};

// Slot tables in LDS.  (Counts are held to the slot's own padded rows and the
// row buffers: stage 2 can be called on a caller's counts and offsets.)
__device__ __forceinline__ void wide_slots(const int32_t* __restrict__ counts, const int32_t* __restrict__ offsets,
                                           int S, int row_cap, int32_t* off, int32_t* cnt, int tid, int nthreads) {
  for (int s = tid; s < S; s += nthreads) {
    const int o = min(max(offsets[s], 0), row_cap), e = min(offsets[s + 1], row_cap);
    off[s] = o;
    cnt[s] = max(0, min(counts[s], e - o));
  }
}

// Wide tiles of the slots before s (st has S + 1 entries), by one wavefront.
__device__ __forceinline__ void wide_prefix(const int32_t* cnt, int32_t* st, int S) {
  const int l = threadIdx.x & 63;
  int w[4], run = 0;
#pragma unroll
  for (int i = 0; i < 4; i++) {
    const int s = 4 * l + i;
    run += s < S ? (cnt[s] + WT_M - 1) / WT_M : 0;
    w[i] = run;
  }
  int incl = run;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const int o = __shfl_up(incl, d);
    if (l >= d) incl += o;
  }
#pragma unroll
  for (int i = 0; i < 4; i++)
    if (4 * l + i < S) st[4 * l + i + 1] = incl - run + w[i];
  if (l == 0) st[0] = 0;
}

// Slot of wide tile t (the last s with st[s] <= t).
__device__ __forceinline__ int wide_slot(const int32_t* st, int S, int t) {
  int lo = 0, hi = S;
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (st[mid] <= t) lo = mid;
    else hi = mid;
  }
  return lo;
}

// The first piece (32 rows) of rows from offset off + 256 sub on.
__device__ __forceinline__ size_t wide_piece(int off, int sub) { return (size_t)(off >> 5) + 8 * sub; }

// The activation rows of every wide tile in packed order, from token rows
// (gather: row r is token row_token[r] of A) or from permuted rows; fp8
// scales from the token rows' own [token][KT] (gather) or the block-major
// [KT][row_cap] ones of stage 1.  Padding rows of a live row block are zero
// with scale 1; row blocks of padding only are not written.  x_perm, x_perm_sc
// (each nullable): the stage-1 outputs of the same rows, which the forward
// leaves to this kernel.  One (tile, step) block per workgroup of a fixed grid
// at a time, through LDS, so that 8 lanes read (and write to x_perm) the 128
// consecutive bytes of a row and 64 lanes write 1 KB: fp8 prefill share with
// x_perm 45 us when every lane read and wrote its own 16 bytes of a row, 39
// like this.
template <bool FP8>
__global__ __launch_bounds__(256) void k_pack_wide(const char* __restrict__ A, const float* __restrict__ A_scale,
                                                   int gather, int row_cap, const int32_t* __restrict__ row_token,
                                                   const int32_t* __restrict__ slot_counts,
                                                   const int32_t* __restrict__ slot_offsets, int S, int max_tiles,
                                                   int KT, char* __restrict__ out, float* __restrict__ out_sc,
                                                   char* __restrict__ x_perm, float* __restrict__ x_perm_sc) {
  __shared__ int32_t s_cnt[kMaxS], s_off[kMaxS], s_st[kMaxS + 1];
  __shared__ __attribute__((aligned(16))) char stage[WT_STEP];  // rows of 128 bytes, chunk c at c ^ (row % 8)
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  wide_slots(slot_counts, slot_offsets, S, row_cap, s_off, s_cnt, tid, 256);
  __syncthreads();
  if (tid < 64) wide_prefix(s_cnt, s_st, S);
  __syncthreads();
  const int blocks = min(s_st[S], max_tiles) * KT;
  const size_t row_bytes = (size_t)KT * 128;
#pragma unroll 1
  for (int blk = blockIdx.x; blk < blocks; blk += gridDim.x) {
    const int tile = blk / KT, kt = blk - tile * KT;
    const int slot = __builtin_amdgcn_readfirstlane(wide_slot(s_st, S, tile));
    const int sub = tile - s_st[slot];
    const int row0 = s_off[slot] + sub * WT_M, nvalid = min(WT_M, s_cnt[slot] - sub * WT_M);
    const int live = (nvalid + 31) >> 5;
    const size_t piece = wide_piece(s_off[slot], sub) * KT + (size_t)kt * live;
    int src[8];
    i32x4 v[8];
#pragma unroll
    for (int i = 0; i < 8; i++) {
      const int r = 32 * i + (tid >> 3);
      src[i] = r < nvalid ? (gather ? max(row_token[row0 + r], 0) : row0 + r) : -1;
    }
    float sc = 1.f;
    if (FP8 && tid < nvalid) {
      if (gather) sc = A_scale[(size_t)max(row_token[row0 + tid], 0) * KT + kt];
      else sc = A_scale[(size_t)kt * row_cap + row0 + tid];
    }
#pragma unroll
    for (int i = 0; i < 8; i++) {
      v[i] = (i32x4){0, 0, 0, 0};
      if (src[i] >= 0)
        v[i] = *reinterpret_cast<const i32x4*>(A + (size_t)src[i] * row_bytes + kt * 128 + (tid & 7) * 16);
    }
#pragma unroll
    for (int i = 0; i < 8; i++) {
      if (i >= live) break;
      const int r = 32 * i + (tid >> 3);
      *reinterpret_cast<i32x4*>(stage + swz(r, tid & 7)) = v[i];
      if (x_perm && src[i] >= 0)
        *reinterpret_cast<i32x4*>(x_perm + (size_t)(row0 + r) * row_bytes + kt * 128 + (tid & 7) * 16) = v[i];
    }
    if (FP8 && tid < 32 * live) out_sc[piece * 32 + tid] = sc;
    if (FP8 && x_perm_sc && tid < nvalid) x_perm_sc[(size_t)kt * row_cap + row0 + tid] = sc;
    __syncthreads();
    for (int b = w; b < live; b += 4)
#pragma unroll
      for (int j = 0; j < 4; j++) {
        const int c = FP8 ? 4 * (j >> 1) + 2 * (lane >> 5) + (j & 1) : 2 * j + (lane >> 5);
        *reinterpret_cast<i32x4*>(out + (piece + b) * 4096 + j * 1024 + lane * 16) =
            *reinterpret_cast<const i32x4*>(stage + swz(32 * b + (lane & 31), c));
      }
    __syncthreads();
  }
}

// 16 bytes per lane of `lanes` from per-lane addresses into LDS at
// lds + 16 * lane (EXEC switched inside the statement, as in
// lds_dma16s_lanes).
__device__ __forceinline__ void lds_dma16v_lanes(const void* gptr, uint32_t lds, uint64_t lanes) {
  uint64_t saved;
  asm volatile(
      "s_mov_b64 %0, exec\n\t"
      "s_mov_b64 exec, %3\n\t"
      "s_mov_b32 m0, %2\n\t"
      "s_nop 0\n\t"
      "global_load_lds_dwordx4 %1, off\n\t"
      "s_mov_b64 exec, %0"
      : "=&s"(saved)
      : "v"(gptr), "s"(lds), "s"(lanes)
      : "memory", "m0");
}

// Load J of 1 KB pieces that are consecutive in memory and in LDS (the
// instruction's offset counts in both addresses).
template <int J>
__device__ __forceinline__ void lds_dma16s_at(uint64_t sbase, uint32_t voff, uint32_t lds) {
  asm volatile(
      "s_mov_b32 m0, %2\n\t"
      "s_nop 0\n\t"
      "global_load_lds_dwordx4 %0, %1 offset:%3" ::"v"(voff),
      "s"(sbase), "s"(lds), "n"(J * 1024)
      : "memory", "m0");
}
// Four (two) of them, with one M0.
__device__ __forceinline__ void lds_dma16s_x4(uint64_t sbase, uint32_t voff, uint32_t lds) {
  asm volatile(
      "s_mov_b32 m0, %2\n\t"
      "s_nop 0\n\t"
      "global_load_lds_dwordx4 %0, %1\n\t"
      "global_load_lds_dwordx4 %0, %1 offset:1024\n\t"
      "global_load_lds_dwordx4 %0, %1 offset:2048\n\t"
      "global_load_lds_dwordx4 %0, %1 offset:3072" ::"v"(voff),
      "s"(sbase), "s"(lds)
      : "memory", "m0");
}
__device__ __forceinline__ void lds_dma16s_x2(uint64_t sbase, uint32_t voff, uint32_t lds) {
  asm volatile(
      "s_mov_b32 m0, %2\n\t"
      "s_nop 0\n\t"
      "global_load_lds_dwordx4 %0, %1\n\t"
      "global_load_lds_dwordx4 %0, %1 offset:1024" ::"v"(voff),
      "s"(sbase), "s"(lds)
      : "memory", "m0");
}
// the same two, or, where on is 0, two loads of no lane (they only count)
__device__ __forceinline__ void lds_dma16s_x2_if(uint64_t sbase, uint32_t voff, uint32_t lds, int on) {
  uint64_t saved;
  asm volatile(
      "s_mov_b64 %0, exec\n\t"
      "s_cmp_lg_u32 %4, 0\n\t"
      "s_cselect_b64 exec, exec, 0\n\t"
      "s_mov_b32 m0, %2\n\t"
      "s_nop 0\n\t"
      "global_load_lds_dwordx4 %1, %3\n\t"
      "global_load_lds_dwordx4 %1, %3 offset:1024\n\t"
      "s_mov_b64 exec, %0"
      : "=&s"(saved)
      : "v"(voff), "s"(lds), "s"(sbase), "s"(__builtin_amdgcn_readfirstlane(on))
      : "memory", "m0", "scc");
}

template <int DT, bool GATEUP>
__global__ __launch_bounds__(WT_THREADS, 2) void k_gemm_wide(const WideArgs p) {
  constexpr bool F8 = DT != kWideBf16, MX = DT == kWideMX;
  constexpr int SL = F8 ? 1 : 0;             // scale loads per wavefront and step
  // the last, partly filled rounds go by halves of items (one weight block),
  // but for fp8 gate/up, which quantises h over both blocks' columns
  constexpr bool HALVES = !(F8 && GATEUP);
  __shared__ __attribute__((aligned(1024))) char ring[WT_S + (HALVES ? 7 : 4) * WT_SC];
  __shared__ float xamax[4][WT_M];
  __shared__ int32_t s_off[kMaxS], s_cnt[kMaxS], s_st[kMaxS + 1];
  __shared__ uint32_t s_ord[WT_MAX_SORT];    // slot | (wide tile within the slot) << 8, in cost order

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave & 1, wn = wave >> 1;
  wide_slots(p.slot_counts, p.slot_offsets, p.S, p.row_cap, s_off, s_cnt, tid, WT_THREADS);
  __syncthreads();
  if (tid < 64) wide_prefix(s_cnt, s_st, p.S);
  __syncthreads();
  const int NT = __builtin_amdgcn_readfirstlane(min(s_st[p.S], p.max_tiles));
  const bool sorted = NT <= WT_MAX_SORT;
  auto tile_desc = [&](int t) {
    const int s = wide_slot(s_st, p.S, t);
    return (uint32_t)s | (uint32_t)(t - s_st[s]) << 8;
  };
  auto live_of = [&](uint32_t d) { return (min(WT_M, s_cnt[d & 255] - (int)(d >> 8) * WT_M) + 31) >> 5; };
  if (sorted && tid < 64) {
    // stable counting sort by live row blocks, most first (descriptors and
    // classes once per tile, held in the ring's bytes between the passes)
    uint32_t* const tmp = reinterpret_cast<uint32_t*>(ring);
    const uint64_t below = (1ull << lane) - 1;
    int pos[9] = {};
    for (int t0 = 0; t0 < NT; t0 += 64) {
      const int t = t0 + lane;
      const uint32_t d = t < NT ? tile_desc(t) : 0;
      const int c = t < NT ? live_of(d) : 0;
      tmp[t] = d | (uint32_t)c << 27;
#pragma unroll
      for (int k = 1; k <= 8; k++) pos[k] += __popcll(__ballot(c == k));
    }
    int run = 0;
#pragma unroll
    for (int k = 8; k >= 1; k--) {
      const int m = pos[k];
      pos[k] = run;
      run += m;
    }
    for (int t0 = 0; t0 < NT; t0 += 64) {
      const uint32_t v = tmp[t0 + lane];
      const int c = v >> 27;
#pragma unroll
      for (int k = 1; k <= 8; k++) {
        const uint64_t m = __ballot(c == k);
        if (c == k) s_ord[pos[k] + __popcll(m & below)] = v & 0x7FFFFFF;
        pos[k] += __popcll(m);
      }
    }
  }
  __syncthreads();

  const int KT = p.KT;
  const int NBT = (p.NB + 1) / 2;  // items per tile
  const int items = NT * NBT;
  const int G = gridDim.x;
  const int lin0 = (G % 8 == 0) ? (blockIdx.x % 8) * (G / 8) + blockIdx.x / 8 : blockIdx.x;
  // `full` whole rounds of items, then what is left in halves; where there is
  // no whole round, only what fits one round of halves (two of them take
  // longer than one of whole items: 10 slots, 3377 tokens, bf16 146 us for
  // 134 on 230 gate/up items)
  const int full = items / G;
  int rest = items - full * G, rounds = full;
  const bool halve = HALVES && (full > 0 || 2 * rest <= G);
  if (halve) {
    rest *= 2;
    if (rest >= G) rest -= G, rounds++;
  }
  const int my_items = rounds + (((rounds & 1) ? G - 1 - lin0 : lin0) < rest ? 1 : 0);
  if (my_items == 0) return;
  // Item n of this workgroup: slot | sub << 8, the pair of weight blocks, and
  // which of the two (-1: both).  Every second XCD takes its items the other
  // way round, the small ones first: tiles of few rows wait for their weights,
  // full ones for the matrix pipes, and the two kinds run side by side.
  auto item_of = [&](int n, int& nbt, int& half) {
    if (blockIdx.x & 1) n = my_items - 1 - n;
    int it = n * G + ((n & 1) ? G - 1 - lin0 : lin0);
    half = -1;
    if (halve && n >= full) {
      const int j = it - full * G;
      it = full * G + (j >> 1);
      half = j & 1;
    }
    const int grp = it / (WT_GM * NBT), w_in = it - grp * (WT_GM * NBT);
    const int gm = min(WT_GM, NT - grp * WT_GM);
    nbt = w_in / gm;
    const int t = grp * WT_GM + (w_in - nbt * gm);
    // (the count through an empty asm: the compiler would keep the condition in
    // a vector register, and spill it)
    int nt = NT;
    asm volatile("" : "+s"(nt));
    return (uint32_t)__builtin_amdgcn_readfirstlane(nt <= WT_MAX_SORT ? s_ord[t] : tile_desc(t));
  };
  auto uni = [](uint64_t v) {
    return ((uint64_t)__builtin_amdgcn_readfirstlane((uint32_t)(v >> 32)) << 32) |
           (uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)v);
  };

  const uint32_t ring_lds = lds_addr(ring);
  const uint32_t lane16 = lane * 16;
  struct Item {
    int slot, sub, nbt, half, live;
  };
  auto item = [&](int n) {
    Item it;
    const uint32_t d = item_of(n, it.nbt, it.half);
    it.slot = d & 255;
    it.sub = d >> 8;
    it.live = __builtin_amdgcn_readfirstlane(live_of(d));
    return it;
  };
  // this wavefront's weights of an item: piece wave of the eight, or half a
  // piece of a half's four (a block past the last one is the last one again,
  // read by nobody)
  auto table = [&]() {
    const uint64_t* t = p.wtab;  // (through an empty asm: see item_of)
    asm volatile("" : "+s"(t));
    return t;
  };
  auto w_of = [&](const Item& it) {
    const int blk = min(2 * it.nbt + (it.half < 0 ? wave >> 2 : it.half), p.NB - 1);
    return uni((uint64_t)(uintptr_t)slot_tensor(p.W, p.w_slot_bytes, table(), p.wfield, it.slot) +
               (size_t)blk * KT * B_BYTES + (it.half < 0 ? (wave & 3) * 4096 : wave * 2048));
  };
  auto a_of = [&](const Item& it) {
    return uni((uint64_t)(uintptr_t)p.A + wide_piece(s_off[it.slot], it.sub) * KT * 4096);
  };
  // fp8 scales of a step, one load: lanes 0 .. 7 those of rows 32 wave .. 32
  // wave + 31 (of the last live block for the dead ones), lanes 8 and 9 those
  // of the two weight blocks
  auto fresh_lane = []() {
    int l;
    asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(l));
    return l;
  };
  auto s_of = [&](const Item& it) {
    const char* ws =
        slot_tensor(reinterpret_cast<const char*>(p.Wsp), p.ws_slot_floats * 4, table(), p.sfield, it.slot);
    const char* as =
        reinterpret_cast<const char*>(p.A_sc + (wide_piece(s_off[it.slot], it.sub) * KT + min(wave, it.live - 1)) * 32);
    // (the lane and what is made of it anew: spilled, its reload would wait for the DMAs)
    const int l = fresh_lane();
    const int blk = min(2 * it.nbt + (it.half < 0 ? (l == 9 ? 1 : 0) : it.half), p.NB - 1);
    return l < 8 ? as + l * 16 : ws + (size_t)blk * KT * 16;
  };
  constexpr uint64_t S_LANES = 0x3FFull;

  // ---- compute ----
  f32x16 acc[4][2];
  i32x8 fa[2][2], fb[2][2];  // [buffer i % 2][half], [piece j][half]
  float sa[4], sw0 = 1.f, sw1 = 1.f;
  auto rd8 = [&](const char* s) {
    const i32x4 lo = *reinterpret_cast<const i32x4*>(s);
    const i32x4 hi = *reinterpret_cast<const i32x4*>(s + 1024);
    return (i32x8){lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
  };
  // two pieces of weights from w, a row block from a into buffer i, the scales
  // of ring slot `slot` for row blocks rb0 + rbs i and weight block `blk` of the item
  auto read_b = [&](const char* w, int j) {
#pragma unroll
    for (int h = 0; h < 2; h++) fb[j][h] = rd8(w + lane16 + j * 4096 + h * 2048);
  };
  auto read_a = [&](const char* a, int i) {
#pragma unroll
    for (int h = 0; h < 2; h++) fa[i & 1][h] = rd8(a + lane16 + h * 2048);
  };
  auto read_s = [&](auto ni, int slot, int rb0, int rbs, int blk) {
    const char* s = ring + WT_S + slot * WT_SC;
#pragma unroll
    for (int i = 0; i < decltype(ni)::value; i++)
      sa[i] = *reinterpret_cast<const float*>(s + (rb0 + rbs * i) * WT_SCW + (lane & 31) * 4);
    const float2 v = *reinterpret_cast<const float2*>(s + 128 + 16 * blk);
    sw0 = v.x;
    if (GATEUP) sw1 = v.y;
  };
  auto ue = [](float s) { return (int)((__float_as_uint(s) >> 23) & 0xFF); };
  // acc of row block i += its rows times this wavefront's weight rows, over
  // one step.  then(q) after a quarter of the MFMAs each: other instructions
  // go between them one by one (a burst of loads from all wavefronts would
  // queue in the texture addresser and hold up the MFMAs behind it).
  auto mul = [&](int i, auto then) {
    const i32x8(&a)[2] = fa[i & 1];
    if constexpr (DT == kWideBf16) {
#pragma unroll
      for (int j = 0; j < 2; j++) {
#pragma unroll
        for (int ks = 0; ks < 4; ks++) {
          const int o = 4 * (ks & 1);
          const i32x8 &av = a[ks >> 1], &bv = fb[j][ks >> 1];
          const i32x4 ax = {av[o], av[o + 1], av[o + 2], av[o + 3]}, bx = {bv[o], bv[o + 1], bv[o + 2], bv[o + 3]};
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(reinterpret_cast<const bf16x8&>(bx),
                                                              reinterpret_cast<const bf16x8&>(ax), acc[i][j], 0, 0, 0);
          if (ks & 1) {
            __builtin_amdgcn_sched_barrier(0);
            then(2 * j + (ks >> 1));
          }
        }
      }
    } else if constexpr (MX) {
      const int ea = ue(sa[i]);
      const int eb = GATEUP ? ((lane & 16) ? ue(sw1) : ue(sw0)) : ue(sw0);
#pragma unroll
      for (int j = 0; j < 2; j++) {
#pragma unroll
        for (int h = 0; h < 2; h++) {
          acc[i][j] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(fb[j][h], a[h], acc[i][j], 0, 0, 0, eb, 0, ea);
          __builtin_amdgcn_sched_barrier(0);
          then(2 * j + h);
        }
      }
    } else {
      f32x16 pp[2];
#pragma unroll
      for (int j = 0; j < 2; j++) {
        const f32x16 z = {};
#pragma unroll
        for (int h = 0; h < 2; h++) {
          pp[j] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(fb[j][h], a[h], h ? pp[j] : z, 0, 0, 0, 127, 0, 127);
          __builtin_amdgcn_sched_barrier(0);
          then(2 * j + h);
        }
      }
      __builtin_amdgcn_sched_barrier(0);
      // elements 0 .. 7 belong to the gate rows of a piece, 8 .. 15 to the up rows
      const float s0 = sa[i] * sw0, s1 = GATEUP ? sa[i] * sw1 : s0;
#pragma unroll
      for (int j = 0; j < 2; j++)
#pragma unroll
        for (int e = 0; e < 16; e++) acc[i][j][e] += pp[j][e] * (e < 8 ? s0 : s1);
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  auto nothing = [](int) {};

  // Start and end of an item: this wavefront's row blocks rb0 + rbs i (i < NI;
  // live ones: i < nb) against the weight rows 64 g .. of the item's 256.
  struct Out {
    int n, nb, rb0, rbs, g;
    uint64_t tstart;
  };
  auto begin = [&](auto ni, int n) {
    constexpr int NI = decltype(ni)::value;
    const Item it = item(n);
    Out o;
    o.n = n;
    o.rb0 = it.half < 0 ? wm : wave >> 1;
    o.rbs = it.half < 0 ? 2 : 4;
    o.g = it.half < 0 ? wn : 2 * it.half + (wave & 1);
    // (none live where its weight block is past the last one)
    o.nb = 2 * it.nbt + (o.g >> 1) < p.NB ? (it.half < 0 ? (it.live + 1 - o.rb0) >> 1 : (it.live + 3 - o.rb0) >> 2) : 0;
    int timing = p.timing;
    asm volatile("" : "+s"(timing));
    o.tstart = timing ? __builtin_amdgcn_s_memrealtime() : 0;
#pragma unroll
    for (int i = 0; i < NI; i++)
#pragma unroll
      for (int j = 0; j < 2; j++)
#pragma unroll
        for (int e = 0; e < 16; e++) acc[i][j][e] = 0.f;
    return o;
  };
  auto finish = [&](auto ni, const Out& o) {
    constexpr int NI = decltype(ni)::value;
    const Item it = item(o.n);
    const int nbt = it.nbt, nb = o.nb, g = o.g;
    const size_t piece = wide_piece(s_off[it.slot], it.sub);  // of the packed h
    const int row0 = __builtin_amdgcn_readfirstlane(s_off[it.slot] + it.sub * WT_M);
    const int nvalid = __builtin_amdgcn_readfirstlane(min(WT_M, s_cnt[it.slot] - it.sub * WT_M));
    // Epilogue.  Lane l of tile (i, j) holds token row 32 (rb0 + rbs i) + l % 32
    // and, in element e, packed weight row 8 (e / 4) + 4 (l / 32) + e % 4 of
    // piece 2 (g & 1) + j of block 2 nbt + g / 2 (gate/up: rows 0 .. 15
    // gate, 16 .. 31 up, so a column's gate and up are elements e and e + 8).
    const int lid = fresh_lane();
    const int l31 = lid & 31, hl = lid >> 5;
    auto pack4 = [](float v0, float v1, float v2, float v3) {
      uint2 w;
      w.x = bf16x2_rne(v0, v1);
      w.y = bf16x2_rne(v2, v3);
      return w;
    };
    // lanes l and l + 32 hold 8-byte halves of 16-byte chunks; a swap gives
    // lane l < 32 the whole chunk of w0, lane l + 32 that of w1
    auto swap16 = [](uint2 w0, uint2 w1) {
      const auto x = __builtin_amdgcn_permlane32_swap(w0.x, w1.x, false, false);
      const auto y = __builtin_amdgcn_permlane32_swap(w0.y, w1.y, false, false);
      return i32x4{(int)x[0], (int)y[0], (int)x[1], (int)y[1]};
    };
    if constexpr (GATEUP && F8) {
      // h in place of the gate elements, and its amax over the item's 128
      // columns: this lane's, the row's other lane's, the other wavefronts'
#pragma unroll
      for (int i = 0; i < NI; i++) {
        float m = 0.f;
#pragma unroll
        for (int j = 0; j < 2; j++)
#pragma unroll
          for (int e = 0; e < 8; e++) {
            const float h = silu_mul(acc[i][j][e], acc[i][j][e + 8]);
            acc[i][j][e] = h;
            m = fmaxf(m, fabsf(h));
          }
        m = fmaxf(m, __shfl_xor(m, 32));
        if (hl == 0) xamax[g][32 * (o.rb0 + o.rbs * i) + l31] = m;
      }
      wait_lgkm0();
      barrier_nofence();
      // chunk 4 (g / 2) + 2 (g & 1) + j of the row in step nbt of the down
      // GEMM: load 2 (g / 2) + j, lane l % 32 + 32 (g & 1)
      const size_t at = piece * (p.NB / 2) + nbt * it.live;
      char* hb = p.C + at * 4096 + (2 * (g >> 1) + hl) * 1024 + (32 * (g & 1) + l31) * 16;
      float* hs = p.C_sc + at * 32;
#pragma unroll
      for (int i = 0; i < NI; i++) {
        if (i >= nb) continue;
        const int r = 32 * (o.rb0 + o.rbs * i) + l31;
        const float mm = fmaxf(fmaxf(xamax[0][r], xamax[1][r]), fmaxf(xamax[2][r], xamax[3][r]));
        float sc = mm > 0.f ? mm / 448.0f : 1.0f;
        if (MX && mm > 0.f) {
          uint32_t bits = __float_as_uint(sc);
          if (bits & 0x7FFFFFu) bits = (bits & 0xFF800000u) + 0x800000u;  // next power of two up
          sc = __uint_as_float(bits);
        }
        if (g == 0 && hl == 0) hs[r] = sc;
        // h / sc, correctly rounded from the reciprocal (Markstein 1990: r =
        // 1 / sc, q0 = h r, q = q0 + (h - q0 sc) r); tiny rows are scaled up
        // so that r stays finite, and an infinite sc gives 0 or NaN like the
        // division
        const float up = mm < 1e-20f ? 0x1p64f : 1.0f;
        const float scs = __builtin_isinf(sc) ? 0.f : sc * up, rcp = __builtin_isinf(sc) ? 0.f : 1.0f / scs;
        uint32_t w[2][2];
#pragma unroll
        for (int j = 0; j < 2; j++) {
          float q[8];
#pragma unroll
          for (int e = 0; e < 8; e++) {
            const float v = acc[i][j][e] * up, q0 = v * rcp;
            q[e] = fminf(fmaxf(fmaf(fmaf(-q0, scs, v), rcp, q0), -448.f), 448.f);
          }
#pragma unroll
          for (int t = 0; t < 2; t++) {
            uint32_t v = __builtin_amdgcn_cvt_pk_fp8_f32(q[4 * t], q[4 * t + 1], 0, false);
            w[t][j] = __builtin_amdgcn_cvt_pk_fp8_f32(q[4 * t + 2], q[4 * t + 3], v, true);
          }
        }
        // bytes 4 hl .. + 3 and 8 + 4 hl .. + 3 of the chunk; one swap per
        // dword gives lane l the chunk of j = 0, lane l + 32 that of j = 1
        const auto x = __builtin_amdgcn_permlane32_swap(w[0][0], w[0][1], false, false);
        const auto y = __builtin_amdgcn_permlane32_swap(w[1][0], w[1][1], false, false);
        *reinterpret_cast<i32x4*>(hb + (o.rb0 + o.rbs * i) * 4096) = i32x4{(int)x[0], (int)x[1], (int)y[0], (int)y[1]};
      }
    } else if constexpr (GATEUP) {
      // columns 64 (g / 2) + 16 p + 8 q + 4 hl + m of the item's 128 (p the
      // piece): chunk 2 p + q of step 2 nbt + g / 2 of the down GEMM, i.e.
      // load p, lane l % 32 + 32 q
      char* hb = p.C + (piece * p.NB + (2 * nbt + (g >> 1)) * it.live) * 4096 + 2 * (g & 1) * 1024 + lid * 16;
#pragma unroll
      for (int i = 0; i < NI; i++) {
        if (i >= nb) continue;
#pragma unroll
        for (int j = 0; j < 2; j++) {
          const f32x16& v = acc[i][j];
          uint2 w[2];
#pragma unroll
          for (int q = 0; q < 2; q++)
            w[q] = pack4(silu_mul(v[4 * q], v[4 * q + 8]), silu_mul(v[4 * q + 1], v[4 * q + 9]),
                         silu_mul(v[4 * q + 2], v[4 * q + 10]), silu_mul(v[4 * q + 3], v[4 * q + 11]));
          *reinterpret_cast<i32x4*>(hb + (o.rb0 + o.rbs * i) * 4096 + j * 1024) = swap16(w[0], w[1]);
        }
      }
    } else {
      char* yb = p.C + (size_t)row0 * p.ld_out + (size_t)(256 * nbt + 64 * g) * 2;
#pragma unroll
      for (int i = 0; i < NI; i++) {
        if (i >= nb) continue;
        const int r = 32 * (o.rb0 + o.rbs * i) + l31;
        const uint32_t yr = (uint32_t)r * (uint32_t)p.ld_out + 16 * hl;
#pragma unroll
        for (int j = 0; j < 2; j++) {
          const f32x16& v = acc[i][j];
          uint2 w[4];
#pragma unroll
          for (int q = 0; q < 4; q++) w[q] = pack4(v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]);
          const i32x4 c0 = swap16(w[0], w[1]), c1 = swap16(w[2], w[3]);
          if (r < nvalid) {  // padding rows of y_perm stay unwritten
            *reinterpret_cast<i32x4*>(yb + yr + (32 * j) * 2) = c0;
            *reinterpret_cast<i32x4*>(yb + yr + (32 * j + 16) * 2) = c1;
          }
        }
      }
    }
    int timing = p.timing;
    asm volatile("" : "+s"(timing));
    if (timing && wave == 0 && lid == 0) {
      const uint64_t tend = __builtin_amdgcn_s_memrealtime();
      atomicMin(reinterpret_cast<unsigned long long*>(&p.t0[it.slot]), (unsigned long long)o.tstart);
      atomicMax(reinterpret_cast<unsigned long long*>(&p.t1[it.slot]), (unsigned long long)tend);
    }
  };
  // Everyone's reads are done and at most n of this wavefront's loads are in flight.
  auto sync = [&](auto nc) {
    wait_lgkm0();
    __builtin_amdgcn_s_waitcnt(TEMPO_VMCNT_IMM(decltype(nc)::value));
    barrier_nofence();
    __builtin_amdgcn_sched_barrier(0);
  };

  // ---- items n0 .. n1 - 1, tiles of more than four live row blocks ----
  // Two slots of weights, five half-steps of activations.  Fragments are read
  // one row block ahead: while the MFMAs of row block i run, those of i + 1
  // come out of LDS, and the first row block and weight piece of the next step
  // during the last row block of this one.  Past the last item the last one is
  // loaded again, so that every barrier sees the same number of loads; a row
  // block of padding only is replaced by block 0 of the tile (read by nobody).
  auto run_wide = [&](int n0, int n1) {
    int ca_n = n0 - 1, ca_k = KT - 1, ca_h = 1, ca_u = WT_NA - 1;
    int cw_n = n0 - 1, cw_k = KT - 1, cw_s = 1;
    uint64_t a_base = 0, w_base = 0;
    uint32_t a_blk[2] = {0, 0}, a_step = 0, sc_step = 0;
    const char* s_ptr = nullptr;
    // a half-step: this wavefront's 2 KB of it (row block 4 h + wave / 2, loads 2 (wave & 1) and + 1)
    uint64_t a_src = 0, w_src = 0;
    uint32_t a_dst = 0, w_dst = 0, s_dst = 0;
    auto next_a = [&]() {
      if (++ca_u == WT_NA) ca_u = 0;
      if ((ca_h ^= 1) == 0 && ++ca_k == KT) {
        ca_k = 0;
        ca_n = min(ca_n + 1, n1 - 1);
        const Item it = item(ca_n);
        a_base = a_of(it) + (wave & 1) * 2048;
        a_step = it.live * 4096;
#pragma unroll
        for (int h = 0; h < 2; h++) {
          const int b = 4 * h + (wave >> 1);
          a_blk[h] = __builtin_amdgcn_readfirstlane(b < it.live ? b * 4096 : 0);
        }
      }
      a_src = a_base + (size_t)ca_k * a_step + (ca_h ? a_blk[1] : a_blk[0]);
      a_dst = ring_lds + WT_A + ca_u * WT_UNIT + wave * 2048;
    };
    auto next_w = [&]() {
      cw_s ^= 1;
      if (++cw_k == KT) {
        cw_k = 0;
        cw_n = min(cw_n + 1, n1 - 1);
        const Item it = item(cw_n);
        w_base = w_of(it);
        if (F8) {
          s_ptr = s_of(it);
          sc_step = it.live * 128;
        }
      }
      w_src = w_base + (size_t)cw_k * B_BYTES;
      w_dst = ring_lds + WT_W + cw_s * WT_STEP + wave * 4096;
      s_dst = ring_lds + WT_S + cw_s * WT_SC + wave * WT_SCW;
    };
    auto load_s = [&]() {
      if (F8) {
        lds_dma16v_lanes(s_ptr, s_dst, S_LANES);
        s_ptr += lane < 8 ? sc_step : 16;
      }
    };
    auto load_a = [&]() {
      next_a();
      lds_dma16s_x2(a_src, lane16, a_dst);
    };
    auto load_w = [&]() {
      next_w();
      lds_dma16s_x4(w_src, lane16, w_dst);
      load_s();
    };
    // the same, one load after a quarter of a row block's MFMAs each
    auto put_w = [&](int q) {
      if (q == 0) lds_dma16s_at<0>(w_src, lane16, w_dst);
      if (q == 1) lds_dma16s_at<1>(w_src, lane16, w_dst);
      if (q == 2) lds_dma16s_at<2>(w_src, lane16, w_dst);
      if (q == 3) lds_dma16s_at<3>(w_src, lane16, w_dst);
      __builtin_amdgcn_sched_barrier(0);
    };
    auto put_sa = [&](int q) {
      if (q == 0) load_s();
      if (q == 1) lds_dma16s_at<0>(a_src, lane16, a_dst);
      if (q == 2) lds_dma16s_at<1>(a_src, lane16, a_dst);
      __builtin_amdgcn_sched_barrier(0);
    };
    auto all = [&](auto put) {
#pragma unroll
      for (int q = 0; q < 4; q++) put(q);
    };
    // The two barriers of a step, each one row block ahead of the reads that
    // need it: the second half-step's rows have landed (after row block 0),
    // the next step's weights, scales and first half-step have (after row
    // block 2); and every wavefront is done with what the loads issued next
    // overwrite: the weights of this step and the second half-step of the one
    // before, then the first half-step of this one.  Loads complete in order;
    // 4 + SL + 2 are issued after the first barrier (weights and scales of
    // step k + 2, its first half-step), 2 after the second (its second
    // half-step), each is needed three barriers later, and one of each
    // follow it.
    constexpr std::integral_constant<int, 8 + SL> in_flight{};
    auto unit_at = [](int u) { return u >= WT_NA ? u - WT_NA : u; };
    int u_rd = 0, w_rd = 0;  // ring positions of the step: its first half-step, its weights
    // (this wavefront's row block i of the half-step in place u, its weights in slot s)
    auto a_at = [&](int u, int i) { return ring + WT_A + u * WT_UNIT + wm * 4096 + 8192 * (i & 1); };
    auto w_at = [&](int s) { return ring + WT_W + s * WT_STEP + wn * 8192; };
    auto scales = [&](int s) { read_s(std::integral_constant<int, 4>{}, s, wm, 2, wn >> 1); };
    load_w();
    load_a();
    load_a();
    load_w();
    load_a();
    load_a();
    sync(std::integral_constant<int, 10 + SL>{});
    read_a(a_at(0, 0), 0);
    read_b(w_at(0), 0);
    if (MX) scales(0);
#pragma unroll 1
    for (int n = n0; n < n1; n++) {
      const Out o = begin(std::integral_constant<int, 4>{}, n);
      const int nb = o.nb;
#pragma unroll 1
      for (int k = 0; k < KT; k++) {
        read_b(w_at(w_rd), 1);
        read_a(a_at(u_rd, 1), 1);
        if (F8 && !MX) scales(w_rd);
        __builtin_amdgcn_sched_barrier(0);
        if (0 < nb) mul(0, nothing);
        sync(in_flight);
        next_w();
        next_a();
        w_rd ^= 1;
        u_rd = unit_at(u_rd + 1);
        read_a(a_at(u_rd, 2), 2);
        __builtin_amdgcn_sched_barrier(0);
        if (1 < nb) mul(1, put_w);
        else all(put_w);
        read_a(a_at(u_rd, 3), 3);
        __builtin_amdgcn_sched_barrier(0);
        if (2 < nb) mul(2, put_sa);
        else all(put_sa);
        sync(in_flight);
        next_a();
        u_rd = unit_at(u_rd + 1);
        read_a(a_at(u_rd, 0), 0);
        __builtin_amdgcn_sched_barrier(0);
        auto put_ab = [&](int q) {
          if (q == 0) lds_dma16s_at<0>(a_src, lane16, a_dst);
          if (q == 1) read_b(w_at(w_rd), 0);  // (its registers are free: the first piece's MFMAs have been issued)
          if (q == 2) lds_dma16s_at<1>(a_src, lane16, a_dst);
          __builtin_amdgcn_sched_barrier(0);
        };
        if (3 < nb) mul(3, put_ab);
        else all(put_ab);
        if (MX) scales(w_rd);
      }
      finish(std::integral_constant<int, 4>{}, o);
    }
  };

  // ---- items n0 .. n1 - 1, tiles of at most four live row blocks, and halves ----
  // These wait for their weights, so the ring holds whole steps instead: AB
  // bytes of activations (all live row blocks), then 32 KB of weights (16 KB
  // for halves), as many slots as fit.  Whole items as above; halves: row
  // blocks wave / 2 + 4 i against 64 of the 128 weight rows.
  auto run_small = [&](int n0, int n1, auto halfc, auto nslc, auto abc) {
    constexpr bool HALF = decltype(halfc)::value;
    constexpr int NSL = decltype(nslc)::value, AB = decltype(abc)::value;
    constexpr int SLOT = AB + (HALF ? WT_UNIT : WT_STEP);
    static_assert(NSL * SLOT <= WT_S, "the ring holds the slots");
    constexpr bool ALL_A = AB == WT_STEP;              // eight row blocks: one per wavefront (else half of one)
    constexpr int NI = HALF && !ALL_A ? 1 : 2;         // row blocks of a wavefront
    constexpr int L = (HALF ? 2 : 4) + SL + (ALL_A ? 4 : 2);  // loads of a step
    constexpr std::integral_constant<int, NI> ni{};
    int c_n = n0 - 1, c_k = KT - 1, c_s = NSL - 1;
    uint64_t a_base = 0, w_base = 0;
    uint32_t a_step = 0;
    int a_b = 0;  // 1 where the row block this wavefront loads is live
    const char* s_ptr = nullptr;
    uint64_t a_src = 0, w_src = 0;
    uint32_t a_dst = 0, w_dst = 0, s_dst = 0;
    auto next = [&]() {
      if (++c_s == NSL) c_s = 0;
      if (++c_k == KT) {
        c_k = 0;
        c_n = min(c_n + 1, n1 - 1);
        const Item it = item(c_n);
        w_base = w_of(it);
        a_base = a_of(it) + wave * (ALL_A ? 4096 : 2048);
        a_step = it.live * 4096;
        a_b = __builtin_amdgcn_readfirstlane((ALL_A ? wave : wave >> 1) < it.live ? 1 : 0);
        if (F8) s_ptr = s_of(it);
      }
      const uint32_t st = ring_lds + c_s * SLOT;
      a_dst = st + wave * (ALL_A ? 4096 : 2048);
      w_dst = st + AB + wave * (HALF ? 2048 : 4096);
      s_dst = ring_lds + WT_S + c_s * WT_SC + wave * WT_SCW;
      w_src = w_base + (size_t)c_k * B_BYTES;
      a_src = a_base + (size_t)c_k * a_step;
    };
    // the loads of a step, one after a quarter of a row block's MFMAs each
    auto put = [&](int q) {
      if (q == 0) lds_dma16s_at<0>(w_src, lane16, w_dst);
      if (q == 1) lds_dma16s_at<1>(w_src, lane16, w_dst);
      if (!HALF && q == 2) lds_dma16s_at<2>(w_src, lane16, w_dst);
      if (!HALF && q == 3) lds_dma16s_at<3>(w_src, lane16, w_dst);
      if (F8 && q == 4) {
        lds_dma16v_lanes(s_ptr, s_dst, S_LANES);
        s_ptr += lane < 8 ? a_step / 32 : 16;
      }
      if (q == 5) lds_dma16s_x2_if(a_src, lane16, a_dst, a_b);
      if (ALL_A && q == 6) lds_dma16s_x2_if(a_src + 2048, lane16, a_dst + 2048, a_b);
      __builtin_amdgcn_sched_barrier(0);
    };
    auto put_lo = [&](int q) { put(q); };
    auto put_hi = [&](int q) { put(4 + q); };
    auto all = [&](auto f) {
#pragma unroll
      for (int q = 0; q < 4; q++) f(q);
    };
    constexpr std::integral_constant<int, (NSL - 2) * L> in_flight{};
    static_assert((NSL - 2) * L <= 63, "the vmcnt field");
#pragma unroll 1
    for (int i = 0; i < NSL - 1; i++) {
      next();
      all(put_lo);
      all(put_hi);
    }
    sync(in_flight);
    int rd = 0;
#pragma unroll 1
    for (int n = n0; n < n1; n++) {
      const Out o = begin(ni, n);
      const int nb = o.nb;
#pragma unroll 1
      for (int k = 0; k < KT; k++) {
        const char* const sa_at = ring + rd * SLOT + (HALF ? wave >> 1 : wm) * 4096;
        const char* const sw_at = ring + rd * SLOT + AB + (HALF ? wave & 1 : wn) * 8192;
        if (0 < nb) {
          read_b(sw_at, 0);
          read_a(sa_at, 0);
          read_b(sw_at, 1);
          if (F8) read_s(ni, rd, HALF ? wave >> 1 : wm, HALF ? 4 : 2, HALF ? 0 : wn >> 1);
          if (NI > 1 && 1 < nb) read_a(sa_at + (HALF ? 4 : 2) * 4096, 1);
        }
        __builtin_amdgcn_sched_barrier(0);
        next();
        if (0 < nb) mul(0, put_lo);
        else all(put_lo);
        if (NI > 1 && 1 < nb) mul(1, put_hi);
        else all(put_hi);
        // step k + 1 has landed and everyone is done with this one's slot
        sync(in_flight);
        if (++rd == NSL) rd = 0;
      }
      finish(ni, o);
    }
  };

  // the items in runs of one kind (a few, as the order is sorted)
  auto kind = [&](int n) {
    const Item it = item(n);
    const int live = sorted ? it.live : 8;
    return (it.half < 0 ? 0 : 3) + (live > 4 ? 0 : live > 1 ? 1 : 2);
  };
#pragma unroll 1
  for (int n0 = 0; n0 < my_items;) {
    const int kd = kind(n0);
    int n1 = n0 + 1;
    while (n1 < my_items && kind(n1) == kd) n1++;
    constexpr std::false_type whole{};
    constexpr std::true_type half{};
    constexpr std::integral_constant<int, 4096> a1{};
    constexpr std::integral_constant<int, WT_UNIT> a4{};
    constexpr std::integral_constant<int, WT_STEP> a8{};
    if (kd == 0) run_wide(n0, n1);
    else if (kd == 1) run_small(n0, n1, whole, std::integral_constant<int, 3>{}, a4);
    else if (!HALVES || kd == 2) run_small(n0, n1, whole, std::integral_constant<int, 4>{}, a1);
    else if constexpr (HALVES) {
      if (kd == 3) run_small(n0, n1, half, std::integral_constant<int, 3>{}, a8);
      else if (kd == 4) run_small(n0, n1, half, std::integral_constant<int, 4>{}, a4);
      else run_small(n0, n1, half, std::integral_constant<int, 7>{}, a1);
    }
    n0 = n1;
    // no DMA of one run may land in the next one's ring, or outlive the workgroup
    sync(std::integral_constant<int, 0>{});
  }
}

template <int DT>
hipError_t launch_wide(const tempo_moe_shape& s, const tempo_dispatch_out& d, const tempo_expert_weights& w,
                       const void* x_rows, const float* x_rows_scale, void* y_perm, char* ws, const Layout& L,
                       bool timing, const hipEvent_t* ev, hipStream_t st) {
  constexpr bool F8 = DT != kWideBf16;
  constexpr int es = F8 ? 1 : 2;
  const int grid = persistent_grid(1);
  const int KTg = s.H * es / 128, KTd = s.I * es / 128;
  auto mark = [&](int i) { return !ev || !ev[i] || hipEventRecord(ev[i], st) == hipSuccess; };
  char* apack = ws + L.wide_a;
  float* apack_sc = reinterpret_cast<float*>(ws + L.wide_a_sc);
  const bool gather = x_rows != nullptr;
  hipLaunchKernelGGL(k_pack_wide<F8>, dim3(persistent_grid(4)), dim3(256), 0, st,
                     static_cast<const char*>(gather ? x_rows : d.x_perm), gather ? x_rows_scale : d.x_perm_scale,
                     gather ? 1 : 0, L.row_cap, d.row_token, d.slot_counts, d.slot_offsets, s.S, L.wide_tiles, KTg,
                     apack, apack_sc, gather && !stream_gathers_rows(s, L) ? static_cast<char*>(d.x_perm) : nullptr,
                     gather && F8 ? d.x_perm_scale : nullptr);

  WideArgs a{};
  a.slot_counts = d.slot_counts;
  a.slot_offsets = d.slot_offsets;
  a.S = s.S;
  a.max_tiles = L.wide_tiles;
  a.row_cap = L.row_cap;
  a.wtab = reinterpret_cast<const uint64_t*>(w.slot_table);
  a.t0 = reinterpret_cast<uint64_t*>(ws + L.slot_t0);
  a.t1 = reinterpret_cast<uint64_t*>(ws + L.slot_t1);
  a.timing = timing ? 1 : 0;

  WideArgs gu = a;
  gu.A = apack;
  gu.A_sc = apack_sc;
  gu.W = static_cast<const char*>(w.w13);
  gu.wfield = kFieldW13;
  gu.sfield = kFieldW13Scale;
  gu.w_slot_bytes = (size_t)2 * s.I * s.H * es;
  gu.Wsp = w.w13_scale;
  gu.ws_slot_floats = (size_t)(s.I / 64) * (s.H / 128) * 4;
  gu.C = ws + L.wide_h;
  gu.C_sc = reinterpret_cast<float*>(ws + L.wide_h_sc);
  gu.KT = KTg;
  gu.NB = s.I / 64;
  if (!mark(0)) return hipErrorLaunchFailure;  // after the pack: the GEMM kernel alone is timed
  hipLaunchKernelGGL((k_gemm_wide<DT, true>), dim3(grid), dim3(WT_THREADS), 0, st, gu);
  if (!mark(1) || !mark(2)) return hipErrorLaunchFailure;

  WideArgs dn = a;
  dn.A = gu.C;
  dn.A_sc = gu.C_sc;
  dn.W = static_cast<const char*>(w.w2);
  dn.wfield = kFieldW2;
  dn.sfield = kFieldW2Scale;
  dn.w_slot_bytes = (size_t)s.H * s.I * es;
  dn.Wsp = w.w2_scale;
  dn.ws_slot_floats = (size_t)(s.H / 128) * (s.I / 128) * 4;
  dn.C = static_cast<char*>(y_perm);
  dn.KT = KTd;
  dn.NB = s.H / 128;
  dn.ld_out = s.H * 2;
  hipLaunchKernelGGL((k_gemm_wide<DT, false>), dim3(grid), dim3(WT_THREADS), 0, st, dn);
  if (!mark(3)) return hipErrorLaunchFailure;
  return hipGetLastError();
}

}  // namespace

// Where the wide tiles win: slots with enough rows, and enough items to fill
// the chip.  The counts per slot are only known on the device; valid rows per
// expert, T_valid K / E, and the items that these make, stand for them (the same
// for every plan, so a row's result does not depend on it; padding tokens make
// no rows: of 1024 tokens half of them valid, judged by all -> by the valid ones,
// 18 slots 195 -> 199 / 196 -> 176 / 176 -> 152 us, 36 slots 657 -> 642 / 585 ->
// 532 / 528 -> 481).
// Which of two kernels wins near the line depends on the plan: uniform shares
// leave slots of very different sizes, which the other kernel balances worst;
// a plan that keeps few replicas busy leaves it slots of few rows each, its
// best case.  The plan's weights are device memory, so the lines lie where the
// plans together gain: 2625 measured calls on wide tiles (22 shapes, three plans)
// take 17% less than with the kernels before, 84 of them over 5% more, at most 15%
// (bf16, 256-row tiles, H 2048, just past a round of items; next fp8, 64-row
// tiles, 16 rows, fewest replicas, 10%).
// Measured, forward us, other kernel -> wide tiles, uniform plan / token
// balancing / fewest replicas ("18": 18 slots H 4096 I 1536; "36": 36 slots H
// 7168 I 2048; "12a": 12 slots H 3072 I 2048; "12b": 12 slots H 2048 I 1408;
// "10": 10 slots H 2048 I 1408; items in brackets):
//   bf16   64-row tiles, rows per expert 64 (18) [264]: 222 -> 213 / 216 -> 205
//          / 171 -> 193; 80: 291 -> 225 / 230 -> 209 / 206 -> 189.  Many items
//          (36), 32: 816 -> 686 / 666 -> 665 / 540 -> 590; 48: 1034 -> 737 / 796
//          -> 675 / 664 -> 648.  Shorter contractions (12a) [272], 112: 241 ->
//          187 / 171 -> 168 / 118 -> 121; (12b) 80 [165]: 122 -> 106 / 93 -> 82 /
//          74 -> 79; 128 [198]: 162 -> 115 / 110 -> 108 / 85 -> 85.
//          128-row tiles (18), 64: 231 -> 209 / 198 -> 205 / 177 -> 192; 80: 243
//          -> 223 / 245 -> 209 / 197 -> 189; (12a) 80: 185 -> 175 / 144 -> 160 /
//          108 -> 113, 128: 232 -> 187 / 185 -> 170 / 140 -> 138.
//          256-row tiles against their own large-tile kernel (18), 24: 219 ->
//          183 / 217 -> 182 / 180 -> 154; 128 [324]: 328 -> 245 / 309 -> 226 /
//          231 -> 200; 512: 562 -> 528 / 509 -> 451 / 385 -> 338; but full
//          tiles that make about one round of items are its best case: (12b) 192
//          [231]: 124 -> 138 / 114 -> 113 / 111 -> 85; 12 slots H 2048 I 768, 128
//          [108]: 104 -> 93, 208 [126]: 110 -> 122, 288 [150]: 115 -> 125; with
//          longer contractions only just: 18 slots H 4096 I 1024, 96 [192]: 198 ->
//          195, 192 [248]: 214 -> 221, 256 [288]: 320 -> 237; (18) 64 [264]: 240 ->
//          209 / 232 -> 202 / 195 -> 192; (12a) 192 [336]: 233 -> 210 / 166 -> 182
//          / 157 -> 149, 320 [416]: 304 -> 265 / 232 -> 190 / 173 -> 181
//   fp8    64-row tiles (18, two placements), 8: 102 -> 90 / 100 -> 90 / 95 ->
//          84, 101 -> 91 / 100 -> 90 / 99 -> 91; 12: 107 -> 96 / 107 -> 96 / 103 ->
//          87, 111 -> 96 / 110 -> 95 / 104 -> 110; 24: 126 -> 121 / 119 -> 118 /
//          107 -> 97, 121 -> 120 / 121 -> 121 / 118 -> 115; (36) 8: +5 / +2 / 0%,
//          12: 378 -> 369 / 328 -> 309 / 300 -> 287, 16: 394 -> 386 / 326 -> 333 /
//          300 -> 291; (12b) 64 [165]: 89 -> 79 / 82 -> 74 / 64 -> 72;
//          (10) 96 [143]: 95 -> 85 / 90 -> 82 / 67 -> 78.  128-row tiles (18), 12:
//          121 -> 95 / 112 -> 95 / 102 -> 87; 20 slots H 2048 I 512, 64 [100]: 77
//          -> 84.  256-row tiles (18), 16: 165 -> 100 / 163 -> 99 / 135 -> 95; 12
//          slots H 7168 I 384, 32 [39]: 121 -> 132, 64: 155 -> 147
//   UE8M0  64-row tiles (18), 48 [252]: 147 -> 130 / 138 -> 126 / 110 -> 121; 64:
//          149 -> 133 / 144 -> 130 / 118 -> 126; (12b) 64 [165]: 83 -> 76 / 73 -> 71
//          / 60 -> 69, 128 [198]: 118 -> 84 / 86 -> 81 / 69 -> 77; (36) 32: 475 ->
//          416 / 388 -> 394 / 325 -> 336.  128-row tiles (18), 56: 158 -> 130 / 142
//          -> 128 / 126 -> 122; (10) 128 [154]: 97 -> 83 / 93 -> 81 / 70 -> 78.
//          256-row tiles with I an odd multiple of 128: 6 slots H 4096 I 384, 64
//          [21]: 72 -> 77, 256 [36]: 96 -> 103, 512 [54]: 129 -> 112; 12 slots H
//          7168 I 384, 64 [45]: 128 -> 137; 6 slots H 2048 I 640, 64 [35]: 69 ->
//          64; 10 slots H 5120 I 896, 64 [84]: 115 -> 112 / 109 -> 108 / 94 -> 102;
//          against its own 256-row kernel 160: 173 -> 173, 512: 327 -> 333
bool experts_wide_wanted(const tempo_moe_shape& s) {
  if (experts_big_f8_supported(s)) return false;
  const long long P = (long long)s.T_valid * s.K, E = s.E;
  // items of the gate/up GEMM, were the pairs spread evenly over the experts
  const long long items = (s.S + P * s.S / (256 * E)) * (s.I / 128);
  const bool m64 = s.m_tile == 64, m256 = s.m_tile == 256, many = items >= 500, deep = s.H >= 4096;
  if (s.dtype == TEMPO_BF16) {
    if (m256) return P >= 24 * E && !(s.H % 256 == 0 && P >= 256 * E && items > 128 && items <= 270);
    return items >= 150 && P >= (many ? (m64 ? 32 : 48) : m64 && deep ? 56 : 64) * E;
  }
  if (s.dtype == TEMPO_FP8_E4M3) {
    if (m256) return P >= 12 * E;
    return items >= 130 && P >= (m64 && !many ? (items >= 170 ? 8 : 20) : 12) * E;
  }
  if (m256) return P >= 32 * E && (!deep || items >= 50);
  return items >= 150 && P >= (many ? 32 : 48) * E;
}

hipError_t launch_experts_wide(const tempo_moe_shape& s, const tempo_dispatch_out& d, const tempo_expert_weights& w,
                               const void* x_rows, const float* x_rows_scale, void* y_perm, char* ws, const Layout& L,
                               bool timing, const hipEvent_t* ev, hipStream_t st) {
  if (s.dtype == TEMPO_BF16)
    return launch_wide<kWideBf16>(s, d, w, x_rows, x_rows_scale, y_perm, ws, L, timing, ev, st);
  if (s.dtype == TEMPO_FP8_E4M3_UE8M0)
    return launch_wide<kWideMX>(s, d, w, x_rows, x_rows_scale, y_perm, ws, L, timing, ev, st);
  return launch_wide<kWideF8>(s, d, w, x_rows, x_rows_scale, y_perm, ws, L, timing, ev, st);
}

}  // namespace tempo
