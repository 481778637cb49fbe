// Stage 2, bf16: the stream-K grouped GEMM of gemm_stream.h with bf16
// operands and fp32 accumulation; h is rounded to bf16 (round to nearest
// even) after SwiGLU, y_perm to bf16 after the down projection.
#include <cmath>

#include "gemm_stream.h"

namespace tempo {
namespace {

using namespace gemm;

template <int BM>
hipError_t launch_bm(const tempo_moe_shape& s, const tempo_dispatch_out& d, const tempo_expert_weights& w,
                     const void* x_rows, void* y_perm, char* ws, const Layout& L, bool timing, const hipEvent_t* ev,
                     hipStream_t st) {
  const int grid = persistent_grid(1);
  GemmArgs a{};
  a.as_ld = L.row_cap;
  a.part = reinterpret_cast<float*>(ws + L.part);
  a.fix = reinterpret_cast<int32_t*>(ws + L.fix);
  a.slot_counts = d.slot_counts;
  a.slot_offsets = d.slot_offsets;
  a.S = s.S;
  a.max_tiles = L.row_cap / BM;
  a.t0 = reinterpret_cast<uint64_t*>(ws + L.slot_t0);
  a.t1 = reinterpret_cast<uint64_t*>(ws + L.slot_t1);
  a.timing = timing ? 1 : 0;
  char* h = ws + L.h;

  // gate/up + SwiGLU -> h [row_cap, I] bf16
  GemmArgs gu = a;
  gu.A = static_cast<const char*>(x_rows ? x_rows : d.x_perm);
  gu.row_src = x_rows ? d.row_token : nullptr;
  gu.W = static_cast<const char*>(w.w13);
  gu.wtab = reinterpret_cast<const uint64_t*>(w.slot_table);
  gu.wfield = kFieldW13;
  gu.sfield = kFieldW13Scale;
  gu.w_slot_bytes = (size_t)2 * s.I * s.H * 2;
  gu.C = h;
  gu.Kd = s.H;
  gu.Nout = s.I;
  gu.cmax = GATEUP_CHUNKS;
  gu.whole = stream_whole_items(s) ? 1 : 0;
  auto mark = [&](int i) { return !ev || !ev[i] || hipEventRecord(ev[i], st) == hipSuccess; };
  if (!mark(0)) return hipErrorLaunchFailure;
  hipLaunchKernelGGL((k_gemm<false, BM, true>), dim3(grid), dim3(GEMM_THREADS), 0, st, gu);
  if (!mark(1)) return hipErrorLaunchFailure;
  // (without split items there is nothing to complete)
  if (!gu.whole)
    hipLaunchKernelGGL((k_fixup<false, BM, true>), dim3(grid * (BM / 8)), dim3(256), 0, st, gu, grid);
  if (!mark(2)) return hipErrorLaunchFailure;

  // down -> y_perm [row_cap, H] bf16
  GemmArgs dn = a;
  dn.A = h;
  dn.W = static_cast<const char*>(w.w2);
  dn.wtab = reinterpret_cast<const uint64_t*>(w.slot_table);
  dn.wfield = kFieldW2;
  dn.sfield = kFieldW2Scale;
  dn.w_slot_bytes = (size_t)s.H * s.I * 2;
  dn.C = y_perm;
  dn.Kd = s.I;
  dn.Nout = s.H;
  dn.cmax = DOWN_CHUNKS;
  hipLaunchKernelGGL((k_gemm<false, BM, false>), dim3(grid), dim3(GEMM_THREADS), 0, st, dn);
  if (!mark(3)) return hipErrorLaunchFailure;
  if (dn.cmax > 1)
    hipLaunchKernelGGL((k_fixup<false, BM, false>), dim3(grid * (BM / 8)), dim3(256), 0, st, dn, grid);
  return hipGetLastError();
}

}  // namespace

bool experts_gather_rows(const tempo_moe_shape& s, const Layout& L) {
  // the wide- and large-tile kernels pack the token rows themselves
  return L.wide_tiles || stream_gathers_rows(s, L);
}

bool stream_gathers_rows(const tempo_moe_shape& s, const Layout& L) {
  if (experts_big_supported(s) || experts_big_f8_supported(s)) return true;
  // upper bound of the M-tiles one workgroup range of the gate/up GEMM spans
  const int grid = persistent_grid(1);
  const int NB = s.I / 64;
  const long long groups = geo_groups(NB, grid), wpx = grid / groups;
  // ranges balance weighted chunks; a range holds at most 1/wpx of the total
  // weight, which is largest when every tile is full, and its tiles weigh at
  // least W_BASE + 1 each
  const long long max_tiles = L.row_cap / s.m_tile;
  const long long wfull = W_BASE + s.m_tile / 32, wmin = W_BASE + 1;
  const long long tiles = (max_tiles * wfull + wpx * wmin - 1) / (wpx * wmin) + 2;
  return tiles <= nrowt_of(s.m_tile);
}

// No partial tiles and no fixup launch, against a coarser balance of the
// ranges: what whole items lose grows with the time of an item, what they save
// does not.  64-row tiles wait for their weights, an item's time goes with its
// steps; larger ones for the MFMAs too, its time goes with H.  64-row tiles
// with long contractions gain where the items are about as many as the workgroups
// or more, and lose where a fraction of the workgroups holds them all.  The
// slots that will be active are only known on the device; the expected number,
// were the valid pairs spread evenly over the experts, stands for them (the
// same for every plan).  Measured, forward us split -> whole, by expected
// items over 256 workgroups (x) and rows per expert:
//   64-row tiles   bf16 H 4096 I 1536 18 slots 16 tokens (x 1.07) 77 -> 68, 32
//          (1.46) 89 -> 83, 64 (1.66) 106 -> 110, 256 (1.69) 155 -> 152, 512 203 ->
//          198; H 7168 I 2048 36 slots (2.9 .. 4.5) -2.5 .. +2.5%; H 3072 I 1024
//          (48 steps) 1 row (0.40) 48 -> 52, 8 (0.62) 63 -> 56; H 2048 I 512 (0.62)
//          55 -> 51; H 5120 I 2048 (80 steps) 8 (0.62) 68 -> 74, 32: 93 -> 86; H
//          7168 I 2048 2 slots (0.25) 64 -> 75; H 1152 (18 steps) 48 -> 43; fp8 H
//          3072 (24 steps) (0.4 .. 0.6) -6 .. +2 us
//   128-row tiles  bf16 H 1152 68 -> 60, fp8 63 -> 55; H 2048 bf16 10 slots 32 rows
//          81 -> 72, 48: 83 -> 84; fp8 12 slots 48 rows 79 -> 71; H 3072 10 slots
//          48 rows 96 -> 87, 128: 113 -> 128; H 4096 18 slots -12 .. +11 us, 6
//          slots +6 .. +17
//   256-row tiles  H 1152 -6 .. 0 us; H 2048 fp8 10 slots 8 rows 70 -> 63; H 4096
//          fp8 18 slots 0 .. +14 us
bool stream_whole_items(const tempo_moe_shape& s) {
  if (s.m_tile > 64) return s.H <= 2048;
  const int KT = s.H / (s.dtype == TEMPO_BF16 ? 64 : 128);
  const double active = s.S * (1.0 - std::pow(1.0 - 1.0 / s.E, (double)s.T_valid * s.K));
  return KT <= 24 || active * (s.I / 64) >= (KT <= 48 ? 0.5 : 0.7) * 256;
}

hipError_t launch_experts_bf16(const tempo_moe_shape& s, const tempo_dispatch_out& d, const tempo_expert_weights& w,
                               const void* x_rows, void* y_perm, char* ws, const Layout& L, bool timing, const hipEvent_t* ev,
                               hipStream_t st) {
  if (L.wide_tiles) return launch_experts_wide(s, d, w, x_rows, nullptr, y_perm, ws, L, timing, ev, st);
  if (s.m_tile == 128) return launch_bm<128>(s, d, w, x_rows, y_perm, ws, L, timing, ev, st);
  if (s.m_tile == 64) return launch_bm<64>(s, d, w, x_rows, y_perm, ws, L, timing, ev, st);
  if (s.m_tile == 256) {
    if (experts_big_supported(s)) return launch_experts_big(s, d, w, x_rows, y_perm, ws, L, timing, ev, st);
    return launch_bm<256>(s, d, w, x_rows, y_perm, ws, L, timing, ev, st);
  }
  if (s.m_tile == 192) return launch_bm<192>(s, d, w, x_rows, y_perm, ws, L, timing, ev, st);
  return hipErrorInvalidValue;
}

}  // namespace tempo
