// K1 -- KV-append scatter (arxiv 2502.11517, Section 3, "Efficiency"; Figure 2c):
// every active thread's new K/V row goes to the next free slot of the shared pool, so rows
// of concurrently decoding threads end up in neighbouring slots.  A pure copy in 16-byte pieces.
// With the rotary option the K pieces are turned by the row's position id on the way (V never).
//
// Where the rows go travels as RUNS: consecutive rows of the call that belong to one request take
// consecutive slots, so a whole prompt is one run and a batch's token step one run per request.  (A list of
// destination rows had to be written, pinned and copied to the device ahead of the launch, in two launches for
// 8192 rows: 44 us per layer for a prompt of 8192 rows, 8 heads x 128 bf16, of which the kernels took 22; with
// runs 14.)  A call with more runs than fit the kernel arguments still sends the list.
// What bounds it: memory, for a prompt: a thread moves four pieces of K and four of V, all requested before the first is
// stored.  Smaller calls are a chain of latencies on a chip that is not full, and a thread moves one piece of each.
#pragma once
#include "k_rope.hpp"
#include "mfma_util.hpp"

namespace pasta {

constexpr int kAppendInline = 32;  // most rows of an append that a decode launch can take along, or that patches lists
constexpr int kAppendRuns = 64;    // runs that travel in the kernel arguments
constexpr int kPatchMax = 64;      // most entries of the device-resident lists one launch brings up to date

struct AppendRun { int32_t row0, req, slot0, pos0; };  // rows row0 ..: slots slot0 .. of request req, position ids pos0 ..

struct AppendParams {
  const u32x4* k_new;   // [n_rows][Hkv][D] as 16-byte pieces
  const u32x4* v_new;
  void* k;              // layer base
  void* v;
  const int32_t* page_table;
  const int32_t* dst_rows;  // physical row per appended row (device), or null: the runs say it
  const int32_t* pos_rows;  // position id per appended row (device; with dst_rows and the rotation)
  Layout lay;
  int n_rows, Hkv, n_runs;
  int pph_log2;         // log2 of the 16-byte pieces per head row
  int elem_shift;       // log2(elem_bytes)
  const double* rope_tab;   // theta^(-2f/D) / (2 pi), f < D/2 (device): the rotating form
  AppendRun runs[kAppendRuns];
  // The append also extends the device-resident visibility lists (the lists that decode steps in
  // maintained mode read): entries of the range arena and of the range index that this call's rows
  // changed or created, computed by the host from its mirror.
  DevRange* arena;
  int32_t* cidx;
  int n_rpatch, n_cpatch;
  int32_t rp_idx[kPatchMax];
  DevRange rp_val[kPatchMax];
  int32_t cp_idx[kPatchMax];
  int32_t cp_val[kPatchMax];
};

static_assert(sizeof(AppendParams) <= 4096, "kernel arguments are limited to 4 KB");

// ROPE: a thread takes both pieces of a pair of partner pieces (D / 2 elements apart), so that a plane's
// angle is worked out once.
constexpr int append_units(bool rope) { return rope ? 2 : 4; }  // pieces (pairs of pieces) per thread, beyond ...
// ... this many pieces (pairs) per call; up to it one per thread.  Launches in a graph, 8 heads x 128, many / one per thread (us):
//   bf16          8 rows 2.6 / 1.9, 512 3.0 / 2.2, 4096 (2^19 pieces) 6.4 / 5.9;  fp32 2048 (2^19) 6.4 / 5.7, 4096 9.0 / 9.5
//   bf16, rotated 8 rows 4.2 / 2.8, 512 4.6 / 3.3, 4096 8.2 / 7.8;  fp32, rotated 8 rows 3.1 / 2.4, 4096 (2^19 pairs) 10.0 / 9.8
constexpr long long kAppendThin = 1ll << 19;

template <bool ROPE, int UNR>
__global__ __launch_bounds__(256) void k_append(AppendParams p) {
  constexpr int PART = ROPE ? 2 : 1;
  const uint32_t t = blockIdx.x * 256u + threadIdx.x;
  if (t < (uint32_t)p.n_rpatch) p.arena[p.rp_idx[t]] = p.rp_val[t];
  else if (t < (uint32_t)(p.n_rpatch + p.n_cpatch)) p.cidx[p.cp_idx[t - p.n_rpatch]] = p.cp_val[t - p.n_rpatch];
  const int unit_log2 = p.pph_log2 - (ROPE ? 1 : 0);  // units per head row
  const uint32_t total = ((uint32_t)p.n_rows * (uint32_t)p.Hkv) << unit_log2;
  const uint32_t part = 1u << unit_log2;              // a unit's second piece
  auto unit = [&](int n) { return (blockIdx.x * UNR + n) * 256u + threadIdx.x; };
  u32x4 kv[UNR][2][PART];
#pragma unroll
  for (int n = 0; n < UNR; ++n) {
    const uint32_t u = min(unit(n), total - 1);  // past the end: the last unit again, stored below by its owner only
    const uint32_t src = ((u >> unit_log2) << p.pph_log2) + (u & (part - 1));
#pragma unroll
    for (int x = 0; x < PART; ++x) {
      kv[n][0][x] = p.k_new[src + x * part];
      kv[n][1][x] = p.v_new[src + x * part];
    }
  }
  int row[UNR];
  AppendRun run[UNR];  // the run that holds the row
#pragma unroll
  for (int n = 0; n < UNR; ++n) {
    row[n] = (int)((min(unit(n), total - 1) >> unit_log2) / (uint32_t)p.Hkv);
    run[n] = p.runs[0];
  }
  if constexpr (UNR > 1) {  // (the chip is full: other waves cover the reads)
    for (int k = 1; k < p.n_runs; ++k) {  // (the same run for every lane: scalar loads)
      const AppendRun rk = p.runs[k];
#pragma unroll
      for (int n = 0; n < UNR; ++n)
        if (row[n] >= rk.row0) run[n] = rk;
    }
  } else if (p.n_runs > 1) {
    // Lane k has run k.  A wave's rows go up with its lanes, so it looks at the runs of its first to its last row only,
    // one as a rule.  (All runs in turn, one dependent read each: 32 rotated rows of as many threads, 8 heads x 128
    // bf16, an append after the other, 7.6 us; this way 4.6, which is the host's call.  The rows of sixteen requests,
    // append and decode step: 64 -> 60.5 us.)
    const int lane = threadIdx.x & 63;
    const AppendRun mine = p.runs[min(lane, p.n_runs - 1)];
    const int begins = lane < p.n_runs ? mine.row0 : INT32_MAX;
    auto run_of = [&](int k) { return AppendRun{__builtin_amdgcn_readlane(mine.row0, k), __builtin_amdgcn_readlane(mine.req, k),
                                                __builtin_amdgcn_readlane(mine.slot0, k), __builtin_amdgcn_readlane(mine.pos0, k)}; };
    const int first = __popcll(__ballot(begins <= __builtin_amdgcn_readlane(row[0], 0))) - 1;  // (run 0 begins at row 0)
    const int last = __popcll(__ballot(begins <= __builtin_amdgcn_readlane(row[0], 63))) - 1;
    run[0] = run_of(first);
    for (int k = first + 1; k <= last; ++k) {
      const AppendRun rk = run_of(k);
      if (row[0] >= rk.row0) run[0] = rk;
    }
  }
#pragma unroll
  for (int n = 0; n < UNR; ++n) {
    const uint32_t u = unit(n);
    if (u >= total) continue;
    const uint32_t piece = u & (part - 1);
    const int g = (int)((u >> unit_log2) % (uint32_t)p.Hkv);
    int phys, pos = 0;
    if (p.dst_rows) {
      phys = p.dst_rows[row[n]];
      if (ROPE) pos = p.pos_rows[row[n]];
    } else {
      phys = phys_row(p.lay, p.page_table, run[n].req, run[n].slot0 + (row[n] - run[n].row0));
      pos = run[n].pos0 + (row[n] - run[n].row0);
    }
    const long long dst = (elem_off(p.lay, phys, g) << p.elem_shift) + (long long)piece * 16;
    if constexpr (ROPE) {
      const u32x4 a4 = kv[n][0][0], b4 = kv[n][0][1];
      const uint32_t a[4] = {a4[0], a4[1], a4[2], a4[3]}, b[4] = {b4[0], b4[1], b4[2], b4[3]};
      uint32_t lo[4], hi[4];
      if (p.elem_shift == 2) {
        rope_piece_f32(a, b, lo, false, (int)piece * 4, pos, p.rope_tab);
        rope_piece_f32(b, a, hi, true, (int)piece * 4, pos, p.rope_tab);
      } else {
        rope_piece_bf16<true>(a, b, lo, false, (int)piece * 8, pos, p.rope_tab);
        rope_piece_bf16<true>(b, a, hi, true, (int)piece * 8, pos, p.rope_tab);
      }
      kv[n][0][0] = u32x4{lo[0], lo[1], lo[2], lo[3]};
      kv[n][0][1] = u32x4{hi[0], hi[1], hi[2], hi[3]};
    }
#pragma unroll
    for (int x = 0; x < PART; ++x) {
      *reinterpret_cast<u32x4*>(reinterpret_cast<char*>(p.k) + dst + (long long)x * part * 16) = kv[n][0][x];
      *reinterpret_cast<u32x4*>(reinterpret_cast<char*>(p.v) + dst + (long long)x * part * 16) = kv[n][1][x];
    }
  }
}

// Carries a piece of a decode step's plan, or of an append's list of rows, to the device inside its own kernel
// arguments: how calls under stream capture send what is too large for the arguments of the launch that reads it,
// since a captured launch must not depend on what later calls leave in host memory.
constexpr int kRelayWords = 960;
struct RelayParams {
  int32_t* dst;
  int n_words;
  int32_t words[kRelayWords];
};
static_assert(sizeof(RelayParams) <= 4096, "kernel arguments are limited to 4 KB");

__global__ __launch_bounds__(256) void k_meta_relay(RelayParams p) {
  typedef const char __attribute__((address_space(4))) * kernarg_ptr;
  kernarg_ptr ka = (kernarg_ptr)__builtin_amdgcn_kernarg_segment_ptr();
  const int32_t __attribute__((address_space(4)))* src =
      (const int32_t __attribute__((address_space(4)))*)(ka + __builtin_offsetof(RelayParams, words));
  for (int i = threadIdx.x; i < p.n_words; i += 256) p.dst[i] = src[i];
}

}  // namespace pasta
