// The partials launch for element types and head widths other than bf16 x 128 (fp32 pools of either
// width, bf16 with 64-wide heads): the same work items, split and partial rows as k_attn, other kernel.
//
// Operands go STRAIGHT from memory into the registers in which the matrix instructions want them; no K
// or V ever passes through LDS.  A wave owns whole blocks of tokens and works in 16-row tiles (a private
// item has at most 8 live rows, so 32-row tiles would double its matrix work -- and fp32 matrix
// instructions are slow enough for that to show):
//   * S^T[16 tok x 16 rows] = K Q^T.  A operand: lane (i = lane % 16, q = lane / 16) holds pieces
//     4 kk + q (16 bytes each) of token i's row, so one load instruction fetches 64 contiguous bytes of
//     16 rows, and the same lanes of Q's rows are the B operand;
//   * the accumulator then holds, per lane (row i, quarter q), tokens 4 q + r of each 16-token tile, which
//     is the B operand of the next product for that token order;
//   * O^T += V^T P^T.  The lanes of quarter q load exactly those tokens' V rows, whole rows per 16 lanes.
//     fp32: a loaded element IS an A operand (one per token and M-tile).  bf16: the eight tokens of a lane
//     are interleaved in registers, one byte-permute per operand register, and a weight is three bf16 operands.  Element c of a lane's piece
//     belongs to M-tile c, so M-tile c is the head dims { (D / 16) m + c } -- a free renaming, undone when
//     the rows leave through LDS.
// The rows' addresses are worked out once per item (one thread per token) and left in LDS as 32-bit codes,
// whatever the list looks like -- contiguous, strided, listed, paged, rows of a deferred append.
//
// What bounds it: like k_attn, the latency of a step's one pass over its rows.  It replaces the vector-ALU
// walker (k_private), whose cost was a chain of lane shuffles per row, which read a shared prefix once per
// stream and could not take a deferred append along.  Append and decode step, walker -> this kernel (us):
//   fp32, 4 query heads on 1 x 64, 256 + 2 x 16 tokens           28.7 ->  9.1
//   fp32, 32 heads on 8 x 128, 1024 tokens + 4 x 32 .. 256       45.8 -> 11.4
//   bf16, 32 heads on 8 x 64, 4096 tokens + 8 x 64 .. 512        27.9 -> 10.9
// One block per wave in registers: with 32 stacked queries fp32 rows need 244 of the 256 registers without a second
// one, and chunks are short enough here that most waves have only one.  (The rotated forms over 128 dims, which work
// out angles between the loads, do not fit: 9 vector registers spilled in bf16, 17 in fp32.)
#pragma once
#include "k_plan.hpp"
#include "k_rope.hpp"

namespace pasta {

constexpr int kDirWin = 1024;    // tokens whose address codes are in LDS at a time
constexpr uint32_t kPendBit = 0x80000000u;  // address code: (byte offset / 16) | kPendBit for a deferred row

// One lane's share of a block of kTok tokens.
template <typename T, int D> struct DirBlock;
template <int D> struct DirBlock<uint16_t, D> {
  static constexpr int kTok = 32, kNT = 2, kNP = D / 32, kNV = 8, kVP = 1;  // kNP pieces of a K row per lane
  typedef std::conditional_t<D == 128, u32x4, u32x2> vec;
  u32x4 k[kNT][kNP];
  vec v[kNV][kVP];
};
template <int D> struct DirBlock<float, D> {
  static constexpr int kTok = D == 64 ? 32 : 16, kNT = kTok / 16, kNP = D / 16, kNV = kTok / 4, kVP = D / 64;
  typedef f32x4 vec;
  u32x4 k[kNT][kNP];
  vec v[kNV][kVP];
};

// LDS of a work-group of NW waves, row tiles up to RT: address codes and ranges on the way in, the waves'
// O on the way out ([wave][group of 64 lanes x 16 bytes], groups one piece apart from a multiple of the
// bank period, so that a row can be read back across groups without conflicts).
template <int D, int RT, int NW> struct DirLds {
  static constexpr int kGroups = RT * 4 * (D / 64);
  f32x4 o[NW][kGroups * 65];
  float mw[NW][16 * RT], lw[NW][16 * RT];
  uint32_t off[kDirWin];
  DevRange ranges[kGatherMax];
};
// ... and of k_one: the rows that are turned once per work-group (a stream's query rows; behind them its newest row where that
// is a deferred one).
constexpr int kMostHeads = 8;  // query heads per kv head
constexpr int kMostDeferred = (int)(sizeof(DecodeParams::pend_pos) / sizeof(int32_t));
template <typename T, int D, int NW, bool ROPE> struct OneLds : DirLds<D, 1, NW> {};
template <typename T, int D, int NW> struct OneLds<T, D, NW, true> : DirLds<D, 1, NW> {
  static constexpr int kPieces = D * (int)sizeof(T) / 16;
  u32x4 turned[kMostHeads + 1][kPieces + 1];
};

// Turns the planes of a row whose pieces 4 kk + q are spread over the quarters' lanes: piece kk and piece
// kk + NP / 2 of a lane are each other's partners.  The same arithmetic as rope_row_piece.
template <typename T, int NP>
__device__ __forceinline__ void rope_lane(u32x4 (&x)[NP], int q, int pos, const double* tab) {
#pragma unroll
  for (int kk = 0; kk < NP / 2; ++kk) {
    const uint32_t a[4] = {x[kk][0], x[kk][1], x[kk][2], x[kk][3]};
    const uint32_t b[4] = {x[kk + NP / 2][0], x[kk + NP / 2][1], x[kk + NP / 2][2], x[kk + NP / 2][3]};
    uint32_t lo[4], hi[4];
    if constexpr (sizeof(T) == 4) {
      const int f0 = (4 * kk + q) * 4;
      rope_piece_f32(a, b, lo, false, f0, pos, tab);
      rope_piece_f32(b, a, hi, true, f0, pos, tab);
    } else {
      const int f0 = (4 * kk + q) * 8;
      rope_piece_bf16<true>(a, b, lo, false, f0, pos, tab);
      rope_piece_bf16<true>(b, a, hi, true, f0, pos, tab);
    }
    x[kk] = u32x4{lo[0], lo[1], lo[2], lo[3]};
    x[kk + NP / 2] = u32x4{hi[0], hi[1], hi[2], hi[3]};
  }
}

// What an item's rows are made of.
struct DirItem {
  int n_tok, R, g;
  long long part_row0;
  const_words req_streams;     // shared-prefix item: the request's streams (null: stack block s is stream s)
  int row0;                    // ... its first stacked row
  int q_stream;                // private item: its stream
  int q_pos;                   // (WHOLE) its query's position id,
  int own_row, own_pos;        // ... the row of its newest token in a deferred append that is to be turned (-1: none), that one's id,
  bool more_deferred;          // ... and whether the token before that may be such a row, too
};

// One item, once code_of(j) -- the address code of token j -- can be asked for.  GATHER: the rows are the G
// heads of one stream; otherwise rows row0 .. of the request's stack.
// WHOLE: the item is all that its stream sees, and what is written is the result instead of a partial row.
template <typename T, int D, int RT, int NW, bool GATHER, bool ROPE, bool WHOLE, class Lds, class CodeOf>
__device__ __forceinline__ void direct_rows(const DecodeParams& p, Lds& lds, const_words meta, const DirItem& it, CodeOf code_of) {
  typedef DirBlock<T, D> Blk;
  constexpr int kTok = Blk::kTok, kNT = Blk::kNT, kNP = Blk::kNP, kMT = D / 16;
  constexpr int kPieceRow = D * (int)sizeof(T) / 16;
  // fp32 lists read whole: a wave has several blocks and their sums meet without a merge, so every block is summed from 0, rescaled and
  // added with one rounding, and the waves' sums are added in pairs.  (Relative error against 64 bits, 8 streams over 112 / 160 / 288 /
  // 416 tokens of 128 dims, 1e-7: split form 1.59 / 1.63 / 1.71 / 1.75, in one chain 1.62 / 1.72 / 1.90 / 2.01, this way 1.59 / 1.63 / 1.69 / 1.71;
  // 64 dims, 288 / 416: 1.61 / 1.66, 1.65 / 1.69, 1.60 / 1.62.  Append and decode step of 8 streams of 128 dims, in one chain -> this way:
  // 110 tokens 8.1 -> 8.2 us, 280 12.2 -> 12.2; rotated 110 9.3 -> 9.4, 400 17.1 -> 16.9.)
  constexpr bool kFine = WHOLE && sizeof(T) == 4;
  constexpr bool kExact = sizeof(T) == 4 || D == 64 || !WHOLE;  // (otherwise k_attn's arithmetic, see weigh)
  const int tid = threadIdx.x, lane = tid & 63, i = lane & 15, q = lane >> 4;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int G = p.Hq / p.Hkv;
  const int n_tok = it.n_tok, R = it.R, g = it.g;

  // ---- Q: the B operands, straight into registers (rows past R repeat row 0: computed, never stored)
  u32x4 qf[RT][kNP];
  int qpos[RT];
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) {
    const int rr = rt * 16 + i < R ? rt * 16 + i : 0;
    int s = it.q_stream, hq = rr;
    if constexpr (!GATHER) {
      const int ra = it.row0 + rr;
      s = it.req_streams ? it.req_streams[ra / G] : ra / G;
      hq = ra % G;
    }
    const char* src = reinterpret_cast<const char*>(p.q) + (long long)(s * p.Hq + g * G + hq) * (D * sizeof(T)) + q * 16;
#pragma unroll
    for (int kk = 0; kk < kNP; ++kk) qf[rt][kk] = *reinterpret_cast<const u32x4*>(src + kk * 64);
    qpos[rt] = 0;
    if constexpr (ROPE) {
      if (!WHOLE && p.rope_q) qpos[rt] = record<DevStream>(meta + p.off_streams, s).pos;
    }
  }

  // A whole stream's rows are turned once per work-group, a plane per lane, and go to the waves through LDS: the last wave
  // turns the stream's newest row, the others the query rows.  Requested here, turned behind the requests for the rows.
  // A launch this short runs its code once, so what the turning costs is code to fetch as much as arithmetic: with every
  // lane turning the planes of its operand registers in place, by a table of angles and, for deferred rows, by angles of
  // its own, 300 + 3 x 20 .. 60 tokens, 16 layers of append and decode step, took 172.8 us; this way 138.4.
  // (A second copy of the block's code, with two blocks requested together, was measured on that form alone: 189.)
  // More deferred rows than that -- the newest slots of their request, so the list's last -- are spread over the waves and go
  // to the place of the waves' O, free until they meet.  (One at a time, by the wave whose block holds them, they took 0.2 us
  // each: 16 tokens of one stream over 64, 8 kv heads, append and decode step, fp32 x 64 9.9 us, bf16 x 64 8.3; this way 7.3
  // and 6.1.  32 rows and one query: 14.2 and 12.1, 7.6 and 6.6.  Steps of one such row per list measure the same.)
  constexpr int kUnits = ROPE && WHOLE ? (kMostHeads + NW - 2) / (NW - 1) : 1;
  constexpr int kTurnedRow = kPieceRow + 1;
  static_assert(!(ROPE && WHOLE) || sizeof(lds.o) >= sizeof(u32x4) * kMostDeferred * kTurnedRow, "more deferred rows than the waves' O hold");
  u32x4* const more_rows = reinterpret_cast<u32x4*>(&lds.o[0][0]);  // deferred row k >= 1, counted from the list's end: row k - 1
  const int plane = lane & (D / 2 - 1);
  Plane<T> unit[kUnits];
  double per_pos = 0.0;
  int n_def = 0;  // deferred rows of the list that are to be turned, where they are more than the newest
  if constexpr (ROPE && WHOLE) {
    per_pos = p.rope_tab[plane];
    if (w == NW - 1) {
      if (it.own_row >= 0) unit[0] = plane_load<T>(reinterpret_cast<const char*>(p.k_pend) + (long long)(it.own_row * p.Hkv + g) * (D * sizeof(T)), plane, D / 2);
    } else if (p.rope_q) {
#pragma unroll
      for (int n = 0; n < kUnits; ++n)
        if (w + n * (NW - 1) < R)
          unit[n] = plane_load<T>(reinterpret_cast<const char*>(p.q) + (long long)(it.q_stream * p.Hq + g * G + w + n * (NW - 1)) * (D * sizeof(T)), plane, D / 2);
    }
  }

  const char* kb = reinterpret_cast<const char*>(p.k);
  const char* vb = reinterpret_cast<const char*>(p.v);
  const char* kpend = reinterpret_cast<const char*>(p.k_pend);
  const char* vpend = reinterpret_cast<const char*>(p.v_pend);
  auto at = [&](uint32_t code, const char* pool, const char* pend) -> const char* {
    return ((int)code < 0 ? pend : pool) + ((unsigned long long)(code & ~kPendBit) << 4);
  };
  auto load_k = [&](Blk& x, int b) {
#pragma unroll
    for (int t = 0; t < kNT; ++t) {
      const char* src = at(lds.off[b * kTok + 16 * t + i], kb, kpend) + q * 16;
#pragma unroll
      for (int kk = 0; kk < kNP; ++kk) x.k[t][kk] = *reinterpret_cast<const u32x4*>(src + kk * 64);
    }
    __builtin_amdgcn_sched_barrier(0);  // (addresses of later loads are not worked out ahead: they would cost the registers the rows need)
  };
  auto load_v = [&](Blk& x, int b) {
#pragma unroll
    for (int t = 0; t < kNT; ++t) {
      const u32x4 c = *reinterpret_cast<const u32x4*>(&lds.off[b * kTok + 16 * t + 4 * q]);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const char* src = at(c[r], vb, vpend) + i * (int)sizeof(typename Blk::vec);
#pragma unroll
        for (int h = 0; h < Blk::kVP; ++h) x.v[4 * t + r][h] = *reinterpret_cast<const typename Blk::vec*>(src + h * 256);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  };

  f32x4 O[RT][kMT];
  // Row rt * 16 + i; l_run covers this lane's quarter of the tokens.  The maximum starts at the lowest finite value: a
  // block whose scores are all -inf in log2 units then has weights of 0 (from -inf on, -inf - -inf would make them NaN).
  float m_run[RT], l_run[RT], corr[RT];
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) {
    m_run[rt] = -__FLT_MAX__;
    l_run[rt] = 0.f;
#pragma unroll
    for (int c = 0; c < kMT; ++c) O[rt][c] = f32x4{0.f, 0.f, 0.f, 0.f};
  }

  // S^T of block x, online softmax in log2 units (the scale is applied inside the exponent); what is left in
  // `pr` are the weights, fp32
  auto scores = [&](Blk& x, int b, int n_here, f32x4 (&pr)[kNT][RT]) {
    if constexpr (ROPE) {  // deferred rows that are to be turned on their way into the pool
      if (p.pend_rope) {
#pragma unroll
        for (int t = 0; t < kNT; ++t) {
          const uint32_t code = lds.off[b * kTok + 16 * t + i];
          if (__builtin_amdgcn_ballot_w64((int)code < 0)) {
            if constexpr (WHOLE) {  // they stand in LDS by now
              if ((int)code < 0) {
                const int k = max(n_here - 1 - (b * kTok + 16 * t + i), 0);
                const u32x4* src = (k == 0 ? lds.turned[kMostHeads] : more_rows + (k - 1) * kTurnedRow) + q;
#pragma unroll
                for (int kk = 0; kk < kNP; ++kk) x.k[t][kk] = src[4 * kk];
              }
            } else {
              const int row = (int)((code & ~kPendBit) / (uint32_t)(p.Hkv * kPieceRow));
              if ((int)code < 0) rope_lane<T, kNP>(x.k[t], q, pend_pos_of(p)[row], p.rope_tab);
            }
          }
        }
      }
    }
#pragma unroll
    for (int t = 0; t < kNT; ++t)
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) pr[t][rt] = f32x4{0.f, 0.f, 0.f, 0.f};
    if constexpr (sizeof(T) == 2) {
#pragma unroll
      for (int kk = 0; kk < kNP; ++kk)
#pragma unroll
        for (int t = 0; t < kNT; ++t)
#pragma unroll
          for (int rt = 0; rt < RT; ++rt)
            pr[t][rt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, x.k[t][kk]), __builtin_bit_cast(bf16x8, qf[rt][kk]), pr[t][rt], 0, 0, 0);
    } else {
      // eight sums of D / 8 products each, added up in pairs: one chain over all of D rounds as often as it has products.  (Relative
      // error of the results against 64 bits, 300 .. 3000 tokens: D = 128 4.0e-7 in one chain, 1.9e-7 this way, 2.1e-7 by the
      // vector-ALU walker; D = 64 3.3e-7, 1.8e-7, 1.9e-7.  Append and decode step, 1024 + 4 x 32 .. 256 tokens: 11.2 and 11.4 us.)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        f32x4 part[2][kNT][RT];
#pragma unroll
        for (int kk = 0; kk < kNP; ++kk)
#pragma unroll
          for (int t = 0; t < kNT; ++t)
#pragma unroll
            for (int rt = 0; rt < RT; ++rt)
              part[kk & 1][t][rt] = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(x.k[t][kk][e]), __uint_as_float(qf[rt][kk][e]),
                                                                         kk < 2 ? f32x4{0.f, 0.f, 0.f, 0.f} : part[kk & 1][t][rt], 0, 0, 0);
#pragma unroll
        for (int t = 0; t < kNT; ++t)
#pragma unroll
          for (int rt = 0; rt < RT; ++rt) pr[t][rt] += part[0][t][rt] + part[1][t][rt];
        if (RT > 1) __builtin_amdgcn_sched_barrier(0);  // (more of them at once would cost registers)
      }
    }
    if ((b + 1) * kTok > n_here) {  // tokens past the item's end are hidden (a block holds at least one that exists)
      const int left = n_here - (b * kTok + 4 * q);
#pragma unroll
      for (int t = 0; t < kNT; ++t)
#pragma unroll
        for (int rt = 0; rt < RT; ++rt)
#pragma unroll
          for (int r = 0; r < 4; ++r) pr[t][rt][r] = 16 * t + r < left ? pr[t][rt][r] : -INFINITY;
    }
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
      float mx = -INFINITY;
#pragma unroll
      for (int t = 0; t < kNT; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r) mx = fmaxf(mx, pr[t][rt][r]);
      mx = fmaxf(mx, __shfl_xor(mx, 16, kWave));
      mx = fmaxf(mx, __shfl_xor(mx, 32, kWave));
      const float mn = fmaxf(m_run[rt], mx * p.scale_log2e);
      const float by = fast_exp2(m_run[rt] - mn);
      if (kFine) corr[rt] = by;
      m_run[rt] = mn;
      float ps = 0.f;
#pragma unroll
      for (int t = 0; t < kNT; ++t) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          pr[t][rt][r] = fast_exp2(fmaf(pr[t][rt][r], p.scale_log2e, -mn));
          if (!kFine) ps += pr[t][rt][r];
        }
        if (kFine) ps += (pr[t][rt][0] + pr[t][rt][1]) + (pr[t][rt][2] + pr[t][rt][3]);
      }
      l_run[rt] = l_run[rt] * by + ps;
      if (!kFine && !__all(by == 1.f)) {  // (kFine: by weigh)
#pragma unroll
        for (int c = 0; c < kMT; ++c) O[rt][c] *= by;
      }
    }
  };

  // O^T += V^T P^T.  The weights of a bf16 block go in as bf16 terms, cut off one behind the other (each product is exact in
  // the fp32 accumulator): three hold all their 24 bits, where the vector-ALU walker had fp32 weights.  Where k_attn would
  // round them to bf16 it takes two: one alone left the results 0.4 % further off than k_attn's, since a weight's rounding
  // depends on how far the maximum reaches (here 32 tokens of one wave).  Lower terms are 2^-126 at least: a term of 0
  // would make NaN of an infinite element of V.
  // (Per layer, 8 streams over 4096 tokens of 64 dims: one term 10.6 us, three 10.9; k_one over 128 dims, 300 + 3 x 20 .. 60
  // tokens, rotated: one 10.7, two 10.8.)
  auto weigh = [&](const Blk& x, const f32x4 (&pr)[kNT][RT]) {
    if constexpr (sizeof(T) == 2) {
      constexpr int kTerms = kExact ? 3 : 2;
      typedef __attribute__((ext_vector_type(2))) uint16_t u16x2;
      u32x4 pb[kTerms][RT];
#pragma unroll
      for (int rt = 0; rt < RT; ++rt)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          float u = pr[e >> 1][rt][2 * (e & 1)], v = pr[e >> 1][rt][2 * (e & 1) + 1];
#pragma unroll
          for (int n = 0; n < kTerms; ++n) {
            const uint32_t iu = __float_as_uint(u), iv = __float_as_uint(v);
            uint32_t term = __builtin_amdgcn_perm(iv, iu, 0x07060302u);
            if (n > 0) term = __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(u16x2, term), u16x2{0x0080, 0x0080}));
            pb[n][rt][e] = term;
            u -= __uint_as_float(iu & 0xffff0000u);
            v -= __uint_as_float(iv & 0xffff0000u);
          }
        }
#pragma unroll
      for (int c = 0; c < kMT; ++c) {
        u32x4 a;
#pragma unroll
        for (int e = 0; e < 4; ++e)  // element c of tokens 2 e and 2 e + 1
          a[e] = __builtin_amdgcn_perm(x.v[2 * e + 1][0][c / 2], x.v[2 * e][0][c / 2], (c & 1) ? 0x07060302u : 0x05040100u);
#pragma unroll
        for (int n = 0; n < kTerms; ++n)
#pragma unroll
          for (int rt = 0; rt < RT; ++rt) O[rt][c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, pb[n][rt]), O[rt][c], 0, 0, 0);
      }
    } else {
#pragma unroll
      for (int c = 0; c < kMT; ++c)
#pragma unroll
        for (int t = 0; t < kNT; ++t)
#pragma unroll
          for (int rt = 0; rt < RT; ++rt) {
            f32x4 sum = kNT > 1 || kFine ? f32x4{0.f, 0.f, 0.f, 0.f} : O[rt][c];  // (16 tokens at a time, for the same reason)
#pragma unroll
            for (int r = 0; r < 4; ++r)
              sum = __builtin_amdgcn_mfma_f32_16x16x4f32(x.v[4 * t + r][c / 4][c % 4], pr[t][rt][r], sum, 0, 0, 0);
            if constexpr (kFine) {
#pragma unroll
              for (int r = 0; r < 4; ++r) O[rt][c][r] = fmaf(O[rt][c][r], t == 0 ? corr[rt] : 1.f, sum[r]);
            } else {
              O[rt][c] = kNT > 1 ? O[rt][c] + sum : sum;
            }
          }
    }
  };

  // ---- the item's tokens, in windows of kDirWin
  bool q_turned = false;
  for (int w0 = 0; w0 < n_tok; w0 += kDirWin) {
    const int n_here = min(kDirWin, n_tok - w0);
    const int nb = (n_here + kTok - 1) / kTok;
    if (w0) lds_barrier();  // everybody is done with the last window's codes
    for (int j = tid; j < nb * kTok; j += NW * 64) lds.off[j] = code_of(w0 + min(j, n_here - 1));  // past the end: the last token again
    lds_barrier();
    auto turn_q = [&]() {
      if constexpr (ROPE && WHOLE) {  // (by all waves, with a block or without, once)
        float c, sn;
        rope_cos_sin_by<sizeof(T) == 2>(per_pos, w == NW - 1 ? it.own_pos : it.q_pos, c, sn);
        if (lane < D / 2) {
          if (w == NW - 1) {
            if (it.own_row >= 0) plane_store<T>(lds.turned[kMostHeads], plane, D / 2, unit[0], c, sn);
          } else if (p.rope_q) {
#pragma unroll
            for (int n = 0; n < kUnits; ++n)
              if (w + n * (NW - 1) < R) plane_store<T>(lds.turned[w + n * (NW - 1)], plane, D / 2, unit[n], c, sn);
          }
        }
        if (__builtin_expect(it.more_deferred, 0)) {
          n_def = __builtin_popcountll(__builtin_amdgcn_ballot_w64(lane < min(n_here, kMostDeferred) && (int)lds.off[max(n_here - 1 - lane, 0)] < 0));
          for (int k = 1 + w; k < n_def; k += NW) {
            const uint32_t at = (uint32_t)__builtin_amdgcn_readfirstlane((int)lds.off[n_here - 1 - k]) & ~kPendBit;
            const Plane<T> x = plane_load<T>(kpend + ((unsigned long long)at << 4), plane, D / 2);
            rope_cos_sin_by<sizeof(T) == 2>(per_pos, pend_pos_of(p)[at / (uint32_t)(p.Hkv * kPieceRow)], c, sn);
            plane_store<T>(more_rows + (k - 1) * kTurnedRow, plane, D / 2, x, c, sn);
          }
        }
        lds_barrier();
        if (p.rope_q) {
#pragma unroll
          for (int kk = 0; kk < kNP; ++kk) qf[0][kk] = lds.turned[i < R ? i : 0][4 * kk + q];
        }
      } else if constexpr (ROPE) {
        if (p.rope_q && !q_turned) {
#pragma unroll
          for (int rt = 0; rt < RT; ++rt) rope_lane<T, kNP>(qf[rt], q, qpos[rt], p.rope_tab);
        }
        q_turned = true;
      }
    };
    constexpr bool kAllTurn = ROPE && WHOLE;  // (one copy of turn_q's code for waves with a block and without)
    if (!kAllTurn && w >= nb) continue;
    const int last = nb - 1 - (nb - 1 - w) % NW;  // this wave's last block, where it has one
    Blk A;
    f32x4 pr[kNT][RT];
    if (!kAllTurn || w < nb) {
      load_k(A, w);
      load_v(A, w);
    }
    turn_q();
    if (kAllTurn && w >= nb) continue;
    for (int b = w; b < last; b += NW) {  // the next block is requested half by half, as this one's places fall free
      scores(A, b, n_here, pr);
      load_k(A, b + NW);
      weigh(A, pr);
      load_v(A, b + NW);
    }
    scores(A, last, n_here, pr);
    if (kExact && (last + 1) * kTok > n_here) {  // places past the end hold the last token again: 0 x its infinities would be NaN
      const int left = n_here - (last * kTok + 4 * q);
#pragma unroll
      for (int t = 0; t < kNT; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
          for (int h = 0; h < Blk::kVP; ++h)
            if (16 * t + r >= left) A.v[4 * t + r][h] = typename Blk::vec(0);
    }
    weigh(A, pr);
  }

  if (ROPE && WHOLE && __builtin_expect(it.more_deferred, 0)) lds_barrier();  // every wave is done with the rows that stand in the place of O
  // ---- the waves meet once.  Group (rt, r, cg) of a lane: head dims of M-tiles 4 cg .. 4 cg + 3 at m = 4 q + r.
  const int n_act = min(NW, (min(kDirWin, n_tok) + kTok - 1) / kTok);  // waves that had a block
  if (w < n_act) {
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
      if (rt * 16 + i < R) {
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
          for (int cg = 0; cg < D / 64; ++cg)
            lds.o[w][((rt * 4 + r) * (D / 64) + cg) * 65 + lane] = f32x4{O[rt][4 * cg][r], O[rt][4 * cg + 1][r], O[rt][4 * cg + 2][r], O[rt][4 * cg + 3][r]};
      }
      float l = l_run[rt] + __shfl_xor(l_run[rt], 16, kWave);
      l += __shfl_xor(l, 32, kWave);
      if (q == 0) { lds.mw[w][rt * 16 + i] = m_run[rt]; lds.lw[w][rt * 16 + i] = l; }
    }
  }
  __syncthreads();
  constexpr int kPR = D / 4, kRows = NW * 64 / kPR;  // pieces of 4 floats per row, rows per pass
  const int pc = tid % kPR;
  // which group and quarter piece pc of a row sits in
  int cg, qq, r;
  if constexpr (sizeof(T) == 2 && D == 128) { qq = pc >> 3; r = (pc >> 1) & 3; cg = pc & 1; }
  else { cg = pc >> 4; qq = (pc >> 2) & 3; r = pc & 3; }
#pragma unroll
  for (int pass = 0; pass < (16 * RT + kRows - 1) / kRows; ++pass) {
    if (pass * kRows >= R) break;
    const int rr = pass * kRows + tid / kPR;
    if (kRows > 16 * RT && rr >= 16 * RT) break;
    const int slot = (((rr >> 4) * 4 + r) * (D / 64) + cg) * 65 + 16 * qq + (rr & 15);
    float mk[NW], ma = -INFINITY;
#pragma unroll
    for (int k = 0; k < NW; ++k) {
      mk[k] = k < n_act ? lds.mw[k][rr] : -INFINITY;
      ma = fmaxf(ma, mk[k]);
    }
    f32x4 acc = f32x4{0.f, 0.f, 0.f, 0.f};
    float l = 0.f;
    if constexpr (kFine) {
      f32x4 two[NW / 2];
      float two_l[NW / 2];
#pragma unroll
      for (int k = 0; k < NW; ++k) {
        if (k % 2 == 0) { two[k / 2] = f32x4{0.f, 0.f, 0.f, 0.f}; two_l[k / 2] = 0.f; }
        if (k < n_act) {
          const float sc = fast_exp2(mk[k] - ma);
          two[k / 2] += lds.o[k][slot] * sc;
          two_l[k / 2] = fmaf(lds.lw[k][rr], sc, two_l[k / 2]);
        }
      }
#pragma unroll
      for (int n = NW / 4; n > 0; n /= 2)
#pragma unroll
        for (int k = 0; k < n; ++k) { two[k] += two[k + n]; two_l[k] += two_l[k + n]; }
      acc = two[0];
      l = two_l[0];
    } else {
#pragma unroll
      for (int k = 0; k < NW; ++k) {
        if (k < n_act) {
          const float sc = fast_exp2(mk[k] - ma);
          acc += lds.o[k][slot] * sc;
          l = fmaf(lds.lw[k][rr], sc, l);
        }
      }
    }
    if (rr >= R) continue;
    if constexpr (WHOLE) {
      const long long row = (long long)it.q_stream * p.Hq + g * G + rr;
      if (l == 0.f) acc = f32x4{0.f, 0.f, 0.f, 0.f};  // (nothing weighed anything: 0 / 0, as behind the merge)
      const float o[4] = {acc[0] / l, acc[1] / l, acc[2] / l, acc[3] / l};
      if constexpr (sizeof(T) == 4) reinterpret_cast<f32x4*>(p.out)[row * kPR + pc] = f32x4{o[0], o[1], o[2], o[3]};
      else reinterpret_cast<u32x2*>(p.out)[row * kPR + pc] = u32x2{pack_bf16x2(o[0], o[1]), pack_bf16x2(o[2], o[3])};
      if (p.lse && pc == 0) p.lse[row] = (ma + __log2f(l)) * kLn2;
    } else {
      *reinterpret_cast<f32x4*>(p.part_acc + (it.part_row0 + rr) * D + 4 * pc) = acc;
      if (pc == 0) p.part_ml[it.part_row0 + rr] = make_float2(l > 0.f ? ma : -INFINITY, l);
    }
  }
}

// The copy of a deferred append's rows into the pool (no work-group of the launch reads those pool rows: lists
// that name them are served from k_pend / v_pend), spread thin over the work-groups' first 16 threads; fewer
// work-groups than that take more each.  ROPE: K rows are turned on the way.
template <typename T, int D, bool ROPE>
__device__ __forceinline__ void direct_copy_pending(const DecodeParams& p, int wg, int n_wgs) {
  constexpr int kPieceRow = D * (int)sizeof(T) / 16;
  const int row_pieces = p.Hkv * kPieceRow, total = p.pend_n * row_pieces;
  const bool thin = 2 * total <= n_wgs * 16;
  const int step = thin ? 2 * total : n_wgs * (int)blockDim.x;
  for (int t = thin ? (threadIdx.x < 16 ? wg * 16 + (int)threadIdx.x : 2 * total) : wg * (int)blockDim.x + (int)threadIdx.x;
       t < 2 * total; t += step) {
    const bool is_v = t >= total;
    const int u = is_v ? t - total : t;
    const int row = u / row_pieces, g = (u % row_pieces) / kPieceRow, piece = u % kPieceRow;
    const uint4* src = reinterpret_cast<const uint4*>(is_v ? p.v_pend : p.k_pend);
    uint4 val;
    if (ROPE && p.pend_rope && !is_v)
      val = rope_row_piece(src + (u - piece), piece, kPieceRow, sizeof(T) == 4, pend_pos_of(p)[row], p.rope_tab);
    else
      val = src[u];
    char* dst = reinterpret_cast<char*>(const_cast<void*>(is_v ? p.v : p.k));
    *reinterpret_cast<uint4*>(dst + elem_off(p.lay, pend_dst_of(p)[row], g) * (long long)sizeof(T) + piece * 16) = val;
  }
}

// Address code of logical slot `slot` of request `req`, kv head g (deferred rows: their place in k_new / v_new).
template <typename T, int D>
__device__ __forceinline__ uint32_t direct_code(const DecodeParams& p, int req, int slot, int g, int pend0, int pend_src0, int& phys) {
  phys = phys_row(p.lay, p.page_table, req, slot);
  if (slot >= pend0) return kPendBit | (uint32_t)(((pend_src0 + (slot - pend0)) * p.Hkv + g) * (D * (int)sizeof(T) / 16));
  return (uint32_t)((unsigned long long)(elem_off(p.lay, phys, g) * (long long)sizeof(T)) >> 4);
}

template <typename T, int D, bool ROPE>
__global__ __launch_bounds__(kAttnThreads, 2) void k_direct(DecodeParams p) {
  __shared__ DirLds<D, 2, 4> lds;
  const const_words meta = meta_words(p);
  const int tid = threadIdx.x;
  if (p.pend_n > 0) direct_copy_pending<T, D, ROPE>(p, (int)blockIdx.x, (int)gridDim.x);
  const int n_prefix_wgs = (int)gridDim.x - p.n_mfma_items * p.Hkv;
  const int G = p.Hq / p.Hkv;
  DirItem it;
  it.req_streams = nullptr;
  it.row0 = 0;
  it.q_stream = 0;
  if ((int)blockIdx.x < n_prefix_wgs) {  // a chunk of a request's common prefix, up to 32 stacked rows (work-group order as in k_attn)
    const int wi = blockIdx.x;
    DevReq rq;
    if (p.single_req) {
      rq = p.req0;
    } else {
      rq = record<DevReq>(meta + p.off_reqs, request_of(p, meta, wi));
      it.req_streams = meta + p.off_req_streams + rq.stream0;
    }
    const int R_all = rq.n_streams * G, n_rg = (R_all + 31) >> 5;
    const int wl = wi - rq.wg_begin, t = wl / p.Hkv;
    const int c = __builtin_amdgcn_readfirstlane(t / n_rg);
    it.row0 = __builtin_amdgcn_readfirstlane((t % n_rg) * 32);
    it.g = __builtin_amdgcn_readfirstlane(wl % p.Hkv);
    it.R = __builtin_amdgcn_readfirstlane(min(32, R_all - it.row0));
    const int slot0 = c * rq.chunk_tokens;
    it.n_tok = __builtin_amdgcn_readfirstlane(min(rq.chunk_tokens, rq.pc - slot0));
    it.part_row0 = rq.part_base + (long long)(it.g * rq.n_chunks + c) * R_all + it.row0;
    const bool report = p.dbg_rows && it.g == 0 && it.row0 == 0;
    auto code_of = [&](int j) -> uint32_t {
      int phys;
      const uint32_t code = direct_code<T, D>(p, rq.req, slot0 + j, it.g, rq.pend0, rq.pend_src0, phys);
      if (report)
        for (int k = 0; k < rq.n_streams; ++k)
          p.dbg_rows[record<DevStream>(meta + p.off_streams, it.req_streams ? it.req_streams[k] : k).gather_base + slot0 + j] = phys;
      return code;
    };
    if (it.R > 16) direct_rows<T, D, 2, 4, false, ROPE, false>(p, lds, meta, it, code_of);
    else direct_rows<T, D, 1, 4, false, ROPE, false>(p, lds, meta, it, code_of);
    return;
  }
  // ---- a piece of one stream's private list
  const int wi = (int)blockIdx.x - n_prefix_wgs;
  const int item = __builtin_amdgcn_readfirstlane(wi / p.Hkv);
  it.g = __builtin_amdgcn_readfirstlane(wi % p.Hkv);
  const bool kept = p.codes != nullptr;  // a plan kept on the device: its tokens' rows are written out
  const DevItem di = record<DevItem>(kept ? words_at(p.items) : meta + p.off_items, item);
  const int32_t* codes = p.codes + (long long)item * p.priv_chunk;
  const int nr = !kept && di.n_ranges > 1 ? di.n_ranges : 0;
  int req = 0, pend0 = INT32_MAX, pend_src0 = 0;
  if (kept) {
  } else if (p.single_req) {
    req = p.req0.req; pend0 = p.req0.pend0; pend_src0 = p.req0.pend_src0;
  } else {
    const DevStream st = record<DevStream>(meta + p.off_streams, di.stream);
    req = st.req; pend0 = st.pend0; pend_src0 = st.pend_src0;
  }
  if (nr > 0) {  // the ranges the piece overlaps -> LDS
    for (int k = tid; k < nr; k += kAttnThreads) lds.ranges[k] = record<DevRange>(meta + p.off_ranges, di.range_first + k);
    __syncthreads();
  }
  it.n_tok = __builtin_amdgcn_readfirstlane(di.tok_count);
  it.R = G;
  it.q_stream = di.stream;
  it.part_row0 = p.priv_part_base + (long long)(item * p.Hkv + it.g) * G;
  const bool report = p.dbg_rows && it.g == 0;
  auto code_of = [&](int j) -> uint32_t {
    int slot;
    if (kept) {
      const int row = codes[j];
      if (report) p.dbg_rows[di.gather_pos + j] = phys_of_code(p, row);
      if (row < 0) return kPendBit | (uint32_t)(((-1 - row) * p.Hkv + it.g) * (D * (int)sizeof(T) / 16));
      return (uint32_t)((unsigned long long)(elem_off(p.lay, row, it.g) * (long long)sizeof(T)) >> 4);
    }
    if (nr > 0) {  // the last range with cum <= tok
      const int tok = di.tok_begin + j;
      int lo = 0, hi = nr - 1;
      while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (lds.ranges[mid].cum <= tok) lo = mid; else hi = mid - 1;
      }
      slot = lds.ranges[lo].start + (tok - lds.ranges[lo].cum) * lds.ranges[lo].stride;
    } else {
      slot = di.slot0 + j * di.stride;
    }
    int phys;
    const uint32_t code = direct_code<T, D>(p, req, slot, it.g, pend0, pend_src0, phys);
    if (report) p.dbg_rows[di.gather_pos + j] = phys;
    return code;
  };
  direct_rows<T, D, 1, 4, true, ROPE, false>(p, lds, meta, it, code_of);
}

// A small step in ONE launch: a work-group takes everything that one stream sees of one kv head and writes the
// result, so that neither partial rows nor a merge launch -- nor, with rotary embedding, the launch that turns Q and
// the deferred rows ahead of k_attn -- stand on the step's path.  All dtypes and widths.
// What bounds it: the rate at which one CU takes in the rows (eight waves with a block each in flight), which is why
// it is for short lists only, and every stream reads the shared prefix by itself (from its XCD's L2: work-group mod
// Hkv is the kv head).  The copy of a deferred append's rows has work-groups of its own behind the others.
// Append and decode step, split form -> this one (us): bf16, 8 kv heads x 128, 128 + 3 x 20 .. 60 tokens 10.0 -> 6.4, with
// rotary embedding, 300 + 3 x 20 .. 60 tokens 13.8 -> 8.6; 8 streams over 300 tokens 11.7 -> 8.0; bf16 x 64, 3 streams over 300 tokens 8.9 -> 6.4.
constexpr int kOneWaves = 8;
template <typename T, int D, bool ROPE>
__global__ __launch_bounds__(kOneWaves * 64) void k_one(DecodeParams p) {
  __shared__ OneLds<T, D, kOneWaves, ROPE> lds;
  static_assert(2 * sizeof(lds) <= 160 * 1024, "two work-groups per CU: the copy's stand beside the streams'");
  const int tid = threadIdx.x;
  const int n_rows_wgs = p.n_mfma_items * p.Hkv;  // (one item per stream)
  if ((int)blockIdx.x >= n_rows_wgs) {
    direct_copy_pending<T, D, ROPE>(p, (int)blockIdx.x - n_rows_wgs, (int)gridDim.x - n_rows_wgs);
    return;
  }
  // The plan always rides in the kernel arguments here (small_step): its records are read with scalar loads
  // (8 kv heads x 128, 128 .. 300 + 1 .. 8 x 20 .. 60 tokens: 0.3 us of 6.4 .. 8.4).
  typedef const_words words;
  typedef const char __attribute__((address_space(4))) * kernarg_ptr;
  const words meta = (words)((kernarg_ptr)__builtin_amdgcn_kernarg_segment_ptr() + __builtin_offsetof(DecodeParams, inline_meta));
  const int item = __builtin_amdgcn_readfirstlane((int)blockIdx.x / p.Hkv);
  const words di = meta + p.off_items + item * (int)(sizeof(DevItem) / 4);
  auto item_word = [&](size_t byte) { return di[byte / 4]; };
  const int stream = item_word(offsetof(DevItem, stream)), gather_pos = item_word(offsetof(DevItem, gather_pos));
  const words ds = meta + p.off_streams + stream * (int)(sizeof(DevStream) / 4);
  const int req = ds[offsetof(DevStream, req) / 4], pend0 = ds[offsetof(DevStream, pend0) / 4], pend_src0 = ds[offsetof(DevStream, pend_src0) / 4];
  DirItem it;
  it.req_streams = nullptr;
  it.row0 = 0;
  it.part_row0 = 0;
  it.g = __builtin_amdgcn_readfirstlane((int)blockIdx.x % p.Hkv);
  it.n_tok = item_word(offsetof(DevItem, tok_count));
  it.R = p.Hq / p.Hkv;
  it.q_stream = stream;
  it.q_pos = ds[offsetof(DevStream, pos) / 4];
  const int nr = item_word(offsetof(DevItem, n_ranges));
  const words ranges = meta + p.off_ranges + item_word(offsetof(DevItem, range_first)) * (int)(sizeof(DevRange) / 4);
  it.own_row = -1;
  it.own_pos = 0;
  it.more_deferred = false;
  if (ROPE && p.pend_rope) {
    const words newest = ranges + 4 * (nr - 1);
    const int left = it.n_tok - 1 - newest[3], slot = newest[0] + left * newest[2];
    if (slot >= pend0) {
      it.own_row = pend_src0 + (slot - pend0);
      it.own_pos = pend_pos_of(p)[it.own_row];
      it.more_deferred = it.n_tok > 1 && slot - (left > 0 ? newest[2] : 1) >= pend0;
    }
  }
  for (int k = tid; k < nr; k += kOneWaves * 64) lds.ranges[k] = DevRange{ranges[4 * k], ranges[4 * k + 1], ranges[4 * k + 2], ranges[4 * k + 3]};
  __syncthreads();
  const bool report = p.dbg_rows && it.g == 0;
  auto code_of = [&](int j) -> uint32_t {  // the last range with cum <= j
    int lo = 0, hi = nr - 1;
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (lds.ranges[mid].cum <= j) lo = mid; else hi = mid - 1;
    }
    int phys;
    const int slot = lds.ranges[lo].start + (j - lds.ranges[lo].cum) * lds.ranges[lo].stride;
    const uint32_t code = direct_code<T, D>(p, req, slot, it.g, pend0, pend_src0, phys);
    if (report) p.dbg_rows[gather_pos + j] = phys;
    return code;
  };
  direct_rows<T, D, 1, kOneWaves, true, ROPE, true>(p, lds, nullptr, it, code_of);
}

}  // namespace pasta
