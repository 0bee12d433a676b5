// Rotary position embedding by GIVEN position ids.  In PASTA a token decoded after a promise
// gets an estimated position id, because the asynchronous block before it has only a predicted
// length (arxiv 2502.11517, Section 4, "Training a PASTA-SFT model"; appendix "Positional
// Embedding"); the ids are the caller's, the rotation is the base model's.  It is applied to K
// on its way into the pool (K1) and, in a decode step, to Q and to the K rows of a deferred append: in a small launch
// ahead of k_attn (k_rope_prep), as they are loaded in k_direct and k_one.  Half-split planes over the whole head dim: plane
// f = (x[f], x[f + D/2]) turns by position * theta^(-2f/D).
//
// Precision: position * frequency reaches tens of thousands of radians, so the product is
// taken in fp64 from a table of theta^(-2f/D) / (2 pi) (fp64, D/2 entries, in the workspace)
// and reduced to a fraction of a revolution before it becomes fp32; the rotation itself is
// fp32, rounded once to the pool dtype.
#pragma once
#include "pasta_dev.hpp"

namespace pasta {

// FAST: the hardware's v_cos_f32 / v_sin_f32 (argument in revolutions), good to about 1e-6
// absolute -- ample under a bf16 rounding.  Otherwise the library's sincospi (about 1 ulp).
template <bool FAST>
__device__ __forceinline__ void rope_cos_sin_by(double per_pos, int pos, float& c, float& s) {  // per_pos: revolutions per position
  const double rev = (double)pos * per_pos;
  const float fr = (float)(rev - __builtin_floor(rev));
  if constexpr (FAST) {
    c = __builtin_amdgcn_cosf(fr);
    s = __builtin_amdgcn_sinf(fr);
  } else {
    sincospif(2.f * fr, &s, &c);
  }
}
template <bool FAST>
__device__ __forceinline__ void rope_cos_sin(const double* tab, int f, int pos, float& c, float& s) {
  rope_cos_sin_by<FAST>(tab[f], pos, c, s);
}

// One 16-byte piece of a bf16 head row (8 elements, first plane index f0), `par` the piece D/2
// elements away; `upper` says that `own` holds the second components of its planes.
template <bool FAST>
__device__ __forceinline__ void rope_piece_bf16(const uint32_t (&own)[4], const uint32_t (&par)[4],
                                                uint32_t (&out)[4], bool upper, int f0, int pos,
                                                const double* tab) {
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    float r[2];
#pragma unroll
    for (int hf = 0; hf < 2; ++hf) {
      const float x = hf ? bf16_hi(own[w]) : bf16_lo(own[w]);
      const float y = hf ? bf16_hi(par[w]) : bf16_lo(par[w]);
      float c, s;
      rope_cos_sin<FAST>(tab, f0 + 2 * w + hf, pos, c, s);
      r[hf] = upper ? x * c + y * s : x * c - y * s;
    }
    out[w] = (uint32_t)f32_to_bf16_rne(r[0]) | ((uint32_t)f32_to_bf16_rne(r[1]) << 16);
  }
}

// The same for an fp32 row: 4 elements per piece.
__device__ __forceinline__ void rope_piece_f32(const uint32_t (&own)[4], const uint32_t (&par)[4],
                                               uint32_t (&out)[4], bool upper, int f0, int pos,
                                               const double* tab) {
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    const float x = __uint_as_float(own[w]), y = __uint_as_float(par[w]);
    float c, s;
    rope_cos_sin<false>(tab, f0 + w, pos, c, s);
    out[w] = __float_as_uint(upper ? x * c + y * s : x * c - y * s);
  }
}

// A piece of either dtype, addressed inside a [..][D] array of 16-byte pieces: `src` points at
// piece 0 of the head row, `piece` < pieces_per_head.
__device__ __forceinline__ uint4 rope_row_piece(const uint4* src, int piece, int pieces_per_head, bool is_f32,
                                                int pos, const double* tab) {
  const int half = pieces_per_head >> 1;
  const bool upper = piece >= half;
  const uint4 o = src[piece], q = src[upper ? piece - half : piece + half];
  const uint32_t own[4] = {o.x, o.y, o.z, o.w}, par[4] = {q.x, q.y, q.z, q.w};
  uint32_t out[4];
  const int f0 = (upper ? piece - half : piece) * (is_f32 ? 4 : 8);
  if (is_f32) rope_piece_f32(own, par, out, upper, f0, pos, tab);
  else rope_piece_bf16<true>(own, par, out, upper, f0, pos, tab);  // the same arithmetic wherever bf16 keys are turned
  return make_uint4(out[0], out[1], out[2], out[3]);
}

// Plane f of a row of 2 * half elements, turned by (c, sn) on its way from `src` to `dst`: a lane per plane.
template <typename T> struct Plane { T a, b; };
template <typename T>
__device__ __forceinline__ Plane<T> plane_load(const void* src, int f, int half) {
  return {static_cast<const T*>(src)[f], static_cast<const T*>(src)[f + half]};
}
template <typename T>
__device__ __forceinline__ void plane_store(void* dst, int f, int half, const Plane<T>& x, float c, float sn) {
  typedef T __attribute__((may_alias)) elem;
  elem* const out = static_cast<elem*>(dst);
  if constexpr (sizeof(T) == 4) {
    out[f] = x.a * c - x.b * sn;
    out[f + half] = x.b * c + x.a * sn;
  } else {
    const float u = __uint_as_float((uint32_t)x.a << 16), v = __uint_as_float((uint32_t)x.b << 16);
    out[f] = f32_to_bf16_rne(u * c - v * sn);
    out[f + half] = f32_to_bf16_rne(v * c + u * sn);
  }
}

// What a decode step with a k_attn launch has to turn before it, in one small launch: the Q rows
// (into q_rot, [n][Hq][D]) and the K rows of a deferred rotating append (into k_rot,
// [pend_n][Hkv][D]; the attention launch then reads and copies those instead of the caller's
// unrotated rows).  A lane per plane, rows [0, n_q_rows) are Q's: the launch is a chain of a position, a row and a store, and
// runs its code once, so little code and many lanes (a lane per 16-byte piece, eight angles each: 8 streams over 4096 tokens, append and decode step, 17.4 us; this way 16.1;
// 3 over 1024 15.8 and 15.4, 8 over 8192 19.8 and 18.9).  Rotating
// inside the attention kernel was tried first and costs more than this launch: with loads that
// go straight into LDS in flight the compiler makes every other wait a wait for all of them.
// DecodeParams comes first (the metadata may ride inside it).  half = 1 << half_log: planes of a row.
template <typename T>
__global__ __launch_bounds__(256) void k_rope_prep(DecodeParams p, T* q_rot, T* k_rot, int half_log, int n_q_rows) {
  const int half = 1 << half_log, f = (int)threadIdx.x & (half - 1);
  const double per_pos = p.rope_tab[f];
  const int t = (int)blockIdx.x * (256 >> half_log) + ((int)threadIdx.x >> half_log);
  const int n_k_rows = p.pend_rope ? p.pend_n * p.Hkv : 0;
  if (t >= n_q_rows + n_k_rows) return;
  const bool is_q = t < n_q_rows;
  const int row = is_q ? t : t - n_q_rows;
  const T* src = static_cast<const T*>(is_q ? p.q : p.k_pend) + (long long)row * 2 * half;
  const Plane<T> x = plane_load<T>(src, f, half);
  const int pos = is_q ? meta_of(p)[p.off_streams + row / p.Hq * (int)(sizeof(DevStream) / 4) + (int)(offsetof(DevStream, pos) / 4)]
                       : pend_pos_of(p)[row / p.Hkv];
  float c, sn;
  rope_cos_sin_by<sizeof(T) == 2>(per_pos, pos, c, sn);
  plane_store<T>((is_q ? q_rot : k_rot) + (long long)row * 2 * half, f, half, x, c, sn);
}

}  // namespace pasta
