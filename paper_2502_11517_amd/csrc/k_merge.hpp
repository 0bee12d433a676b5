// K4 -- log-sum-exp merge of the split partials.  Splitting a stream's visible set between
// the shared-prefix chunks and the private-segment items is this build's device; the
// identity used is  sum_t e^{z_t} v_t = sum_i e^{m_i} acc_i  over the parts i, so
//   m = max_i m_i,  l = sum_i l_i 2^{m_i - m},  out = sum_i acc_i 2^{m_i - m} / l
// (m in log2 units).  Parts with l_i = 0 (nothing visible in them) contribute nothing.
// One work-group of NT threads per (stream, query head): the threads form NT / (D / 4) groups,
// group k takes parts k, k + groups, ... with four head-dim elements per thread (a part's
// row is read as one coalesced 4D-byte line).  The kernel is a chain of memory round
// trips, kept to one -- what it needs of up to 32 streams rides in the kernel arguments -- or
// two (the stream's record, then all its parts in one list).  The maximum
// and the sum over the groups are taken by group 0 after one LDS exchange.
// What bounds it is that chain and the start of its wavefronts, so a row gets the fewest threads that hold the parts
// of the launch's longest row in one batch.  One head-dim element per thread, 1024 threads per row and the plan's 4 KB of arguments took 3.6 us in a kernel trace (17
// parts on each of 128 rows), this form takes 2.9.  Append and decode step of a layer by 256 / 128 / 64 threads (us; the form before):
//   18 parts, 32 rows        7.9 / 7.8 / 8.3 (8.3)       35 parts, 64 rows     14.0 / 14.4 / 15.0 (14.4)
//   17 parts, 512 rows      17.5 / 17.3 / 17.5 (18.4)    9 parts, 1024 rows    43.5 / 42.9 / 42.2 (43.3)
//   36 parts, 256 rows of 64 dims 11.1 / 10.9 / 11.2 (11.8)   130 parts, 4 rows 10.3 / 11.7 / 14.5 (11.3)
#pragma once
#include "mfma_util.hpp"

namespace pasta {

constexpr int kMergeRecs = 32;
constexpr int kMergeBatch = 8;  // parts per thread and batch
constexpr int merge_batch(int threads, int D) { return threads / (D / 4) * kMergeBatch; }  // parts that a work-group takes in one

struct MergeRec {  // a stream's parts: shared-prefix part i of (kv head g, head gi) is row pre0 + (g * n_pre + i) * R + gi,
  int32_t pre0, n_pre, R;       // private part j is row priv_part_base + ((item_begin + j) * Hkv + g) * G + gi
  int32_t item_begin, n_priv;
};
struct MergeParams {
  void* out;              // [n][Hq][D]
  float* lse;             // [n][Hq] or null
  const float* part_acc;  // [rows][D]
  const float2* part_ml;  // [rows] (m in log2 units, l)
  const int32_t* meta;    // null: the records are in `rec`; else the plan's words, in device memory
  int off_streams, priv_part_base, Hkv, G;
  MergeRec rec[kMergeRecs];
};

template <typename T, int D, int NT>
__global__ __launch_bounds__(NT) void k_merge(MergeParams p) {
  constexpr int kLanes = D / 4, kGroups = NT / kLanes;
  constexpr int kBatch = kMergeBatch;
  __shared__ f32x4 osum[kGroups][kLanes];
  __shared__ float msum[kGroups], lsum[kGroups];
  const int tid = threadIdx.x;
  const int grp = tid / kLanes, d = tid % kLanes;
  // grid (Hkv, G, streams): the linear work-group index is (s * G + gi) * Hkv + g, whose remainder
  // mod Hkv is the kv head, as in the attention launch, so that with 8 kv heads the partials are
  // read on the XCD whose L2 holds them (three grid dimensions spare the kernel the divisions)
  const int g = blockIdx.x, gi = blockIdx.y, s = blockIdx.z;
  typedef const int32_t __attribute__((address_space(4))) * words;
  typedef const char __attribute__((address_space(4))) * kernarg_ptr;
  int pre0, n_pre, R, item_begin, n_priv;
  if (!p.meta) {
    const words r = (words)((kernarg_ptr)__builtin_amdgcn_kernarg_segment_ptr() + __builtin_offsetof(MergeParams, rec)) + s * (int)(sizeof(MergeRec) / 4);
    pre0 = r[0]; n_pre = r[1]; R = r[2]; item_begin = r[3]; n_priv = r[4];
  } else {
    const words r = (words)(uintptr_t)p.meta + p.off_streams + s * (int)(sizeof(DevStream) / 4);
    pre0 = r[offsetof(DevStream, m_pre0) / 4]; n_pre = r[offsetof(DevStream, m_n_pre) / 4]; R = r[offsetof(DevStream, m_R) / 4];
    item_begin = r[offsetof(DevStream, item_begin) / 4];
    n_priv = r[offsetof(DevStream, item_end) / 4] - item_begin;
  }
  // parts [0, n_pre) and [n_pre, n) as ONE list
  const int n = n_pre + n_priv, step_b = p.Hkv * p.G;
  const int a0 = pre0 + g * n_pre * R + gi, b0 = p.priv_part_base + (item_begin * p.Hkv + g) * p.G + gi;
  // The running state of this thread: max-free accumulation is not possible, so each batch
  // is folded with the running max of what the thread has seen (one more online softmax).
  // No early exit and no branch on the loaded values: with one, the compiler requests a part's
  // accumulator only after its (m, l) has arrived and been looked at -- two memory round trips
  // per batch instead of one.
  float m_t = -INFINITY, l_t = 0.f;
  f32x4 o_t = f32x4{0.f, 0.f, 0.f, 0.f};
  for (int i0 = grp; i0 < n; i0 += kGroups * kBatch) {
    float2 ml[kBatch];
    f32x4 a[kBatch];
#pragma unroll
    for (int u = 0; u < kBatch; ++u) {
      ml[u] = make_float2(-INFINITY, 0.f);
      a[u] = f32x4{0.f, 0.f, 0.f, 0.f};
      const int i = i0 + u * kGroups;
      if (i < n) {  // (nothing stands in for a part that is not there: 0 times an infinity of another's would be NaN)
        const int row = i < n_pre ? a0 + i * R : b0 + (i - n_pre) * step_b;
        ml[u] = p.part_ml[row];
        a[u] = *reinterpret_cast<const f32x4*>(p.part_acc + (long long)row * D + 4 * d);
      }
    }
    float mb = m_t;
#pragma unroll
    for (int u = 0; u < kBatch; ++u) mb = fmaxf(mb, ml[u].y > 0.f ? ml[u].x : -INFINITY);
    const float mref = mb == -INFINITY ? 0.f : mb;  // nothing seen yet: every weight below is 0
    const float c = fast_exp2(m_t - mref);          // 0 when m_t was -inf
    l_t *= c;
    o_t *= c;
    m_t = mb;
#pragma unroll
    for (int u = 0; u < kBatch; ++u) {
      const float wgt = ml[u].y > 0.f ? fast_exp2(ml[u].x - mref) : 0.f;
      l_t = fmaf(ml[u].y, wgt, l_t);
#pragma unroll
      for (int e = 0; e < 4; ++e) o_t[e] = fmaf(a[u][e], wgt, o_t[e]);
    }
  }

  // ---- the groups meet once: each leaves its (m, l, o) in LDS as it is, group 0 takes the common
  // max, rescales and adds (a group's m and l are the same for all its head-dim elements)
  osum[grp][d] = o_t;
  if (d == 0) { msum[grp] = m_t; lsum[grp] = l_t; }
  __syncthreads();
  if (grp == 0) {
    float mg[kGroups], mx = -INFINITY;
#pragma unroll
    for (int k = 0; k < kGroups; ++k) { mg[k] = msum[k]; mx = fmaxf(mx, mg[k]); }
    f32x4 o = f32x4{0.f, 0.f, 0.f, 0.f};
    float L = 0.f;
#pragma unroll
    for (int k = 0; k < kGroups; ++k) {
      const float c = (mg[k] == -INFINITY) ? 0.f : fast_exp2(mg[k] - mx);
      const f32x4 x = osum[k][d];
#pragma unroll
      for (int e = 0; e < 4; ++e) o[e] = fmaf(x[e], c, o[e]);
      L = fmaf(lsum[k], c, L);
    }
    const long long row = (long long)s * p.Hkv * p.G + g * p.G + gi;
    // (`out` may be any multiple of 4 bytes)
    if constexpr (sizeof(T) == 4) {
      typedef f32x4 __attribute__((aligned(4))) quad;
      *reinterpret_cast<quad*>(reinterpret_cast<float*>(p.out) + row * D + 4 * d) = f32x4{o[0] / L, o[1] / L, o[2] / L, o[3] / L};
    } else {
      typedef u32x2 __attribute__((aligned(4))) pair;
      uint32_t x[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) x[e] = f32_to_bf16_rne(o[e] / L);
      *reinterpret_cast<pair*>(reinterpret_cast<uint16_t*>(p.out) + row * D + 4 * d) = u32x2{x[0] | x[1] << 16, x[2] | x[3] << 16};
    }
    if (p.lse && d == 0) p.lse[row] = (mx + __log2f(L)) * kLn2;
  }
}

}  // namespace pasta
