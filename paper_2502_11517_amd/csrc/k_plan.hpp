// Puts a decode step's plan on the device, once for all the layers that use it.
//
// A plan that does not fit the kernel arguments (many streams, or lists of many short ranges) is the same for
// every layer of a token step.  The host writes it to pinned memory once, this launch copies it to device
// memory and expands it: work-group b resolves private item b -- which stream, which ranges, which physical
// row for every token -- so that the attention launches find their rows in one read.  Later calls with an
// identical plan use what is there.
// Before, every layer's call sent its records in one or two launches of their own, and every one of the item's
// Hkv work-groups derived the item by itself, some ten dependent reads ahead of its first K/V request.
#pragma once
#include "mfma_util.hpp"

namespace pasta {

// Pieces of the device-resident lists on their way from pinned host memory to their places in the workspace.
// (One asynchronous copy per list and index took some 10 us each on the stream: 600 us for the first step of 32
// streams after a prefill.)
struct ListPiece { long long dst_word; int32_t src_word, n_words; };

__global__ __launch_bounds__(256) void k_lists(const ListPiece* pieces, const int32_t* words, int32_t* workspace) {
  const ListPiece lp = pieces[blockIdx.x];
  for (int i = threadIdx.x; i < lp.n_words; i += 256) workspace[lp.dst_word + i] = words[lp.src_word + i];
}

// A plan of up to kPlanWords words travels in the kernel arguments, a larger one lies in pinned host memory --
// where a read takes a microsecond, so a work-group makes two at most, one behind the other.
constexpr int kPlanWords = 960;
struct PlanParams {
  const int32_t* src;    // null: `words`
  int32_t* dst;          // the plan's place on the device
  DevItem* items;        // one per private item, its ranges resolved: one that lies inside a single range has n_ranges =
                         // -(its request), range_first and tok_begin = its stream's pend0 and pend_src0
  int32_t* codes;        // priv_chunk per item: physical row of every token, or -(1 + row) of a deferred append
  const int32_t* page_table;
  const DevRange* arena; // device-resident lists
  const int32_t* cidx;
  Layout lay;
  int n_words;           // words to copy (the source holds off_items beyond them, with device-resident lists)
  int n_items, priv_chunk;
  int dev_tables;        // 1: no ranges in the plan; off_items holds the stream of every item
  int off_streams, off_ranges, off_items;
  int32_t words[kPlanWords];
};
static_assert(sizeof(PlanParams) <= 4096, "kernel arguments are limited to 4 KB");

__global__ __launch_bounds__(256) void k_plan(PlanParams p) {
  __shared__ DevRange lr[kGatherMax];
  __shared__ int sel[2];
  typedef const char __attribute__((address_space(4))) * kernarg_ptr;
  const int32_t* src = p.src ? p.src : (const int32_t*)((kernarg_ptr)__builtin_amdgcn_kernarg_segment_ptr() + __builtin_offsetof(PlanParams, words));
  const int tid = threadIdx.x, b = blockIdx.x;
  for (int i = b * 256 + tid; i < p.n_words; i += gridDim.x * 256) p.dst[i] = src[i];
  if (b >= p.n_items) return;
  DevItem it;
  DevStream st;
  int nr = 0, range0 = 0;
  if (!p.dev_tables) {
    it = reinterpret_cast<const DevItem*>(src + p.off_items)[b];
    st = reinterpret_cast<const DevStream*>(src + p.off_streams)[it.stream];
    if (it.n_ranges > 1) { nr = it.n_ranges; range0 = it.range_first; }
  } else {
    const int si = src[p.off_items + b];
    st = reinterpret_cast<const DevStream*>(src + p.off_streams)[si];
    bool in_ranges;
    it = dev_item(p, st, si, b, in_ranges);
    if (in_ranges) range0 = dev_item_candidates(p, st, it.tok_begin, it.tok_count, kGatherMax, nr);
  }
  const int tok_base = it.tok_begin;
  const DevRange* ranges = reinterpret_cast<const DevRange*>(src + p.off_ranges);
  for (int k = tid; k < nr; k += 256) lr[k] = p.dev_tables ? dev_range_at(p, st, range0 + k) : ranges[range0 + k];  // (thread k reads its own entries below)
  if (p.dev_tables && nr > 0) {  // which candidates hold the item's first and last token
    const int t_lo = it.tok_begin, t_hi = it.tok_begin + it.tok_count - 1;
    for (int k = tid; k < nr; k += 256) {
      if (lr[k].cum <= t_lo && t_lo < lr[k].cum + lr[k].count) sel[0] = k;
      if (lr[k].cum <= t_hi && t_hi < lr[k].cum + lr[k].count) sel[1] = k;
    }
  }
  __syncthreads();
  if (tid == 0) {
    DevItem out = it;
    if (p.dev_tables && nr > 0) {
      const DevRange r0 = lr[sel[0]];
      out.slot0 = r0.start + (tok_base - r0.cum) * r0.stride;
      out.stride = r0.stride;
      out.n_ranges = sel[1] - sel[0] + 1;
    }
    if (out.n_ranges == 1) {  // tokens slot0 + j * stride: what the attention launch needs to address them by arithmetic
      out.n_ranges = -st.req;
      out.range_first = st.pend0;
      out.tok_begin = st.pend_src0;
    }
    p.items[b] = out;
  }
  for (int j = tid; j < it.tok_count; j += 256) {
    int slot = it.slot0 + j * it.stride;
    if (nr > 0) {
      const int tok = tok_base + j;
      int lo = 0, hi = nr - 1;  // last range with cum <= tok
      while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (lr[mid].cum <= tok) lo = mid; else hi = mid - 1;
      }
      slot = lr[lo].start + (tok - lr[lo].cum) * lr[lo].stride;
    }
    p.codes[(long long)b * p.priv_chunk + j] = slot >= st.pend0 ? -1 - (st.pend_src0 + (slot - st.pend0)) : phys_row(p.lay, p.page_table, st.req, slot);
  }
}

// The physical row behind a row code.
__device__ __forceinline__ int phys_of_code(const DecodeParams& p, int code) { return code >= 0 ? code : pend_dst_of(p)[-1 - code]; }

}  // namespace pasta
