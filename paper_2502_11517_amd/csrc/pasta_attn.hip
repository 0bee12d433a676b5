// C-ABI library of the multi-stream decode-attention step (include/pasta_attn.h).
// Host side: argument validation, the visibility lists kept per (request, stream)
// (arxiv 2502.11517, Section 3 "Efficiency": ancestor rule of Figure 2b), slot assignment
// at the pool tail (Figure 2c), and the launch plan.  Every step of the arithmetic runs in
// the gfx950 kernels included below.
#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <new>
#include <unordered_map>
#include <vector>

#include "../../include/pasta_attn.h"
#include "k_append.hpp"
#include "k_attn.hpp"
#include "k_direct.hpp"
#include "k_merge.hpp"
#include "k_private.hpp"
#include "staging_ring.hpp"

using namespace pasta;

namespace {

constexpr uint32_t kMagic = 0x50415354u;  // "PAST"
constexpr int kRing = 8;                  // metadata staging buffers in flight
constexpr int64_t kPlanCodesMax = (int64_t)1 << 22;  // most private tokens of a plan that is kept on the device (16 MiB of row codes;
                                                     // more where the streams of a no-alloc call can have more between them)
constexpr int kOneTokens = 1024;          // most tokens of a work-group of k_one (it holds their addresses at once)
constexpr int kManyChunk = 512;           // tokens: chunks of several requests' prefixes are not cut down below this
constexpr int kNumCUs = 256;              // MI355X; planning default until the device has been asked
constexpr int kTargetPrefixWgs = 768;     // most shared-prefix work-groups budgeted for

struct Range { int32_t start, count, stride; };

struct StreamState {
  bool open = false;
  int32_t prefix_len = 0;        // visible head [0, prefix_len)
  std::vector<Range> ranges;     // then these, span-ascending
  int64_t range_tokens = 0;      // tokens in `ranges`
  // The copy of the range list that lives on the device (workspace): ranges with running token counts in
  // the arena, and an index "range that holds range token 32 j".  Small appends patch it through the K1
  // launch, everything else (prefill, fork, join, relocation) marks it dirty and it is rebuilt from this
  // mirror at the next decode step that wants it.  The newest range is never relied on: it grows with
  // every append and rides with each call instead.
  int32_t seg_off = -1, seg_cap = 0;    // arena segment (DevRange entries)
  int32_t cseg_off = -1, cseg_cap = 0;  // index segment (int32 entries)
  int32_t dev_ranges = 0;        // arena entries [0, dev_ranges) are exact
  int32_t dev_cidx = 0;          // index entries [0, dev_cidx) are on the device; all later ones lie in the newest range
  bool dirty = true;
};

inline size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

struct ListView {  // one stream's visible list for this call
  int32_t prefix_len;
  const Range* ranges;   // maintained mode
  int32_t n_ranges;
  const int32_t *start, *count, *stride;  // explicit mode (ranges == nullptr)
  int64_t range_tokens;      // tokens in the ranges
  Range at(int k) const { return ranges ? ranges[k] : Range{start[k], count[k], stride[k]}; }
};



// Host buffers of one decode_step's plan.  They live in the handle and keep their capacity from
// call to call, so that a step in a serving loop touches no allocator; create reserves what a
// plan small enough to ride in the kernel arguments can need.
struct PlanBuf {
  std::vector<ListView> lv;
  std::vector<Range> trim;               // the lists that causal_skip shortens (never grown past its reserve: views point into it)
  std::vector<uint8_t> seen, mask;
  std::vector<int32_t> mask_base, req_idx_of, stream_req_idx, stream_local, req_streams, blob;
  std::vector<DevReq> reqs;
  std::vector<DevStream> streams;
  std::vector<DevRange> ranges;
  std::vector<DevItem> items;
};

}  // namespace

struct pasta_attn {
  uint32_t magic = kMagic;
  pasta_attn_config cfg{};
  int G = 1, elem = 2, page_shift = 31;
  int64_t rows_per_layer = 0, layer_elems = 0, req_capacity = 0;
  Layout lay{};
  std::vector<int32_t> page_table;
  std::vector<int32_t> req_pages;        // paged mode: pages assigned to each request (its capacity)
  std::vector<int64_t> tail;             // per request
  std::vector<int64_t> tail_before;      // tails before the latest layer-0 append
  std::vector<StreamState> streams;      // [max_requests * max_streams]
  // workspace carve-up (byte offsets)
  size_t off_page_table = 0, off_meta = 0, meta_bytes = 0, off_ml = 0, off_acc = 0;
  size_t off_rope = 0, off_qrot = 0, off_krot = 0;  // rope_theta > 0: rotary table (fp64, D/2 entries), rotated Q,
                                                   // rotated K rows of a deferred append
  size_t off_mask = 0, mask_bytes = 0;  // dense-mask comparison mode: one byte per (stream, slot)
  uint8_t* mask_pinned = nullptr;       // its host staging, allocated at first use
  hipEvent_t mask_ev{};
  bool mask_ev_used = false;
  int64_t part_rows_cap = 0;
  // a deferred append (PASTA_APPEND_DEFER): its copy is done by the next decode_step's launch
  struct Pending {
    bool active = false;
    int layer = 0, n_rows = 0;
    const void *k_new = nullptr, *v_new = nullptr;
    int32_t dst_rows[kAppendInline]{};
    bool rope = false;                 // PASTA_APPEND_ROPE: K still to be rotated by pos
    int32_t pos[kAppendInline]{};
    std::vector<AppendRun> runs;       // the same rows as runs, for the launch that copies them if no decode step does
    std::vector<int32_t> req_pend0, req_src0;  // per request: first deferred slot, its row in k_new
    std::vector<int32_t> stage_p0, stage_s0, stage_last;  // (their buffers while a call is looked at)
  } pending;
  PlanBuf pb;
  // device-resident lists: carve-up and bump allocation (entries)
  size_t off_arena = 0, off_cidx = 0;
  // the plan kept on the device (k_plan): its words, its items and their tokens' rows; and what it was made of
  size_t off_plan[2] = {}, off_plan_items[2] = {}, off_plan_codes[2] = {};  // [1]: of calls under stream capture
  int64_t plan_items_cap = 0, plan_codes_cap = 0;
  std::vector<int32_t> plan_words;       // the words it was made from (empty: none there)
  uint64_t lists_epoch = 0;              // counts the changes of the maintained lists
  int64_t arena_cap = 0, cidx_cap = 0, arena_top = 0, cidx_top = 0;
  bool tables_reset = false;             // the segments ran out: start over at the next call (all streams dirty)
  bool lists_in_use = false;             // a decode step has read the device copy: appends keep it current from then on
                                         // (before that they only mark what changed, and may be deferred freely)
  std::vector<DevRange> stage_r;         // staging of one stream's lists for a rebuild
  std::vector<int32_t> stage_c;
  std::vector<ListPiece> stage_pieces;   // ... and of all the lists that one call sends
  std::vector<int32_t> stage_words;
  struct Undo { int64_t key; bool open; int32_t prefix_len; int32_t n_ranges; Range last; int64_t range_tokens;
                int32_t dev_ranges, dev_cidx; bool dirty; bool replaced; std::vector<Range> saved; };
  std::vector<Undo> undo;                // append_kv: what to restore if a later row of the call fails
  std::vector<int64_t> t2;
  std::vector<int32_t> dst_rows;         // destination rows of a call whose runs do not fit the kernel arguments
  std::vector<AppendRun> runs;           // append_kv: the call's rows as runs
  int tune_prefix_chunk = 0, tune_priv_chunk = 0;  // forced chunk sizes (tokens; 0 = heuristic): set only by -DPASTA_TUNING builds
  // device-side readiness (deferred so that the host logic works without a GPU)
  bool device_ready = false;
  char* pinned = nullptr;                // kRing * meta_bytes
  hipEvent_t ring_ev[2]{};               // one per half of the ring
  int ring_ev_made = 0;                  // events created so far (both once the device is ready)
  int device = 0, n_cus = kNumCUs;       // the device current at first use and its compute-unit count
  StagingRing<kRing> ring;
  int relay_next = 0;
};

namespace {

int64_t meta_words_cap(const pasta_attn_config& c) {
  // streams + reqs + req_streams + ranges (+1 per stream for the uncommon prefix tail) + items
  const int64_t ns = (int64_t)c.max_requests * c.max_streams;
  const int64_t ranges = (int64_t)c.max_ranges + ns;
  const int64_t cap_tokens = c.page_tokens ? (int64_t)c.pages_per_request * c.page_tokens : c.pool_tokens;
  // items: every stream can split its private list into chunks; bounded by total tokens/chunk + streams
  const int64_t items = ns * ((cap_tokens + kPrivChunk - 1) / kPrivChunk + 1);
  return ns * (int64_t)(sizeof(DevStream) / 4) + (int64_t)c.max_requests * (sizeof(DevReq) / 4) + ns +
         ranges * 4 + std::min<int64_t>(items, (int64_t)1 << 22) * (int64_t)(sizeof(DevItem) / 4) + 64;
}

int validate_cfg(const pasta_attn_config* c) {
  if (!c || c->struct_size != sizeof(pasta_attn_config)) return PASTA_E_INVAL;
  if (c->dtype != PASTA_F32 && c->dtype != PASTA_BF16) return PASTA_E_INVAL;
  if (c->n_q_heads < 1 || c->n_kv_heads < 1 || c->n_q_heads % c->n_kv_heads) return PASTA_E_INVAL;
  const int G = c->n_q_heads / c->n_kv_heads;
  if (G != 1 && G != 2 && G != 4 && G != 8) return PASTA_E_INVAL;
  if (c->head_dim != 64 && c->head_dim != 128) return PASTA_E_INVAL;
  if (c->n_layers < 1 || c->max_requests < 1 || c->max_streams < 1 || c->max_ranges < 1) return PASTA_E_INVAL;
  if (c->kv_layout != PASTA_LAYOUT_TOKEN_MAJOR && c->kv_layout != PASTA_LAYOUT_HEAD_MAJOR) return PASTA_E_INVAL;
  if (!(c->softmax_scale > 0.f) || !std::isfinite(c->softmax_scale)) return PASTA_E_INVAL;
  if (!(c->rope_theta >= 0.f) || !std::isfinite(c->rope_theta) || (c->rope_theta > 0.f && c->rope_theta < 1.f))
    return PASTA_E_INVAL;
  if (c->page_tokens == 0) {
    if (c->pool_tokens < 1) return PASTA_E_INVAL;
    if ((int64_t)c->max_requests * c->pool_tokens >= ((int64_t)1 << 31)) return PASTA_E_INVAL;
  } else {
    if (c->page_tokens < 1 || (c->page_tokens & (c->page_tokens - 1))) return PASTA_E_INVAL;
    if (c->n_phys_pages < 1 || c->pages_per_request < 1) return PASTA_E_INVAL;
    if ((int64_t)c->n_phys_pages * c->page_tokens >= ((int64_t)1 << 31)) return PASTA_E_INVAL;
  }
  return PASTA_OK;
}

// Partial-row budget: enough for the split-K parallelism aimed for at the largest stacked
// row count, plus one row per (private item, query head).
int64_t part_rows_budget(const pasta_attn_config& c) {
  const int64_t ns = (int64_t)c.max_requests * c.max_streams;
  const int64_t cap_tokens = c.page_tokens ? (int64_t)c.pages_per_request * c.page_tokens : c.pool_tokens;
  const int64_t prefix = (int64_t)(kTargetPrefixWgs + c.n_kv_heads * c.max_requests) * c.max_streams *
                         (c.n_q_heads / c.n_kv_heads) * 2;
  const int64_t items = std::min<int64_t>(ns * ((cap_tokens + kPrivChunk - 1) / kPrivChunk + 1),
                                          (int64_t)c.max_requests * cap_tokens / 16 + ns * 2);
  return prefix + items * c.n_q_heads;
}

void carve(pasta_attn* h) {
  const pasta_attn_config& c = h->cfg;
  size_t off = 0;
  h->off_page_table = off;
  off += align_up((size_t)c.max_requests * (c.page_tokens ? c.pages_per_request : 0) * 4 + 4, 256);
  h->meta_bytes = align_up((size_t)meta_words_cap(c) * 4, 256);
  h->off_meta = off;
  off += h->meta_bytes * kRing;
  h->part_rows_cap = part_rows_budget(c);
  h->off_ml = off;
  off += align_up((size_t)h->part_rows_cap * sizeof(float2), 256);
  h->off_acc = off;
  off += align_up((size_t)h->part_rows_cap * c.head_dim * sizeof(float), 256);
  {
    const int64_t cap_tokens = c.page_tokens ? (int64_t)c.pages_per_request * c.page_tokens : c.pool_tokens;
    h->mask_bytes = align_up((size_t)c.max_requests * c.max_streams * (size_t)cap_tokens + 256, 256);
    h->off_mask = off;
    off += h->mask_bytes;
  }
  {  // device-resident lists: room for every range twice over (segments grow by doubling) and for the index
    const int64_t ns = (int64_t)c.max_requests * c.max_streams;
    const int64_t cap_tokens = c.page_tokens ? (int64_t)c.pages_per_request * c.page_tokens : c.pool_tokens;
    h->arena_cap = std::min<int64_t>(4 * ((int64_t)c.max_ranges + ns * 16), (int64_t)1 << 26);
    h->cidx_cap = std::min<int64_t>(2 * (ns * (cap_tokens / kCidxTokens + 16)), (int64_t)1 << 26);
    h->off_arena = off;
    off += align_up((size_t)h->arena_cap * sizeof(DevRange), 256);
    h->off_cidx = off;
    off += align_up((size_t)h->cidx_cap * 4, 256);
  }
  {  // the plan kept on the device; one with more private tokens is made from the host's lists and read where it lies
    const int64_t ns = (int64_t)c.max_requests * c.max_streams;
    const int64_t cap_tokens = c.page_tokens ? (int64_t)c.pages_per_request * c.page_tokens : c.pool_tokens;
    const int64_t per_stream = cap_tokens + 2 * kGatherMax;
    h->plan_codes_cap = std::min<int64_t>(ns * per_stream, std::max<int64_t>(kPlanCodesMax, kInlineMetaWords / (sizeof(DevStream) / 4) * per_stream));
    h->plan_items_cap = h->plan_codes_cap / kPrivChunk;
    for (int at = 0; at < 2; ++at) {
      h->off_plan[at] = off;
      off += h->meta_bytes;
      h->off_plan_items[at] = off;
      off += align_up((size_t)h->plan_items_cap * sizeof(DevItem), 256);
      h->off_plan_codes[at] = off;
      off += align_up((size_t)h->plan_codes_cap * 4, 256);
    }
  }
  if (c.rope_theta > 0.f) {
    h->off_rope = off;
    off += align_up((size_t)(c.head_dim / 2) * sizeof(double), 256);
    h->off_qrot = off;
    off += align_up((size_t)c.max_requests * c.max_streams * c.n_q_heads * c.head_dim * h->elem, 256);
    h->off_krot = off;
    off += align_up((size_t)kAppendInline * c.n_kv_heads * c.head_dim * h->elem, 256);
  }
  h->cfg.workspace_bytes = off;
}

int ensure_device(pasta_attn* h) {
  if (h->device_ready) return PASTA_OK;
  // every step is skipped on re-entry once it has succeeded, so a failure leaks nothing
  if (!h->pinned && hipHostMalloc((void**)&h->pinned, h->meta_bytes * kRing, hipHostMallocDefault) != hipSuccess) {
    (void)hipGetLastError();
    h->pinned = nullptr;
    return PASTA_E_DEVICE;
  }
  for (; h->ring_ev_made < 2; ++h->ring_ev_made)
    if (hipEventCreateWithFlags(&h->ring_ev[h->ring_ev_made], hipEventDisableTiming) != hipSuccess) {
      (void)hipGetLastError();
      return PASTA_E_DEVICE;
    }
  int n_cu = 0;
  if (hipGetDevice(&h->device) != hipSuccess ||
      hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, h->device) != hipSuccess || n_cu < 1) {
    (void)hipGetLastError();
    return PASTA_E_DEVICE;
  }
  h->n_cus = n_cu;
  if (h->cfg.page_tokens) {
    if (hipMemcpy((char*)h->cfg.workspace + h->off_page_table, h->page_table.data(),
                  h->page_table.size() * 4, hipMemcpyHostToDevice) != hipSuccess) {
      (void)hipGetLastError();
      return PASTA_E_DEVICE;
    }
  }
  if (h->cfg.rope_theta > 0.f) {  // theta^(-2f/D) / (2 pi) in fp64: angles are taken in revolutions
    const int D = h->cfg.head_dim;
    std::vector<double> tab(D / 2);
    for (int f = 0; f < D / 2; ++f)
      tab[f] = std::pow((double)h->cfg.rope_theta, -2.0 * f / D) / 6.283185307179586476925286766559;
    if (hipMemcpy((char*)h->cfg.workspace + h->off_rope, tab.data(), tab.size() * sizeof(double),
                  hipMemcpyHostToDevice) != hipSuccess) {
      (void)hipGetLastError();
      return PASTA_E_DEVICE;
    }
  }
  h->device_ready = true;
  return PASTA_OK;
}

int ring_take(pasta_attn* h, int* slot, char** host) {
  if (!h->ring.take(slot, [&](int half) { return hipEventSynchronize(h->ring_ev[half]) == hipSuccess; },
                    [&] { return hipStreamSynchronize((hipStream_t)h->cfg.hip_stream) == hipSuccess; })) return PASTA_E_DEVICE;
  *host = h->pinned + (size_t)*slot * h->meta_bytes;
  return PASTA_OK;
}
int ring_give(pasta_attn* h) {  // the work that reads the slot has been enqueued
  return h->ring.give([&](int half) { return hipEventRecord(h->ring_ev[half], (hipStream_t)h->cfg.hip_stream) == hipSuccess; }) ? PASTA_OK : PASTA_E_DEVICE;
}

bool stream_capturing(const pasta_attn* h) {
  hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing((hipStream_t)h->cfg.hip_stream, &cap) != hipSuccess) { (void)hipGetLastError(); return false; }
  return cap != hipStreamCaptureStatusNone;
}

// Host words to the next device staging slot inside the arguments of as many small launches as it takes.
int relay_words(pasta_attn* h, const int32_t* src, size_t n, const int32_t** dev_out) {
  const int s = h->relay_next;
  h->relay_next = (s + 1) % kRing;
  int32_t* dev = (int32_t*)((char*)h->cfg.workspace + h->off_meta + (size_t)s * h->meta_bytes);
  for (size_t lo = 0; lo < n; lo += kRelayWords) {
    RelayParams rp;
    rp.dst = dev + lo;
    rp.n_words = (int)std::min<size_t>(kRelayWords, n - lo);
    std::memcpy(rp.words, src + lo, (size_t)rp.n_words * 4);
    k_meta_relay<<<dim3(1), 256, 0, (hipStream_t)h->cfg.hip_stream>>>(rp);
    if (hipGetLastError() != hipSuccess) return PASTA_E_DEVICE;
  }
  *dev_out = dev;
  return PASTA_OK;
}

// Copies n words of host metadata to the next device staging slot, asynchronously on the
// caller's stream; returns the device address.  A slot is reused only after the copy that
// last read its pinned half has completed.  (Under stream capture the words are recorded with the launches
// that carry them: a replay finds a pinned slot as later calls have left it.)
int upload_meta(pasta_attn* h, const int32_t* src, size_t n, const int32_t** dev_out) {
  const size_t bytes = n * 4;
  if (bytes > h->meta_bytes) return PASTA_E_CAPACITY;
  if (stream_capturing(h)) return relay_words(h, src, n, dev_out);
  int s;
  char* host;
  const int rc = ring_take(h, &s, &host);
  if (rc != PASTA_OK) return rc;
  std::memcpy(host, src, bytes);
  char* dev = (char*)h->cfg.workspace + h->off_meta + (size_t)s * h->meta_bytes;
  hipStream_t st = (hipStream_t)h->cfg.hip_stream;
  if (hipMemcpyAsync(dev, host, bytes, hipMemcpyHostToDevice, st) != hipSuccess) return PASTA_E_DEVICE;
  *dev_out = (const int32_t*)dev;
  return ring_give(h);
}

// Sends the staged pieces of lists to their places in the workspace: one pinned slot, one launch (never under capture).
int flush_lists(pasta_attn* h) {
  std::vector<ListPiece>& ps = h->stage_pieces;
  std::vector<int32_t>& words = h->stage_words;
  if (ps.empty()) return PASTA_OK;
  hipStream_t st = (hipStream_t)h->cfg.hip_stream;
  int sl;
  char* host;
  const int rc = ring_take(h, &sl, &host);
  if (rc != PASTA_OK) return rc;
  std::memcpy(host, ps.data(), ps.size() * sizeof(ListPiece));
  std::memcpy(host + ps.size() * sizeof(ListPiece), words.data(), words.size() * 4);
  k_lists<<<dim3((unsigned)ps.size()), 256, 0, st>>>((const ListPiece*)host, (const int32_t*)(host + ps.size() * sizeof(ListPiece)), (int32_t*)h->cfg.workspace);
  if (hipGetLastError() != hipSuccess) return PASTA_E_DEVICE;
  ps.clear();
  words.clear();
  return ring_give(h);
}

// Stages n words for place `off` (bytes, a multiple of 4) of the workspace, in pieces of a few KB each.
int stage_list(pasta_attn* h, size_t off, const int32_t* src, size_t n) {
  const size_t piece = std::min<size_t>(2048, h->meta_bytes / 4 - sizeof(ListPiece) / 4);
  for (size_t lo = 0; lo < n; lo += piece) {
    const size_t k = std::min(piece, n - lo);
    if ((h->stage_pieces.size() + 1) * sizeof(ListPiece) + (h->stage_words.size() + k) * 4 > h->meta_bytes) {
      const int rc = flush_lists(h);
      if (rc != PASTA_OK) return rc;
    }
    h->stage_pieces.push_back(ListPiece{(long long)(off / 4 + lo), (int32_t)h->stage_words.size(), (int32_t)k});
    h->stage_words.insert(h->stage_words.end(), src + lo, src + lo + k);
  }
  return PASTA_OK;
}

constexpr int kNoRoom = 1;  // rebuild_tables: the segments ran out (not an error: the call plans from the host lists)

// Stages the device copy of one stream's range list and range index, from the mirror; flush_lists sends it.
int rebuild_tables(pasta_attn* h, StreamState& st) {
  const int64_t n = (int64_t)st.ranges.size();
  const int64_t n_c = (st.range_tokens + kCidxTokens - 1) / kCidxTokens;
  if (n > st.seg_cap) {
    const int64_t cap = std::max<int64_t>(16, 2 * n);
    if (h->arena_top + cap > h->arena_cap) { h->tables_reset = true; return kNoRoom; }
    st.seg_off = (int32_t)h->arena_top;
    st.seg_cap = (int32_t)cap;
    h->arena_top += cap;
  }
  if (n_c > st.cseg_cap) {
    const int64_t cap = std::max<int64_t>(16, 2 * n_c);
    if (h->cidx_top + cap > h->cidx_cap) { h->tables_reset = true; return kNoRoom; }
    st.cseg_off = (int32_t)h->cidx_top;
    st.cseg_cap = (int32_t)cap;
    h->cidx_top += cap;
  }
  std::vector<DevRange>& sr = h->stage_r;
  std::vector<int32_t>& sc = h->stage_c;
  sr.resize((size_t)n);
  sc.resize((size_t)n_c);
  int64_t cum = 0, tok = 0;
  for (int64_t k = 0; k < n; ++k) {
    const Range& g = st.ranges[(size_t)k];
    sr[(size_t)k] = DevRange{g.start, g.count, g.stride, (int32_t)cum};
    for (; tok < cum + g.count; tok += kCidxTokens) sc[(size_t)(tok / kCidxTokens)] = (int32_t)k;
    cum += g.count;
  }
  int rc = PASTA_OK;
  if (n) rc = stage_list(h, h->off_arena + (size_t)st.seg_off * sizeof(DevRange), (const int32_t*)sr.data(), (size_t)n * (sizeof(DevRange) / 4));
  if (rc == PASTA_OK && n_c) rc = stage_list(h, h->off_cidx + (size_t)st.cseg_off * 4, sc.data(), (size_t)n_c);
  if (rc != PASTA_OK) return rc;
  st.dev_ranges = (int32_t)n;
  st.dev_cidx = (int32_t)n_c;
  st.dirty = true;  // until the pieces have been sent
  return PASTA_OK;
}

inline StreamState& sstate(pasta_attn* h, int req, int sid) {
  return h->streams[(size_t)req * h->cfg.max_streams + sid];
}

// logical slot -> physical row on the host (same formula as the header states)
inline int64_t host_phys(const pasta_attn* h, int req, int64_t slot) {
  if (!h->cfg.page_tokens) return (int64_t)req * h->cfg.pool_tokens + slot;
  const int64_t pp = h->page_table[(size_t)req * h->cfg.pages_per_request + (slot >> h->page_shift)];
  return (pp << h->page_shift) | (slot & (h->cfg.page_tokens - 1));
}

// Adds an owned slot to a stream's list (slots arrive in increasing order).
void add_slot(StreamState& s, int32_t slot) {
  if (s.ranges.empty() && slot == s.prefix_len) { s.prefix_len++; return; }
  s.range_tokens++;
  if (!s.ranges.empty()) {
    Range& r = s.ranges.back();
    if (r.count == 1 && slot > r.start) { r.stride = slot - r.start; r.count = 2; return; }
    if (slot == r.start + (int64_t)r.count * r.stride) { r.count++; return; }
  }
  s.ranges.push_back({slot, 1, 1});
}

// Adds n slots from `slot` on.
void add_slots(StreamState& s, int32_t slot, int32_t n) {
  int32_t k = 0;
  for (; k < n && k < 3; ++k) add_slot(s, slot + k);
  if (k == n) return;
  // three consecutive slots behind each other: the newest range ends in them with stride 1, or all is still the head
  if (s.ranges.empty()) { s.prefix_len += n - k; return; }
  s.ranges.back().count += n - k;
  s.range_tokens += n - k;
}

template <typename T, int D>
int launch_private_g(int G, dim3 grid, hipStream_t st, const DecodeParams& p) {
  switch (G) {
    case 1: k_private<T, D, 1><<<grid, 256, 0, st>>>(p); break;
    case 2: k_private<T, D, 2><<<grid, 256, 0, st>>>(p); break;
    case 4: k_private<T, D, 4><<<grid, 256, 0, st>>>(p); break;
    case 8: k_private<T, D, 8><<<grid, 256, 0, st>>>(p); break;
    default: return PASTA_E_INVAL;
  }
  return PASTA_OK;
}
template <typename T, int D>
void launch_merge_g(dim3 grid, hipStream_t st, const MergeParams& p, int64_t parts) {
  if (parts <= merge_batch(64, D)) k_merge<T, D, 64><<<grid, 64, 0, st>>>(p);
  else if (parts <= merge_batch(128, D)) k_merge<T, D, 128><<<grid, 128, 0, st>>>(p);
  else k_merge<T, D, 256><<<grid, 256, 0, st>>>(p);
}

int launch_private(const pasta_attn* h, dim3 grid, hipStream_t st, const DecodeParams& p) {
  const int D = h->cfg.head_dim;
  if (h->cfg.dtype == PASTA_F32)
    return D == 64 ? launch_private_g<float, 64>(h->G, grid, st, p) : launch_private_g<float, 128>(h->G, grid, st, p);
  return D == 64 ? launch_private_g<uint16_t, 64>(h->G, grid, st, p)
                 : launch_private_g<uint16_t, 128>(h->G, grid, st, p);
}
// grid = (Hkv, G, n); parts = the most partial rows that one of its output rows reads: such rows end the launch.  By the mean instead, rows
// of few parts beside them leave them too few threads: append and decode step of a layer by the mean / by the most parts (us), 8 kv heads:
//   16384 tokens and three requests of 512      26.2 / 24.7      32768 and fifteen of 512    41.0 / 38.4
//   the same in fp32                            44.9 / 43.2      16384 and seven of 300, 2 streams each    27.0 / 25.4
// (where both give one width, or all rows have as many parts, the same within noise).
void launch_merge(const pasta_attn* h, dim3 grid, hipStream_t st, const MergeParams& p, int64_t parts) {
  if (h->cfg.dtype == PASTA_F32) {
    if (h->cfg.head_dim == 64) launch_merge_g<float, 64>(grid, st, p, parts);
    else launch_merge_g<float, 128>(grid, st, p, parts);
  } else {
    if (h->cfg.head_dim == 64) launch_merge_g<uint16_t, 64>(grid, st, p, parts);
    else launch_merge_g<uint16_t, 128>(grid, st, p, parts);
  }
}

struct ListPatches {  // entries of the device-resident lists that an append brings up to date
  int n_r = 0, n_c = 0;
  int32_t r_idx[kPatchMax];
  DevRange r_val[kPatchMax];
  int32_t c_idx[kPatchMax];
  int32_t c_val[kPatchMax];
};

// Most rows of one K1 launch: the kernel numbers its pieces in 32 bits.
size_t append_rows_max(const pasta_attn* h, bool rope) {
  return (size_t)(((int64_t)1 << 30) / ((int64_t)h->cfg.n_kv_heads * h->cfg.head_dim * h->elem / 16 / (rope ? 2 : 1)));
}
// Whether an append sends its destination rows as a list: more runs than travel in the kernel arguments, or more rows than one launch takes.
bool append_as_list(const pasta_attn* h, size_t n_runs, int n_rows, bool rope) {
  return n_runs > (size_t)kAppendRuns || (size_t)n_rows > append_rows_max(h, rope);
}

// Launches K1 for n_rows rows that form the given runs.  positions: rotate K by them.
int launch_append(pasta_attn* h, int layer, int n_rows, const void* k_new, const void* v_new, const std::vector<AppendRun>& runs,
                  const int32_t* positions = nullptr, const ListPatches* patches = nullptr) {
  const pasta_attn_config& c = h->cfg;
  hipStream_t st = (hipStream_t)c.hip_stream;
  AppendParams p{};
  p.arena = (DevRange*)((char*)c.workspace + h->off_arena);
  p.cidx = (int32_t*)((char*)c.workspace + h->off_cidx);
  p.page_table = (const int32_t*)((const char*)c.workspace + h->off_page_table);
  p.k = (char*)c.k_pool + (size_t)layer * h->layer_elems * h->elem;
  p.v = (char*)c.v_pool + (size_t)layer * h->layer_elems * h->elem;
  p.lay = h->lay;
  p.Hkv = c.n_kv_heads;
  p.elem_shift = h->elem == 4 ? 2 : 1;
  while ((16 << p.pph_log2) < c.head_dim * h->elem) p.pph_log2++;
  const size_t row_bytes = (size_t)c.n_kv_heads * c.head_dim * h->elem;
  const bool rope = positions != nullptr;
  p.rope_tab = rope ? (const double*)((const char*)c.workspace + h->off_rope) : nullptr;
  const long long units_per_row = (long long)row_bytes / 16 / (rope ? 2 : 1);
  auto launch = [&](size_t lo, size_t n) -> int {  // rows [lo, lo + n) of the call
    p.n_rows = (int)n;
    p.k_new = (const u32x4*)((const char*)k_new + lo * row_bytes);
    p.v_new = (const u32x4*)((const char*)v_new + lo * row_bytes);
    const long long units = (long long)n * units_per_row;
    const int per = units <= kAppendThin ? 1 : append_units(rope);
    const dim3 grid((unsigned)((units + 256 * per - 1) / (256 * per)));
    if (rope) { if (per == 1) k_append<true, 1><<<grid, 256, 0, st>>>(p); else k_append<true, append_units(true)><<<grid, 256, 0, st>>>(p); }
    else { if (per == 1) k_append<false, 1><<<grid, 256, 0, st>>>(p); else k_append<false, append_units(false)><<<grid, 256, 0, st>>>(p); }
    return hipGetLastError() == hipSuccess ? PASTA_OK : PASTA_E_DEVICE;
  };
  if (!append_as_list(h, runs.size(), n_rows, rope)) {
    p.n_runs = (int)runs.size();
    std::memcpy(p.runs, runs.data(), runs.size() * sizeof(AppendRun));
    if (patches) {
      p.n_rpatch = patches->n_r;
      p.n_cpatch = patches->n_c;
      std::memcpy(p.rp_idx, patches->r_idx, sizeof(int32_t) * patches->n_r);
      std::memcpy(p.rp_val, patches->r_val, sizeof(DevRange) * patches->n_r);
      std::memcpy(p.cp_idx, patches->c_idx, sizeof(int32_t) * patches->n_c);
      std::memcpy(p.cp_val, patches->c_val, sizeof(int32_t) * patches->n_c);
    }
    return launch(0, (size_t)n_rows);
  }
  // the destination rows as a list, in pieces of one staging slot
  std::vector<int32_t>& dst = h->dst_rows;  // (append_kv has reserved it)
  dst.resize((size_t)n_rows);
  for (size_t k = 0; k < runs.size(); ++k) {
    const int32_t end = k + 1 < runs.size() ? runs[k + 1].row0 : n_rows;
    for (int32_t i = runs[k].row0; i < end; ++i) dst[(size_t)i] = (int32_t)host_phys(h, runs[k].req, runs[k].slot0 + (i - runs[k].row0));
  }
  const size_t per = std::min(h->meta_bytes / 4, append_rows_max(h, rope));
  for (size_t lo = 0; lo < (size_t)n_rows; lo += per) {
    const size_t n = std::min(per, (size_t)n_rows - lo);
    int rc = upload_meta(h, dst.data() + lo, n, &p.dst_rows);
    if (rc == PASTA_OK && rope) rc = upload_meta(h, positions + lo, n, &p.pos_rows);
    if (rc == PASTA_OK) rc = launch(lo, n);
    if (rc != PASTA_OK) return rc;
  }
  return PASTA_OK;
}

// Performs a deferred append's copy with K1 (when no decode_step took it along).
int flush_pending(pasta_attn* h) {
  if (!h->pending.active) return PASTA_OK;
  h->pending.active = false;
  return launch_append(h, h->pending.layer, h->pending.n_rows, h->pending.k_new, h->pending.v_new,
                       h->pending.runs, h->pending.rope ? h->pending.pos : nullptr);
}

}  // namespace

// =============================================================================== create
extern "C" int32_t pasta_attn_create(pasta_attn_config* cfg, pasta_attn** out) {
  int rc = validate_cfg(cfg);
  if (rc != PASTA_OK) return rc;
  pasta_attn* h = new (std::nothrow) pasta_attn();
  if (!h) return PASTA_E_NOMEM;
  h->cfg = *cfg;
  h->G = cfg->n_q_heads / cfg->n_kv_heads;
  h->elem = cfg->dtype == PASTA_F32 ? 4 : 2;
  const int64_t D = cfg->head_dim, H = cfg->n_kv_heads;
  if (cfg->page_tokens) {
    h->page_shift = 0;
    while ((1 << h->page_shift) < cfg->page_tokens) h->page_shift++;
    h->rows_per_layer = (int64_t)cfg->n_phys_pages * cfg->page_tokens;
    h->req_capacity = (int64_t)cfg->pages_per_request * cfg->page_tokens;
  } else {
    h->rows_per_layer = (int64_t)cfg->max_requests * cfg->pool_tokens;
    h->req_capacity = cfg->pool_tokens;
  }
  h->layer_elems = h->rows_per_layer * H * D;
  Layout& L = h->lay;
  L.paged = cfg->page_tokens ? 1 : 0;
  L.pages_per_request = cfg->pages_per_request;
  L.pool_tokens = (int)cfg->pool_tokens;
  L.page_shift = cfg->page_tokens ? h->page_shift : 31;
  L.page_mask = cfg->page_tokens ? cfg->page_tokens - 1 : 0x7fffffff;
  if (cfg->kv_layout == PASTA_LAYOUT_TOKEN_MAJOR) {
    L.slot_stride = (int)(H * D);
    L.head_stride = D;
    L.page_stride = cfg->page_tokens ? (int64_t)cfg->page_tokens * H * D : 0;
  } else if (!cfg->page_tokens) {
    L.slot_stride = (int)D;
    L.head_stride = h->rows_per_layer * D;
    L.page_stride = 0;
  } else {
    L.slot_stride = (int)D;
    L.head_stride = (int64_t)cfg->page_tokens * D;
    L.page_stride = (int64_t)cfg->page_tokens * H * D;
  }
  const uint64_t given = cfg->workspace_bytes;
  carve(h);
  if (!out) {  // query mode
    cfg->workspace_bytes = h->cfg.workspace_bytes;
    delete h;
    return PASTA_OK;
  }
  auto fail = [&](int code) { delete h; return code; };
  if (!cfg->k_pool || !cfg->v_pool || !cfg->workspace) return fail(PASTA_E_INVAL);
  if (((uintptr_t)cfg->workspace & 255) || ((uintptr_t)cfg->k_pool & 15) || ((uintptr_t)cfg->v_pool & 15))
    return fail(PASTA_E_INVAL);
  if (given < h->cfg.workspace_bytes) return fail(PASTA_E_CAPACITY);
  h->cfg.workspace_bytes = given;
  if (cfg->page_tokens) {
    if (!cfg->page_table) return fail(PASTA_E_INVAL);
    const size_t n = (size_t)cfg->max_requests * cfg->pages_per_request;
    try {
      h->page_table.assign(cfg->page_table, cfg->page_table + n);
      // a request's assigned pages come first, -1 ("no page") after them; assigned pages must be
      // distinct over the whole table: a page named twice would alias two logical pages
      std::vector<uint8_t> taken((size_t)cfg->n_phys_pages, 0);
      h->req_pages.assign(cfg->max_requests, 0);
      for (int r = 0; r < cfg->max_requests; ++r) {
        bool ended = false;
        for (int k = 0; k < cfg->pages_per_request; ++k) {
          const int32_t pp = h->page_table[(size_t)r * cfg->pages_per_request + k];
          if (pp == -1) { ended = true; continue; }
          if (ended || pp < 0 || pp >= cfg->n_phys_pages || taken[pp]) return fail(PASTA_E_INVAL);
          taken[pp] = 1;
          h->req_pages[r] = k + 1;
        }
      }
    } catch (const std::bad_alloc&) { return fail(PASTA_E_NOMEM); }
    h->cfg.page_table = nullptr;  // the caller's array is not kept
  }
#ifdef PASTA_TUNING  // tuning builds only: forced chunk sizes from the environment
  if (const char* e = std::getenv("PASTA_PREFIX_CHUNK")) h->tune_prefix_chunk = std::atoi(e);
  if (const char* e = std::getenv("PASTA_PRIV_CHUNK")) h->tune_priv_chunk = std::atoi(e);
#endif
  try {
    h->tail.assign(cfg->max_requests, 0);
    h->tail_before.assign(cfg->max_requests, 0);
    h->streams.resize((size_t)cfg->max_requests * cfg->max_streams);
    for (auto* v : {&h->pending.req_pend0, &h->pending.req_src0, &h->pending.stage_p0, &h->pending.stage_s0, &h->pending.stage_last}) v->reserve(cfg->max_requests);
    // plan buffers: what a plan that rides in the kernel arguments can need (larger plans grow them on demand)
    const size_t ns = (size_t)cfg->max_requests * cfg->max_streams, nsc = std::min<size_t>(ns, 65535);
    PlanBuf& pb = h->pb;
    pb.lv.reserve(nsc); pb.mask_base.reserve(nsc); pb.stream_req_idx.reserve(nsc); pb.stream_local.reserve(nsc);
    pb.req_streams.reserve(nsc); pb.streams.reserve(nsc);
    pb.seen.reserve(ns);
    pb.req_idx_of.reserve(cfg->max_requests); pb.reqs.reserve(cfg->max_requests);
    pb.ranges.reserve(std::min<size_t>((size_t)cfg->max_ranges + nsc, kInlineMetaWords));
    pb.items.reserve(kInlineMetaWords / (sizeof(DevItem) / 4));
    pb.blob.reserve(kInlineMetaWords + 16 + (size_t)h->plan_items_cap);  // (and an entry per private item: device-resident lists)
    h->plan_words.reserve(kInlineMetaWords + 16 + (size_t)h->plan_items_cap);
  } catch (...) { return fail(PASTA_E_NOMEM); }
#if defined(PASTA_TUNING) && PASTA_TUNING >= 2
  std::fprintf(stderr, "PASTA_CLOCKS byte offset in workspace: %zu\n", h->off_ml + (size_t)(h->part_rows_cap - 16 * PASTA_CLK_WGS) * 8);
#endif
  *out = h;
  return PASTA_OK;
}

extern "C" int32_t pasta_attn_destroy(pasta_attn* h) {
  if (!h) return PASTA_OK;
  if (h->magic != kMagic) return PASTA_E_STATE;
  if (h->device_ready) (void)flush_pending(h);  // a deferred append still owes its copy
  h->magic = 0;
  for (int i = 0; i < h->ring_ev_made; ++i) (void)hipEventDestroy(h->ring_ev[i]);
  if (h->pinned) (void)hipHostFree(h->pinned);
  if (h->mask_pinned) { (void)hipHostFree(h->mask_pinned); (void)hipEventDestroy(h->mask_ev); }
  delete h;
  return PASTA_OK;
}

// =============================================================================== append
// How many of n entries lead for which differs(k) is 0, looked at 16 at a time without a branch between them (the compiler does that in
// vector registers).  One at a time, these looks were most of a rotated prompt's call: 6480 rows 11.2 or 12.0 us, by where the loop's code
// came to lie, now 3.7; 8192 rows that are not rotated 5.2 or 6.6, now 1.9.  The first kFew rows are looked at one at a time (by the
// caller): the rows of interleaved streams rarely go on for longer.
constexpr int kFew = 32;
template <class Differs>
__attribute__((noinline)) int leading(int n, Differs differs) {
  constexpr int kBlock = 16;
  int k = 0;
  for (; k + kBlock <= n; k += kBlock) {
    uint32_t any = 0;
    for (int j = 0; j < kBlock; ++j) any |= differs(k + j);
    if (any) break;
  }
  while (k < n && !differs(k)) ++k;
  return k;
}

extern "C" int32_t pasta_attn_append_kv(pasta_attn* h, const pasta_append_args* a) {
  if (!h || h->magic != kMagic) return PASTA_E_STATE;
  if (!a || a->struct_size != sizeof(pasta_append_args)) return PASTA_E_INVAL;
  const pasta_attn_config& c = h->cfg;
  if (a->layer < 0 || a->layer >= c.n_layers) return PASTA_E_STATE;
  if (a->n_rows < 0) return PASTA_E_INVAL;
  if (a->n_rows == 0) return PASTA_OK;
  const bool reserve_only = a->flags & PASTA_APPEND_RESERVE_ONLY;
  if (!a->request_id || !a->stream_id) return PASTA_E_INVAL;
  if (!reserve_only && (!a->k_new || !a->v_new)) return PASTA_E_INVAL;
  if (!reserve_only && (((uintptr_t)a->k_new & 15) || ((uintptr_t)a->v_new & 15))) return PASTA_E_INVAL;
  const bool rope = a->flags & PASTA_APPEND_ROPE;
  if (rope) {
    if (reserve_only || !a->position || !(c.rope_theta > 0.f)) return PASTA_E_INVAL;
    int32_t all = 0;  // (negative if one of them is; no exit within, so that the compiler takes several at once)
    for (int i = 0; i < a->n_rows; ++i) all |= a->position[i];
    if (all < 0) return PASTA_E_INVAL;
  }
  const bool commit = a->layer == 0;  // layer 0 assigns the slots; other layers replay them

  // ---- the rows, one by one, on the live state; what a failing call has to put back is logged
  // (per touched stream: its state at first touch -- an append only ever changes a list's newest range
  // or adds ranges behind it)
  std::vector<int64_t>& t2 = h->t2;
  std::vector<AppendRun>& runs = h->runs;
  std::vector<pasta_attn::Undo>& undo = h->undo;
  auto roll_back = [&]() {
    for (size_t u = undo.size(); u-- > 0;) {
      pasta_attn::Undo& e = undo[u];
      StreamState& st = h->streams[(size_t)e.key];
      if (e.replaced) st.ranges = std::move(e.saved);
      st.ranges.resize((size_t)e.n_ranges);
      if (e.n_ranges) st.ranges.back() = e.last;
      st.open = e.open; st.prefix_len = e.prefix_len; st.range_tokens = e.range_tokens;
      st.dev_ranges = e.dev_ranges; st.dev_cidx = e.dev_cidx; st.dirty = e.dirty;
    }
    undo.clear();
  };
  try {
    t2 = commit ? h->tail : h->tail_before;
    runs.clear();
    undo.clear();
    auto touch = [&](int req, int sid) -> StreamState& {  // logs the stream's state the first time it is touched
      const int64_t key = (int64_t)req * c.max_streams + sid;
      StreamState& st = h->streams[(size_t)key];
      for (const auto& e : undo)
        if (e.key == key) return st;
      pasta_attn::Undo e{};
      e.key = key; e.open = st.open; e.prefix_len = st.prefix_len; e.n_ranges = (int32_t)st.ranges.size();
      if (e.n_ranges) e.last = st.ranges.back();
      e.range_tokens = st.range_tokens; e.dev_ranges = st.dev_ranges; e.dev_cidx = st.dev_cidx; e.dirty = st.dirty;
      undo.push_back(std::move(e));
      return st;
    };
    auto fail = [&](int code) { roll_back(); return code; };
    // rows are taken in groups: one stream's consecutive rows, of which only the first may open it
    for (int i = 0, end; i < a->n_rows; i = end) {
      const int r = a->request_id[i], s = a->stream_id[i];
      const int par = a->parent_stream ? a->parent_stream[i] : -1;
      if (r < 0 || r >= c.max_requests || s < 0 || s >= c.max_streams) return fail(PASTA_E_INVAL);
      if (par < -1 || par >= c.max_streams || par == s) return fail(PASTA_E_INVAL);
      end = i + 1;
      for (const int few = std::min(a->n_rows, i + kFew); end < few && a->request_id[end] == r && a->stream_id[end] == s && (!a->parent_stream || a->parent_stream[end] == -1);) end++;
      if (end == i + kFew) {
        const int32_t *const reqs = a->request_id + end, *const sids = a->stream_id + end, *const pars = a->parent_stream ? a->parent_stream + end : nullptr;
        end += leading(a->n_rows - end, [=](int k) { return (uint32_t)((reqs[k] ^ r) | (sids[k] ^ s) | (pars ? ~pars[k] : 0)); });
      }
      const int n_g = end - i;
      const int64_t slot = t2[r];
      const int64_t room = c.page_tokens ? (int64_t)h->req_pages[r] << h->page_shift : h->req_capacity;
      if (slot >= room) return fail(PASTA_E_CAPACITY);  // (the errors are those of the first row that cannot be taken)
      t2[r] = slot + n_g;
      // the copy's runs: one as long as the request stays the same (and the position ids go on by one)
      for (int k = i; k < end;) {
        int ke = end;
        if (rope) {
          const int few = std::min(end, k + kFew);
          for (ke = k + 1; ke < few && a->position[ke] == a->position[ke - 1] + 1;) ke++;
          if (ke == k + kFew) {
            const int32_t* const pos = a->position + ke;
            ke += leading(end - ke, [=](int j) { return (uint32_t)pos[j] ^ ((uint32_t)pos[-1] + 1u + (uint32_t)j); });
          }
        }
        if (k == 0 || a->request_id[k - 1] != r || (rope && a->position[k] != a->position[k - 1] + 1))
          runs.push_back(AppendRun{k, r, (int32_t)(slot + (k - i)), rope ? a->position[k] : 0});
        k = ke;
      }
      if (!commit) {  // replay: same slots as the layer-0 call, lists untouched
        if (slot + n_g > h->tail[r]) return fail(h->tail[r] >= room ? PASTA_E_CAPACITY : PASTA_E_STATE);
        continue;
      }
      StreamState& st = touch(r, s);
      if (par >= 0 || !st.open) {  // the first row opens the stream: as a fork of `par`, or as a root (empty visible set)
        if (par >= 0 && st.open) return fail(PASTA_E_INVAL);  // parent only on the row that opens the stream
        const StreamState* ps = nullptr;
        if (par >= 0) {
          ps = &sstate(h, r, par);
          if (!ps->open) return fail(PASTA_E_INVAL);
        }
        pasta_attn::Undo* ue = nullptr;
        for (auto& e : undo)
          if (e.key == (int64_t)r * c.max_streams + s) ue = &e;
        if (!ue->replaced) { ue->replaced = true; ue->saved = std::move(st.ranges); st.ranges.clear(); }
        if (ps) {  // ancestor rule: inherit what the parent sees now
          st.prefix_len = ps->prefix_len;
          st.ranges = ps->ranges;
          st.range_tokens = ps->range_tokens;
        } else {
          st.prefix_len = 0;
          st.ranges.clear();
          st.range_tokens = 0;
        }
        st.open = true;
        st.dirty = true;  // the device copy is rebuilt from the mirror when a decode step wants it
        st.dev_ranges = st.dev_cidx = 0;
      }
      if (slot + n_g > room) return fail(PASTA_E_CAPACITY);
      add_slots(st, (int32_t)slot, n_g);
      if ((int64_t)st.ranges.size() > c.max_ranges) return fail(PASTA_E_CAPACITY);
    }
    if (!reserve_only && append_as_list(h, runs.size(), a->n_rows, rope)) h->dst_rows.reserve((size_t)a->n_rows);  // (the launch below must not throw)
  } catch (...) { roll_back(); return PASTA_E_NOMEM; }

  // ---- what the call changes in the device-resident lists.  A stream whose ranges only GREW needs
  // nothing (its newest range rides with every decode call, and index entries that are not on the device
  // mean "the newest range").  A stream that got NEW ranges has its arena and index entries brought up to
  // date by this call's K1 launch when they are few and the launch exists; otherwise its copy is marked
  // for a rebuild.
  ListPatches patches;
  bool need_k1 = false;  // patches exist: the copy cannot be left to a later decode launch
  if (commit) {
    const bool k1_possible = !reserve_only && a->n_rows <= kAppendInline;
    for (auto& e : undo) {
      StreamState& st = h->streams[(size_t)e.key];
      const int32_t nb = e.n_ranges, na = (int32_t)st.ranges.size();
      if (st.dirty) continue;
      if (!h->lists_in_use) {  // no step has read the device copy so far: nothing to keep current
        if (na != nb) st.dirty = true;
        continue;
      }
      if (na == nb) {  // growth only
        st.dev_ranges = std::min(st.dev_ranges, std::max(na - 1, 0));
        continue;
      }
      const int64_t n_cidx = (st.range_tokens + kCidxTokens - 1) / kCidxTokens;
      const int32_t k0 = std::min(st.dev_ranges, std::max(nb - 1, 0));  // first arena entry to (re)write
      const int64_t want_r = na - k0, want_c = n_cidx - st.dev_cidx;
      if (!k1_possible || na > st.seg_cap || n_cidx > st.cseg_cap || patches.n_r + want_r > kPatchMax ||
          patches.n_c + want_c > kPatchMax) {
        st.dirty = true;
        continue;
      }
      int64_t cum = st.range_tokens;  // tokens before range k, walking down from the end
      for (int32_t k = na - 1; k >= k0; --k) cum -= st.ranges[k].count;
      int64_t tok = (int64_t)st.dev_cidx * kCidxTokens;  // next index entry's token (lies at or behind range k0's start)
      for (int32_t k = k0; k < na; ++k) {
        const Range& g = st.ranges[k];
        patches.r_idx[patches.n_r] = st.seg_off + k;
        patches.r_val[patches.n_r++] = DevRange{g.start, g.count, g.stride, (int32_t)cum};
        for (; tok < cum + g.count && tok < st.range_tokens; tok += kCidxTokens) {
          patches.c_idx[patches.n_c] = st.cseg_off + (int32_t)(tok / kCidxTokens);
          patches.c_val[patches.n_c++] = k;
        }
        cum += g.count;
      }
      st.dev_ranges = na;
      st.dev_cidx = (int32_t)n_cidx;
      need_k1 = true;
    }
  }

  // ---- enqueue K1, or leave the copy to the next decode_step (PASTA_APPEND_DEFER)
  int rc = PASTA_OK;
  bool runs_left_to_pending = false;
  auto fail_dev = [&](int code) { if (commit) roll_back(); return code; };
  // At most one deferred append is outstanding, and the slots it covers are the newest of their
  // requests: any later append -- also one that only reserves slots for the caller's own kernel --
  // first sends the deferred rows to the pool (a deferred append exists only on a ready device).
  rc = flush_pending(h);
  if (rc != PASTA_OK) return fail_dev(rc);
  if (!reserve_only) {
    rc = ensure_device(h);
    if (rc != PASTA_OK) return fail_dev(rc);
    bool defer = (a->flags & PASTA_APPEND_DEFER) && a->n_rows <= kAppendInline && !need_k1;
    std::vector<int32_t>&p0 = h->pending.stage_p0, &s0 = h->pending.stage_s0;
    if (defer) {  // rows of one request must be consecutive in the call: slot t <-> row src0 + (t - pend0)
      p0.assign(c.max_requests, INT32_MAX);
      s0.assign(c.max_requests, 0);
      std::vector<int32_t>& last = h->pending.stage_last;
      last.assign(c.max_requests, -2);
      for (size_t k = 0; k < runs.size() && defer; ++k) {
        const AppendRun& rn = runs[k];
        if (p0[rn.req] == INT32_MAX) { p0[rn.req] = rn.slot0; s0[rn.req] = rn.row0; }
        else if (last[rn.req] != rn.row0 - 1) defer = false;
        last[rn.req] = (k + 1 < runs.size() ? runs[k + 1].row0 : a->n_rows) - 1;
      }
    }
    if (defer) {
      pasta_attn::Pending& pd = h->pending;
      pd.active = true;
      pd.layer = a->layer;
      pd.n_rows = a->n_rows;
      pd.k_new = a->k_new;
      pd.v_new = a->v_new;
      pd.runs.swap(runs);
      for (size_t k = 0; k < pd.runs.size(); ++k) {
        const AppendRun& rn = pd.runs[k];
        const int32_t end = k + 1 < pd.runs.size() ? pd.runs[k + 1].row0 : a->n_rows;
        for (int32_t i = rn.row0; i < end; ++i) pd.dst_rows[i] = (int32_t)host_phys(h, rn.req, rn.slot0 + (i - rn.row0));
      }
      pd.rope = rope;
      if (rope) std::memcpy(pd.pos, a->position, (size_t)a->n_rows * 4);
      pd.req_pend0.swap(p0);
      pd.req_src0.swap(s0);
      runs_left_to_pending = true;
    } else {
      rc = launch_append(h, a->layer, a->n_rows, a->k_new, a->v_new, runs, rope ? a->position : nullptr,
                         need_k1 ? &patches : nullptr);
      if (rc != PASTA_OK) return fail_dev(rc);
    }
  }

  // ---- commit
  if (a->out_slot) {
    const std::vector<AppendRun>& rs = runs_left_to_pending ? h->pending.runs : runs;
    for (size_t k = 0; k < rs.size(); ++k)
      for (int32_t i = rs[k].row0, end = k + 1 < rs.size() ? rs[k + 1].row0 : a->n_rows; i < end; ++i) a->out_slot[i] = rs[k].slot0 + (i - rs[k].row0);
  }
  if (commit) {
    h->lists_epoch++;
    h->tail_before = h->tail;
    h->tail.swap(t2);
    undo.clear();
  }
  return PASTA_OK;
}

// =============================================================================== sync
// Union of visible sets, rebuilt slot by slot in ascending order so that the result is in the
// same canonical form as a list grown by appends (contiguous head in prefix_len, then strided
// descriptors).  Host work proportional to the number of visible slots; a sync is rare.
extern "C" int32_t pasta_attn_sync(pasta_attn* h, const pasta_sync_args* a) {
  if (!h || h->magic != kMagic) return PASTA_E_STATE;
  if (!a || a->struct_size != sizeof(pasta_sync_args)) return PASTA_E_INVAL;
  const pasta_attn_config& c = h->cfg;
  const bool retire = a->flags & PASTA_SYNC_RETIRE;
  if (a->request_id < 0 || a->request_id >= c.max_requests) return PASTA_E_INVAL;
  if (a->n_join < 1 || !a->join_stream) return PASTA_E_INVAL;
  if (a->stream_id < -1 || a->stream_id >= c.max_streams || (a->stream_id == -1 && !retire)) return PASTA_E_INVAL;
  for (int i = 0; i < a->n_join; ++i) {
    const int j = a->join_stream[i];
    if (j < 0 || j >= c.max_streams || j == a->stream_id) return PASTA_E_INVAL;
    for (int k = 0; k < i; ++k)
      if (a->join_stream[k] == j) return PASTA_E_INVAL;
    if (!sstate(h, a->request_id, j).open) return PASTA_E_STATE;
  }
  h->lists_epoch++;
  try {
    if (a->stream_id >= 0) {
      StreamState& dst = sstate(h, a->request_id, a->stream_id);
      if (!dst.open) return PASTA_E_STATE;
      // k-way merge of the lists' slots (each list ascending), duplicates dropped
      struct Cursor { const StreamState* s; int64_t next; size_t ri; int32_t k; };  // next < prefix_len: in the head
      std::vector<Cursor> cur;
      cur.push_back({&dst, 0, 0, 0});
      for (int i = 0; i < a->n_join; ++i) cur.push_back({&sstate(h, a->request_id, a->join_stream[i]), 0, 0, 0});
      auto peek = [](const Cursor& q) -> int64_t {
        if (q.next < q.s->prefix_len) return q.next;
        if (q.ri < q.s->ranges.size()) return (int64_t)q.s->ranges[q.ri].start + (int64_t)q.k * q.s->ranges[q.ri].stride;
        return INT64_MAX;
      };
      auto advance = [](Cursor& q) {
        if (q.next < q.s->prefix_len) { q.next++; return; }
        if (++q.k >= q.s->ranges[q.ri].count) { q.k = 0; q.ri++; }
      };
      // the common head [0, min prefix_len) needs no merging
      int64_t head = INT64_MAX;
      for (auto& q : cur) head = std::min<int64_t>(head, q.s->prefix_len);
      StreamState merged;
      merged.open = true;
      merged.prefix_len = (int32_t)head;
      for (auto& q : cur) q.next = head;
      for (;;) {
        int64_t lo = INT64_MAX;
        for (auto& q : cur) lo = std::min(lo, peek(q));
        if (lo == INT64_MAX) break;
        add_slot(merged, (int32_t)lo);
        for (auto& q : cur)
          if (peek(q) == lo) advance(q);
        if ((int64_t)merged.ranges.size() > c.max_ranges) return PASTA_E_CAPACITY;
      }
      merged.range_tokens = 0;
      for (const Range& g : merged.ranges) merged.range_tokens += g.count;
      merged.seg_off = dst.seg_off; merged.seg_cap = dst.seg_cap;      // the device copy keeps its segments
      merged.cseg_off = dst.cseg_off; merged.cseg_cap = dst.cseg_cap;  // and is rebuilt from the joined list
      dst = std::move(merged);                                         // when a decode step next wants it
    }
    if (retire)
      for (int i = 0; i < a->n_join; ++i) {
        StreamState& js = sstate(h, a->request_id, a->join_stream[i]);
        js.open = false;
        js.prefix_len = 0;
        js.ranges.clear();
        js.range_tokens = 0;
        js.dirty = true;
        js.dev_ranges = js.dev_cidx = 0;
      }
  } catch (const std::bad_alloc&) {
    return PASTA_E_NOMEM;
  }
  return PASTA_OK;
}

extern "C" int32_t pasta_attn_stream_list(pasta_attn* h, int32_t request_id, int32_t stream_id, int32_t* prefix_len,
                                          int32_t* n_ranges, int32_t cap, int32_t* start, int32_t* count,
                                          int32_t* stride) {
  if (!h || h->magic != kMagic) return PASTA_E_STATE;
  const pasta_attn_config& c = h->cfg;
  if (request_id < 0 || request_id >= c.max_requests || stream_id < 0 || stream_id >= c.max_streams) return PASTA_E_INVAL;
  if (!prefix_len || !n_ranges || cap < 0 || (cap > 0 && (!start || !count || !stride))) return PASTA_E_INVAL;
  const StreamState& s = sstate(h, request_id, stream_id);
  if (!s.open) return PASTA_E_STATE;
  *prefix_len = s.prefix_len;
  *n_ranges = (int32_t)s.ranges.size();
  for (int32_t k = 0; k < cap && k < (int32_t)s.ranges.size(); ++k) {
    start[k] = s.ranges[k].start;
    count[k] = s.ranges[k].count;
    stride[k] = s.ranges[k].stride;
  }
  return PASTA_OK;
}

// =============================================================================== decode
namespace {

// The scratch of the entry point that allocates nothing: partial (m, l) and accumulator rows of one
// decode step.  One array per GPU that the library runs on, held until the process ends; host code
// reaches it only through the address that hipGetSymbolAddress returns for the current device.
constexpr size_t kScratchBytes = (size_t)16 << 20;
constexpr int kMaxDevices = 64;
static __device__ __align__(256) unsigned char scratch[kScratchBytes];
void* g_scratch_ptr[kMaxDevices] = {};

// Steps that k_one takes: every stream sees few enough bytes of K and V per kv head that one CU reads them sooner than the
// merge launch (and, with rotary embedding ahead of k_attn, the small launch for it) takes.  One launch takes longer with the
// list -- by rounds of eight waves' blocks -- and hardly with anything else.  The split form takes longer with a second stream, and
// with more than 16 rows stacked over a shared prefix, where k_direct computes two row tiles.  Hence a line per kind and column:
// [one stream, or few (stream, kv head) pairs; others; others of more than 16 stacked rows].  Each lies where both forms take about
// the same time on the device -- the mean of warm pools and of pools that come from HBM -- and called eagerly one launch is
// still some twentieth the sooner one.  The measured lists next to each line, append and decode step of a layer, 8 kv heads of 4 query
// heads, 20 .. 60 own tokens per stream: tokens: us split / one, replayed graphs of 16 warm layers (of 600 MB of layers) [called]
//                  1 stream                                      3 streams                                     8 streams
//   bf16 x 128     384: 7.0 / 7.4 (7.8 / 8.0) [7.8 / 7.7]        512: 9.7 / 9.4 (9.9 / 10.2) [10.3 / 9.3]      512: 10.3 / 9.5 (11.0 / 10.5) [10.1 / 9.2]
//                  448: 7.4 / 8.5 (8.0 / 9.0) [7.9 / 8.5]        576: 9.8 / 10.1 (10.0 / 11.2) [10.4 / 10.1]   576: 10.3 / 10.2 (11.0 / 11.3) [10.1 / 10.0]
//    rotated       512: 10.6 / 10.2 (10.7 / 10.6) [10.8 / 10.0]  768: 12.8 / 12.7 (13.6 / 14.3) [13.7 / 12.6]  768: 13.3 / 12.9 (14.3 / 14.3) [14.1 / 12.7]
//                  576: 11.0 / 10.8 (11.0 / 11.9) [10.9 / 10.6]  832: 12.9 / 13.3 (13.8 / 15.1) [13.8 / 13.1]  (plans too large)
//   bf16 x 64      768: 6.6 / 7.8 (7.7 / 8.2) [7.6 / 8.2]        768: 8.1 / 8.3 (8.4 / 8.5) [9.3 / 9.0]        768: 9.1 / 8.8 (9.5 / 9.0) [10.1 / 9.3]
//    rotated       960: 10.8 / 10.8 (11.1 / 11.0) [11.5 / 10.8]  960: 11.6 / 11.1 (11.7 / 11.4) [12.3 / 11.1]  768: 12.4 / 9.8 (12.8 / 10.2) [13.2 / 9.8]
//   fp32 x 128      96: 7.8 / 6.6 (8.9 / 7.1) [9.3 / 7.8]        192: 9.5 / 9.6 (9.8 / 9.8) [10.3 / 9.8]       288: 13.2 / 12.7 (13.9 / 13.2) [13.5 / 12.5]
//                  128: 8.1 / 6.9 (8.9 / 7.2) [9.6 / 8.1]        224: 9.9 / 11.2 (10.0 / 11.4) [10.5 / 11.1]   320: 13.2 / 13.0 (13.8 / 13.7) [13.5 / 12.9]
//    rotated       256: 12.2 / 11.9 (12.5 / 12.4) [12.7 / 11.9]  256: 13.5 / 12.7 (13.8 / 13.4) [13.8 / 12.6]  416: 19.4 / 17.4 (20.2 / 18.5) [19.4 / 17.2]
//                  288: 12.2 / 13.9 (12.5 / 14.5) [12.6 / 13.9]  288: 13.4 / 14.1 (14.1 / 14.9) [13.9 / 14.0]  448: 19.5 / 17.8 (20.3 / 18.9) [19.6 / 17.6]
//   fp32 x 64      224: 7.5 / 7.0 (8.6 / 7.3) [9.3 / 8.1]        288: 8.2 / 8.6 (9.3 / 9.0) [10.3 / 9.3]       448: 11.4 / 11.5 (12.0 / 12.0) [11.8 / 11.4]
//                  256: 7.6 / 7.1 (8.6 / 7.5) [9.3 / 8.1]        320: 8.1 / 8.8 (9.3 / 9.2) [10.2 / 9.5]       480: 11.4 / 11.5 (12.3 / 12.0) [11.9 / 11.5]
//    rotated       384: 10.4 / 10.4 (11.6 / 11.0) [11.9 / 10.8]  448: 12.2 / 12.5 (12.5 / 12.7) [12.9 / 12.4]  512: 14.1 / 13.3 (15.1 / 14.3) [14.3 / 13.1]
//                  416: 10.3 / 11.6 (11.3 / 12.2) [12.0 / 12.0]  480: 12.4 / 12.6 (12.6 / 13.4) [12.8 / 12.5]  544: 14.0 / 14.5 (15.1 / 15.3) [14.3 / 14.3]
// (the first column's plain lines are older than the table: bf16 x 64 past, fp32 short of where both are even.)  More pairs do not
// count: 4 streams x 16 heads are as 3 x 8 (fp32 x 128 over 288 10.2 / 12.5, 8 streams x 8 heads 13.2 / 12.7), one stream of 32 heads as one
// of 8 (bf16 x 128 over 448 8.6 / 9.3).  8 query heads per kv head: 3 streams as 8 of 4 (fp32 x 64 over 384 10.8 / 9.4).  Six requests of
// one stream: better than 3 streams (bf16 x 128 over 576 11.3 / 10.1).  One kv head: as 8 (bf16 x 128 over 500, called, 1 stream 8.1 / 8.5, 4
// streams 9.8 / 8.9): few pairs of several streams stay in the first column, on the safe side.
constexpr int kFewPairs = 24, kOneRowTile = 16;
constexpr int kOneKiB[4][2][3] = {  // [bf16 x 128, bf16 x 64, fp32 x 128, fp32 x 64][rotated][column]
    {{192, 272, 288}, {272, 384, 384}},
    {{192, 192, 208}, {240, 240, 240}},
    {{112, 192, 288}, {256, 256, 416}},
    {{112, 144, 224}, {192, 224, 256}},
};
bool small_step(const pasta_attn* h, const pasta_decode_args* a, const std::vector<ListView>& lv, const std::vector<DevReq>& reqs) {
  const pasta_attn_config& c = h->cfg;
  const int n = a->n_streams;
  // what asks for a certain form, its partials or a plan alone gets the split one
  if ((a->flags & ~(uint32_t)(PASTA_DECODE_ROPE_Q)) || a->dbg_part_ml) return false;
  if (n * c.n_kv_heads > h->n_cus) return false;
  const bool rope = (a->flags & PASTA_DECODE_ROPE_Q) || (h->pending.active && h->pending.rope);
  int stacked = 0;  // most rows over one shared prefix
  for (const DevReq& q : reqs)
    if (q.pc >= kTile) stacked = std::max(stacked, q.n_streams * h->G);
  const int column = n == 1 || n * c.n_kv_heads < kFewPairs ? 0 : stacked <= kOneRowTile ? 1 : 2;
  int64_t most = kOneKiB[(c.dtype == PASTA_F32 ? 2 : 0) + (c.head_dim == 64 ? 1 : 0)][rope ? 1 : 0][column];
  most = std::min<int64_t>(kOneTokens, (most << 10) / ((int64_t)c.head_dim * h->elem * 2));
  int64_t words = (int64_t)n * (sizeof(DevStream) / 4 + 1) + (int64_t)reqs.size() * (sizeof(DevReq) / 4) + 16;  // of the split plan at least: it has to ride in the kernel arguments
  for (int i = 0; i < n; ++i) {
    const ListView& v = lv[i];
    if (v.prefix_len > most || v.n_ranges >= kGatherMax) return false;
    int64_t seen = v.prefix_len;
    for (int k = 0; k < v.n_ranges; ++k) seen += v.at(k).count;
    if (seen > most) return false;
    words += ((int64_t)v.n_ranges + 1) * (sizeof(DevRange) / 4) + (seen + 127) / 128 * (sizeof(DevItem) / 4);
  }
  if (words > kInlineMetaWords) return false;
  // results are written while other work-groups still read: only where they lie apart from what is read
  // (Q itself excepted, whose rows a work-group has read before it writes the same rows), in whole pieces
  const size_t out_bytes = (size_t)n * c.n_q_heads * c.head_dim * h->elem, lse_bytes = (size_t)n * c.n_q_heads * sizeof(float);
  auto apart = [](const void* x, size_t nx, const void* y, size_t ny) {
    return !x || !y || (uintptr_t)x + nx <= (uintptr_t)y || (uintptr_t)y + ny <= (uintptr_t)x;
  };
  if ((uintptr_t)a->out & 15) return false;
  if (a->out != a->q && !apart(a->out, out_bytes, a->q, out_bytes)) return false;
  if (!apart(a->out_lse, lse_bytes, a->q, out_bytes)) return false;
  if (h->pending.active) {
    const size_t pend_bytes = (size_t)h->pending.n_rows * c.n_kv_heads * c.head_dim * h->elem;
    for (const void* src : {(const void*)h->pending.k_new, (const void*)h->pending.v_new})
      if (!apart(a->out, out_bytes, src, pend_bytes) || !apart(a->out_lse, lse_bytes, src, pend_bytes)) return false;
  }
  return true;
}

// `no_alloc`: the partials go to the static scratch array instead of the workspace, and the call
// must get by without any allocation, device or host (see pasta_attn_decode_step_noalloc).
int32_t decode_impl(pasta_attn* h, const pasta_decode_args* a, const bool no_alloc) {
  if (!h || h->magic != kMagic) return PASTA_E_STATE;
  if (!a || a->struct_size != sizeof(pasta_decode_args)) return PASTA_E_INVAL;
  const pasta_attn_config& c = h->cfg;
  if (a->layer < 0 || a->layer >= c.n_layers) return PASTA_E_STATE;
  const int n = a->n_streams;
  if (n < 1 || n > c.max_requests * c.max_streams) return PASTA_E_INVAL;
  if (n > 65535) return PASTA_E_CAPACITY;  // one grid dimension of the merge launch counts the query rows
  if (!a->request_id || !a->stream_id) return PASTA_E_INVAL;
  const bool plan_only = a->flags & PASTA_DECODE_PLAN_ONLY;
  if (!plan_only && (!a->q || !a->out)) return PASTA_E_INVAL;
  if (!plan_only && (((uintptr_t)a->q & 15) || ((uintptr_t)a->out & 3))) return PASTA_E_INVAL;
  const bool rope_q = a->flags & PASTA_DECODE_ROPE_Q;
  if (rope_q) {
    if (!a->position || !(c.rope_theta > 0.f)) return PASTA_E_INVAL;
    for (int i = 0; i < n; ++i)
      if (a->position[i] < 0) return PASTA_E_INVAL;
  }
  const bool explicit_mode = a->range_offsets != nullptr;
  if (explicit_mode && !a->prefix_len) return PASTA_E_INVAL;
  if (explicit_mode && a->causal_skip) return PASTA_E_INVAL;  // the lists say it all there
  const bool no_share = a->flags & (PASTA_DECODE_NO_SHARE | PASTA_DECODE_DENSE_MASK);
  const bool dense = a->flags & PASTA_DECODE_DENSE_MASK;
  const bool probe = a->flags & PASTA_DECODE_READ_PROBE;
  const bool partials_only = a->flags & PASTA_DECODE_PARTIALS_ONLY, merge_only = a->flags & PASTA_DECODE_MERGE_ONLY;
  if ((partials_only && merge_only) || ((partials_only || merge_only) && probe)) return PASTA_E_INVAL;
  if ((a->dbg_part_ml == nullptr) != (a->dbg_part_acc == nullptr)) return PASTA_E_INVAL;
  if (a->dbg_part_ml && (no_alloc || ((uintptr_t)a->dbg_part_ml & 7) || ((uintptr_t)a->dbg_part_acc & 15))) return PASTA_E_INVAL;
  if (probe && (dense || no_alloc || (a->flags & PASTA_DECODE_NO_MFMA))) return PASTA_E_INVAL;
  if (dense && (c.dtype != PASTA_BF16 || c.head_dim != 128 || (a->flags & PASTA_DECODE_NO_MFMA))) return PASTA_E_INVAL;
  const int G = h->G, D = c.head_dim, Hkv = c.n_kv_heads;
  float2* part_ml = nullptr;   // where this call's partials go
  float* part_acc = nullptr;
  int64_t part_rows_cap = h->part_rows_cap;
  if (no_alloc) {
    // nothing here may allocate: the handle must have been through its set-up (any append_kv does
    // that), the plan must fit the kernel arguments, and the comparison mode with its host staging is out
    if (plan_only || dense) return PASTA_E_INVAL;
    if (!h->device_ready) return PASTA_E_STATE;
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) { (void)hipGetLastError(); return PASTA_E_DEVICE; }
    if (!g_scratch_ptr[dev]) {  // once per device, with that device current
      void* ptr = nullptr;
      if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) { (void)hipGetLastError(); return PASTA_E_DEVICE; }
      g_scratch_ptr[dev] = ptr;
    }
    part_rows_cap = (int64_t)(kScratchBytes / (sizeof(float2) + (size_t)D * sizeof(float)));
    part_ml = (float2*)g_scratch_ptr[dev];
    part_acc = (float*)((char*)g_scratch_ptr[dev] + align_up((size_t)part_rows_cap * sizeof(float2), 256));
    part_rows_cap -= 64;  // (the alignment gap between the two arrays)
  } else if (!plan_only) {  // before planning: the plan is sized to the device's compute-unit count
    const int rc0 = ensure_device(h);
    if (rc0 != PASTA_OK) return rc0;
    part_ml = (float2*)((char*)c.workspace + h->off_ml);
    part_acc = (float*)((char*)c.workspace + h->off_acc);
    if (a->dbg_part_ml) { part_ml = (float2*)a->dbg_part_ml; part_acc = a->dbg_part_acc; }
  }
  // a buffer of the plan may grow only where allocation is allowed
  auto room = [&](const auto& v, size_t want) { return !no_alloc || want <= v.capacity(); };

  try {
    // ---- lists + validation
    PlanBuf& pb = h->pb;
    if (!room(pb.lv, n) || !room(pb.mask_base, n) || !room(pb.stream_req_idx, n) || !room(pb.streams, n)) return PASTA_E_CAPACITY;
    std::vector<ListView>& lv = pb.lv;
    lv.resize(n);
    std::vector<Range>& trim = pb.trim;    // storage of the views that causal_skip shortens (stable: never past its reserve)
    trim.clear();
    if (a->causal_skip && trim.capacity() < (size_t)c.max_ranges) {
      if (no_alloc) return PASTA_E_CAPACITY;
      trim.reserve((size_t)c.max_ranges);
    }
    std::vector<uint8_t>& seen = pb.seen;
    seen.assign((size_t)c.max_requests * c.max_streams, 0);  // (reserved at create)
    int64_t total_ranges = 0;
    for (int i = 0; i < n; ++i) {
      const int r = a->request_id[i], s = a->stream_id[i];
      if (r < 0 || r >= c.max_requests || s < 0 || s >= c.max_streams) return PASTA_E_INVAL;
      uint8_t& sn = seen[(size_t)r * c.max_streams + s];
      if (sn && !explicit_mode && !a->causal_skip) return PASTA_E_INVAL;  // one query token per stream, unless said otherwise
      sn = 1;
      ListView& v = lv[i];
      if (explicit_mode) {
        const int32_t r0 = a->range_offsets[i], r1 = a->range_offsets[i + 1];
        if (r0 < 0 || r1 < r0 || (i == 0 && r0 != 0)) return PASTA_E_INVAL;
        if (r1 > r0 && (!a->range_start || !a->range_count || !a->range_stride)) return PASTA_E_INVAL;
        v = ListView{a->prefix_len[i], nullptr, r1 - r0, a->range_start + r0, a->range_count + r0,
                     a->range_stride + r0, 0};
        const int64_t tail = h->tail[r];
        if (v.prefix_len < 0 || v.prefix_len > tail) return PASTA_E_INVAL;
        int64_t last = (int64_t)v.prefix_len - 1;
        for (int k = 0; k < v.n_ranges; ++k) {
          const Range g = v.at(k);
          if (g.count < 1 || g.stride < 1 || g.start <= last) return PASTA_E_INVAL;
          last = (int64_t)g.start + (int64_t)(g.count - 1) * g.stride;
          if (last >= tail) return PASTA_E_INVAL;
          v.range_tokens += g.count;
        }
        if (v.prefix_len == 0 && v.n_ranges == 0) return PASTA_E_INVAL;
      } else {
        const StreamState& ss = sstate(h, r, s);
        if (!ss.open) return PASTA_E_STATE;
        v = ListView{ss.prefix_len, ss.ranges.data(), (int32_t)ss.ranges.size(), nullptr, nullptr, nullptr, ss.range_tokens};
        const int skip = a->causal_skip ? a->causal_skip[i] : 0;
        if (skip < 0) return PASTA_E_INVAL;
        if (skip > 0) {  // a view without the stream's `skip` newest rows: they are the largest slots of its list
          if (trim.size() + ss.ranges.size() > (size_t)c.max_ranges) return PASTA_E_CAPACITY;
          const size_t t0 = trim.size();
          trim.insert(trim.end(), ss.ranges.begin(), ss.ranges.end());
          int left = skip;
          while (left > 0 && trim.size() > t0) {
            const int take = std::min(left, trim.back().count);
            trim.back().count -= take;
            left -= take;
            if (trim.back().count == 0) trim.pop_back();
          }
          if (left > ss.prefix_len) return PASTA_E_INVAL;
          v = ListView{ss.prefix_len - left, trim.data() + t0, (int32_t)(trim.size() - t0), nullptr, nullptr, nullptr, ss.range_tokens - (skip - left)};
        }
        if (v.prefix_len == 0 && v.n_ranges == 0) return PASTA_E_INVAL;
      }
      total_ranges += v.n_ranges;
    }
    if (total_ranges > c.max_ranges) return PASTA_E_CAPACITY;

    // ---- dense-mask comparison mode: the lists become one 0/1 byte per (stream, slot), and every
    // stream's list becomes "all slots of its request"
    std::vector<uint8_t>& mask = pb.mask;
    std::vector<int32_t>& mask_base = pb.mask_base;
    mask_base.assign(n, 0);
    if (dense) {
      size_t total = 0;
      for (int i = 0; i < n; ++i) {
        mask_base[i] = (int32_t)total;
        total += (size_t)h->tail[a->request_id[i]];
      }
      if (total + 256 > h->mask_bytes) return PASTA_E_CAPACITY;
      mask.assign(total + 256, 0);
      for (int i = 0; i < n; ++i) {
        uint8_t* m = mask.data() + mask_base[i];
        std::memset(m, 1, (size_t)lv[i].prefix_len);
        for (int k = 0; k < lv[i].n_ranges; ++k) {
          const Range g = lv[i].at(k);
          for (int j = 0; j < g.count; ++j) m[(int64_t)g.start + (int64_t)j * g.stride] = 1;
        }
        lv[i] = ListView{(int32_t)h->tail[a->request_id[i]], nullptr, 0, nullptr, nullptr, nullptr, 0};
      }
      total_ranges = 0;
    }

    // ---- group by request (order of first appearance)
    std::vector<int32_t>& req_idx_of = pb.req_idx_of;
    req_idx_of.assign(c.max_requests, -1);  // (reserved at create, as is reqs)
    std::vector<DevReq>& reqs = pb.reqs;
    reqs.clear();
    std::vector<int32_t>&stream_req_idx = pb.stream_req_idx, &stream_local = pb.stream_local;
    stream_req_idx.resize(n);
    stream_local.resize(n);
    for (int i = 0; i < n; ++i) {
      const int r = a->request_id[i];
      if (req_idx_of[r] < 0) {
        req_idx_of[r] = (int32_t)reqs.size();
        DevReq q{};
        q.req = r;
        q.pc = INT32_MAX;
        q.pend0 = INT32_MAX;
        reqs.push_back(q);
      }
      DevReq& q = reqs[req_idx_of[r]];
      stream_req_idx[i] = req_idx_of[r];
      stream_local[i] = q.n_streams++;
      q.pc = std::min(q.pc, lv[i].prefix_len);
    }
    std::vector<int32_t>& req_streams = pb.req_streams;
    req_streams.resize(n);
    {
      int32_t pos = 0;
      for (auto& q : reqs) { q.stream0 = pos; pos += q.n_streams; }
      for (int i = 0; i < n; ++i) req_streams[reqs[stream_req_idx[i]].stream0 + stream_local[i]] = i;
    }

    // ---- shared-prefix plan: only what the matrix-core kernel takes; the rest is private
    // (the matrix-core kernel addresses a layer's pool and the query rows with 32-bit byte offsets)
    const bool mfma = c.dtype == PASTA_BF16 && !(a->flags & PASTA_DECODE_NO_MFMA) && attn_kernel_supports(D, G) &&
                      h->layer_elems * h->elem < ((int64_t)1 << 32) - 65536 &&
                      (int64_t)n * c.n_q_heads * D * h->elem < ((int64_t)1 << 31);
    if ((dense || probe) && !mfma) return PASTA_E_INVAL;  // the mask and the read-only form belong to that kernel
    // Everything else -- fp32, 64-wide heads, layers too large for 32-bit offsets -- goes through the kernel that
    // takes its operands straight from memory (its address codes count 16-byte pieces in 31 bits).  The vector-ALU
    // walker is left with NO_MFMA and what is larger still.
    const bool fits_direct = !(a->flags & PASTA_DECODE_NO_MFMA) && h->layer_elems * h->elem < ((int64_t)1 << 35);
    // (k_one rounds the weights of bf16 x 128 as k_attn does; layers that k_attn does not address keep fp32's)
    const bool one = fits_direct && (mfma || c.dtype == PASTA_F32 || D == 64) && small_step(h, a, lv, reqs);
    const bool direct = fits_direct && (one || !mfma);
    const bool matrix = mfma || direct;
    int64_t pc_total = 0, pc_weighted = 0;  // the second counts a prefix once per work-group that reads it
    for (auto& q : reqs) {
      if (!matrix || q.pc < kTile || no_share || one) q.pc = 0;
      pc_total += q.pc;
    }
    // More than 32 stacked rows per request: the rows go in groups of 32.  When EVERY request with a
    // shared prefix is that wide, the launch may take the form whose work-groups serve four row groups
    // each (one per wave, over shared tiles); otherwise each row group is a work-group of its own.
    // The wide form pays where its waves are busy and its work-groups are long -- every such request keeps three of four waves
    // computing on average, and a chunk is 512 tokens, four times the ring of tiles, or more -- and loses elsewhere; the caller may
    // force either form.  Append and decode step of a layer, 8 kv heads, four groups per work-group / one (us; streams x heads per kv head):
    //   not taken: 8k tokens 12 x 4 20.6 / 17.9, 24 x 4 28.7 / 25.9, 32 x 4 34.8 / 29.8; 16k 16 x 4 28.4 / 28.0; 32k 16 x 4 37.0 / 37.2, 40 x 4 67.5 / 69.7
    //   taken: 16k 24 x 4 35.2 / 34.1 (on the line), 32 x 4 38.9 / 40.5, 12 x 8 29.0 / 31.3; 32k 20 x 4 40.6 / 46.8, 24 x 4 42.4 / 51.8,
    //     32 x 4 48.0 / 59.8, 48 x 4 68.3 / 75.9
    bool wide = mfma && !dense && pc_total > 0 && !(a->flags & PASTA_DECODE_ROW_GROUPS);
    const bool force_wide = a->flags & PASTA_DECODE_FOUR_GROUPS;
    if ((a->flags & PASTA_DECODE_ROW_GROUPS) && force_wide) return PASTA_E_INVAL;
    for (auto& q : reqs) {
      if (q.pc <= 0) continue;
      const int R_all = q.n_streams * G;
      if (R_all <= 32) wide = false;
      const int n_rg = (R_all + 31) / 32, n_quads = (n_rg + 3) / 4;
      if (!force_wide && n_rg < 3 * n_quads) wide = false;  // on average fewer than three of a work-group's four waves would compute
    }
    auto row_units = [&](const DevReq& q) -> int64_t {  // shared-prefix work-groups per (chunk, kv head)
      const int64_t n_rg = (q.n_streams * G + 31) / 32;
      return wide ? (n_rg + 3) / 4 : n_rg;
    };
    if (wide && !force_wide) {  // the chunk the wide form would get: at least sixteen tiles of 32 tokens?
      int64_t pw = 0;
      for (auto& q : reqs) pw += (int64_t)q.pc * row_units(q);
      if (pw * Hkv / h->n_cus < 16 * 32) wide = false;
    }
    for (auto& q : reqs) pc_weighted += (int64_t)q.pc * row_units(q);
    // Chunking.  Every chunk costs one partial row per stacked query row (written here, read
    // by the merge), so chunks should be long; but the step wants at least one shared-prefix
    // work-group per CU to keep enough loads in flight.  Tokens per chunk = the largest
    // multiple of the 64-token tile that still gives kNumCUs prefix work-groups.  Private
    // items stay at 128 tokens: they are few and their rows are scattered.
    int64_t priv_chunk = kPrivChunk, chunk_tokens = kTile;
    if (matrix) {
      chunk_tokens = std::max<int64_t>(kTile, pc_weighted * Hkv / h->n_cus / kTile * kTile);
      // Several prefixes rarely end with a chunk: their remainders make more work-groups than there are CUs, some CUs then have two
      // long ones and end the launch alone.  Chunks of two thirds spread that out; where the chunks come out one per CU they only
      // add partial rows.  So the line is the number of work-groups, those of an eighth of a chunk or less not counted.
      // Append and decode step, one per CU -> two thirds (us; 150 drawn batches and 80 of equal prefixes, geometric means 0.93 and
      // 0.94 by this rule, 1.01 at most; two thirds for every batch: up to 1.19):
      //   bf16 x 128, 8 kv heads, 16 requests of 256 .. 4096 tokens   60.3 -> 56.1 (chunks of 512: 57.1, of 256: 64.3)
      //   fp32 x 128, 13 requests of 941 .. 6604                     108.9 -> 84.9
      //   bf16 x 64, 10 requests of 5120                              42.5 -> 31.6
      //   not taken: bf16 x 128, 16 x 2 streams over 4096 60.8 (64.5), bf16 x 64 37.1 (43.4), fp32 x 128 8 x 8 over 8192 195 (233)
      if (!wide && chunk_tokens >= kManyChunk) {
        int64_t n_prefixes = 0, n_wgs = 0;
        for (auto& q : reqs) {
          n_prefixes += q.pc > 0;
          n_wgs += (q.pc / chunk_tokens + (q.pc % chunk_tokens > chunk_tokens / 8)) * Hkv * row_units(q);
        }
        if (n_prefixes > 1 && n_wgs > h->n_cus) chunk_tokens = std::max<int64_t>(kManyChunk, chunk_tokens * 2 / 3 / kTile * kTile);
      }
      priv_chunk = wide ? 256 : 128;  // (beside the long wide work-groups the private items get one slot per CU: longer items keep more in flight there)
      if (direct && !one && c.dtype == PASTA_F32 && D == 128) {
        // The blocks of this kind are 16 tokens: pieces of 64 give each of four waves one, as 128 do elsewhere.  Not where they make more
        // CUs take a first or a second work-group than there are, where beyond that they are more than 1.4 times as many, or where they make
        // the plan too large for the kernel arguments.  Append and decode step of 8 kv heads, pieces of 128 -> 64 (us; work-groups):
        //   1024 + 4 x 64 .. 512 tokens 10.9 -> 9.9 (176 -> 216), 4096 + 8 x 64 .. 512 20.4 -> 18.8 (384 -> 496), six requests of
        //     1024 + 4 x 64 .. 256 30.3 -> 25.8 (600 -> 832)
        //   not taken: 1024 + 6 x 64 .. 512 12.2 -> 14.4 (216 -> 288), 4096 + 8 x 300 .. 512 20.5 -> 22.6 (472 -> 656), six requests of
        //     1024 + 4 x 300 .. 512 35.9 -> 37.2 (960 -> 1560)
        // Nor where the call has no room for the additional items and rows that it has for 128's (kept plan, metadata, partial rows).
        struct At { int64_t words, wgs, items, rows; };
        const int64_t stream_words = (int64_t)n * (int64_t)(sizeof(DevStream) / 4 + 1) + (int64_t)reqs.size() * (int64_t)(sizeof(DevReq) / 4);
        const bool maintained = !explicit_mode && !a->causal_skip;
        int64_t whole_heads = 0;  // streams without a range of their own for what their prefix has beyond the common one
        auto plan_at = [&](int64_t piece) {
          At at{stream_words, 0, 0, 0};
          whole_heads = 0;
          for (int i = 0; i < n; ++i) {
            const ListView& v = lv[i];
            const int32_t pc = reqs[stream_req_idx[i]].pc;
            const int64_t priv = (int64_t)v.prefix_len - pc + v.range_tokens;
            whole_heads += v.prefix_len == pc;
            at.words += ((int64_t)v.n_ranges + (v.prefix_len > pc)) * (int64_t)(sizeof(DevRange) / 4);
            at.items += (priv + piece - 1) / piece;
          }
          at.words += at.items * (int64_t)(sizeof(DevItem) / 4);
          at.wgs = at.items * Hkv;
          at.rows = at.items * c.n_q_heads;
          for (auto& q : reqs) {
            const int64_t chunks = (q.pc + chunk_tokens - 1) / chunk_tokens * Hkv;
            at.wgs += chunks * row_units(q);
            at.rows += chunks * q.n_streams * G;
          }
          return at;
        };
        const At by_64 = plan_at(64), by_128 = plan_at(128);
        auto turn = [&](int64_t wgs) { return std::min<int64_t>((wgs + h->n_cus - 1) / h->n_cus, 3); };
        // Counted as it is (the launch), with 8 words more (the no-alloc entry) and with a further range per stream (the choice of the lists
        // on the device, below): by none of these may the plan be within the arguments with pieces of 128 and beyond them with 64.
        const int64_t counted_more = 8 + whole_heads * (int64_t)(sizeof(DevRange) / 4);
        auto leaves = [&](int64_t more) { return by_64.words + more > kInlineMetaWords && by_128.words + more <= kInlineMetaWords; };
        const bool left_inline = !leaves(0) && !(no_alloc && leaves(8)) && !(maintained && leaves(counted_more));
        // Nor may a captured plan leave the arguments of k_plan: its words are relayed by a launch of their own then, on every replay (4 streams
        // of 108 random-order tokens over 512, 2 kv heads: 14.9 us per replayed step, 12.3 by pieces of 128).
        auto relayed = [&](int64_t w64, int64_t w128) { return w64 > kPlanWords && w128 <= kPlanWords; };
        const bool relay_64 = (relayed(by_64.words + 1, by_128.words + 1) || (maintained && relayed(stream_words + by_64.items + 3, stream_words + by_128.items + 3))) &&
                              !plan_only && stream_capturing(h);
        // (a list on the device can have an item more than here, its prefix's rest and its ranges apart; an entry per item goes with the words)
        const bool inline_64 = by_64.words + (maintained ? counted_more : 0) <= kInlineMetaWords && !(a->flags & PASTA_DECODE_DEVICE_LISTS);
        const bool fits_64 = (inline_64 || by_64.items + n <= h->plan_items_cap || by_128.items > h->plan_items_cap) &&
                             (by_64.words + by_64.items + counted_more + n) * 4 <= (int64_t)h->meta_bytes && by_64.rows + (int64_t)n * c.n_q_heads <= part_rows_cap;
        if (fits_64 && left_inline && !relay_64 && turn(by_64.wgs) == turn(by_128.wgs) && (turn(by_64.wgs) < 3 || 5 * by_64.wgs <= 7 * by_128.wgs)) priv_chunk = 64;
      }
      if (h->tune_prefix_chunk >= kTile) chunk_tokens = h->tune_prefix_chunk / kTile * kTile;
      if (one) priv_chunk = kOneTokens;  // a stream's whole list
      else if (h->tune_priv_chunk >= 32) priv_chunk = std::min<int64_t>(h->tune_priv_chunk / 32 * 32, kGatherMax);  // whole 32-token blocks
    }
    // ---- where the lists come from.  Maintained lists have a copy on the device (range arena + range
    // index, kept up to date by the appends): a step may then send a fixed-size record per stream and let
    // the kernels derive the private work items, instead of sending every range and item.  A plan small
    // enough to ride in the kernel arguments is sent whole all the same -- its items then cost the
    // kernels no dependent loads -- unless the caller asks for the device lists.
    bool dev_lists = false, plan_fits = true;
    if (!explicit_mode && !a->causal_skip && !dense) {
      int64_t dev_items = 0;
      int64_t words = (int64_t)n * (sizeof(DevStream) / 4 + 1) + (int64_t)reqs.size() * (sizeof(DevReq) / 4) + 8;
      for (int i = 0; i < n; ++i) {
        const StreamState& ss = sstate(h, a->request_id[i], a->stream_id[i]);
        const int64_t priv = (int64_t)lv[i].prefix_len - reqs[stream_req_idx[i]].pc + ss.range_tokens;
        words += ((int64_t)lv[i].n_ranges + 1) * 4 + (priv + priv_chunk - 1) / priv_chunk * (sizeof(DevItem) / 4);
        dev_items += (priv + priv_chunk - 1) / priv_chunk + 1;
      }
      dev_lists = (a->flags & PASTA_DECODE_DEVICE_LISTS) || words > kInlineMetaWords;
      plan_fits = dev_items <= h->plan_items_cap && dev_items * priv_chunk <= h->plan_codes_cap;
      if (!plan_fits) dev_lists = false;  // (k_plan has no room)
    } else if (a->flags & PASTA_DECODE_DEVICE_LISTS) {
      return PASTA_E_INVAL;
    }
    if (dev_lists && !plan_only) {  // the copies this step reads must be current (all but each list's newest range)
      auto stale = [](const StreamState& ss) { return ss.dirty || ss.dev_ranges < (int32_t)ss.ranges.size() - 1; };
      bool rebuild = h->tables_reset;
      for (int i = 0; i < n && !rebuild; ++i) rebuild = stale(sstate(h, a->request_id[i], a->stream_id[i]));
      // No rebuild where nothing may be allocated (it stages through buffers that may have to grow), nor under stream
      // capture: a replay would find the pinned slot as later calls left it, and put back lists of another time.
      if (rebuild && (no_alloc || stream_capturing(h))) rebuild = dev_lists = false;
      if (rebuild) {
        h->stage_pieces.clear();  // (what a failed call may have left)
        h->stage_words.clear();
        if (h->tables_reset) {  // the segments ran out earlier: start over
          h->tables_reset = false;
          h->arena_top = h->cidx_top = 0;
          for (StreamState& ss : h->streams) { ss.seg_off = ss.cseg_off = -1; ss.seg_cap = ss.cseg_cap = 0; ss.dirty = true; }
        }
        for (int i = 0; i < n && dev_lists; ++i) {
          StreamState& ss = sstate(h, a->request_id[i], a->stream_id[i]);
          if (!stale(ss)) continue;
          const int rb = rebuild_tables(h, ss);
          if (rb == kNoRoom) dev_lists = false;
          else if (rb != PASTA_OK) return rb;
        }
        const int fl = flush_lists(h);
        if (fl != PASTA_OK) return fl;
        for (int i = 0; i < n && dev_lists; ++i) sstate(h, a->request_id[i], a->stream_id[i]).dirty = false;  // (kNoRoom: staged again next time)
      }
      if (dev_lists) h->lists_in_use = true;
    }
    if (!dev_lists && plan_fits && (a->flags & PASTA_DECODE_DEVICE_LISTS)) return PASTA_E_CAPACITY;
    // private items
    std::vector<DevStream>& streams = pb.streams;
    std::vector<DevRange>& ranges = pb.ranges;
    std::vector<DevItem>& items = pb.items;
    streams.assign(n, DevStream{});
    ranges.clear();
    items.clear();
    if (!dev_lists) {
      if (!room(ranges, (size_t)total_ranges + n)) return PASTA_E_CAPACITY;
      ranges.reserve((size_t)total_ranges + n);
    }
    int64_t gather_total = 0, n_items_total = 0;
    for (int i = 0; i < n; ++i) {
      DevStream& ds = streams[i];
      const DevReq& q = reqs[stream_req_idx[i]];
      ds.req = q.req;
      ds.req_idx = stream_req_idx[i];
      ds.local = stream_local[i];
      ds.pos = rope_q ? a->position[i] : 0;
      ds.mask_base = mask_base[i];
      ds.pc = q.pc;
      ds.pend0 = INT32_MAX;
      if (dev_lists) {
        const StreamState& ss = sstate(h, a->request_id[i], a->stream_id[i]);
        const int64_t extra = (int64_t)lv[i].prefix_len - q.pc, T = ss.range_tokens;
        if (gather_total + q.pc + extra + T > INT32_MAX) return PASTA_E_CAPACITY;
        ds.extra = (int32_t)extra;
        ds.n_ranges = (int32_t)ss.ranges.size();
        ds.seg_off = ss.seg_off;
        ds.range_tokens = (int32_t)T;
        ds.cseg_off = ss.cseg_off;
        ds.n_cidx = ss.dev_cidx;
        if (ds.n_ranges) {
          const Range& g = ss.ranges.back();
          ds.last[0] = g.start; ds.last[1] = g.count; ds.last[2] = g.stride; ds.last[3] = (int32_t)(T - g.count);
        }
        ds.item_begin = (int32_t)n_items_total;
        n_items_total += (extra + priv_chunk - 1) / priv_chunk + (T + priv_chunk - 1) / priv_chunk;
        ds.item_end = (int32_t)n_items_total;
        ds.gather_base = (int32_t)gather_total;
        if (a->dbg_gather_offsets) a->dbg_gather_offsets[i] = gather_total;
        gather_total += (int64_t)q.pc + extra + T;
        continue;
      }
      const int32_t range_begin = (int32_t)ranges.size();
      int32_t cum = 0;
      if (lv[i].prefix_len > q.pc) {
        ranges.push_back({q.pc, lv[i].prefix_len - q.pc, 1, 0});
        cum = lv[i].prefix_len - q.pc;
      }
      for (int k = 0; k < lv[i].n_ranges; ++k) {
        const Range g = lv[i].at(k);
        ranges.push_back({g.start, g.count, g.stride, cum});
        cum += g.count;
      }
      const int32_t range_end = (int32_t)ranges.size();
      ds.item_begin = (int32_t)items.size();
      int32_t rcur = range_begin;
      for (int32_t t = 0; t < cum; t += (int32_t)priv_chunk) {
        while (rcur + 1 < range_end && ranges[rcur + 1].cum <= t) rcur++;
        DevItem it{};
        it.stream = i;
        it.tok_begin = t;
        it.tok_count = std::min<int32_t>((int32_t)priv_chunk, cum - t);
        it.range_first = rcur;
        int32_t rlast = rcur;
        while (rlast + 1 < range_end && ranges[rlast + 1].cum < t + it.tok_count) rlast++;
        it.n_ranges = rlast - rcur + 1;
        it.gather_pos = (int32_t)(gather_total + q.pc + t);
        it.slot0 = ranges[rcur].start + (t - ranges[rcur].cum) * ranges[rcur].stride;
        it.stride = it.n_ranges == 1 ? ranges[rcur].stride : 0;  // 0: rows come from the expanded list
        if (!room(items, items.size() + 1)) return PASTA_E_CAPACITY;
        items.push_back(it);
      }
      ds.item_end = (int32_t)items.size();
      n_items_total = (int64_t)items.size();
      if (gather_total + q.pc + cum > INT32_MAX) return PASTA_E_CAPACITY;
      ds.gather_base = (int32_t)gather_total;
      if (a->dbg_gather_offsets) a->dbg_gather_offsets[i] = gather_total;
      gather_total += (int64_t)q.pc + cum;
    }
    if (a->dbg_gather_offsets) a->dbg_gather_offsets[n] = gather_total;

    // split-K chunks of the common prefixes; grow the chunk until the partial rows fit
    const int64_t priv_rows = n_items_total * c.n_q_heads;
    int64_t n_prefix_wgs = 0, prefix_rows = 0;
    if (pc_total > 0) {
      for (;; chunk_tokens += kTile) {
        n_prefix_wgs = 0;
        prefix_rows = 0;
        for (auto& q : reqs) {
          q.n_chunks = q.pc ? (int32_t)((q.pc + chunk_tokens - 1) / chunk_tokens) : 0;
          q.chunk_tokens = (int32_t)chunk_tokens;
          q.wg_begin = (int32_t)n_prefix_wgs;
          q.part_base = (int32_t)prefix_rows;
          n_prefix_wgs += (int64_t)q.n_chunks * Hkv * row_units(q);
          prefix_rows += (int64_t)q.n_chunks * Hkv * q.n_streams * G;
        }
        if (prefix_rows + priv_rows <= part_rows_cap) break;
        if (chunk_tokens > (int64_t)1 << 30) return PASTA_E_CAPACITY;
      }
    } else {
      for (auto& q : reqs) { q.n_chunks = 0; q.chunk_tokens = kTile; q.wg_begin = 0; q.part_base = 0; }
      if (priv_rows > part_rows_cap) return PASTA_E_CAPACITY;
    }

    for (int i = 0; i < n; ++i) {  // the merge's view of each stream's request (known now that the chunks are)
      const DevReq& q = reqs[stream_req_idx[i]];
      streams[i].m_pre0 = q.part_base + streams[i].local * G;
      streams[i].m_n_pre = q.n_chunks;
      streams[i].m_R = q.n_streams * G;
    }
    // ---- metadata blob
    std::vector<int32_t>& blob = pb.blob;
    blob.clear();
    {
      const size_t words = (streams.size() * sizeof(DevStream) + reqs.size() * sizeof(DevReq) + req_streams.size() * 4 +
                            ranges.size() * sizeof(DevRange) + items.size() * sizeof(DevItem)) / 4 + 8;
      if (no_alloc && words > (size_t)kInlineMetaWords) return PASTA_E_CAPACITY;  // larger plans need the pinned staging
      if (!room(blob, words)) return PASTA_E_CAPACITY;
      blob.reserve(words);
    }
    DecodeParams p{};
    auto put = [&](const void* src, size_t bytes) -> int {
      const int off = (int)blob.size();
      blob.resize(blob.size() + (bytes + 3) / 4);
      if (bytes) std::memcpy(blob.data() + off, src, bytes);
      return off;
    };
    p.off_streams = put(streams.data(), streams.size() * sizeof(DevStream));
    p.off_reqs = put(reqs.data(), reqs.size() * sizeof(DevReq));
    p.off_req_streams = put(req_streams.data(), req_streams.size() * 4);
    p.off_ranges = put(ranges.data(), ranges.size() * sizeof(DevRange));
    p.off_items = put(items.data(), items.size() * sizeof(DevItem));
    if (blob.size() * 4 > h->meta_bytes) return PASTA_E_CAPACITY;
    const size_t plan_size = blob.size();  // the words the attention and merge launches read

    if (a->dbg_plan) {
      int64_t tiles = 0;
      for (auto& q : reqs) tiles += (int64_t)(q.pc + kTile - 1) / kTile * Hkv;
      a->dbg_plan[0] = tiles;
      a->dbg_plan[1] = n_prefix_wgs;
      a->dbg_plan[2] = n_items_total;
      a->dbg_plan[3] = one ? 0 : prefix_rows + priv_rows;
      a->dbg_plan[4] = pc_total ? chunk_tokens : 0;
      a->dbg_plan[5] = pc_total;
      a->dbg_plan[6] = (int64_t)blob.size() * 4;
      a->dbg_plan[7] = prefix_rows;
    }
    if (plan_only) return PASTA_OK;

    // ---- enqueue
    int rc = PASTA_OK;
    hipStream_t st = (hipStream_t)c.hip_stream;
    int meta_slot = -1;  // pinned staging slot that this call's kernels read, if any
    // a deferred append rides along with the partials launch of its layer; otherwise K1 runs now
    const bool take_pending = h->pending.active && matrix && h->pending.layer == a->layer && !probe && !merge_only;
    if (h->pending.active && !take_pending) {
      rc = flush_pending(h);
      if (rc != PASTA_OK) return rc;
    }
    if (take_pending) {
      const pasta_attn::Pending& pd = h->pending;
      for (auto& q : reqs) { q.pend0 = pd.req_pend0[q.req]; q.pend_src0 = pd.req_src0[q.req]; }
      p.k_pend = pd.k_new;
      p.v_pend = pd.v_new;
      p.pend_n = pd.n_rows;
      std::memcpy(p.pend_dst, pd.dst_rows, sizeof(p.pend_dst));
      if (pd.rope) {  // turned by the small launch ahead of k_attn (below), or by k_direct / k_one as they load them
        p.pend_rope = 1;
        std::memcpy(p.pend_pos, pd.pos, sizeof(p.pend_pos));
      }
      for (auto& ds : streams) { ds.pend0 = pd.req_pend0[ds.req]; ds.pend_src0 = pd.req_src0[ds.req]; }
      // the blob was built before these fields were known: patch the tables in place
      std::memcpy(blob.data() + p.off_reqs, reqs.data(), reqs.size() * sizeof(DevReq));
      std::memcpy(blob.data() + p.off_streams, streams.data(), streams.size() * sizeof(DevStream));
    }
    if (dense) {  // the masks travel like the paper's mask tensors: host -> device, every step
      if (!h->mask_pinned) {
        if (hipHostMalloc((void**)&h->mask_pinned, h->mask_bytes, hipHostMallocDefault) != hipSuccess) {
          (void)hipGetLastError();
          h->mask_pinned = nullptr;
          return PASTA_E_DEVICE;
        }
        if (hipEventCreateWithFlags(&h->mask_ev, hipEventDisableTiming) != hipSuccess) return PASTA_E_DEVICE;
      }
      if (h->mask_ev_used && hipEventSynchronize(h->mask_ev) != hipSuccess) return PASTA_E_DEVICE;
      std::memcpy(h->mask_pinned, mask.data(), mask.size());
      uint8_t* dev_mask = (uint8_t*)c.workspace + h->off_mask;
      if (hipMemcpyAsync(dev_mask, h->mask_pinned, mask.size(), hipMemcpyHostToDevice, st) != hipSuccess) return PASTA_E_DEVICE;
      if (hipEventRecord(h->mask_ev, st) != hipSuccess) return PASTA_E_DEVICE;
      h->mask_ev_used = true;
      p.dense_mask = dev_mask;
    }
    p.page_table = (const int32_t*)((const char*)c.workspace + h->off_page_table);
    p.lay = h->lay;
    p.n_streams = n;
    p.n_items = (int)n_items_total;
    p.priv_chunk = (int)priv_chunk;
    if (!dev_lists && blob.size() <= (size_t)kInlineMetaWords) {  // small plan: rides in the kernel arguments
      p.meta = nullptr;
      std::memcpy(p.inline_meta, blob.data(), blob.size() * 4);
    } else {
      // A larger plan is put on the device once and used by every call that makes the same one -- all layers of
      // a token step do (k_plan).  "The same" is decided by its words; for device-resident lists, whose ranges
      // are not among them, the words end with the count of changes the lists have seen.  A captured call
      // writes a place of its own every time it is replayed: what it leaves says nothing about later calls.
      const bool keep = n_items_total <= h->plan_items_cap && n_items_total * priv_chunk <= h->plan_codes_cap;
      if (dev_lists) {
        if (!room(blob, blob.size() + (size_t)n_items_total + 4)) return PASTA_E_CAPACITY;
        for (int i = 0; i < n; ++i) blob.insert(blob.end(), (size_t)(streams[i].item_end - streams[i].item_begin), i);
        p.off_items = (int)plan_size;
        blob.push_back((int32_t)(h->lists_epoch & 0xffffffffu));
        blob.push_back((int32_t)(h->lists_epoch >> 32));
      }
      blob.push_back((int32_t)priv_chunk);
      if (blob.size() * 4 > h->meta_bytes) return PASTA_E_CAPACITY;
      const bool capturing = stream_capturing(h);
      const int at = capturing ? 1 : 0;
      int32_t* dev = (int32_t*)((char*)c.workspace + h->off_plan[at]);
      DevItem* d_items = (DevItem*)((char*)c.workspace + h->off_plan_items[at]);
      int32_t* d_codes = (int32_t*)((char*)c.workspace + h->off_plan_codes[at]);
      if (!keep || capturing || blob != h->plan_words) {
        if (keep && !capturing) h->plan_words.clear();  // (what is there is about to be overwritten)
        PlanParams pp{};
        if (keep && blob.size() <= (size_t)kPlanWords) {
          std::memcpy(pp.words, blob.data(), blob.size() * 4);
        } else if (capturing) {
          rc = relay_words(h, blob.data(), blob.size(), &pp.src);
          if (rc != PASTA_OK) return rc;
          p.meta = pp.src;
        } else {  // through pinned memory; the slot is reused only after the launches that read it have completed
          char* host = nullptr;
          rc = ring_take(h, &meta_slot, &host);
          if (rc != PASTA_OK) return rc;
          std::memcpy(host, blob.data(), blob.size() * 4);
          p.meta = pp.src = (const int32_t*)host;
        }
        if (keep) {
          pp.dst = dev;
          pp.items = d_items;
          pp.codes = d_codes;
          pp.page_table = p.page_table;
          pp.arena = (const DevRange*)((const char*)c.workspace + h->off_arena);
          pp.cidx = (const int32_t*)((const char*)c.workspace + h->off_cidx);
          pp.lay = h->lay;
          pp.n_words = (int)plan_size;
          pp.n_items = (int)n_items_total;
          pp.priv_chunk = (int)priv_chunk;
          pp.dev_tables = dev_lists ? 1 : 0;
          pp.off_streams = p.off_streams;
          pp.off_ranges = p.off_ranges;
          pp.off_items = p.off_items;
          const size_t wgs = std::max<size_t>((size_t)n_items_total, (plan_size + 255) / 256);
          k_plan<<<dim3((unsigned)wgs), 256, 0, st>>>(pp);
          if (hipGetLastError() != hipSuccess) return PASTA_E_DEVICE;
          if (meta_slot >= 0) {
            rc = ring_give(h);
            if (rc != PASTA_OK) return rc;
            meta_slot = -1;
          }
          if (!capturing) {
            if (!room(h->plan_words, blob.size())) return PASTA_E_CAPACITY;
            h->plan_words.assign(blob.begin(), blob.end());
          }
        }
      }
      if (keep) {
        p.meta = dev;
        p.items = d_items;
        p.codes = d_codes;
      }  // (else: a plan of millions of private tokens is read where it lies)
    }
    p.k = (const char*)c.k_pool + (size_t)a->layer * h->layer_elems * h->elem;
    p.v = (const char*)c.v_pool + (size_t)a->layer * h->layer_elems * h->elem;
    p.q = a->q;
    p.out = a->out;
    p.lse = a->out_lse;
    p.dbg_rows = a->dbg_gather_rows;
    p.part_acc = part_acc;
    p.part_ml = part_ml;
    p.n_reqs = (int)reqs.size();
    p.n_mfma_items = matrix ? (int)n_items_total : 0;
    p.n_prefix_wgs = (int)n_prefix_wgs;
    p.priv_part_base = (int)prefix_rows;
    p.Hq = c.n_q_heads;
    p.Hkv = Hkv;
    p.scale_log2e = c.softmax_scale * kLog2e;
#if defined(PASTA_TUNING) && PASTA_TUNING >= 2
    p.clock_row0 = h->part_rows_cap - 16 * PASTA_CLK_WGS + (a->layer & 1) * 8 * PASTA_CLK_WGS;  // the tail of the (m, l) array, two halves
#endif
    p.single_req = reqs.size() == 1 ? 1 : 0;
    p.req0 = reqs[0];

    const bool rope = rope_q || p.pend_rope;
    if (rope && direct) {  // that kernel turns what it has to as it loads it
      p.rope_tab = (const double*)((const char*)c.workspace + h->off_rope);
      p.rope_q = rope_q ? 1 : 0;
    } else if (rope) {
      // one small launch turns what has to be turned: Q into its buffer, the deferred K rows into theirs
      p.rope_tab = (const double*)((const char*)c.workspace + h->off_rope);
      p.rope_q = rope_q ? 1 : 0;
      void* const q_rot = (char*)c.workspace + h->off_qrot;
      void* const k_rot = (char*)c.workspace + h->off_krot;
      const int half_log = D == 128 ? 6 : 5, per_wg = 256 >> half_log;
      const int64_t nq = rope_q ? (int64_t)n * c.n_q_heads : 0, nk = p.pend_rope ? (int64_t)p.pend_n * Hkv : 0;
      const dim3 grid((unsigned)((nq + nk + per_wg - 1) / per_wg));
      if (c.dtype == PASTA_F32) k_rope_prep<float><<<grid, 256, 0, st>>>(p, (float*)q_rot, (float*)k_rot, half_log, (int)nq);
      else k_rope_prep<uint16_t><<<grid, 256, 0, st>>>(p, (uint16_t*)q_rot, (uint16_t*)k_rot, half_log, (int)nq);
      if (rope_q) p.q = q_rot;
      if (p.pend_rope) { p.k_pend = k_rot; p.pend_rope = 0; }
    }
    // Profiling events: the matrix-core launch hands them to the dispatch itself, so they carry the
    // start and the end of that kernel's execution (what a kernel trace reports) and put no packet of
    // their own on the stream; around the vector-ALU form they are recorded on the stream.
    const hipEvent_t ev0 = (hipEvent_t)a->prof_event_start, ev1 = (hipEvent_t)a->prof_event_stop;
    const bool ev_in_dispatch = matrix && ev0 && ev1;
    if (ev0 && !ev_in_dispatch && hipEventRecord(ev0, st) != hipSuccess) return PASTA_E_DEVICE;
    if (merge_only) {
      // (kernel-isolated test of the merge: the partial buffers are taken as they are)
    } else if (matrix) {
      unsigned grid = (unsigned)(n_items_total * Hkv + n_prefix_wgs);
      if (one) grid += (unsigned)((2ll * p.pend_n * Hkv * D * h->elem / 16 + kOneWaves * 64 - 1) / (kOneWaves * 64));  // the deferred rows' copy
      auto launch = [&](auto kernel, int threads = kAttnThreads) {
        if (ev_in_dispatch) hipExtLaunchKernelGGL(kernel, dim3(grid), dim3(threads), 0, st, ev0, ev1, 0, p);
        else kernel<<<dim3(grid), threads, 0, st>>>(p);
      };
      if (one) {
        auto by_rope = [&](auto turned) {
          if (c.dtype == PASTA_F32) { if (D == 64) launch(k_one<float, 64, turned.value>, kOneWaves * 64); else launch(k_one<float, 128, turned.value>, kOneWaves * 64); }
          else { if (D == 64) launch(k_one<uint16_t, 64, turned.value>, kOneWaves * 64); else launch(k_one<uint16_t, 128, turned.value>, kOneWaves * 64); }
        };
        if (rope) by_rope(std::true_type{}); else by_rope(std::false_type{});
      } else if (direct) {
        if (c.dtype == PASTA_F32) {
          if (D == 64) { if (rope) launch(k_direct<float, 64, true>); else launch(k_direct<float, 64, false>); }
          else { if (rope) launch(k_direct<float, 128, true>); else launch(k_direct<float, 128, false>); }
        } else {
          if (D == 64) { if (rope) launch(k_direct<uint16_t, 64, true>); else launch(k_direct<uint16_t, 64, false>); }
          else { if (rope) launch(k_direct<uint16_t, 128, true>); else launch(k_direct<uint16_t, 128, false>); }
        }
      } else if (dense) {  // the variant that carries the dense-mask mode
        if (p.codes) { if (h->lay.paged) launch(k_attn<true, true, true>); else launch(k_attn<true, false, true>); }
        else { if (h->lay.paged) launch(k_attn<false, true, true>); else launch(k_attn<false, false, true>); }
      } else {
        // prefix chunks of more than two 32-token blocks per wave: the variant whose loop has the
        // cheap addressing of plain blocks
        const bool long_items = n_prefix_wgs > 0 && chunk_tokens > 2 * 4 * 32;
        auto by_form = [&](auto kept, auto paged, auto prb) {
          if (wide) launch(k_attn<kept.value, paged.value, false, false, prb.value, true>);
          else if (long_items) launch(k_attn<kept.value, paged.value, false, true, prb.value>);
          else launch(k_attn<kept.value, paged.value, false, false, prb.value>);
        };
        auto by_probe = [&](auto kept, auto paged) {
          if (probe) by_form(kept, paged, std::true_type{});
          else by_form(kept, paged, std::false_type{});
        };
        auto by_pool = [&](auto kept) {
          if (h->lay.paged) by_probe(kept, std::true_type{});
          else by_probe(kept, std::false_type{});
        };
        if (p.codes) by_pool(std::true_type{});
        else by_pool(std::false_type{});
      }
      if (take_pending) h->pending.active = false;
    } else if (n_items_total > 0) {
      const unsigned waves = (unsigned)n_items_total * Hkv;
      rc = launch_private(h, dim3((waves + 3) / 4), st, p);
      if (rc != PASTA_OK) return rc;
    }
    if (ev1 && !ev_in_dispatch && hipEventRecord(ev1, st) != hipSuccess) return PASTA_E_DEVICE;
    int64_t merge_parts = 0;  // every output row reads its request's prefix chunks and its stream's items: the most of them
    for (int i = 0; i < n; ++i)
      merge_parts = std::max<int64_t>(merge_parts, reqs[stream_req_idx[i]].n_chunks + streams[i].item_end - streams[i].item_begin);
    if (!probe && !partials_only && !one) {
      MergeParams mp;  // (what is not filled in is not read)
      mp.out = p.out;
      mp.lse = p.lse;
      mp.part_acc = p.part_acc;
      mp.part_ml = p.part_ml;
      static_assert(kInlineMetaWords / (sizeof(DevStream) / 4) <= kMergeRecs, "a plan of more streams lies on the device");
      mp.meta = n <= kMergeRecs ? nullptr : p.meta;
      mp.off_streams = p.off_streams;
      mp.priv_part_base = p.priv_part_base;
      mp.Hkv = Hkv;
      mp.G = G;
      for (int i = 0; i < n && n <= kMergeRecs; ++i)
        mp.rec[i] = MergeRec{streams[i].m_pre0, streams[i].m_n_pre, streams[i].m_R, streams[i].item_begin, streams[i].item_end - streams[i].item_begin};
      launch_merge(h, dim3((unsigned)Hkv, (unsigned)G, (unsigned)n), st, mp, merge_parts);
    }
    if (meta_slot >= 0) {
      rc = ring_give(h);
      if (rc != PASTA_OK) return rc;
    }
    if (hipGetLastError() != hipSuccess) return PASTA_E_DEVICE;
    return PASTA_OK;
  } catch (const std::bad_alloc&) {
    return PASTA_E_NOMEM;
  }
}

}  // namespace

extern "C" int32_t pasta_attn_decode_step(pasta_attn* h, const pasta_decode_args* a) { return decode_impl(h, a, false); }

extern "C" int32_t pasta_attn_decode_step_noalloc(pasta_attn* h, const pasta_decode_args* a) {
  return decode_impl(h, a, true);
}

#include "replay.hpp"
