// Internal declarations shared by the host planner, the launchers and the kernels.
// Not part of the public ABI (that is include/cronus.h).
#pragma once

#include <stddef.h>
#include <stdint.h>

#include "cronus.h"

#if defined(__HIP__)
#define CRONUS_HOST_DEVICE __host__ __device__
#else
#define CRONUS_HOST_DEVICE
#endif

namespace cronus {

constexpr int kBlock = 16;          // tokens per KV block (N_size of Algorithm 1)
constexpr int kThreads = 512;       // 8 wavefronts of 64 lanes per work-group: two per SIMD
constexpr int kWaves = 8;
constexpr int kNarrowRows = 32;     // one MFMA column tile: a decode's (token, head) rows
constexpr int kWideKvTile = 64;     // keys staged in LDS per step of a wide (chunk) tile
constexpr int kNarrowKvStep = 32 * kWaves;  // keys covered by the waves of a narrow item per step
constexpr int kQueues = 8;          // work queues of a launch: one per XCD of an MI355X (each XCD has its own L2)
// int32 between the queue heads of a set: 256 bytes, so that no two lie in one 128-byte line.  Every ticket and look of the 256
// work-groups goes to memory, whose lines take them one at a time, and with 64 bytes two queues and all looks at either shared a
// line.  us a pass at 64 / 128 / 256 / 512 / 1024 bytes: 16 decodes of 281 .. 2407 29.3 / 25.3 / 25.1 / 25.2 / 25.2, 40 of 2717 .. 5329
// (7 heads a KV head) 71.9 / 69.8 / 69.8 / 69.9 / 69.9, 4 chunks of 512 next to 64 decodes 127.0 / 124.1 / 124.3 / 124.0 / 124.3, fp8, a chunk
// of 201 next to 48 87.1 / 84.8 / 84.6 / 84.7 / 84.6; launches with no more items than work-groups take no tickets: no difference.
constexpr int kCounterStride = 64;
// Row groups whose results are merged from key spans, per launch at most: each has kWaves arrival
// counters in the set.  A launch with more rows to split leaves its shortest ones whole (build_plan).
constexpr int kMaxMergeGroups = 4096;
constexpr int kQueueSetInts = (kQueues + 1) * kCounterStride + kMaxMergeGroups * kWaves;  // a set: the heads, the count of finished work-groups, the arrival counters
constexpr int kQueueSets = 9;       // sets of queue heads per device: one per plan buffer of the ring, one for the static entry point

// Per-sequence record of the batch (section 4.4: one iteration = chunks + decodes).
struct SeqInfo {
  int32_t prefix_len;  // keys cached before this chunk ("length already processed", section 4.2)
  int32_t chunk_len;   // query rows of this iteration (1 = decode)
  int32_t q_off;       // index of the sequence's first row in q/out
  int32_t n_blocks;    // ceil((prefix+chunk)/16): table entries that may be read
};

// One work-group's job.
struct WorkItem {
  int32_t seq;
  int32_t kv_head;
  int32_t head0;     // first q head of the group handled here
  int32_t n_heads;   // q heads handled (all read kv_head)
  int32_t q_tok0;    // first chunk token of the tile
  int32_t n_tok;     // tokens in the tile; rows = n_tok * n_heads
  int32_t kv_begin;  // keys [kv_begin, kv_end) are processed by this item
  int32_t kv_end;
  int32_t partial;   // < 0: writes final output; else index of its (wide: first of kWaves) partial-result slot(s)
  int32_t wide;      // 1: chunk tile staged through LDS; >= 2: the same, reading the bf16 copy of an fp8
                     // sequence's K/V whose first block in the copy is wide - 2; 0: narrow (<= 32 rows),
                     // waves split keys; -1: nothing to do (a work-group's "no item left" marker)
  // copy of the sequence's record, so that a work-group needs one dependent load less
  // before it can address Q and the block table
  int32_t prefix_len, chunk_len, q_off;
  union {
    int32_t n_blocks;  // wide: as in the sequence's record
    int32_t peers;     // narrow: < 0: its K/V is read the ordinary way; else a bit for each sequence near by whose table has
                       // the item's column (peer_column, peer_offset)
  };
  // partial >= 0: first partial slot of the item's row group, and n_split * kMaxMergeGroups +
  // the group's index among those of the launch
  int32_t first_partial, merge_key;
};
static_assert(sizeof(WorkItem) == 64, "one work item = one 64-byte line");

// A narrow item whose K/V no other item reads keeps it out of the caches.  The host knows of the others where there are more
// head groups of a KV head than one, and where the item is the tail of a chunk, whose tiles read the same keys.  Whether
// decodes share blocks is seen in the block tables only: the item compares its block at three quarters of its keys with that
// of the 16 sequences before and the 15 behind it in the batch, where they attend in this launch and have as many blocks (no
// other entry of their rows is read).  As many as a record has bits for; the sign says whether to look (a flag among the
// kernel's arguments cost each narrow item a scalar load, 0.5 us).  With 8 on either side, 64 decodes of the same 4 k keys in
// groups of 7, nine places apart, took 101 us instead of 71, and 8 prefixes dealt at random 84 instead of 75.
constexpr int kPeersBefore = 16, kPeers = 31;
CRONUS_HOST_DEVICE inline int32_t peer_column(int32_t kv_begin, int32_t kv_end) {
  return (int32_t)(((uint32_t)kv_begin + (uint32_t)(kv_end - kv_begin) / 4 * 3) / kBlock);
}
CRONUS_HOST_DEVICE inline int32_t peer_offset(int32_t bit) { return bit < kPeersBefore ? bit - kPeersBefore : bit - kPeersBefore + 1; }

// The K/V of a launch's decodes passes the caches from this many bytes on: less of it may still lie there from its last use, three such
// batches in turn fit into 256 MB.  us a pass, ordinary / past the caches, over the same three batches in turn and cold:
// 2 decodes of 1000 keys (8 MB) 15.6 / 17.8 and 18.6 / 18.3, 4 of 2000 (33 MB) 17.4 / 19.3 and 20.8 / 20.1, 76 of 150 (47 MB) 29.9 / 31.2 and
// 34.0 / 32.5, 8 of 1500 (49 MB) 20.6 / 21.7 and 23.8 / 22.5, 128 of 130 (68 MB) 42.6 / 45.4 and 48.0 / 46.0, 100 of 200 (82 MB) 39.5 / 40.8
// and 43.7 / 41.9, 33 of 700 (95 MB) 34.3 / 34.5 and 37.9 / 35.2, 12 of 2000 (98 MB) 33.2 / 32.6 and 36.0 / 33.4, 200 of 120 (98 MB) 63.8 / 62.5 and
// 66.1 / 63.2, 16 of 2000 (131 MB) 36.1 / 32.6 and 36.8 / 33.0.  Cold batches below the line give up 4 to 8 % for it.
constexpr long long kPastCacheBytes = 90'000'000;
// And whatever there is of it where the chunks' products take this long (at 1.2 PFLOP/s): the decodes are not what such a launch
// waits for, and their K/V would push out what the chunk tiles read again.  us a pass, ordinary / past the caches: 4 decodes of 2000
// next to 500 tokens behind 8000 (products 56 us) 99.6 / 98.2, next to 3 x 400 behind 4000 (69) 118.4 / 117.8; fp8, 8 of 1100 next to 4 whole prompts
// of 700 (27) 75.0 / 72.0.  The other side: 4 of 2000 next to 64 tokens behind 200 (0.2) 17.2 / 18.8; 7 heads a KV head, 8 of 1100 next to
// 256 behind 1000 (4) 30.0 / 30.7; 8 of 1100 next to 4 whole prompts of 700 (13) 46.2 / 46.9.
constexpr double kPastCacheProductsUs = 20;

// Compact form of the work list: the items of one tile of a sequence differ only by KV head and
// key span, so an item is a number (unit << head_bits | kv_head) << span_bits | span (2 bytes
// when all fit) and a unit holds the rest.  expand_unit() is the one definition of what an item then is:
// the device builds the records with it, and the host accepts the compact form only if it gives back
// every record.  No divisions: the device expands an item each time that a work-group takes one.
struct CompactUnit {
  int32_t seq, prefix_len, chunk_len, q_off;
  uint32_t tile;      // tile of the chunk | head group << 24
  uint32_t per;       // keys per span | wide << 31
  uint32_t partial;   // first partial slot of KV head 0 | slots per KV head << 16
  uint32_t merge;     // merge group of KV head 0 | groups per KV head << 12 | spans << 24
};
static_assert(sizeof(CompactUnit) == 32, "two 16-byte vectors");
struct CompactPlan {
  int32_t n_items, n_units, head_bits, span_bits;
  int32_t group_heads, heads_per_kv, wide_tok, ref_bytes;  // ref_bytes: 2 or 4
  int32_t past_cache;                                      // Plan::past_cache
};
CRONUS_HOST_DEVICE inline uint32_t unit_of_ref(const CompactPlan& c, uint32_t ref) { return ref >> (c.head_bits + c.span_bits); }
CRONUS_HOST_DEVICE inline WorkItem expand_unit(const CompactPlan& c, const CompactUnit& u, uint32_t ref) {
  const int32_t span = (int32_t)(ref & ((1u << c.span_bits) - 1)), kvh = (int32_t)(ref >> c.span_bits & ((1u << c.head_bits) - 1));
  const int32_t first_head = (int32_t)(u.tile >> 24) * c.group_heads, per = (int32_t)(u.per & 0x7fffffffu);
  const int32_t n_split = (int32_t)(u.merge >> 24);
  const bool wide = u.per >> 31;
  WorkItem w;
  w.seq = u.seq;
  w.kv_head = kvh;
  w.head0 = kvh * c.heads_per_kv + first_head;
  w.n_heads = c.heads_per_kv - first_head < c.group_heads ? c.heads_per_kv - first_head : c.group_heads;
  w.q_tok0 = (int32_t)(u.tile & 0xffffffu) * c.wide_tok;
  w.n_tok = u.chunk_len - w.q_tok0 < c.wide_tok ? u.chunk_len - w.q_tok0 : c.wide_tok;
  const int32_t kv_total = u.prefix_len + w.q_tok0 + w.n_tok;
  w.kv_begin = span * per;
  w.kv_end = kv_total - w.kv_begin < per ? kv_total : w.kv_begin + per;
  w.first_partial = (int32_t)(u.partial & 0xffffu) + kvh * (int32_t)(u.partial >> 16);
  w.partial = n_split > 1 ? w.first_partial + span * (wide ? kWaves : 1) : -1;
  w.merge_key = n_split * kMaxMergeGroups + (int32_t)(u.merge & 0xfffu) + kvh * (int32_t)(u.merge >> 12 & 0xfffu);
  w.wide = wide;
  w.prefix_len = u.prefix_len;
  w.chunk_len = u.chunk_len;
  w.q_off = u.q_off;
  if (wide) w.n_blocks = (u.prefix_len + u.chunk_len + kBlock - 1) / kBlock;
  else w.peers = c.past_cache && w.n_tok == u.chunk_len ? 0 : -1;  // no peers yet
  return w;
}
// Units lie in the order of their sequences, so a decode's peers are found beside its own unit, where the sequences
// between them have one unit each.
CRONUS_HOST_DEVICE inline bool is_peer(const CompactUnit& v, int32_t seq, int32_t offset, int32_t column) {
  return (v.seq == seq + offset) & (column * kBlock < v.prefix_len + v.chunk_len);
}
CRONUS_HOST_DEVICE inline WorkItem expand_item(const CompactPlan& c, const CompactUnit* units, uint32_t ref) {
  const int32_t unit = (int32_t)unit_of_ref(c, ref);
  WorkItem w = expand_unit(c, units[unit], ref);
  if (!w.wide && w.peers == 0) {
    const int32_t column = peer_column(w.kv_begin, w.kv_end);
    for (int32_t b = 0; b < kPeers; ++b) {
      const int32_t v = unit + peer_offset(b);
      if (v >= 0 && v < c.n_units && is_peer(units[v], w.seq, peer_offset(b), column)) w.peers |= 1 << b;
    }
  }
  return w;
}
// A static call's list of at most this many bytes and with 2-byte references travels in the main kernel's own arguments (up to
// kShortListBytes in a smaller set of them).  More do not fit in 4 KiB next to the other arguments.
constexpr int kListBytes = 3840, kShortListBytes = 1280;
// A call of cronus_attn_mixed or cronus_iteration with at most this many items passes their records in the main kernel's arguments
// (3 KiB; new rows and the other arguments take 0.6 of the 4 KiB that there are).  us a pass, records in host memory / in the
// arguments: 12 items, a chunk of 64 next to 4 decodes 12.9 / 11.4; 3 decodes, 7 heads a KV head 11.2 / 8.4; a decode of 300, 8 KV heads
// 10.6 / 9.2; 40 items, 5 decodes 10.9 / 9.6; 8 of 64 .. 700, 7 heads 13.0 / 10.4; two chunk tiles a KV head next to 2 decodes 14.9 / 13.5.  Room for
// 16, 32 or 48: 12 items 11.6 / 11.8 / 11.7.
constexpr int kFewItems = 48;

// Rows whose partial results (split over key spans) are combined, for inspection (the kernels
// find what they need in the work items):
// rows row0 .. row0 + n_rows - 1 of the tile (row r = token r / n_heads, head r % n_heads);
// span s left them in partial slot first_partial + s * stride, at slot rows 0 .. n_rows - 1.
// A narrow item fills one slot (stride 1, row0 0); a split wide tile fills kWaves slots
// per span, one per wavefront (stride kWaves, row0 = 32 * wavefront).
struct MergeItem {
  int32_t first_partial;
  int32_t n_split;
  int32_t seq;
  int32_t kv_head;
  int32_t head0;
  int32_t n_heads;
  int32_t q_tok0;
  int32_t n_tok;
  int32_t row0;
  int32_t n_rows;
  int32_t stride;
  int32_t q_off;  // the sequence's first row in q/out (copy of SeqInfo::q_off: one dependent load less)
};

// A sequence of an fp8 cache whose chunk has many tiles: its K/V blocks 0 .. n_blocks - 1 are
// converted to bf16 once per launch, into blocks blk0 .. of a copy in the workspace (same
// layout as the cache, 2 bytes per element), and its wide tiles read that copy.
struct StageSeq {
  int32_t seq;
  int32_t blk0;
  int32_t n_blocks;
  int32_t pad;
};

struct Plan {
  // sizes
  int64_t n_items = 0, n_wide = 0, n_partials = 0, n_merge = 0, n_merge_rows = 0;
  int32_t n_seqs = 0;
  int32_t wide_rows = 0;  // rows per wide tile (compile-time choice of the kernel instance)
  int32_t past_cache = 0;  // 1: the decodes' K/V passes the caches (WorkItem::peers; one head group, kPastCacheBytes or kPastCacheProductsUs)
  int32_t n_stage_seqs = 0;
  int64_t n_stage_blocks = 0;
  // The work items form kQueues queues, stored one after the other: queue x is items
  // q_base[x] .. q_base[x] + q_len[x] - 1 in the order in which they should be taken.  The
  // main kernel runs n_workgroups resident work-groups that take items from the queue of the
  // XCD they run on until it is empty, then from the others.
  int32_t q_base[kQueues] = {0}, q_len[kQueues] = {0};
  int32_t n_workgroups = 0;
  // byte offsets inside the plan image (host-built metadata that the kernels read:
  // [WorkItem x n_items | MergeItem x n_merge | StageSeq x n_stage_seqs]) and its size
  size_t off_items = 0, off_merge = 0, off_stage = 0, image_bytes = 0;
  // byte offsets inside the caller's workspace (partial results; fp8: the bf16 copy) and its size
  size_t off_partials = 0, off_stage_k = 0, off_stage_v = 0, total_bytes = 0;
};

// Number of floats of one partial slot: O (32 x D), then (m, l) of 32 rows.
inline size_t partial_floats(int head_dim) { return (size_t)kNarrowRows * (head_dim + 2); }

// Rows per wide tile for a head shape (must match the kernel instance that is launched).
int wide_rows_for(int head_dim, int kv_dtype);

// Builds the work decomposition (sizes and offsets into *plan; the work list itself stays
// in a per-thread scratch).  write_plan() then copies that list into host_buf, which must
// hold plan->image_bytes bytes; it must follow build_plan() on the same thread.
// allow_stage = false: an fp8 cache gets no bf16 copy (every chunk tile converts codes on
// the fly), so the workspace holds partial results only.  scratch_limit > 0: the wide tiles of a
// launch that picks its span length get no cut whose list and partial results exceed that many bytes.
// lean: the cut that library versions up to 505 chose, for a workspace that is too small for the faster one.
int build_plan(const cronus_kv_cache* cache, const int32_t* prefix_lens, const int32_t* chunk_lens,
               int32_t n_seqs, int32_t max_blocks_per_seq, int n_cus, Plan* plan, bool allow_stage = true,
               size_t scratch_limit = 0, bool lean = false);
void write_plan(const Plan* plan, void* host_buf);
// The same list in compact form ([CompactUnit x n_units | references], *bytes of buf used, a
// multiple of 16), when it can be expressed (it holds every record) and fits in `capacity`.
// Checking every record costs the host less than the launches it saves the static entry point (host time of a
// call there, records / compact: 512 items 66 / 26 us, 1024 110 / 49, 2800 246 / 119).  The other one writes its
// records to host memory: a compact list as an argument saves it 0.5 us of device time a launch, but costs the host 1.6 us more for
// 264 items, 2.9 for 552 and 8 on a first pass.
bool compact_plan(const cronus_kv_cache* cache, const Plan* plan, CompactPlan* c, void* buf, size_t capacity, size_t* bytes);

// Whether the rows of such an iteration are stored past the caches (cronus_iteration).
bool rows_past_cache(const cronus_kv_cache* cache, const int32_t* prefix_lens, const int32_t* chunk_lens, int32_t n_seqs);

// An iteration of at most this many decodes whose one set has a row for each places them in its attention launch: one lane a row, and
// a block is compared with all rows at once.  One launch less and no wait for its last work-group: 1.5 .. 3 us a pass, two launches / one:
// a decode of 8000 keys 18.2 / 16.4, 16 of 500 .. 1500 21.2 / 19.9 (7 heads a KV head 17.5 / 15.3), 64 of 20 .. 250 20.9 / 19.4 (D = 64, 2 KV heads
// 12.7 / 10.1); fp8, 8 of 300 .. 2000 15.9 / 13.6, 64 of 500 .. 1000 32.3 / 31.1.
// The compares come before an item's first requests, about 0.4 us an item and 0.5 us per 1000 keys of what a CU works on, so the rows of launches
// with more than kPlacingKeysPerCu keys a CU, a row counting as kPlacingRowKeys, are scattered: 64 of 4000 .. 8000, 8 KV heads, would take 247.8 / 250.7,
// 64 of 500 .. 1000, 32 KV heads 142.0 / 148.4 (fp8 95.8 / 103.6), 32 of 500 .. 3000 146.4 / 150.6.  Of 187 sets of 1 .. 64 decodes, 2 .. 64 KV heads,
// 134 are within the line, 0.99 .. 1.37 times as fast as with a scatter (10 % less time on average), and of the others none would gain more than 1.3 us.
// Rows that are not one a sequence are stored one after the other by whoever reads their block, so they are scattered too: one KV head a query
// head, 2 chunks of 32 15.7 / 27.3; 4 heads, 16 chunks of 4 22.7 / 26.3, 8 of 8 18.5 / 20.9 (but 8 of 2 18.3 / 16.9); 64 rows of one sequence
// next to a decode 10.9 / 22.8, and 10.8 / 35.0 where no item reads them; decodes of which half have a row 54.1 / 56.0.  Where sequences are skipped,
// a row's sequence is looked for among all, one after the other: with half of the sequences or one skipped, 2 to 8 of 20 .. 3000 keys take
// 0.73 .. 1.02 of what they take with a scatter, 16 up to 1.04, 32 1.08, 64 1.23, so they may be kPlacingSkippedSeqs at most.  (The host knows
// their number only: 20 rows of one sequence next to 20 decodes pass for theirs, and take 25.5 / 30.6.)
constexpr int kMaxNewRows = 64, kPlacingRowKeys = 900, kPlacingKeysPerCu = 4400, kPlacingSkippedSeqs = 8;
bool rows_in_launch(const cronus_kv_cache* cache, const cronus_kv_rows* first, const cronus_kv_rows* second, const int32_t* prefix_lens,
                    const int32_t* chunk_lens, int32_t n_seqs, int n_cus);

struct AttnLaunch {
  const cronus_kv_cache* cache;
  const void* q;
  void* out;
  const int32_t* block_tables;
  int32_t max_blocks_per_seq;
  float sm_scale;
  void* workspace;  // device; holds the partial results at plan->off_partials
  const void* plan_image;  // device-visible [WorkItem | MergeItem | StageSeq] image at the plan's offsets
  const WorkItem* records;  // host; the items of a launch of at most kFewItems, which travel in the arguments, or nullptr
  const void* list;  // host, kListBytes long; the compact list that takes the place of the image's items (copied by
                     // the launch), or nullptr
  CompactPlan compact;
  size_t list_bytes;
  const cronus_kv_rows* rows;  // rows that the main kernel places (rows_in_launch, and no list), or nullptr
  const int32_t* prefix_lens;  // of the call, where there are such rows
  const int32_t* chunk_lens;
  const Plan* plan;
  void* stream;
  int* queue_set;  // device; this call's set of queue heads (kQueueSetInts ints, all zero between launches)
  uint32_t* done_flag;  // device-visible host memory; receives done_value when the main kernel is done with the plan
                        // image and the queue set, or nullptr
  uint32_t done_value;
  // optional hipEvent_t handles (measurement aid): [0], [1] start and stop of the main
  // kernel's dispatch; [2] start of the call's first kernel when that is another one (the
  // fp8 copy); [3] recorded behind the main kernel when that merges results of key spans
  void* ev[4];
};

// One-time set-up of the attention kernels on the current device (dynamic LDS limits);
// call before the first launch_attn() there.
int prepare_attn_kernels();
// *main_launched: whether the main kernel, which reports the end of the call, has been enqueued.
int launch_attn(const AttnLaunch& a, bool* main_launched);

// The no-allocation variant's device memory: a static array in the library's device image
// (attn_mixed.hip).  static_scratch_resolve() looks up its address on the current device
// (once per device, at set-up); static_scratch_upload() enqueues the copy of `bytes` bytes of
// host data to `dst` inside it as kernel arguments (no staging buffer, nothing allocated; the
// host data may be reused as soon as the call returns).
constexpr size_t kStaticScratchBytes = (size_t)64 << 20;
int static_scratch_resolve(void** device_ptr);
// Address, on the current device, of the library's kQueueSets sets of queue heads (a small
// static device array, zero when the library is loaded; every launch leaves its set zero).
int queue_sets_resolve(int** device_ptr);
int static_scratch_upload(void* dst, const void* host_src, size_t bytes, void* stream);
// Enqueues the launches that build the work items of a compact list at `items` (device), through `staging`
// (device, 16-byte aligned, `bytes` bytes): for a list of more than kListBytes.
int static_scratch_expand(void* items, void* staging, const CompactPlan& c, const void* host_src, size_t bytes, void* stream);
constexpr int kMaxScatterHeads = 65535;  // KV heads that the scatter and the gather accept: their grids' y dimension
// second may be null; past_cache: the rows do not stay in the caches (non-temporal stores)
int launch_kv_append(const cronus_kv_cache* cache, const cronus_kv_rows* first, const cronus_kv_rows* second,
                     const int32_t* block_tables, int32_t max_blocks_per_seq, int32_t n_seqs, void* stream,
                     bool past_cache = false);
int launch_kv_gather(const cronus_kv_cache* cache, void* k_dst, void* v_dst, const int32_t* cu_tokens,
                     const int32_t* start_pos, const int32_t* block_tables, int32_t max_blocks_per_seq,
                     int32_t n_seqs, int32_t n_tokens, void* stream);

// mfma_probe.hip (measurement aid)
int launch_mfma_probe(bool small_shape, int random_operands, int iters, int n_cus, float* sink, void* stream, double* flops);
int mfma_probe_sink_floats(int n_cus);

}  // namespace cronus
