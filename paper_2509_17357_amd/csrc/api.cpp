// C ABI entry points (include/cronus.h): argument checks, plan upload, launches.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstring>
#include <mutex>
#include <vector>

#include "cronus_internal.h"
#include "plan_ring.h"

namespace cronus {
namespace {

int check_cache(const cronus_kv_cache* c) {
  if (!c || !c->k_cache || !c->v_cache || c->num_blocks <= 0) return CRONUS_ERR_INVALID_ARG;
  if (c->num_q_heads <= 0 || c->num_kv_heads <= 0) return CRONUS_ERR_INVALID_ARG;
  if (c->block_size != kBlock) return CRONUS_ERR_UNSUPPORTED;
  if (c->head_dim != 64 && c->head_dim != 128) return CRONUS_ERR_UNSUPPORTED;
  if (c->num_q_heads % c->num_kv_heads) return CRONUS_ERR_UNSUPPORTED;
  if (c->kv_dtype == CRONUS_KV_BF16) {
    if (c->k_scale || c->v_scale) return CRONUS_ERR_INVALID_ARG;
  } else if (c->kv_dtype == CRONUS_KV_FP8_E4M3) {
    if (!c->k_scale || !c->v_scale) return CRONUS_ERR_INVALID_ARG;
  } else {
    return CRONUS_ERR_UNSUPPORTED;
  }
  return CRONUS_OK;
}

// Shape-only variant for the size queries, which need no device pointers.
int check_shape(const cronus_kv_cache* c) {
  if (!c || c->num_q_heads <= 0 || c->num_kv_heads <= 0) return CRONUS_ERR_INVALID_ARG;
  if (c->block_size != kBlock) return CRONUS_ERR_UNSUPPORTED;
  if (c->head_dim != 64 && c->head_dim != 128) return CRONUS_ERR_UNSUPPORTED;
  if (c->num_q_heads % c->num_kv_heads) return CRONUS_ERR_UNSUPPORTED;
  if (c->kv_dtype != CRONUS_KV_BF16 && c->kv_dtype != CRONUS_KV_FP8_E4M3) return CRONUS_ERR_UNSUPPORTED;
  return CRONUS_OK;
}

// Per-device facts and one-time set-up, guarded by g_mu.  Index = HIP device ordinal.
struct DeviceState {
  int n_cus = 0;           // 0: not queried yet
  bool kernels_ready = false;
  void* static_scratch = nullptr;  // this device's address of the library's static scratch array
  int* queue_sets = nullptr;       // and of its sets of queue heads
};
constexpr int kMaxDevices = 64;
DeviceState g_dev[kMaxDevices];
std::mutex g_mu;

// CU count of the current device; 256 (MI355X) when sizes are queried without a device.
int device_cus() {
  int dev = 0, n = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) {
    (void)hipGetLastError();
    return 256;
  }
  std::lock_guard<std::mutex> lock(g_mu);
  if (g_dev[dev].n_cus) return g_dev[dev].n_cus;
  if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) {
    (void)hipGetLastError();
    return 256;
  }
  g_dev[dev].n_cus = n;
  return n;
}

// Set-up that must precede the first launch on the current device (kernel attributes).
// Caller holds g_mu.
int prepare_device_locked(int* device) {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return CRONUS_ERR_HIP;
  *device = dev;
  if (!g_dev[dev].kernels_ready) {
    if (int rc = prepare_attn_kernels()) return rc;
    if (int rc = static_scratch_resolve(&g_dev[dev].static_scratch)) return rc;
    if (int rc = queue_sets_resolve(&g_dev[dev].queue_sets)) return rc;
    g_dev[dev].kernels_ready = true;
  }
  return CRONUS_OK;
}

constexpr size_t kSlotHeader = 256;  // bytes in front of the plan image: the number of the last finished call
void* g_ev[4] = {nullptr, nullptr, nullptr, nullptr};

static_assert(kQueueSets == kSlots + 1, "one set of queue heads per plan buffer, one for the static entry point");
PlanRing g_rings[kMaxDevices];  // a ring per device: a slot's memory is mapped for one

// A captured call runs when its graph does, and again with every replay.
bool is_capturing(hipStream_t stream) {
  hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
  if (stream == nullptr) return false;  // the default stream cannot be captured
  if (hipStreamIsCapturing(stream, &st) != hipSuccess) {
    (void)hipGetLastError();
    return false;
  }
  return st != hipStreamCaptureStatusNone;
}

// A plan buffer of at least `bytes` behind its header, or nullptr.  The caller holds g_mu through `lock`.
Slot* acquire_slot(int dev, size_t bytes, hipStream_t stream, std::unique_lock<std::mutex>& lock) {
  bytes += kSlotHeader;
  Slot* s = wait_for_slot(g_rings[dev], lock, stream, std::chrono::seconds(10), [&] {
    if (is_capturing(stream)) return StreamIs::kBusy;
    const hipError_t e = hipStreamQuery(stream);
    if (e == hipSuccess) return StreamIs::kDone;
    (void)hipGetLastError();
    return e == hipErrorNotReady ? StreamIs::kBusy : StreamIs::kFailed;
  });
  if (!s) return nullptr;
  if (s->cap < bytes) {
    if (s->host) (void)hipHostFree(s->host);
    s->host = s->dev = nullptr;
    s->cap = 0;
    size_t cap = 1 << 16;
    while (cap < bytes) cap <<= 1;
    if (hipHostMalloc(&s->host, cap, hipHostMallocMapped | hipHostMallocPortable) != hipSuccess) return nullptr;
    if (hipHostGetDevicePointer(&s->dev, s->host, 0) != hipSuccess) {
      (void)hipHostFree(s->host);
      s->host = nullptr;
      return nullptr;
    }
    s->cap = cap;
    *static_cast<volatile uint32_t*>(s->host) = s->call;
  }
  return s;
}

}  // namespace
}  // namespace cronus

using namespace cronus;

extern "C" {

int cronus_kv_append(const cronus_kv_cache* cache, const void* k_src, const void* v_src,
                     const int32_t* cu_tokens, const int32_t* start_pos, const int32_t* block_tables,
                     int32_t max_blocks_per_seq, int32_t n_seqs, int32_t n_tokens, void* hip_stream) {
  if (int rc = check_cache(cache)) return rc;
  if (n_seqs < 0 || n_tokens < 0 || max_blocks_per_seq <= 0) return CRONUS_ERR_INVALID_ARG;
  if (n_tokens == 0 || n_seqs == 0) return CRONUS_OK;
  if (!k_src || !v_src || !cu_tokens || !start_pos || !block_tables) return CRONUS_ERR_INVALID_ARG;
  const cronus_kv_rows rows{k_src, v_src, cu_tokens, start_pos, n_tokens};
  return launch_kv_append(cache, &rows, nullptr, block_tables, max_blocks_per_seq, n_seqs, hip_stream);
}

// Checks two sets of rows; then *first is null when there is none, *second when there are not two.
static int check_rows(const cronus_kv_cache* cache, const cronus_kv_rows** first, const cronus_kv_rows** second,
                      const int32_t* block_tables, int32_t max_blocks_per_seq, int32_t n_seqs) {
  if (int rc = check_cache(cache)) return rc;
  if (!*first || !*second || n_seqs < 0 || max_blocks_per_seq <= 0) return CRONUS_ERR_INVALID_ARG;
  for (const cronus_kv_rows* r : {*first, *second}) {
    if (r->n_tokens < 0) return CRONUS_ERR_INVALID_ARG;
    if (r->n_tokens > 0 && n_seqs > 0 && (!r->k_src || !r->v_src || !r->cu_tokens || !r->start_pos || !block_tables))
      return CRONUS_ERR_INVALID_ARG;
  }
  if ((*first)->n_tokens == 0) std::swap(*first, *second);
  if ((*second)->n_tokens == 0 || n_seqs == 0) *second = nullptr;
  if ((*first)->n_tokens == 0 || n_seqs == 0) *first = nullptr;
  return CRONUS_OK;
}

int cronus_kv_append_pair(const cronus_kv_cache* cache, const cronus_kv_rows* first, const cronus_kv_rows* second,
                          const int32_t* block_tables, int32_t max_blocks_per_seq, int32_t n_seqs, void* hip_stream) {
  if (int rc = check_rows(cache, &first, &second, block_tables, max_blocks_per_seq, n_seqs)) return rc;
  if (!first) return CRONUS_OK;
  return launch_kv_append(cache, first, second, block_tables, max_blocks_per_seq, n_seqs, hip_stream);
}

int cronus_kv_gather(const cronus_kv_cache* cache, void* k_dst, void* v_dst, const int32_t* cu_tokens,
                     const int32_t* start_pos, const int32_t* block_tables, int32_t max_blocks_per_seq,
                     int32_t n_seqs, int32_t n_tokens, void* hip_stream) {
  if (int rc = check_cache(cache)) return rc;
  if (n_seqs < 0 || n_tokens < 0 || max_blocks_per_seq <= 0) return CRONUS_ERR_INVALID_ARG;
  if (n_tokens == 0 || n_seqs == 0) return CRONUS_OK;
  if (!k_dst || !v_dst || !cu_tokens || !start_pos || !block_tables) return CRONUS_ERR_INVALID_ARG;
  return launch_kv_gather(cache, k_dst, v_dst, cu_tokens, start_pos, block_tables, max_blocks_per_seq, n_seqs,
                          n_tokens, hip_stream);
}

size_t cronus_probe_mfma_sink_floats(void) { return (size_t)mfma_probe_sink_floats(device_cus()); }

static int probe_mfma(bool small_shape, int random_operands, int iters, float* sink, size_t sink_floats, void* hip_stream,
                      double* flops_host) {
  if (iters < 1 || iters > (1 << 20) || !sink || !flops_host) return CRONUS_ERR_INVALID_ARG;
  const int n_cus = device_cus();
  if (sink_floats < (size_t)mfma_probe_sink_floats(n_cus)) return CRONUS_ERR_WORKSPACE;
  return launch_mfma_probe(small_shape, random_operands, iters, n_cus, sink, hip_stream, flops_host);
}

int cronus_probe_mfma(int random_operands, int iters, float* sink, size_t sink_floats, void* hip_stream,
                      double* flops_host) {
  return probe_mfma(false, random_operands, iters, sink, sink_floats, hip_stream, flops_host);
}

int cronus_probe_mfma_16x16x32(int random_operands, int iters, float* sink, size_t sink_floats, void* hip_stream,
                               double* flops_host) {
  return probe_mfma(true, random_operands, iters, sink, sink_floats, hip_stream, flops_host);
}

size_t cronus_attn_mixed_workspace_bytes(const cronus_kv_cache* cache, const int32_t* prefix_lens,
                                         const int32_t* chunk_lens, int32_t n_seqs) {
  if (check_shape(cache) || n_seqs < 0 || (n_seqs > 0 && (!prefix_lens || !chunk_lens))) return 0;
  Plan plan;
  if (build_plan(cache, prefix_lens, chunk_lens, n_seqs, 0x7fffffff / kBlock, device_cus(), &plan)) return 0;
  return plan.total_bytes;
}

int cronus_attn_mixed_plan_stats(const cronus_kv_cache* cache, const int32_t* prefix_lens,
                                 const int32_t* chunk_lens, int32_t n_seqs, int64_t* stats) {
  if (int rc = check_shape(cache)) return rc;
  if (!stats || n_seqs < 0 || (n_seqs > 0 && (!prefix_lens || !chunk_lens))) return CRONUS_ERR_INVALID_ARG;
  Plan plan;
  if (int rc = build_plan(cache, prefix_lens, chunk_lens, n_seqs, 0x7fffffff / kBlock, device_cus(), &plan))
    return rc;
  stats[0] = plan.n_items;
  stats[1] = plan.n_wide;
  stats[2] = plan.n_partials;
  stats[3] = plan.n_merge_rows;
  stats[4] = plan.n_merge;
  stats[5] = plan.n_stage_blocks;
  return CRONUS_OK;
}

int64_t cronus_attn_mixed_plan_items(const cronus_kv_cache* cache, const int32_t* prefix_lens,
                                     const int32_t* chunk_lens, int32_t n_seqs, int32_t* items, int64_t capacity) {
  if (int rc = check_shape(cache)) return -rc;
  if (n_seqs < 0 || capacity < 0 || (n_seqs > 0 && (!prefix_lens || !chunk_lens)) || (capacity > 0 && !items))
    return -CRONUS_ERR_INVALID_ARG;
  Plan plan;
  if (int rc = build_plan(cache, prefix_lens, chunk_lens, n_seqs, 0x7fffffff / kBlock, device_cus(), &plan)) return -rc;
  std::vector<unsigned char> buf(plan.image_bytes);
  write_plan(&plan, buf.data());
  const int64_t n = std::min<int64_t>(capacity, plan.n_items);
  const WorkItem* wi = reinterpret_cast<const WorkItem*>(buf.data() + plan.off_items);
  int queue = 0;
  for (int64_t i = 0; i < n; ++i) {
    while (queue + 1 < kQueues && i >= plan.q_base[queue] + plan.q_len[queue]) ++queue;
    const WorkItem& w = wi[i];
    const int32_t row[11] = {w.seq, w.kv_head, w.head0, w.n_heads, w.q_tok0, w.n_tok, w.kv_begin, w.kv_end,
                             w.partial, w.wide, queue};
    std::memcpy(items + 11 * i, row, sizeof(row));
  }
  return plan.n_items;
}

namespace {

// Host-side checks shared by the two attention entry points; *total_q = sum of chunk_lens.
int check_attn_args(const cronus_kv_cache* cache, const void* q, const void* out, const int32_t* prefix_lens,
                    const int32_t* chunk_lens, const int32_t* block_tables, int32_t max_blocks_per_seq,
                    int32_t n_seqs, float sm_scale, long long* total_q) {
  *total_q = 0;
  if (int rc = check_cache(cache)) return rc;
  if (n_seqs < 0 || max_blocks_per_seq <= 0) return CRONUS_ERR_INVALID_ARG;
  if (!(sm_scale > 0.f) || !std::isfinite(sm_scale)) return CRONUS_ERR_INVALID_ARG;
  if (n_seqs == 0) return CRONUS_OK;
  if (!prefix_lens || !chunk_lens || !block_tables) return CRONUS_ERR_INVALID_ARG;
  long long total = 0;
  for (int s = 0; s < n_seqs; ++s) {
    if (chunk_lens[s] < 0 || prefix_lens[s] < 0) return CRONUS_ERR_INVALID_ARG;
    total += chunk_lens[s];
  }
  if (total > 0 && (total > 0x7fffffffLL || !q || !out)) return CRONUS_ERR_INVALID_ARG;
  *total_q = total;
  return CRONUS_OK;
}

// What the launches of both attention entry points have in common; the caller holds g_mu.
AttnLaunch attn_launch(const cronus_kv_cache* cache, const void* q, void* out, const int32_t* block_tables, int32_t max_blocks_per_seq,
                       float sm_scale, const Plan& plan, void* hip_stream) {
  AttnLaunch a{};
  a.cache = cache;
  a.q = q;
  a.out = out;
  a.block_tables = block_tables;
  a.max_blocks_per_seq = max_blocks_per_seq;
  a.sm_scale = sm_scale;
  a.plan = &plan;
  a.stream = hip_stream;
  std::copy(g_ev, g_ev + 4, a.ev);
  return a;
}

// Whether an array that the rows are read from shares memory with [p, p + bytes).
bool read_from(const cronus_kv_cache* cache, const cronus_kv_rows* rows, int32_t n_seqs, const void* p, size_t bytes) {
  auto meets = [&](const void* src, size_t n) {
    const uintptr_t a = reinterpret_cast<uintptr_t>(src), b = reinterpret_cast<uintptr_t>(p);
    return a < b + bytes && b < a + n;
  };
  const size_t values = (size_t)rows->n_tokens * cache->num_kv_heads * cache->head_dim * 2, ints = (size_t)n_seqs * sizeof(int32_t);
  return meets(rows->k_src, values) || meets(rows->v_src, values) || meets(rows->cu_tokens, ints + sizeof(int32_t)) || meets(rows->start_pos, ints);
}

bool workspace_refused(const void* workspace) { return !workspace || (reinterpret_cast<uintptr_t>(workspace) & 255u); }

// cronus_attn_mixed behind the placing of the rows of `first` and `second` (null: none).
int attn_mixed(const cronus_kv_cache* cache, const cronus_kv_rows* first, const cronus_kv_rows* second, const void* q, void* out,
               const int32_t* prefix_lens, const int32_t* chunk_lens, const int32_t* block_tables, int32_t max_blocks_per_seq,
               int32_t n_seqs, float sm_scale, void* workspace, size_t workspace_bytes, void* hip_stream) {
  long long total_q = 0;
  if (int rc = check_attn_args(cache, q, out, prefix_lens, chunk_lens, block_tables, max_blocks_per_seq, n_seqs,
                               sm_scale, &total_q))
    return rc;
  if (first) {
    // What build_plan and the workspace refuse: no row is placed for these lengths, whose scatter would read the table
    // beyond the sequence's own entries.
    if (total_q > 0) {
      for (int s = 0; s < n_seqs; ++s)
        if ((long long)prefix_lens[s] + chunk_lens[s] > (long long)max_blocks_per_seq * kBlock) return CRONUS_ERR_INVALID_ARG;
      if (workspace_refused(workspace)) return CRONUS_ERR_WORKSPACE;
    }
  }
  auto place_rows = [&] {
    return launch_kv_append(cache, first, second, block_tables, max_blocks_per_seq, n_seqs, hip_stream,
                            rows_past_cache(cache, prefix_lens, chunk_lens, n_seqs));
  };
  const int n_cus = device_cus();
  // (rows that lie in what the attention writes are read before it starts)
  bool in_launch = total_q > 0 && rows_in_launch(cache, first, second, prefix_lens, chunk_lens, n_seqs, n_cus) &&
                   !read_from(cache, first, n_seqs, out, (size_t)total_q * cache->num_q_heads * cache->head_dim * 2) &&
                   !read_from(cache, first, n_seqs, workspace, workspace_bytes);
  auto refused = [&](int rc) {  // after the checks, with the attention not enqueued: the rows are placed all the same
    const int placed = in_launch ? place_rows() : CRONUS_OK;
    return placed ? placed : rc;
  };
  if (first && !in_launch) {
    // before the plan is built, so that the device works meanwhile (whole prompts, a first pass:
    // 400 us, 446 with the plan first)
    if (int rc = place_rows()) return rc;
  }
  if (total_q == 0) return CRONUS_OK;

  Plan plan;
  if (int rc = build_plan(cache, prefix_lens, chunk_lens, n_seqs, max_blocks_per_seq, n_cus, &plan)) return rc;
  if (workspace_refused(workspace)) return CRONUS_ERR_WORKSPACE;
  // a workspace that served these lengths before the tiles were cut finer still does
  if (workspace_bytes < plan.total_bytes) {
    if (int rc = build_plan(cache, prefix_lens, chunk_lens, n_seqs, max_blocks_per_seq, n_cus, &plan, true, 0, true)) return rc;
  }
  if (workspace_bytes < plan.total_bytes) return refused(CRONUS_ERR_WORKSPACE);
  if (plan.n_items > 0x7fffffffLL) return CRONUS_ERR_INVALID_ARG;
  if (in_launch && plan.n_wide > 0) {  // the kernels that place rows have no chunk tiles; a decode's item is narrow, and the plan has the last word
    if (int rc = place_rows()) return rc;
    in_launch = false;
  }

  hipStream_t stream = static_cast<hipStream_t>(hip_stream);
  std::unique_lock<std::mutex> lock(g_mu);
  // everything that can fail without a launch comes first: kernel attributes, the plan buffer
  int dev = 0;
  if (int rc = prepare_device_locked(&dev)) return refused(rc);
  Slot* slot = acquire_slot(dev, plan.image_bytes, stream, lock);
  if (!slot) return refused(CRONUS_ERR_HIP);
  unsigned char* const host = static_cast<unsigned char*>(slot->host);
  unsigned char* const dev_mem = static_cast<unsigned char*>(slot->dev);
  write_plan(&plan, host + kSlotHeader);
  // the set of queue heads that belongs to this plan buffer: free again when the buffer is
  const int set = (int)(slot - g_rings[dev].slots);
  AttnLaunch a = attn_launch(cache, q, out, block_tables, max_blocks_per_seq, sm_scale, plan, hip_stream);
  a.workspace = workspace;
  a.plan_image = dev_mem + kSlotHeader;
  if (plan.n_items <= std::min<int64_t>(kFewItems, plan.n_workgroups))
    a.records = reinterpret_cast<const WorkItem*>(host + kSlotHeader + plan.off_items);
  if (in_launch) a.rows = first;
  a.prefix_lens = prefix_lens;
  a.chunk_lens = chunk_lens;
  a.queue_set = g_dev[dev].queue_sets + set * kQueueSetInts;
  a.done_flag = reinterpret_cast<uint32_t*>(dev_mem);
  a.done_value = ++slot->call;
  slot->stream = stream;
  slot->state = is_capturing(stream) ? Slot::kLost : Slot::kPending;
  bool main_launched = false;
  const int rc = launch_attn(a, &main_launched);
  if (!main_launched && slot->state == Slot::kPending) {
    lock.unlock();
    (void)hipStreamSynchronize(stream);  // an earlier kernel of the failed call may read the slot
    lock.lock();
    slot->state = Slot::kFree;
  }
  return main_launched ? rc : refused(rc);
}

}  // namespace

int cronus_attn_mixed(const cronus_kv_cache* cache, const void* q, void* out, const int32_t* prefix_lens,
                      const int32_t* chunk_lens, const int32_t* block_tables, int32_t max_blocks_per_seq,
                      int32_t n_seqs, float sm_scale, void* workspace, size_t workspace_bytes, void* hip_stream) {
  return attn_mixed(cache, nullptr, nullptr, q, out, prefix_lens, chunk_lens, block_tables, max_blocks_per_seq, n_seqs, sm_scale,
                    workspace, workspace_bytes, hip_stream);
}

int cronus_iteration(const cronus_kv_cache* cache, const cronus_kv_rows* first, const cronus_kv_rows* second, const void* q,
                     void* out, const int32_t* prefix_lens, const int32_t* chunk_lens, const int32_t* block_tables,
                     int32_t max_blocks_per_seq, int32_t n_seqs, float sm_scale, void* workspace, size_t workspace_bytes,
                     void* hip_stream) {
  if (int rc = check_rows(cache, &first, &second, block_tables, max_blocks_per_seq, n_seqs)) return rc;
  return attn_mixed(cache, first, second, q, out, prefix_lens, chunk_lens, block_tables, max_blocks_per_seq, n_seqs, sm_scale,
                    workspace, workspace_bytes, hip_stream);
}

int cronus_attn_mixed_static(const cronus_kv_cache* cache, const void* q, void* out, const int32_t* prefix_lens,
                             const int32_t* chunk_lens, const int32_t* block_tables, int32_t max_blocks_per_seq,
                             int32_t n_seqs, float sm_scale, void* hip_stream) {
  long long total_q = 0;
  if (int rc = check_attn_args(cache, q, out, prefix_lens, chunk_lens, block_tables, max_blocks_per_seq, n_seqs,
                               sm_scale, &total_q))
    return rc;
  if (total_q == 0) return CRONUS_OK;

  // no bf16 copy of fp8 sequences here: it can take a gigabyte; their chunk tiles convert on the fly
  Plan plan;
  if (int rc = build_plan(cache, prefix_lens, chunk_lens, n_seqs, max_blocks_per_seq, device_cus(), &plan, false))
    return rc;
  if (plan.n_items > 0x7fffffffLL) return CRONUS_ERR_INVALID_ARG;
  // scratch layout: [plan image | partial results]; both sizes are multiples of 256
  auto fits = [&] { return plan.image_bytes <= kStaticScratchBytes && plan.total_bytes <= kStaticScratchBytes - plan.image_bytes; };
  // the fastest cut of the wide tiles may not fit where a coarser one does
  if (!fits()) {
    if (int rc = build_plan(cache, prefix_lens, chunk_lens, n_seqs, max_blocks_per_seq, device_cus(), &plan, false, kStaticScratchBytes))
      return rc;
  }
  if (!fits()) return CRONUS_ERR_WORKSPACE;

  std::lock_guard<std::mutex> lock(g_mu);
  int dev = 0;
  if (int rc = prepare_device_locked(&dev)) return rc;  // first call on a device: looks up its scratch address
  unsigned char* base = static_cast<unsigned char*>(g_dev[dev].static_scratch);
  static thread_local std::vector<unsigned char> image;  // host memory; grows to the largest plan seen
  image.resize(std::max(plan.image_bytes, (size_t)kListBytes));
  // the compact list, when there is one and the scratch has room to stage it behind the rest
  CompactPlan compact{};
  size_t compact_bytes = 0;
  const bool compacted = compact_plan(cache, &plan, &compact, image.data(), plan.image_bytes, &compact_bytes);
  // a short one travels in the main kernel's arguments
  const bool listed = compacted && compact_bytes <= (size_t)kListBytes && compact.ref_bytes == 2;
  if (listed) {
    // nothing to upload
  } else if (compacted && compact_bytes <= kStaticScratchBytes - plan.image_bytes - plan.total_bytes) {
    if (int rc = static_scratch_expand(base + plan.off_items, base + plan.image_bytes + plan.total_bytes, compact, image.data(),
                                       compact_bytes, hip_stream))
      return rc;
  } else {
    write_plan(&plan, image.data());
    if (int rc = static_scratch_upload(base, image.data(), plan.image_bytes, hip_stream)) return rc;
  }
  // Nothing in the scratch has to start at zero: the kernels read the plan image that was just
  // stored and, of the partial slots, exactly the rows that items of this call write first.
  // (The heads of the work queues, which must, live in their own small array, and every
  // launch leaves them zero.)
  AttnLaunch a = attn_launch(cache, q, out, block_tables, max_blocks_per_seq, sm_scale, plan, hip_stream);
  a.workspace = base + plan.image_bytes;
  a.plan_image = base;
  if (listed) {
    a.list = image.data();
    a.list_bytes = compact_bytes;
  }
  a.compact = compact;
  a.queue_set = g_dev[dev].queue_sets + kSlots * kQueueSetInts;
  bool main_launched = false;
  return launch_attn(a, &main_launched);
}

void cronus_profile_events(void* main_start, void* main_stop, void* first_start, void* last_stop) {
  std::lock_guard<std::mutex> lock(g_mu);
  g_ev[0] = main_start;
  g_ev[1] = main_stop;
  g_ev[2] = first_start;
  g_ev[3] = last_stop;
}

const char* cronus_status_string(int status) {
  switch (status) {
    case CRONUS_OK: return "ok";
    case CRONUS_ERR_INVALID_ARG: return "invalid argument";
    case CRONUS_ERR_UNSUPPORTED: return "unsupported shape or dtype";
    case CRONUS_ERR_WORKSPACE: return "workspace missing, misaligned or too small";
    case CRONUS_ERR_HIP: return "HIP runtime error";
    default: return "unknown status";
  }
}

int cronus_version(void) { return 511; }  // 0.5.11: decode iterations place their rows in the attention launch only where that is faster and the rows do not lie in what it writes

}  // extern "C"
