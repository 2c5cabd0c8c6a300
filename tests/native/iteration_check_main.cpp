// Host-only driver of cronus_iteration (api.cpp, plan.cpp as they are; the launches and the HIP calls are the stubs below): which
// launches a call enqueues, in order, and what it returns.  Arguments:
//   <Hq> <Hkv> <D> <fp8 0|1> <failure> <rows of the first set> <of the second> <k_src> <v_src> <cu_tokens> <start_pos> <out>
//   <workspace> <workspace bytes> <n_seqs> P0 C0 P1 C1 ...
// failure: none, setup (kernel attributes), buffer (pinned memory), launch (main kernel), rule (rows_in_launch, which plan.cpp is
// compiled with another name for, says yes to everything).  Addresses are made up, never used.
// Prints the status and, for each launch, "rows" (scatter), "attention" or "attention+rows" (which places them itself).
#include <hip/hip_runtime.h>

#include <cstdio>
#include <cstdlib>
#include <string>
#include <vector>

#include "cronus_internal.h"

static std::string failure, enqueued;
static int queue_sets[1 << 20];

extern "C" {
hipError_t hipGetDevice(int* dev) { return *dev = 0, hipSuccess; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) { return *v = 256, hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipStreamQuery(hipStream_t) { return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* st) { return *st = hipStreamCaptureStatusNone, hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipHostMalloc(void** p, size_t n, unsigned) {
  *p = failure == "buffer" ? nullptr : std::malloc(n);
  return *p ? hipSuccess : hipErrorOutOfMemory;
}
hipError_t hipHostFree(void* p) { return std::free(p), hipSuccess; }
hipError_t hipHostGetDevicePointer(void** d, void* p, unsigned) { return *d = p, hipSuccess; }
}

namespace cronus {
int wide_rows_for(int, int) { return kWaves * 32; }
bool rule_of_plan_cpp(const cronus_kv_cache*, const cronus_kv_rows*, const cronus_kv_rows*, const int32_t*, const int32_t*, int32_t, int);
bool rows_in_launch(const cronus_kv_cache* c, const cronus_kv_rows* first, const cronus_kv_rows* second, const int32_t* P, const int32_t* C,
                    int32_t n, int n_cus) {
  return failure == "rule" || rule_of_plan_cpp(c, first, second, P, C, n, n_cus);
}
int prepare_attn_kernels() { return failure == "setup" ? CRONUS_ERR_HIP : CRONUS_OK; }
int static_scratch_resolve(void** p) { return *p = queue_sets, CRONUS_OK; }
int queue_sets_resolve(int** p) { return *p = queue_sets, CRONUS_OK; }
int static_scratch_upload(void*, const void*, size_t, void*) { std::abort(); }
int static_scratch_expand(void*, void*, const CompactPlan&, const void*, size_t, void*) { std::abort(); }
int launch_kv_append(const cronus_kv_cache* c, const cronus_kv_rows*, const cronus_kv_rows*, const int32_t*, int32_t, int32_t, void*, bool) {
  if (c->num_kv_heads > kMaxScatterHeads) return CRONUS_ERR_INVALID_ARG;  // as kv_append.hip
  enqueued += " rows";
  return CRONUS_OK;
}
int launch_kv_gather(const cronus_kv_cache*, void*, void*, const int32_t*, const int32_t*, const int32_t*, int32_t, int32_t, int32_t, void*) { std::abort(); }
int launch_mfma_probe(bool, int, int, int, float*, void*, double*) { std::abort(); }
int mfma_probe_sink_floats(int) { return 1; }
int launch_attn(const AttnLaunch& a, bool* main_launched) {
  if (failure == "launch") return CRONUS_ERR_HIP;
  enqueued += a.rows ? " attention+rows" : " attention";
  *main_launched = true;
  return CRONUS_OK;
}
}  // namespace cronus

int main(int argc, char** argv) {
  auto num = [&](int i) { return std::strtoull(argv[i], nullptr, 0); };
  auto ptr = [&](int i) { return reinterpret_cast<char*>(num(i)); };
  auto ints = [&](int i) { return reinterpret_cast<int32_t*>(num(i)); };
  if (argc < 16) return 2;
  failure = argv[5];
  cronus_kv_cache c{};
  c.k_cache = c.v_cache = reinterpret_cast<void*>(0x10000000);
  c.num_blocks = 1 << 20;
  c.num_q_heads = (int)num(1);
  c.num_kv_heads = (int)num(2);
  c.head_dim = (int)num(3);
  c.block_size = 16;
  c.kv_dtype = num(4) ? CRONUS_KV_FP8_E4M3 : CRONUS_KV_BF16;
  if (num(4)) c.k_scale = c.v_scale = reinterpret_cast<float*>(0x20000000);
  const cronus_kv_rows first{ptr(8), ptr(9), ints(10), ints(11), (int32_t)num(6)}, second{ptr(8), ptr(9), ints(10), ints(11), (int32_t)num(7)};
  const int n = (int)num(15);
  if (argc < 16 + 2 * n) return 2;
  std::vector<int32_t> P, C;
  for (int i = 0; i < n; ++i) {
    P.push_back((int32_t)num(16 + 2 * i));
    C.push_back((int32_t)num(17 + 2 * i));
  }
  const int rc = cronus_iteration(&c, &first, &second, reinterpret_cast<void*>(0x30000000), ptr(12), P.data(), C.data(),
                                  reinterpret_cast<int32_t*>(0x40000000), 1 << 16, n, 0.125f, ptr(13), num(14), nullptr);
  std::printf("%d%s\n", rc, enqueued.c_str());
  return 0;
}
