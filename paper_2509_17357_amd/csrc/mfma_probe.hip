// Measurement aid, not part of the attention path: the rate of v_mfma_f32_32x32x16_bf16 (decode spans) and of
// v_mfma_f32_16x16x32_bf16 (chunk tiles; each A operand held for two products, as there) that
// this GPU sustains when nothing else runs.  The published dense bf16 peak assumes the matrix
// pipes busy every cycle at the nominal clock; under a chip-wide MFMA load the clock follows
// the power drawn, and that follows the switching activity of the operands.  The probe runs
// the same instruction stream with operand registers that hold small constants or random
// bf16 values, so the difference is the data's.
#include <hip/hip_runtime.h>

#include "cronus_internal.h"

namespace cronus {
namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

constexpr int kProbeThreads = 512;     // 8 wavefronts, two per SIMD, like the attention kernel
constexpr int kProbeMfmaPerIter = 32;  // per wavefront

// Operand registers: small constants, or random bf16 values.
template <bool RANDOM>
__device__ __forceinline__ void fill_operands(u32x4 (&a)[8], u32x4 (&b)[8]) {
  unsigned h = threadIdx.x * 2654435761u + blockIdx.x * 40503u + 12345u;
  auto next = [&]() {
    h ^= h << 13;
    h ^= h >> 17;
    h ^= h << 5;
    // two bf16 values: random sign and mantissa, exponent 0x7b .. 0x7e (magnitude 1/16 .. 1)
    return (h & 0x81ff81ffu) | 0x3d803d80u | ((h >> 3) & 0x01000100u);
  };
#pragma unroll
  for (int i = 0; i < 8; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      a[i][j] = RANDOM ? next() : (unsigned)(i + j);
      b[i][j] = RANDOM ? next() : (unsigned)(2 * i + j);
    }
}

template <bool RANDOM>
__global__ __launch_bounds__(kProbeThreads) void mfma_probe_kernel(float* sink, int iters) {
  f32x16 acc[4];
#pragma unroll
  for (int j = 0; j < 4; ++j)
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[j][i] = 0.f;
  u32x4 a[8], b[8];
  fill_operands<RANDOM>(a, b);
  for (int it = 0; it < iters; ++it) {
#pragma unroll
    for (int s = 0; s < kProbeMfmaPerIter; ++s)
      asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(acc[s & 3]) : "v"(a[s & 7]), "v"(b[(s >> 2) & 7]));
  }
  float r = 0.f;
#pragma unroll
  for (int j = 0; j < 4; ++j)
#pragma unroll
    for (int i = 0; i < 16; ++i) r += acc[j][i];
  sink[(size_t)blockIdx.x * kProbeThreads + threadIdx.x] = r;
}

template <bool RANDOM>
__global__ __launch_bounds__(kProbeThreads) void mfma_probe_16x16x32_kernel(float* sink, int iters) {
  f32x4 acc[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) acc[j] = f32x4{0.f, 0.f, 0.f, 0.f};
  u32x4 a[8], b[8];
  fill_operands<RANDOM>(a, b);
  for (int it = 0; it < iters; ++it) {
#pragma unroll
    for (int s = 0; s < kProbeMfmaPerIter; ++s)
      acc[s & 7] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a[(s >> 1) & 7]),
                                                           __builtin_bit_cast(bf16x8, b[(s ^ (s >> 3)) & 7]), acc[s & 7], 0, 0, 0);
  }
  float r = 0.f;
#pragma unroll
  for (int j = 0; j < 8; ++j) r += (acc[j][0] + acc[j][1]) + (acc[j][2] + acc[j][3]);
  sink[(size_t)blockIdx.x * kProbeThreads + threadIdx.x] = r;
}

}  // namespace

int launch_mfma_probe(bool small_shape, int random_operands, int iters, int n_cus, float* sink, void* stream, double* flops) {
  auto kernel = small_shape ? (random_operands ? mfma_probe_16x16x32_kernel<true> : mfma_probe_16x16x32_kernel<false>)
                            : (random_operands ? mfma_probe_kernel<true> : mfma_probe_kernel<false>);
  hipLaunchKernelGGL(kernel, dim3((unsigned)n_cus), dim3(kProbeThreads), 0, static_cast<hipStream_t>(stream), sink, iters);
  if (hipGetLastError() != hipSuccess) return CRONUS_ERR_HIP;
  *flops = 2.0 * (small_shape ? 16 * 16 * 32 : 32 * 32 * 16) * (double)kProbeMfmaPerIter * (double)iters *
           (kProbeThreads / 64) * (double)n_cus;
  return CRONUS_OK;
}

int mfma_probe_sink_floats(int n_cus) { return n_cus * kProbeThreads; }

}  // namespace cronus
