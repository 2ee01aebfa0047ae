// The two bf16 MFMA shapes under the power limit: v_mfma_f32_32x32x16_bf16 against v_mfma_f32_16x16x32_bf16 on
// the same 64 x 128 block of a product per wave (8 waves per CU, all 256 CUs, gaussian operands), once with the
// operand fragments kept in registers and once with the twelve fragments of a half step read from LDS again
// every time.  The smaller shape moves half the accumulator registers per FLOP.  Prints TFLOP/s of launches
// that together last some 100 ms, three times in turn.
// Measurement aid only: nothing in the library uses it.
//   hipcc --offload-arch=gfx950 -O3 -Xclang -target-feature -Xclang -packed-fp32-ops mfma_shapes.hip -o mfma_shapes && ./mfma_shapes
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>
#include <vector>
typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float floatx16_t __attribute__((ext_vector_type(16)));
typedef float floatx4_t __attribute__((ext_vector_type(4)));

#define CK(x)                                                                   \
  do {                                                                          \
    hipError_t e_ = (x);                                                        \
    if (e_ != hipSuccess) {                                                     \
      printf("HIP error %s at line %d\n", hipGetErrorString(e_), __LINE__);     \
      exit(1);                                                                  \
    }                                                                           \
  } while (0)

constexpr int CHUNKS = 4096;                       // 16-byte chunks in LDS (64 KB) and per read of the source
constexpr size_t SOURCE = (size_t)1 << 20;         // 16-byte chunks of operands in memory

template <bool SMALL, bool FROM_LDS>
__global__ void __launch_bounds__(512) kern(const uint4* src, float* out, int iters) {
  __shared__ uint4 l[CHUNKS];
  for (int i = threadIdx.x; i < CHUNKS; i += 512) l[i] = src[((size_t)blockIdx.x * CHUNKS + i) % SOURCE];
  __syncthreads();
  const int at = (threadIdx.x & 63) + (threadIdx.x >> 6) * 320;
  union Fragment { uint4 u; bf16x8_t b; } fr[12];  // 4 of A, 8 of W
  for (int i = 0; i < 12; ++i) fr[i].u = l[(i * 64 + at) % CHUNKS];
  floatx16_t big[SMALL ? 1 : 8];
  floatx4_t small[SMALL ? 32 : 1];
  if constexpr (SMALL) {
    for (int i = 0; i < 32; ++i) for (int r = 0; r < 4; ++r) small[i][r] = 0.f;
  } else {
    for (int i = 0; i < 8; ++i) for (int r = 0; r < 16; ++r) big[i][r] = 0.f;
  }
  for (int it = 0; it < iters; ++it) {
    if (FROM_LDS)
      for (int i = 0; i < 12; ++i) fr[i].u = l[((i + it * 12) * 64 + at) % CHUNKS];
    if constexpr (SMALL) {
#pragma unroll
      for (int n = 0; n < 32; ++n) {
        const int i = n / 8, j = (i & 1) ? 7 - n % 8 : n % 8;
        small[i * 8 + j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fr[4 + j].b, fr[i].b, small[i * 8 + j], 0, 0, 0);
      }
    } else {
#pragma unroll
      for (int n = 0; n < 16; ++n) {
        const int k = n / 8, i = (n / 4) % 2, j = n % 4;
        big[i * 4 + j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[4 + k * 4 + j].b, fr[k * 2 + i].b, big[i * 4 + j], 0, 0, 0);
      }
    }
    __builtin_amdgcn_sched_barrier(0);
    if (!FROM_LDS) asm volatile("" : "+v"(fr[0].u.x), "+v"(fr[4].u.x));
  }
  float sum = 0.f;
  if constexpr (SMALL) {
    for (int i = 0; i < 32; ++i) for (int r = 0; r < 4; ++r) sum += small[i][r];
  } else {
    for (int i = 0; i < 8; ++i) for (int r = 0; r < 16; ++r) sum += big[i][r];
  }
  out[blockIdx.x * 512 + threadIdx.x] = sum;
}

template <bool SMALL, bool FROM_LDS>
static void run(const char* name, const uint4* src, float* out) {
  const int iters = 1000, launches = 200;
  hipEvent_t a, b;
  CK(hipEventCreate(&a)); CK(hipEventCreate(&b));
  hipLaunchKernelGGL((kern<SMALL, FROM_LDS>), dim3(256), dim3(512), 0, 0, src, out, iters);
  CK(hipEventRecord(a, 0));
  for (int i = 0; i < launches; ++i) hipLaunchKernelGGL((kern<SMALL, FROM_LDS>), dim3(256), dim3(512), 0, 0, src, out, iters);
  CK(hipEventRecord(b, 0)); CK(hipEventSynchronize(b));
  float ms;
  CK(hipEventElapsedTime(&ms, a, b));
  const double flop = 2.0 * 64 * 128 * 32 * iters * 8 * 256 * launches;   // 64 x 128 x 32 per wave and iteration
  printf("%-44s %7.1f ms %8.1f TFLOP/s\n", name, ms, flop / ms * 1e-9);
  fflush(stdout);
  CK(hipEventDestroy(a)); CK(hipEventDestroy(b));
}

int main() {
  std::vector<uint16_t> h(SOURCE * 8);
  uint32_t x = 12345;
  auto uniform = [&]() { x = x * 1664525u + 1013904223u; return ((x >> 8) + 0.5f) / 16777216.0f; };
  for (auto& v : h) {
    const float g = 0.3f * sqrtf(-2 * logf(uniform())) * cosf(6.2831853f * uniform());
    uint32_t bits;
    memcpy(&bits, &g, 4);
    v = (uint16_t)((bits + 0x8000u) >> 16);
  }
  uint4* src; float* out;
  CK(hipMalloc(&src, SOURCE * 16)); CK(hipMalloc(&out, 256 * 512 * sizeof(float)));
  CK(hipMemcpy(src, h.data(), SOURCE * 16, hipMemcpyHostToDevice));
  for (int rep = 0; rep < 3; ++rep) {
    run<false, false>("32x32x16, operands in registers", src, out);
    run<true, false>("16x16x32, operands in registers", src, out);
    run<false, true>("32x32x16, fragments from LDS every time", src, out);
    run<true, true>("16x16x32, fragments from LDS every time", src, out);
  }
  return 0;
}
