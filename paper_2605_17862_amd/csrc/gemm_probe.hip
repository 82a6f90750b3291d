// Timing of the bf16 contraction kernels on one shape.
//
//   gemm_probe [N rows, default 8192] [M, default 151936] [K, default 4096] [row padding in elements, default 0]
//              [groups of 20 back-to-back launches of the shipped loop, default 3] [operand values: 0 (default)
//              magnitudes in [0.5, 1), 1 close to normal with the spread of hidden states and projection weights]
//
// Out[N, M] = Bn[N, K] . Am[M, K]^T with fopd_gemm_nt (the kernel behind two contractions of the loss pass through the
// projection; its loop is that of the projection kernel fused with the log-sum-exp), single launches and launches back to
// back; at the benchmark's M and K also the weight gradient's kernel fopd_gemm_tn.
// Under `rocprofv3 --pmc ...` the same program gives the kernels' counters.

#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>

#include "fopd_gemm.hip"

#define CHECK(x)                                                                     \
  do {                                                                               \
    hipError_t e_ = (x);                                                             \
    if (e_ != hipSuccess) {                                                          \
      fprintf(stderr, "gemm_probe: %s failed: %s\n", #x, hipGetErrorString(e_));     \
      return 1;                                                                      \
    }                                                                                \
  } while (0)

__device__ inline uint32_t gemm_probe_hash(uint32_t x) {
  x ^= x >> 16;
  x *= 0x7feb352du;
  x ^= x >> 15;
  x *= 0x846ca68bu;
  x ^= x >> 16;
  return x;
}

// normal == 0: bf16 values with magnitudes in [0.5, 1): random sign and mantissa, one exponent.
// normal != 0: close to N(0, scale^2) (a sum of 12 uniforms), the spread of the operands the pass sees: the
// rate the part sustains depends on the operand bits (more toggling, more power, a lower clock).
__global__ void gemm_probe_fill(uint16_t* p, size_t n, uint32_t seed, int normal, float scale) {
  for (size_t i = blockIdx.x * static_cast<size_t>(blockDim.x) + threadIdx.x; i < n;
       i += static_cast<size_t>(gridDim.x) * blockDim.x) {
    if (normal == 0) {
      uint32_t h = static_cast<uint32_t>(i) * 2654435761u + seed;
      h ^= h >> 15;
      p[i] = static_cast<uint16_t>(((h & 1u) << 15) | (0x3f00u + ((h >> 8) & 0x7fu)));
    } else {
      float acc = 0.f;
      for (uint32_t k = 0; k < 12u; ++k)
        acc += static_cast<float>(gemm_probe_hash(static_cast<uint32_t>(i) * 12u + k + seed * 0x9e3779b9u) >> 8) *
               (1.0f / 16777216.0f);
      p[i] = static_cast<uint16_t>(__float_as_uint((acc - 6.0f) * scale) >> 16);
    }
  }
}

// `groups` groups of `each` launches back to back, timed apiece.
template <typename Launch>
static int time_groups(const char* name, int groups, int each, double flops, hipEvent_t e0, hipEvent_t e1, Launch launch) {
  for (int group = 0; group < groups; ++group) {
    CHECK(hipEventRecord(e0, 0));
    for (int rep = 0; rep < each; ++rep) launch();
    CHECK(hipGetLastError());
    CHECK(hipEventRecord(e1, 0));
    CHECK(hipEventSynchronize(e1));
    float ms = 0.f;
    CHECK(hipEventElapsedTime(&ms, e0, e1));
    printf("gemm_probe: %s, %d back to back (group %d): avg %.3f ms, %.0f TFLOP/s (%.3f of 2500)\n", name, each, group,
           ms / each, flops / (ms / each) * 1e-9, flops / (ms / each) * 1e-9 / 2500.0);
    fflush(stdout);
  }
  return 0;
}

int main(int argc, char** argv) {
  const int N = (argc > 1) ? atoi(argv[1]) : 8192;
  const int M = (argc > 2) ? atoi(argv[2]) : 151936;
  const int K = (argc > 3) ? atoi(argv[3]) : 4096;
  const int pad = (argc > 4) ? atoi(argv[4]) : 0;       // extra elements per operand row (row pitch K + pad)
  const int groups = (argc > 5) ? atoi(argv[5]) : 3;    // groups of 20 back-to-back launches of the shipped loop
  const int normal = (argc > 6) ? atoi(argv[6]) : 0;    // 1: operands close to N(0, 1) and N(0, (3/64)^2)
  if (N < 1 || N > 65536 || M < 4 || M > 262144 || M % 4 != 0 || K < 64 || K > 16384 || K % 64 != 0 || pad < 0 ||
      pad > 4096 || pad % 8 != 0 || groups < 0 || groups > 64) {
    fprintf(stderr, "gemm_probe: N in [1, 65536], M in [4, 262144] and a multiple of 4, K a multiple of 64 in [64, 16384]\n");
    return 2;
  }
  __bf16 *A = nullptr, *B = nullptr;
  float* out = nullptr;
  const int64_t ld = K + pad;
  CHECK(hipMalloc(&A, static_cast<size_t>(M) * ld * 2));
  CHECK(hipMalloc(&B, static_cast<size_t>(N) * ld * 2));
  CHECK(hipMalloc(&out, static_cast<size_t>(N) * M * 4));
  gemm_probe_fill<<<4096, 256>>>(reinterpret_cast<uint16_t*>(A), static_cast<size_t>(M) * ld, 1u, normal, 0.046875f);
  gemm_probe_fill<<<4096, 256>>>(reinterpret_cast<uint16_t*>(B), static_cast<size_t>(N) * ld, 2u, normal, 1.0f);
  CHECK(hipDeviceSynchronize());
  hipEvent_t e0, e1;
  CHECK(hipEventCreate(&e0));
  CHECK(hipEventCreate(&e1));
  printf("gemm_probe: Out[%d, %d] = Bn[%d, %d] . Am[%d, %d]^T, bf16 in, fp32 out, operand row pitch %ld elements, %s\n", N,
         M, N, K, M, K, static_cast<long>(ld),
         normal ? "operands close to N(0, 1) and N(0, (3/64)^2)" : "operand magnitudes in [0.5, 1)");
  using namespace fopd;
  const int tiles_m = (M + kGemmTile - 1) / kGemmTile, tiles_n = (N + kGemmTile - 1) / kGemmTile;
  const int64_t rounds = (tile_groups(tiles_m, tiles_n) + 7) / 8;
  const bool walk = gemm_walks(static_cast<int64_t>(tiles_m) * tiles_n, K / kLmK, false);
  const unsigned grid = gemm_grid(rounds, walk);
  const double flops = 2.0 * M * static_cast<double>(N) * K;
  auto kern = walk ? fopd_gemm_nt<false, true> : fopd_gemm_nt<false, false>;
  CHECK(hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, kLoopLdsBytes));
  auto nt = [&]() {
    kern<<<grid, kGemmThreads, kLoopLdsBytes>>>(A, ld, M, M, B, ld, N, K, out, M, tiles_m, tiles_n, nullptr, 1, 0);
  };
  if (time_groups("fopd_gemm_nt", 4, 1, flops, e0, e1, nt)) return 1;
  if (time_groups("fopd_gemm_nt", groups, 20, flops, e0, e1, nt)) return 1;
  if (N >= 8192 && M == 151936 && K == 4096 && pad == 0) {
    // the weight gradient's shape, B k-major, in the same buffers: Out[151936, 4096] = sum over 4096 entries of
    // Bk[4096, 151936] (all of buffer A) and Am[4096, 4096] (half of the first 8192 rows of buffer B)
    const int tm = 4096 / kGemmTile, tn = (151936 + kGemmTile - 1) / kGemmTile;
    const int64_t rounds_tn = (tile_groups(tm, tn) + 7) / 8;
    const bool walk_tn = gemm_walks(static_cast<int64_t>(tm) * tn, 4096 / kLmK, false);
    auto kern_tn = walk_tn ? fopd_gemm_tn<false, true> : fopd_gemm_tn<false, false>;
    CHECK(hipFuncSetAttribute(reinterpret_cast<const void*>(kern_tn), hipFuncAttributeMaxDynamicSharedMemorySize,
                              kLoopLdsBytes));
    if (time_groups("fopd_gemm_tn, Out[151936, 4096], K = 4096", 4, 1, 2.0 * 4096 * 151936.0 * 4096, e0, e1, [&]() {
          kern_tn<<<gemm_grid(rounds_tn, walk_tn), kGemmThreads, kLoopLdsBytes>>>(B, 4096, 4096, A, 151936, 151936, 4096, out,
                                                                                 4096, tm, tn, nullptr);
        }))
      return 1;
  }
  CHECK(hipFree(A));
  CHECK(hipFree(B));
  CHECK(hipFree(out));
  return 0;
}
