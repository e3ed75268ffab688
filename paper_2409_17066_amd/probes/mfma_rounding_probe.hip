// How far v_mfma_f32_32x32x16_f16 and v_mfma_f32_16x16x32_f16 are from the exact sum of their products on gfx950, in units of the sum of
// the terms' magnitudes: the constant behind the screening bounds of vq_assign.hip and vq_quantize_loop.hip, which trust a nearest
// centroid only where its score wins by more than the scores can be wrong (they allow 2^-19).  Products of two binary16 numbers are
// exact in binary32, so what is measured is the instruction's own alignment and addition.  Operands below the normal range (2^-14) are
// counted as 2^-14.  Distributions: Gaussian; exponents spread over the whole range; large terms that cancel beside small ones; the
// operands of the screening (elements against |c|^2 / 2 in parts); operands below the normal range; with and without an accumulator.
// Build: hipcc --offload-arch=gfx950 -O3 -o mfma_rounding_probe mfma_rounding_probe.hip ; run without arguments.
#include <hip/hip_runtime.h>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <random>
#include <vector>
#define CK(x) do { hipError_t e = (x); if (e != hipSuccess) { printf("HIP error %s at line %d\n", hipGetErrorString(e), __LINE__); exit(1); } } while (0)

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef float float16v __attribute__((ext_vector_type(16)));
typedef float float4v __attribute__((ext_vector_type(4)));

// A wave per tile of M x M results over K products.  a, b: [tile][M][K], c, d: [tile][M][M]
template <int M>
__global__ __launch_bounds__(64) void mfma_kernel(const _Float16 *a, const _Float16 *b, const float *c, float *d) {
  constexpr int K = M == 32 ? 16 : 32, R = M == 32 ? 16 : 4;
  const int lane = threadIdx.x, row = lane & (M - 1), part = lane / M;
  const size_t tile = blockIdx.x;
  half8 x, y;
  for (int i = 0; i < 8; ++i) { x[i] = a[(tile * M + row) * K + part * 8 + i]; y[i] = b[(tile * M + row) * K + part * 8 + i]; }
  auto place = [&](int r) { return (tile * M + (M == 32 ? 8 * (r >> 2) + 4 * part + (r & 3) : 4 * part + r)) * M + row; };
  if constexpr (M == 32) {
    float16v acc;
    for (int r = 0; r < R; ++r) acc[r] = c[place(r)];
    acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(x, y, acc, 0, 0, 0);
    for (int r = 0; r < R; ++r) d[place(r)] = acc[r];
  } else {
    float4v acc;
    for (int r = 0; r < R; ++r) acc[r] = c[place(r)];
    acc = __builtin_amdgcn_mfma_f32_16x16x32_f16(x, y, acc, 0, 0, 0);
    for (int r = 0; r < R; ++r) d[place(r)] = acc[r];
  }
}

static const char *kKinds[] = {"Gaussian", "exponents over the whole range", "large terms that cancel, small ones beside them",
                               "elements against |c|^2 / 2 in three parts", "operands below the normal range among others",
                               "one large term, the others around its last bits"};

template <int M> void run(int kind, bool accumulate, int tiles) {
  constexpr int K = M == 32 ? 16 : 32;
  std::mt19937 rng(1234 + kind * 2 + accumulate);
  std::normal_distribution<float> normal;
  std::uniform_real_distribution<float> uniform(-1.0f, 1.0f);
  std::vector<_Float16> a((size_t)tiles * M * K), b(a.size());
  std::vector<float> c((size_t)tiles * M * M, 0.0f), d(c.size());
  auto spread = [&](int low, int high) { return (_Float16)std::ldexp(uniform(rng), low + (int)(rng() % (unsigned)(high - low + 1))); };
  for (size_t i = 0; i < a.size(); ++i) {
    const int k = (int)(i % K);
    switch (kind) {
      case 0: a[i] = (_Float16)normal(rng); b[i] = (_Float16)normal(rng); break;
      case 1: a[i] = spread(-13, 15); b[i] = spread(-13, 15); break;
      case 2:                                               // k and k ^ 1 of a are each other's negative, b the same but for its last bit
        a[i] = k & 1 ? (_Float16)-a[i - 1] : (_Float16)std::ldexp(1.0f + (float)(rng() % 1024) / 1024.0f, k < 4 ? 14 : (int)(rng() % 12));
        b[i] = k & 1 ? b[i - 1] : spread(-3, 3);
        if ((k & 1) && rng() % 2) b[i] = (_Float16)((float)b[i] * (1.0f + 0x1p-9f));
        break;
      case 3:
        if (k % 8 < 6) { a[i] = (_Float16)(0.02f * normal(rng)); b[i] = (_Float16)std::ldexp(uniform(rng), 13); }
        else { a[i] = (_Float16)std::ldexp(std::fabs(uniform(rng)), k % 8 == 6 ? 15 : 4); b[i] = (_Float16)std::ldexp(-1.0f, (int)(rng() % 4)); }
        break;
      case 5:                                               // (all of one sign, mantissas of ones: whatever is cut off adds up)
        if (k == (int)(i / K % K)) { a[i] = (_Float16)std::ldexp(1.0f, 14); b[i] = (_Float16)1.0f; }
        else { a[i] = (_Float16)std::ldexp(2.0f - 0x1p-10f, -(int)(i / (K * M) % 12)); b[i] = (_Float16)std::ldexp(2.0f - 0x1p-10f, -(int)(rng() % 6)); }
        break;
      default: a[i] = rng() % 3 ? spread(-24, -15) : spread(-10, 4); b[i] = rng() % 3 ? spread(-24, -15) : spread(-10, 4);
    }
  }
  if (accumulate) for (float &x : c) x = std::ldexp(uniform(rng), kind == 3 ? 15 : (int)(rng() % 20) - 10);
  _Float16 *ga, *gb; float *gc, *gd;
  CK(hipMalloc(&ga, a.size() * 2)); CK(hipMalloc(&gb, b.size() * 2)); CK(hipMalloc(&gc, c.size() * 4)); CK(hipMalloc(&gd, d.size() * 4));
  CK(hipMemcpy(ga, a.data(), a.size() * 2, hipMemcpyHostToDevice)); CK(hipMemcpy(gb, b.data(), b.size() * 2, hipMemcpyHostToDevice));
  CK(hipMemcpy(gc, c.data(), c.size() * 4, hipMemcpyHostToDevice));
  hipLaunchKernelGGL(mfma_kernel<M>, dim3((unsigned)tiles), dim3(64), 0, 0, ga, gb, gc, gd);
  CK(hipGetLastError()); CK(hipMemcpy(d.data(), gd, d.size() * 4, hipMemcpyDeviceToHost));
  CK(hipFree(ga)); CK(hipFree(gb)); CK(hipFree(gc)); CK(hipFree(gd));
  double worst = 0.0;
  const double least = 0x1p-14;
  for (int t = 0; t < tiles; ++t)
    for (int i = 0; i < M; ++i)
      for (int j = 0; j < M; ++j) {
        const size_t at = ((size_t)t * M + i) * M + j;
        double sum = c[at], size = std::fabs((double)c[at]);
        for (int k = 0; k < K; ++k) {
          const double x = (double)(float)a[((size_t)t * M + i) * K + k], y = (double)(float)b[((size_t)t * M + j) * K + k];
          sum += x * y;                                     // (exact: 22 bits a product, exponents within 60 of each other at most)
          size += std::fmax(std::fabs(x), least) * std::fmax(std::fabs(y), least);
        }
        worst = std::fmax(worst, std::fabs((double)d[at] - sum) / size);
      }
  printf("%dx%dx%d  %-48s %-16s largest error 2^%.2f of the terms' magnitudes, %d results\n", M, M, K, kKinds[kind], accumulate ? "accumulator" : "no accumulator",
         worst > 0 ? std::log2(worst) : -99.0, tiles * M * M);
  fflush(stdout);
}

int main() {
  for (int kind = 0; kind < 6; ++kind)
    for (int accumulate = 0; accumulate < 2; ++accumulate) { run<32>(kind, accumulate != 0, 512); run<16>(kind, accumulate != 0, 2048); }
  return 0;
}
