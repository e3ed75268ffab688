// What the two column-loop kernels of vq_quantize_columns share (internal).
#pragma once
#include "vq_common.hpp"

namespace vq {
namespace {

typedef float float16v __attribute__((ext_vector_type(16)));

constexpr int QB = 128;          // most columns per block: two per lane
constexpr int CPL = QB / 64;

// smaller distance, else smaller index: the rule by which the lanes' candidates meet.  Distances are sums of squares, so
// their bit patterns order like the numbers: the smallest pattern first, then the smallest index among its holders.
__device__ __forceinline__ void wave_arg_min(float &d, unsigned &i) {
  const unsigned bits = __float_as_uint(d);
  const unsigned lowest = wave_min_u32(bits);
  i = wave_min_u32(bits == lowest ? i : 0xFFFFFFFFu);
  d = __uint_as_float(lowest);
}

typedef unsigned uint4v __attribute__((ext_vector_type(4)));
typedef unsigned uint2v __attribute__((ext_vector_type(2)));

__device__ __forceinline__ float half_of(unsigned dword, int hi) { return __half2float(__ushort_as_half((unsigned short)(hi ? dword >> 16 : dword & 0xFFFFu))); }

// workgroup barrier that waits for LDS traffic only (rows of H^-1 stay on their way across it)
__device__ __forceinline__ void lds_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

}  // namespace

// The whole loop in one launch, where the tables fit registers and LDS; VQ_ERR_UNSUPPORTED otherwise.  Streams cleared beforehand.
struct LoopArgs {
  float *W; long long ldw; int rows, cols;
  const float *Hinv; long long ldh;
  const __half *cb; int k; const __half *cb_res; int k_res;
  int v, block, P;                     // P: stack positions per workgroup
  int whole;                           // positions of v rows; one more workgroup takes the cut-off one, if there is one
  unsigned *idx; long long idx_dwords; int bits;
  unsigned *idx_res; long long idx_res_dwords; int bits_res;
  float *T; long long ldt;
};
int launch_quantize_loop(LoopArgs a, hipStream_t st);

}  // namespace vq
