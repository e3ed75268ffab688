// Column order of a layer whose stored columns are a permutation of its own (Sec. 3.2.3 "Outlier Elimination": the columns
// that get the outlier codebook are picked by the Hessian's diagonal and stored first; Algorithm 2's outlier step): the two
// data movements that let every other kernel of the library work in stored order.
#include "vq_common.hpp"

namespace vq {

namespace {

typedef unsigned uint4v __attribute__((ext_vector_type(4)));
typedef unsigned uint2v __attribute__((ext_vector_type(2)));
typedef unsigned uint4b __attribute__((ext_vector_type(4), aligned(2)));      // (16 bytes of a row that begins at any half)
typedef unsigned uint4w __attribute__((ext_vector_type(4), aligned(4)));      // (of perm)

// dst[t][c] = src[t][perm[c]]: the activations in the stored order of the columns.  One thread per pair of columns;
// entries of perm outside the row read as zero, no perm is the identity; the pad columns [cols, ld_dst) of dst are cleared when ld_dst - cols < 8.
__global__ __launch_bounds__(256) void gather_cols_kernel(const __half *__restrict__ src, long long ld_src, int cols, const int *__restrict__ perm,
                                                          __half *__restrict__ dst, long long ld_dst, int dst_cols) {
  const int c = (blockIdx.x * 256 + threadIdx.x) * 2;
  if (c >= dst_cols) return;
  const __half *srow = src + (long long)blockIdx.y * ld_src;
  unsigned short h[2] = {0, 0};
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    if (c + j < cols) {
      const int t = perm ? perm[c + j] : c + j;
      if ((unsigned)t < (unsigned)cols) h[j] = __half_as_ushort(srow[t]);
    }
  }
  // dst rows start 4-byte aligned and c is even
  *reinterpret_cast<unsigned *>(dst + (long long)blockIdx.y * ld_dst + c) = (unsigned)h[0] | ((unsigned)h[1] << 16);
}

// W[o][perm[c]] = W[o][c] for every c < cols, one workgroup per row: the row goes to its new places in LDS, and comes
// back in order, in 16-byte pieces, wherever it begins (the tail in single elements).
__global__ __launch_bounds__(1024) void place_cols_kernel(__half *__restrict__ W, long long ldw, int cols, const int *__restrict__ perm) {
  extern __shared__ __attribute__((aligned(16))) __half row[];
  __half *w = W + (long long)blockIdx.x * ldw;
  const int body = cols & ~7;
  for (int c = (int)threadIdx.x * 8; c < body; c += 1024 * 8) {
    const uint4v v = *reinterpret_cast<const uint4b *>(w + c);
    const uint4v t0 = *reinterpret_cast<const uint4w *>(perm + c), t1 = *reinterpret_cast<const uint4w *>(perm + c + 4);
    const unsigned t[8] = {t0.x, t0.y, t0.z, t0.w, t1.x, t1.y, t1.z, t1.w};
    const unsigned d[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int j = 0; j < 8; ++j)
      if (t[j] < (unsigned)cols) row[t[j]] = __ushort_as_half((unsigned short)(d[j >> 1] >> ((j & 1) * 16)));
  }
  for (int c = body + (int)threadIdx.x; c < cols; c += 1024) {
    const unsigned t = (unsigned)perm[c];
    if (t < (unsigned)cols) row[t] = w[c];
  }
  __syncthreads();
  for (int c = (int)threadIdx.x * 8; c < body; c += 1024 * 8) *reinterpret_cast<uint4b *>(w + c) = *reinterpret_cast<const uint4v *>(row + c);
  for (int c = body + (int)threadIdx.x; c < cols; c += 1024) w[c] = row[c];
}

constexpr int PLACE_ROWS = 4;

// Where column t of PLACE_ROWS rows lies in LDS, in bytes: eight bytes a column, the 16-byte pairs of every eight columns in an order that
// changes from one 32 columns to the next, so that 16 lanes with eight columns each read from all banks.
__device__ __forceinline__ unsigned placed(unsigned t) { return (((t >> 1) ^ ((t >> 5) & 3u)) << 4) | ((t & 1u) << 3); }

// The same for four rows to a workgroup.  What bounds place_cols_kernel is its scatter in LDS, an instruction for an element of every lane, and
// perm, of which it reads twice a row's bytes; here a lane writes a column's four elements with one, at the price of one (a wave's 64 places of
// eight bytes meet no more conflicts than 64 of two), and reads perm once for the four.  Rows may begin at any half.  (With the restoring
// kernel in front, v = 6, before -> now: 8064 x 384 17.7 -> 10.3 us, 4096 x 4096 30.4 -> 27, of which 10 are the other kernel's; 5248 x 7936
// 46.3 -> 45.2, 28 of them for the 167 MB of this one, which is memory's rate; 5248 x 7935 82.5 -> 47.8.)
__global__ __launch_bounds__(1024) void place_cols4_kernel(__half *__restrict__ W, long long ldw, int rows, int cols, const int *__restrict__ perm) {
  extern __shared__ __attribute__((aligned(16))) __half row[];
  unsigned char *lds = reinterpret_cast<unsigned char *>(row);
  const int o0 = (int)blockIdx.x * PLACE_ROWS, n = min(PLACE_ROWS, rows - o0), body = cols & ~7, threads = (int)blockDim.x;
  __half *w[PLACE_ROWS];
#pragma unroll
  for (int r = 0; r < PLACE_ROWS; ++r) w[r] = W + (long long)(o0 + min(r, n - 1)) * ldw;
  for (int c = (int)threadIdx.x * 8; c < body; c += threads * 8) {
    uint4v v[PLACE_ROWS];
#pragma unroll
    for (int r = 0; r < PLACE_ROWS; ++r) v[r] = *reinterpret_cast<const uint4b *>(w[r] + c);
    const uint4v t0 = *reinterpret_cast<const uint4w *>(perm + c), t1 = *reinterpret_cast<const uint4w *>(perm + c + 4);
    const unsigned t[8] = {t0.x, t0.y, t0.z, t0.w, t1.x, t1.y, t1.z, t1.w};
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const unsigned sel = j & 1 ? 0x07060302u : 0x05040100u;
      const int d = j >> 1;
      if (t[j] < (unsigned)cols)
        *reinterpret_cast<uint2v *>(lds + placed(t[j])) = uint2v{__builtin_amdgcn_perm(v[1][d], v[0][d], sel), __builtin_amdgcn_perm(v[3][d], v[2][d], sel)};
    }
  }
  for (int c = body + (int)threadIdx.x; c < cols; c += threads) {
    const unsigned t = (unsigned)perm[c];
    if (t < (unsigned)cols)
#pragma unroll
      for (int r = 0; r < PLACE_ROWS; ++r) reinterpret_cast<__half *>(lds + placed(t))[r] = w[r][c];
  }
  __syncthreads();
  for (int c = (int)threadIdx.x * 8; c < body; c += threads * 8) {
    uint4v e[4];
#pragma unroll
    for (int m = 0; m < 4; ++m) e[m] = *reinterpret_cast<const uint4v *>(lds + placed((unsigned)(c + 2 * m)));
#pragma unroll
    for (int r = 0; r < PLACE_ROWS; ++r) {
      const unsigned sel = r & 1 ? 0x07060302u : 0x05040100u;
      const int h = r >> 1;
      if (r < n)
        *reinterpret_cast<uint4b *>(w[r] + c) = uint4b{__builtin_amdgcn_perm(e[0][2 + h], e[0][h], sel), __builtin_amdgcn_perm(e[1][2 + h], e[1][h], sel),
                                                       __builtin_amdgcn_perm(e[2][2 + h], e[2][h], sel), __builtin_amdgcn_perm(e[3][2 + h], e[3][h], sel)};
    }
  }
  for (int c = body + (int)threadIdx.x; c < cols; c += threads)
#pragma unroll
    for (int r = 0; r < PLACE_ROWS; ++r)
      if (r < n) w[r][c] = reinterpret_cast<const __half *>(lds + placed((unsigned)c))[r];
}

}  // namespace

int launch_gather_cols(const __half *src, long long ld_src, int rows, int cols, const int *perm, __half *dst, long long ld_dst, hipStream_t s) {
  if (rows < 1 || rows > 65535 || (ld_dst & 1) || (reinterpret_cast<uintptr_t>(dst) & 3)) return VQ_ERR_UNSUPPORTED;
  const int dst_cols = ld_dst - cols < 8 ? (int)ld_dst : cols + (cols & 1);     // whole pairs; the pad of a row rounded up to 8
  if (dst_cols > ld_dst) return VQ_ERR_UNSUPPORTED;
  hipLaunchKernelGGL(gather_cols_kernel, dim3((unsigned)((dst_cols + 511) / 512), (unsigned)rows), dim3(256), 0, s, src, ld_src, cols, perm, dst,
                     ld_dst, dst_cols);
  return hipGetLastError() == hipSuccess ? VQ_OK : VQ_ERR_HIP;
}

int launch_place_cols(__half *W, long long ldw, int rows, int cols, const int *perm, hipStream_t s) {
  const unsigned lds = (unsigned)(((long long)cols * 2 + 15) & ~15LL);
  if ((long long)cols * 2 > 160 * 1024) return VQ_ERR_UNSUPPORTED;
  // Four rows to a workgroup where that leaves one for every CU, and two of them and more fit a CU's LDS, so that one's loads run beside
  // another's stores.  (Whole vq_dequant, v = 6, one row -> four: 512 rows of 4096 columns 9.1 -> 9.8 us, 1024 12.8 -> 12.9, 2048 19.6 -> 17.9,
  // 4096 30.4 -> 26.7; 4096 rows of 512 14.9 -> 9.2, of 10240 46.4 -> 45.4, of 12288 52.8 -> 58.)
  if (rows >= 1024 && cols <= 10240) {
    VQ_ALLOW_FULL_LDS(place_cols4_kernel);
    const unsigned threads = (unsigned)min(1024, ((cols + 7) / 8 + 63) / 64 * 64);
    hipLaunchKernelGGL(place_cols4_kernel, dim3((unsigned)((rows + PLACE_ROWS - 1) / PLACE_ROWS)), dim3(threads), (unsigned)((cols + 31) / 32 * 32 * 8), s, W, ldw, rows,
                       cols, perm);
    return hipGetLastError() == hipSuccess ? VQ_OK : VQ_ERR_HIP;
  }
  VQ_ALLOW_FULL_LDS(place_cols_kernel);
  hipLaunchKernelGGL(place_cols_kernel, dim3((unsigned)rows), dim3(1024), lds, s, W, ldw, cols, perm);
  return hipGetLastError() == hipSuccess ? VQ_OK : VQ_ERR_HIP;
}

}  // namespace vq
