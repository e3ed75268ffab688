// The padding of index streams (internal).
#pragma once

namespace vq {

// What follows the streams' last dwords, `count` dwords from number `from` on of each of `rows` strides, as zeros for a caller whose buffer is as the
// allocator left it (count = 0: left alone).  Every thread of a launch takes some; a launch of its own that cleared the whole buffer in front took
// 2766 x 384, v = 2, k = 16 1.6 us of 8.9, 2967 x 419, v = 6, k = 256 1.2 of 13.1, 1554 x 448, k = 4096, down the columns 1.5 of 32.3.
struct Padding { unsigned char *idx; long long stride; int rows, from, count; };

// (a thread per vector is more than 2^31 threads of the largest matrices)
__host__ __device__ inline void clear_padding(const Padding &p, unsigned block, unsigned block_threads, unsigned thread, unsigned blocks) {
  if (p.count == 0) return;
  const long long total = (long long)p.rows * p.count, step = (long long)blocks * block_threads;
  for (long long i = (long long)block * block_threads + thread; i < total; i += step) {
    const int number = (int)i;                             // (rows of 2^24 at most, three dwords each)
    reinterpret_cast<unsigned *>(p.idx + (long long)(number / p.count) * p.stride)[p.from + number % p.count] = 0u;
  }
}

}  // namespace vq
