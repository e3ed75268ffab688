// vq_assign: the encode side of the lookup -- index of the nearest centroid of every length-v vector along the
// rows of a weight matrix (Eq. 2 of Sec. 2.2; with a base matrix, the residual stage's equation of Sec. 3.2.2),
// written as the packed index streams that vq_dequant / vq_gemv / vq_gemm read.
//
// The distance decides an integer, so its arithmetic is fixed (include/vq.h): binary32, t_j = W - B as one
// subtraction, per element one subtraction and one fused multiply-add into a sum that starts at +0, elements in
// ascending order, the first of equal distances wins.
//
// Three kernels.  assign_screen_kernel (v <= 13, tables of 64 entries and more) finds for every vector the 16 or 32 centroids among
// which the nearest one must be, on the matrix cores, and computes the distances as defined for those only.  The other two
// compute every distance on the vector ALUs, 2 v + 3 instructions per (vector, centroid) pair: assign_short_kernel for
// tables of fewer entries, assign_kernel for longer vectors.
#include "vq_common.hpp"
#include "vq_padding.hpp"
#include <type_traits>

namespace vq {
namespace {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef float float16v __attribute__((ext_vector_type(16)));
typedef unsigned uint4v __attribute__((ext_vector_type(4)));

// Which vectors a launch takes and where their indices go.  Vector u of row o: element j at
// W[o * row_step + u * vec_step + j * elem_step] (along the rows of W: ld, v, 1; down its columns: v * ld, 1, ld).  Only the first
// `len` elements of vectors and centroids are compared; the rest counts as zeros on both sides, which adds nothing to a distance.
struct Vectors {
  const __half *W, *B;
  long long row_step, vec_step, elem_step;
  int rows, per_row, len;
  unsigned char *idx;
  long long idx_stride;
  // Indices of a row fill its stream from bit 0; the bits of the last dword past them are zeroed, except that bits from
  // `spare_from` on (the index of a cut-off last vector and what follows it) are somebody else's to write.
  long long spare_from;
  // scatter_bit >= 0: there is one row, and the index of its vector u goes into stream u at this bit, the rest of its last
  // dword being zeroed (the cut-off last vectors of all rows).
  long long scatter_bit;
};

__device__ __forceinline__ void clear_padding(const Padding &p) { vq::clear_padding(p, blockIdx.x, blockDim.x, threadIdx.x, gridDim.x); }

// Writes `count` bits of a dword that another lane may be writing other bits of.
__device__ __forceinline__ void put_bits(unsigned *w, unsigned value, int from, int count) {
  const unsigned mask = (count >= 32 ? 0xFFFFFFFFu : (1u << count) - 1u) << from;
  atomicAnd(w, ~mask | (value << from));
  atomicOr(w, value << from);
}

// The index of a cut-off last vector: its bits and the zeros up to the end of its last dword.
__device__ __forceinline__ void scatter_index(const Vectors &a, int u, unsigned index, int bits) {
  unsigned *w = reinterpret_cast<unsigned *>(a.idx + (long long)u * a.idx_stride) + (a.scatter_bit >> 5);
  const int sh = (int)(a.scatter_bit & 31);
  put_bits(w, index, sh, 32 - sh);
  if (sh + bits > 32) w[1] = index >> (32 - sh);
}

// A row's dword number d: all of it, or below the bits that are somebody else's.
__device__ __forceinline__ void store_dword(const Vectors &a, unsigned *w, long long d, unsigned value) {
  const long long left = a.spare_from - 32 * d;
  if (left >= 32) *w = value;
  else put_bits(w, value, 0, (int)left);
}

// Vectors are dealt out in row order, every row's count rounded up to whole segments of seg_len, whose indices fill whole dwords.
__host__ __device__ inline int items_per_row(const Vectors &a, int seg_len) { return (a.per_row + seg_len - 1) / seg_len * seg_len; }
__host__ __device__ inline long long items_of(const Vectors &a, int seg_len) { return (long long)a.rows * items_per_row(a, seg_len); }

// Row and position of the items from number g0 (the same in all lanes of a wave) on; up to 64 of them.
struct Place {
  int row_items, o0, p0;
  __device__ Place(const Vectors &a, long long g0, long long items, int seg_len) : row_items(items_per_row(a, seg_len)) {
    o0 = items <= 0x7fffffffLL ? (int)((unsigned)g0 / (unsigned)row_items) : (int)(g0 / row_items);
    p0 = (int)(g0 - (long long)o0 * row_items);
  }
  __device__ void item(int x, int &o, int &p) const {
    const unsigned q = row_items >= 64 ? (p0 + x >= row_items ? 1u : 0u) : (unsigned)(p0 + x) / (unsigned)row_items;
    o = o0 + (int)q;
    p = p0 + x - (int)q * row_items;
  }
};

// The dword of packed indices that a lane writes out of up to 64 items (whole segments; an index has 16 bits at most): the segment's
// first item, the dword's number in the segment, the first code with bits in it and where that code starts.
struct PackLane {
  int item, word, code, shift, seg_shift;
  __device__ PackLane(int lane, int seg_len, int bits) {
    const int per_seg = seg_len * bits / 32, sg = lane / per_seg;
    item = sg * seg_len; word = lane - sg * per_seg; code = 32 * lane / bits; shift = code * bits - 32 * lane;
    seg_shift = __builtin_ctz(seg_len);                      // 8, 16 or 32
  }
};

// The indices of a wave's first `count` items, a lane per dword.
__device__ __forceinline__ void pack_items(const Vectors &a, const Place &place, int count, const PackLane &lay, int bits, const unsigned *codes, int lane) {
  if (lane >= count * bits / 32) return;
  int o, p;
  place.item(lay.item, o, p);
  const long long at = (long long)(p >> lay.seg_shift) * (bits << lay.seg_shift >> 5) + lay.word;
  if (o >= a.rows || 32 * at >= (long long)a.per_row * bits) return;
  unsigned w = 0;
  for (int i = lay.code, sh = lay.shift; sh < 32; ++i, sh += bits)          // (past a row's end the codes are zero)
    w |= sh >= 0 ? codes[i] << sh : codes[i] >> -sh;
  store_dword(a, reinterpret_cast<unsigned *>(a.idx + (long long)o * a.idx_stride) + at, at, w);
}

// The distance of the definition from t to one centroid.
template <int V, typename Get>
__device__ __forceinline__ float distance(const float (&t)[V], Get element) {
  float d = 0.0f;
#pragma unroll
  for (int j = 0; j < V; ++j) {
    // t - c as one fused operation (the same single rounding: the product c * -1 is exact), which takes a binary16 c as it is
    const float diff = __fmaf_rn(element(j), -1.0f, t[j]);
    d = __fmaf_rn(diff, diff, d);
  }
  return d;
}

// The same to a centroid as the screening planes hold it, eight binary16 elements in 16 bytes (the second 16 bytes: elements 8 on).
// (Inline assembly, as the compiler makes a conversion and a subtraction of the fused operation.)
template <int V>
__device__ __forceinline__ float distance(const float (&t)[V], const half8 &c0, const half8 &c1) {
  const uint4v w0 = __builtin_bit_cast(uint4v, c0), w1 = __builtin_bit_cast(uint4v, c1);
  float d = 0.0f;
#pragma unroll
  for (int j = 0; j < V; ++j) {
    const unsigned w = j < 8 ? w0[j / 2 & 3] : w1[j / 2 & 3];
    float diff;
    if (j & 1) asm("v_fma_mix_f32 %0, %1, -1.0, %2 op_sel:[1,0,0] op_sel_hi:[1,0,0]" : "=v"(diff) : "v"(w), "v"(t[j]));
    else asm("v_fma_mix_f32 %0, %1, -1.0, %2 op_sel_hi:[1,0,0]" : "=v"(diff) : "v"(w), "v"(t[j]));
    d = __fmaf_rn(diff, diff, d);
  }
  return d;
}

// Entries of a table in memory as the planes hold one: V elements, zeros from len on, in loads of as many bytes as divide a row where
// those are aligned (`whole`).
template <int V> constexpr int load_bytes() { return V % 8 == 0 ? 16 : V % 4 == 0 ? 8 : V % 2 == 0 ? 4 : 2; }

// N entries under one branch: with a branch for each the compiler would wait for each before the next.
template <int V, int N>
__device__ __forceinline__ void load_entries(const __half *codebook, const int (&i)[N], int stride, int len, bool whole, half8 (&c0)[N], half8 (&c1)[N]) {
  constexpr int B = load_bytes<V>() / 2;
  typedef _Float16 part __attribute__((ext_vector_type(B)));
  _Float16 c[N][16] = {};
  if (whole) {
#pragma unroll
    for (int n = 0; n < N; ++n)
#pragma unroll
      for (int x = 0; x < V / B; ++x) {
        const part y = reinterpret_cast<const part *>(codebook + (long long)i[n] * stride)[x];
#pragma unroll
        for (int j = 0; j < B; ++j) c[n][x * B + j] = y[j];
      }
  } else {
#pragma unroll
    for (int n = 0; n < N; ++n)
#pragma unroll
      for (int j = 0; j < V; ++j) c[n][j] = __builtin_bit_cast(_Float16, codebook[(long long)i[n] * stride + j]);
  }
  // (whole dwords masked: a choice for every element takes several instructions)
  unsigned mask[8];
#pragma unroll
  for (int d = 0; d < 8; ++d) mask[d] = len > 2 * d + 1 ? 0xFFFFFFFFu : len > 2 * d ? 0xFFFFu : 0u;
#pragma unroll
  for (int n = 0; n < N; ++n) {
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      if (j < 8) c0[n][j] = c[n][j];
      else c1[n][j & 7] = c[n][j];
    }
    uint4v w0 = __builtin_bit_cast(uint4v, c0[n]), w1 = __builtin_bit_cast(uint4v, c1[n]);
#pragma unroll
    for (int d = 0; d < (V + 1) / 2; ++d) {
      if (d < 4) w0[d & 3] &= mask[d];
      else w1[d & 3] &= mask[d];
    }
    c0[n] = __builtin_bit_cast(half8, w0); c1[n] = __builtin_bit_cast(half8, w1);
  }
}

// Distances from t to N entries in memory.
template <int V, int N>
__device__ __forceinline__ void distances_to(const __half *codebook, const int (&i)[N], int stride, int len, bool whole, const float (&t)[V], float (&d)[N]) {
  if constexpr (V % 2 == 0) {
    half8 c0[N], c1[N];
    load_entries<V, N>(codebook, i, stride, len, whole, c0, c1);
#pragma unroll
    for (int n = 0; n < N; ++n) d[n] = distance<V>(t, c0[n], c1[n]);
  } else {                                                   // (loaded one by one, and not packed to be taken apart again)
    float c[N][V];
#pragma unroll
    for (int n = 0; n < N; ++n)
#pragma unroll
      for (int j = 0; j < V; ++j) {
        const float y = __half2float(codebook[(long long)i[n] * stride + j]);
        c[n][j] = j < len ? y : 0.0f;
      }
#pragma unroll
    for (int n = 0; n < N; ++n) d[n] = distance<V>(t, [&](int j) -> float { return c[n][j]; });
  }
}

// The lanes' candidates meet: the smaller distance, else the smaller index.  Distances are sums of squares, so their bits order
// like the numbers.
__device__ __forceinline__ void wave_arg_min(float &d, unsigned &i) {
  const unsigned lowest = wave_min_u32(__float_as_uint(d));
  i = wave_min_u32(__float_as_uint(d) == lowest ? i : 0xFFFFFFFFu);
  d = __uint_as_float(lowest);
}

// ---- screening on the matrix cores ------------------------------------------------------------------------------------
//
// The nearest centroid has the largest score s_i = t . c_i - |c_i|^2 / 2.  One v_mfma_f32_32x32x16_f16 gives the scores of 32
// centroids with 32 vectors: the centroid's row of operand A holds its elements and |c|^2 / 2, scaled by a power of two and
// split into three binary16 parts; the vector's column of operand B holds t and the matching negative power of two.  A t that is
// a difference W - B is no binary16 number: it is scaled and split into two (v <= 6: both in one instruction's 16 k slots,
// against the same elements twice; longer vectors: a second instruction with the same A).  A lane sees 16 rows of every result:
// it keeps the largest score of any such block of 16 (of two results, 32, where a wave holds two tiles of vectors and the table has 4096
// entries or more), that block's number, and the largest score of every other block.
//
// Scores carry rounding errors, so the winning block is only trusted when it wins by more than they can be.  With T = |t|, the
// nearest centroid and whichever centroid has the largest computed score have norms of at most R = T + sqrt(d), d their
// squared distance; |c|^2 / 2 is kept to 2^-39, or 2^-30 of the largest; the products are exact in binary32, and an instruction cuts
// each of its 16 terms and the accumulator where the largest one's binary32 ends: 17 2^-24 of the sum of the terms' magnitudes at most, for two scores
// 34 2^-24 an instruction (probes/mfma_rounding_probe.hip finds up to 9 2^-24 where all terms lose their last bits to the same side, 6 2^-24
// with operands like these; operands below the normal range count as 2^-14); the definition's own roundings move d by (v + 2) 2^-24.  Vectors that fail the test
// -- about 0.3 % with 4096 Gaussian entries --, and all of them when a table has entries that are not finite or huge, are
// compared with every centroid by the wave together.
//
// What bounds it: the vector ALUs, which are busy 89 % of the clocks (profiles/case_counters.txt; at 1.9 GHz: both units' power).  A result (two blocks of
// 16 scores) costs 32 matrix-core clocks and 12 vector instructions of 4 clocks, 10 with blocks of 32; what a vector costs beside the search
// -- operands, distances of the winning block, the test, packing -- is about a fifth of the time at k = 4096 and most of it at 256.  So:
//  - the products of one result run while the largest score of the one before is found;
//  - behind the search a lane has a vector to itself, its operands and results swapped between the two halves of the wave
//    (one instruction a register) instead of both lanes of a vector doing the same;
//  - a workgroup's waves draw their vectors by ticket: with equal shares the waves that a SIMD prefers were done early and on average
//    2.6 of its four were left;
//  - blocks of 32 from 4096 entries on, for waves of two tiles: 8 instructions fewer for every 64 entries and 64 vectors, 16 distances of
//    15 instructions more (k = 4096: 995 -> 950 us; at 2048 the two are equal).
//  - tables of more than 4096 entries are kernels of their own, which keep their registers out of the others (11008 x 4096, k = 256:
//    156 -> 144 us, v = 12 with a base 835 -> 775).
// Measured, 11008 x 4096, v = 6: k = 4096 1152 -> 950 us, k = 256 261 -> 144 us; every distance on the vector ALUs 8.4 ms.
// 4096 x 4096, v = 8, k = 65536, entries loaded together, and whole where they are aligned: 5.1 -> 4.2 ms;
// 2048 x 2048 with a base 1.74 -> 1.42.
constexpr int WAVES = 16;
constexpr int SCREEN_ROWS = 4096;                       // table rows in LDS at once: two planes of 16 bytes each
constexpr int screen_instructions(int v, bool base) { return base && v > 6 ? 2 : 1; }
constexpr int screen_rows(int k) { return k >= SCREEN_ROWS ? SCREEN_ROWS : (k + 127) & ~127; }   // a wave takes up to four tiles of 32 at once

struct TableScale { int f; float h_max; bool fine; };

// Centroids [c0, c0 + rows) into the two planes, rows past the table repeating its last entry; returns the scale.
template <int V>
__device__ TableScale stage_screen_table(const __half *__restrict__ codebook, int stride, int len, int k, int c0, int rows, bool whole, half8 *plane, float *red) {
  constexpr int PER = SCREEN_ROWS / (WAVES * 64);
  const int tid = threadIdx.x, wave = tid >> 6;
  half8 first_half[PER], second_half[PER];
  int which[PER];
#pragma unroll
  for (int r = 0; r < PER; ++r) which[r] = min(c0 + tid + r * (WAVES * 64), k - 1);
  load_entries<V, PER>(codebook, which, stride, len, whole, first_half, second_half);
  float h[PER], most = 0.0f;
  bool fine = true;
#pragma unroll
  for (int r = 0; r < PER; ++r) {
    const int e = tid + r * (WAVES * 64);
    h[r] = 0.0f;
    if (e < rows) {
      const half8 e0 = first_half[r], e1 = second_half[r];
      _Float16 c[V];
#pragma unroll
      for (int j = 0; j < V; ++j) c[j] = j < 8 ? e0[j & 7] : e1[j & 7];
      float q = 0.0f;
#pragma unroll
      for (int j = 0; j < V; ++j) q = __fmaf_rn((float)c[j], (float)c[j], q);
      h[r] = 0.5f * q;
      fine = fine && h[r] < 0x1p28f;                      // (false for entries that are not numbers)
      most = fmaxf(most, h[r]);
      half8 lo = {}, hi = {};
      if constexpr (V <= 6) {
#pragma unroll
        for (int j = 0; j < V; ++j) { lo[j] = c[j]; hi[j] = c[j]; }
      } else {
#pragma unroll
        for (int j = 0; j < V; ++j) { if (j < 8) lo[j & 7] = c[j]; else hi[j & 7] = c[j]; }
      }
      plane[e] = lo;
      plane[rows + e] = hi;
    }
  }
  for (int s = 32; s > 0; s >>= 1) most = fmaxf(most, __shfl_xor(most, s, 64));
  const bool wave_fine = __all(fine);
  if ((tid & 63) == 0) { red[wave] = most; red[WAVES + wave] = wave_fine ? 1.0f : 0.0f; }
  __syncthreads();
  TableScale t;
  t.h_max = 0.0f; t.fine = true;
#pragma unroll
  for (int w = 0; w < WAVES; ++w) { t.h_max = fmaxf(t.h_max, red[w]); t.fine = t.fine && red[WAVES + w] != 0.0f; }
  // |c|^2 / 2 * 2^f below 2^15 and its parts' factor 2^-f a normal binary16 number
  t.f = t.h_max > 0.0f ? min(14, max(-14, 15 - __builtin_amdgcn_frexp_expf(t.h_max))) : 14;
#pragma unroll
  for (int r = 0; r < PER; ++r) {
    const int e = tid + r * (WAVES * 64);
    if (e < rows) {
      const float x = ldexpf(h[r], t.f);
      const _Float16 n1 = (_Float16)x;
      const float x1 = x - (float)n1;
      const _Float16 n2 = (_Float16)x1;
      const _Float16 n3 = (_Float16)(x1 - (float)n2);
      if constexpr (V <= 6) {
        plane[e][6] = n1; plane[e][7] = n2; plane[rows + e][6] = n3;
      } else {
        plane[rows + e][5] = n1; plane[rows + e][6] = n2; plane[rows + e][7] = n3;
      }
    }
  }
  __syncthreads();
  return t;
}

template <int V, bool BASE>
__device__ __forceinline__ void load_vector(const Vectors &a, int o, int u, bool on, float (&t)[V]) {
  const long long at = on ? (long long)o * a.row_step + (long long)u * a.vec_step : 0;
  if (a.elem_step == 1 && a.len == V) {
#pragma unroll
    for (int j = 0; j < V; ++j) {
      float x = __half2float(a.W[at + j]);
      if (BASE) x = __fsub_rn(x, __half2float(a.B[at + j]));
      t[j] = on ? x : 0.0f;
    }
    return;
  }
#pragma unroll
  for (int j = 0; j < V; ++j) {
    const long long c = at + (long long)(j < a.len ? j : 0) * a.elem_step;
    float x = __half2float(a.W[c]);
    if (BASE) x = __fsub_rn(x, __half2float(a.B[c]));
    t[j] = on && j < a.len ? x : 0.0f;
  }
}

template <int V>
__device__ __forceinline__ void load_halves(const Vectors &a, int o, int u, bool on, _Float16 (&t)[V]) {
  const long long at = on ? (long long)o * a.row_step + (long long)u * a.vec_step : 0;
  const _Float16 *from = reinterpret_cast<const _Float16 *>(a.W) + at;
  if (a.elem_step == 1 && a.len == V) {
#pragma unroll
    for (int j = 0; j < V; ++j) t[j] = from[j];
  } else {
#pragma unroll
    for (int j = 0; j < V; ++j) t[j] = from[(j < a.len ? j : 0) * a.elem_step];
#pragma unroll
    for (int j = 0; j < V; ++j) t[j] = j < a.len ? t[j] : (_Float16)0.0f;
  }
#pragma unroll
  for (int j = 0; j < V; ++j) t[j] = on ? t[j] : (_Float16)0.0f;
}

// The upper 32 lanes of x for the lower ones of y
__device__ __forceinline__ void swap_halves(unsigned &x, unsigned &y) {
  const auto z = __builtin_amdgcn_permlane32_swap(x, y, false, false);
  x = z[0]; y = z[1];
}
__device__ __forceinline__ void swap_halves(float &x, float &y) {
  unsigned i = __float_as_uint(x), j = __float_as_uint(y);
  swap_halves(i, j);
  x = __uint_as_float(i); y = __uint_as_float(j);
}
__device__ __forceinline__ void swap_halves(half8 &x, half8 &y) {
  uint4v i = __builtin_bit_cast(uint4v, x), j = __builtin_bit_cast(uint4v, y);
#pragma unroll
  for (int d = 0; d < 4; ++d) { unsigned p = i[d], q = j[d]; swap_halves(p, q); i[d] = p; j[d] = q; }
  x = __builtin_bit_cast(half8, i); y = __builtin_bit_cast(half8, j);
}

// The power of two that scales a difference's elements to below 2^14 (as far as the |c|^2 slots' factor allows).
template <int V>
__device__ __forceinline__ int vector_scale(const float (&t)[V], int f) {
  float most = 0.0f;
#pragma unroll
  for (int j = 0; j < V; ++j) most = fmaxf(most, fabsf(t[j]));
  return most > 0.0f ? min(f + 15, max(f - 14, 14 - __builtin_amdgcn_frexp_expf(most))) : f;
}

// The factor of the |c|^2 slots, -2^(e - f), as binary16; 0 when that is out of its range (the vector is then not trusted).
__device__ __forceinline__ _Float16 slot_factor(int e, int f) {
  const int x = e - f;
  return x >= -14 && x <= 15 ? (_Float16)(-ldexpf(1.0f, x)) : (_Float16)0.0f;
}

template <int V>
__device__ __forceinline__ void set_slots(half8 &b, int half, _Float16 factor) {
  if constexpr (V <= 6) { b[6] = factor; b[7] = half ? (_Float16)0.0f : factor; }
  else if (half) { b[5] = factor; b[6] = factor; b[7] = factor; }
}

// NT: tiles of 32 vectors a wave holds.  WIDE: blocks of 32 centroids.  CHUNKED: more than SCREEN_ROWS entries, a chunk of them after the other.  SPLIT: `split` waves (a power of two) share a tile of vectors, each taking its share
// of the table.  The first last_wgs workgroups take `last`, the others `first`.
template <int V, bool BASE, int NT, bool SPLIT, bool WIDE, bool CHUNKED>
__global__ __launch_bounds__(WAVES * 64, 4) void assign_screen_kernel(Vectors first, Vectors last, Padding padding, int last_wgs, const __half *__restrict__ codebook,
                                                                       int stride, int k, int bits, int seg_len, int split) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  clear_padding(padding);
  const int rows_lds = screen_rows(k);
  half8 *plane = reinterpret_cast<half8 *>(smem);                                     // [2][rows_lds]
  float *red = reinterpret_cast<float *>(smem + (size_t)rows_lds * 32);               // [2 * WAVES]
  unsigned *codes = reinterpret_cast<unsigned *>(red + 2 * WAVES);                    // [WAVES][NT * 32]
  float *meet = reinterpret_cast<float *>(codes + WAVES * NT * 32);                   // SPLIT: [3][WAVES][64]
  int *list = reinterpret_cast<int *>(meet + (SPLIT ? 3 * WAVES * 64 : 0));           // tables of several chunks: how many, then which
  constexpr bool TWO = screen_instructions(V, BASE) == 2;
  constexpr int TU = 2;                                         // tiles of the table taken at once
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), n = lane & 31, half = lane >> 5;
  const bool is_last = (int)blockIdx.x < last_wgs;
  const Vectors a = is_last ? last : first;
  const int n_chunks = CHUNKED ? (k + SCREEN_ROWS - 1) / SCREEN_ROWS : 1;
  const long long items = items_of(a, seg_len);
  const int groups = SPLIT ? WAVES / split : WAVES, part = SPLIT ? wave % split : 0;
  const int block_items = groups * NT * 32;
  const int n_blocks = (int)((items + block_items - 1) / block_items);
  unsigned *my_codes = codes + wave * (NT * 32);
  const PackLane pack(lane, seg_len, bits);
  const bool whole = stride == V && reinterpret_cast<size_t>(codebook) % load_bytes<V>() == 0;
  TableScale ts = {0, 0.0f, true};
  int *ticket = list;
  constexpr bool tickets = !SPLIT && !CHUNKED;
  if (tickets && threadIdx.x == 0) *ticket = 0;           // (seen by all behind the barriers of the next line)
  if constexpr (!CHUNKED) ts = stage_screen_table<V>(codebook, stride, a.len, k, 0, rows_lds, whole, plane, red);

  const int wg0 = is_last ? blockIdx.x : blockIdx.x - last_wgs, wgs = is_last ? last_wgs : gridDim.x - last_wgs;
  for (int turn = 0;; ++turn) {
    int blk = wg0 + turn * wgs, group = SPLIT ? wave / split : wave;
    if (tickets) {
      const int t = __builtin_amdgcn_readfirstlane(lane == 0 ? atomicAdd(ticket, 1) : 0);
      blk = wg0 + t / WAVES * wgs; group = t % WAVES;
    }
    if (blk >= n_blocks) break;
    const long long g0 = (long long)blk * block_items + group * (NT * 32);
    const Place place(a, g0, items, seg_len);
    half8 b[NT], b_lo[TWO ? NT : 1];
    // A lane looks after one vector: number `lane` of two tiles' 64, or n of one tile's 32, which both of its lanes then hold
    const int x = NT == 2 ? lane : n;
    int o, p;
    place.item(x, o, p);
    const bool on = o < a.rows && p < a.per_row, live = on && (NT == 2 || half == 0);
    constexpr bool KEEP = BASE && V <= 6;                    // (short enough to stay in registers across the search)
    float kept[KEEP ? V : 1];
    int e = 0;
    float b1[NT], b2[NT];
    int id[NT];
    bool trusted = true;                                     // (of this lane's vectors: every chunk's factor was in range)
    float h_max = 0.0f;
    for (int ch = 0; ch < n_chunks; ++ch) {
      if constexpr (CHUNKED) {
        __syncthreads();
        ts = stage_screen_table<V>(codebook, stride, a.len, k, ch * SCREEN_ROWS, rows_lds, whole, plane, red);
      }
      h_max = fmaxf(h_max, ts.h_max);
      trusted = trusted && ts.fine;
      if (ch == 0) {
        // the vector's operands in the lower lanes (lo) and in the upper ones (up), of its first and second part
        half8 lo = {}, up = {}, lo2 = {}, up2 = {};
        if constexpr (BASE) {
          float t[V];
          load_vector<V, BASE>(a, o, p, on, t);
          if constexpr (KEEP) {
#pragma unroll
            for (int j = 0; j < V; ++j) kept[j] = t[j];
          }
          e = vector_scale<V>(t, ts.f);
#pragma unroll
          for (int j = 0; j < V; ++j) {
            const float y = ldexpf(t[j], e);
            const _Float16 yh = (_Float16)y, yl = (_Float16)(y - (float)yh);
            if constexpr (V <= 6) { lo[j] = yh; up[j] = yl; }
            else if (j < 8) { lo[j & 7] = yh; lo2[j & 7] = yl; }
            else { up[j & 7] = yh; up2[j & 7] = yl; }
          }
        } else {
          _Float16 t[V];
          load_halves<V>(a, o, p, on, t);
#pragma unroll
          for (int j = 0; j < V; ++j) {
            if (j < 8) lo[j & 7] = t[j];
            else up[j & 7] = t[j];
          }
        }
        if constexpr (NT == 2) {
          swap_halves(lo, up);
          b[0] = lo; b[NT - 1] = up;
          if constexpr (TWO) { swap_halves(lo2, up2); b_lo[0] = lo2; b_lo[NT - 1] = up2; }
        } else {
          b[0] = half ? up : lo;
          if constexpr (TWO) b_lo[0] = half ? up2 : lo2;
        }
#pragma unroll
        for (int u = 0; u < NT; ++u) { b1[u] = -__builtin_inff(); b2[u] = -__builtin_inff(); id[u] = 0; }
      }
      if (ch == 0 || CHUNKED) {
        const _Float16 factor = slot_factor(e, ts.f);
        trusted = trusted && factor != (_Float16)0.0f;
        if constexpr (BASE && NT == 2) {
          unsigned f0 = __builtin_bit_cast(unsigned short, factor), f1 = f0;
          swap_halves(f0, f1);
          set_slots<V>(b[0], half, __builtin_bit_cast(_Float16, (unsigned short)f0));
          set_slots<V>(b[NT - 1], half, __builtin_bit_cast(_Float16, (unsigned short)f1));
        } else {
#pragma unroll
          for (int u = 0; u < NT; ++u) set_slots<V>(b[u], half, factor);
        }
      }
      const int tiles = (min(k - ch * SCREEN_ROWS, SCREEN_ROWS) + 31) >> 5, rounds = (tiles + TU - 1) / TU;
      const int step = SPLIT ? split : 1, round0 = ch * (SCREEN_ROWS / 32 / TU);
      const half8 *mine = plane + (half ? rows_lds : 0) + n;
      // A round's two tiles: the products of one run while the largest score of the other is found
      float16v s0[NT], s1[NT];
      auto products = [&](half8 c, float16v (&s)[NT]) {
#pragma unroll
        for (int u = 0; u < NT; ++u) {
          float16v z;
#pragma unroll
          for (int r = 0; r < 16; ++r) z[r] = 0.0f;
          s[u] = __builtin_amdgcn_mfma_f32_32x32x16_f16(c, b[u], z, 0, 0, 0);
          if constexpr (TWO) s[u] = __builtin_amdgcn_mfma_f32_32x32x16_f16(c, b_lo[u], s[u], 0, 0, 0);
        }
      };
      auto max3 = [](float p_, float q_, float r_) { return fmaxf(fmaxf(p_, q_), r_); };
      auto largest = [&](const float16v &v, float m) {
        const float m0 = max3(v[0], v[1], v[2]), m1 = max3(v[3], v[4], v[5]), m2 = max3(v[6], v[7], v[8]);
        const float m3 = max3(v[9], v[10], v[11]), m4 = max3(v[12], v[13], v[14]);
        return max3(max3(m0, m1, m2), max3(m3, m4, v[15]), m);
      };
      auto take = [&](int u, float m, int number) {
        const bool up = m > b1[u];
        b2[u] = __builtin_amdgcn_fmed3f(b1[u], b2[u], m);
        id[u] = up ? number : id[u];
        b1[u] = up ? m : b1[u];
      };
      auto tile_of = [&](int round, int x) { return mine[(min(round, rounds - 1) * TU + x) * 32]; };
      if constexpr (SPLIT) {                                 // (few rounds a chunk: nothing to run ahead of)
        half8 c0 = tile_of(part, 0), c1 = tile_of(part, 1);
        for (int round = part; round < rounds; round += step) {
          products(c0, s0);
          products(c1, s1);
          c0 = tile_of(round + step, 0);
          c1 = tile_of(round + step, 1);
#pragma unroll
          for (int u = 0; u < NT; ++u) {
            take(u, largest(s0[u], s0[u][0]), (round0 + round) * TU);
            take(u, largest(s1[u], s1[u][0]), (round0 + round) * TU + 1);
          }
        }
        continue;
      }
      half8 c1 = tile_of(part, 1), next = tile_of(part + step, 0);
      products(tile_of(part, 0), s0);
      for (int round = part; round < rounds; round += step) {
        float m[NT];
        products(c1, s1);
        c1 = tile_of(round + step, 1);
#pragma unroll
        for (int u = 0; u < NT; ++u) {
          m[u] = largest(s0[u], s0[u][0]);
          if constexpr (!WIDE) take(u, m[u], (round0 + round) * TU);
        }
        __builtin_amdgcn_sched_barrier(0);
        products(next, s0);
        next = tile_of(round + 2 * step, 0);
#pragma unroll
        for (int u = 0; u < NT; ++u) {
          if constexpr (WIDE) take(u, largest(s1[u], m[u]), round0 + round);
          else take(u, largest(s1[u], s1[u][0]), (round0 + round) * TU + 1);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    if constexpr (SPLIT) {                                   // the waves of a group meet in their first one
      float *m1 = meet, *m2 = meet + WAVES * 64, *mb = meet + 2 * WAVES * 64;
      m1[wave * 64 + lane] = b1[0]; m2[wave * 64 + lane] = b2[0]; mb[wave * 64 + lane] = __int_as_float(id[0]);
      __syncthreads();
      if (part == 0) {
        for (int w = 1; w < split; ++w) {
          const float o1 = m1[(wave + w) * 64 + lane], o2 = m2[(wave + w) * 64 + lane];
          const int ob = __float_as_int(mb[(wave + w) * 64 + lane]);
          b2[0] = fmaxf(fminf(b1[0], o1), fmaxf(b2[0], o2));
          if (o1 > b1[0]) { b1[0] = o1; id[0] = ob; }
        }
      }
      __syncthreads();
    }
    if constexpr (CHUNKED) {
      if (threadIdx.x == 0) list[0] = 0;
      __syncthreads();
    }

    // the distances as defined, for the centroids of the winning block: in the vector's lane, or half of them in each of its two lanes
    if (part == 0) {
      float t[V];
      if constexpr (KEEP) {
#pragma unroll
        for (int j = 0; j < V; ++j) t[j] = kept[j];
      } else if constexpr (BASE) {
        load_vector<V, BASE>(a, o, p, on, t);
      } else {                                               // the operands still hold the vectors: elements 0 .. 7 in the lower lanes
        half8 lo = b[0], up = b[NT - 1];
        if constexpr (NT == 2) {
          swap_halves(lo, up);
        } else {
          const uint4v mine = __builtin_bit_cast(uint4v, b[0]);
          uint4v l, h;
#pragma unroll
          for (int d = 0; d < 4; ++d) { l[d] = __shfl(mine[d], n, 64); h[d] = V > 8 ? __shfl(mine[d], n + 32, 64) : 0u; }
          lo = __builtin_bit_cast(half8, l); up = __builtin_bit_cast(half8, h);
        }
#pragma unroll
        for (int j = 0; j < V; ++j) t[j] = (float)(j < 8 ? lo[j & 7] : up[j & 7]);
      }
      // what the lower and the upper lanes found for the vector
      float s_lo = b1[0], s_up = b1[NT - 1], q_lo = b2[0], q_up = b2[NT - 1];
      unsigned i_lo = (unsigned)id[0], i_up = (unsigned)id[NT - 1];
      if constexpr (NT == 2) {
        swap_halves(s_lo, s_up); swap_halves(q_lo, q_up); swap_halves(i_lo, i_up);
      } else {
        const float s = __shfl_xor(b1[0], 32, 64), q = __shfl_xor(b2[0], 32, 64);
        const unsigned i = (unsigned)__shfl_xor(id[0], 32, 64);
        if (half) { s_lo = s; q_lo = q; i_lo = i; }
        else { s_up = s; q_up = q; i_up = i; }
      }
      const bool lower = s_lo >= s_up;
      const float best_s = fmaxf(s_lo, s_up), second = fmaxf(fminf(s_lo, s_up), fmaxf(q_lo, q_up));
      bool sure = trusted;
      {
        const float c_max = __builtin_amdgcn_sqrtf(2.0f * h_max) * 1.001f;
        float tt = 0.0f;
#pragma unroll
        for (int j = 0; j < V; ++j) tt = __fmaf_rn(t[j], t[j], tt);
        const float T = __builtin_amdgcn_sqrtf(tt) * 1.001f, down = BASE ? ldexpf(1.0f, -e) : 1.0f, q = 0x1p-12f, qt = 0x1p-12f * down;
        const float dist = fmaxf(0.0f, tt - 2.0f * best_s * down) + 0x1p-13f * (tt + c_max * c_max);
        const float R = T + __builtin_amdgcn_sqrtf(dist) * 1.001f;
        const float eps = screen_instructions(V, BASE) * 0x1.2p-19f * ((T + qt) * (R + q) + 0.5f * R * R + 0x1p-26f * (1.0f + down)) + (V + 3) * 0x1p-23f * dist +
                          0x1p-28f * h_max + 0x1p-37f + 0x1p-21f * down * R;
        const float gap = (best_s - second) * down;
        sure = sure && gap > eps;                            // (false when anything is not a number)
      }
      // rows of a lane's results: registers r & 3 of quads of rows 8 apart, the upper lanes' quads 4 below
      // (rows past the table repeat its last entry, which is never preferred to the entry itself)
      constexpr int MINE = (WIDE ? 32 : 16) * NT / 2;
      const int row0 = (int)(lower ? i_lo : i_up) * (WIDE ? 64 : 32) + (lower ? 0 : 4) + (NT == 2 ? 0 : half * 16);
      float best = __builtin_inff();
      int nearest = 0;
      auto consider = [&](float d, int at) {
        const bool closer = d < best;
        best = closer ? d : best;
        nearest = closer ? at : nearest;
      };
      if constexpr (!CHUNKED) {
        const half8 *from = plane + row0, *from2 = from + (V > 8 ? rows_lds : 0);
#pragma unroll
        for (int r = 0; r < MINE; ++r) {
          const int at = (r & 3) + 8 * (r >> 2);
          consider(distance<V>(t, from[at], from2[at]), at);
        }
      } else {
        constexpr int QUADS = NT == 1 ? 2 : 1;
#pragma unroll QUADS
        for (int quad = 0; quad < MINE / 4; ++quad) {
          int which[4];
          float d[4];
#pragma unroll
          for (int r = 0; r < 4; ++r) which[r] = min(row0 + r + 8 * quad, k - 1);
          distances_to<V, 4>(codebook, which, stride, a.len, whole, t, d);
#pragma unroll
          for (int r = 0; r < 4; ++r) consider(d[r], r + 8 * quad);
        }
      }
      unsigned arg = best < __builtin_inff() ? (unsigned)min(row0 + nearest, k - 1) : 0u;
      if constexpr (NT == 1) {
        const float od = __shfl_xor(best, 32, 64);
        const unsigned oa = __shfl_xor(arg, 32, 64);
        if (od < best || (od == best && oa < arg)) { best = od; arg = oa; }
      }
      // vectors whose block is not sure: the wave takes them one at a time, its lanes the centroids in turn
      if constexpr (CHUNKED) {
        if (live && !sure) list[1 + atomicAdd(&list[0], 1)] = group * (NT * 32) + x;
      } else {
        for (unsigned long long todo = __ballot(live && !sure); todo; todo &= todo - 1) {
          const int w = __builtin_ctzll(todo);
          float tv[V];
#pragma unroll
          for (int j = 0; j < V; ++j) tv[j] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(t[j]), w));
          float bd = __builtin_inff();
          unsigned bi = 0xFFFFFFFFu;
          auto compare = [&](int i0, auto entries) {
#pragma unroll
            for (int y = 0; y < decltype(entries)::value; ++y) {
              const int i = i0 + 64 * y;
              const float d = distance<V>(tv, plane[i], plane[V > 8 ? rows_lds + i : i]);
              if (d < bd) { bd = d; bi = (unsigned)i; }
            }
          };
          int i0 = lane;                                       // (rows_lds is a multiple of 128; two at a time 297 x 4231 took 332 us, 298)
          for (; i0 + 192 < rows_lds; i0 += 256) compare(i0, std::integral_constant<int, 4>{});
          if (i0 < rows_lds) compare(i0, std::integral_constant<int, 2>{});
          wave_arg_min(bd, bi);
          if (lane == w) arg = bi == 0xFFFFFFFFu ? 0u : bi;    // (no distance below infinity: the first centroid)
        }
      }
      if (NT == 2 || half == 0) my_codes[x] = live ? arg : 0u;
    }
    if constexpr (CHUNKED) {
      // the vectors that are not sure, against the whole table: every wave takes a share of it
      __syncthreads();
      const int n_list = list[0], share = (k + WAVES * 64 - 1) / (WAVES * 64) * 64, from = wave * share, to = min(k, from + share);
      float *found_d = reinterpret_cast<float *>(plane);                    // [n_list][WAVES], over the last chunk
      unsigned *found_i = reinterpret_cast<unsigned *>(plane) + NT * 32 * WAVES * WAVES;
      for (int x = 0; x < n_list; ++x) {
        const int which = list[1 + x];                                       // group and item of the group
        const Place where(a, (long long)blk * block_items + which / (NT * 32) * (NT * 32), items, seg_len);
        int o, p;
        where.item(which % (NT * 32), o, p);
        float t[V];
        load_vector<V, BASE>(a, o, p, true, t);
        float bd = __builtin_inff();
        unsigned bi = 0xFFFFFFFFu;
        auto compare = [&](int i0, auto entries) {
          constexpr int N = decltype(entries)::value;
          int which[N];
          float d[N];
#pragma unroll
          for (int y = 0; y < N; ++y) which[y] = min(i0 + 64 * y + lane, k - 1);
          distances_to<V, N>(codebook, which, stride, a.len, whole, t, d);
#pragma unroll
          for (int y = 0; y < N; ++y)
            if (d[y] < bd) { bd = d[y]; bi = (unsigned)which[y]; }
        };
        int i0 = from;
        for (; i0 + 256 <= to; i0 += 256) compare(i0, std::integral_constant<int, 4>{});
        for (; i0 < to; i0 += 64) compare(i0, std::integral_constant<int, 1>{});        // (a share need not fill fours: k = 5000, 320)
        wave_arg_min(bd, bi);
        if (lane == 0) { found_d[x * WAVES + wave] = bd; found_i[x * WAVES + wave] = bi; }
      }
      __syncthreads();
      if ((int)threadIdx.x < n_list) {
        float bd = __builtin_inff();
        unsigned bi = 0u;                                    // (no distance below infinity: the first centroid)
        for (int w = 0; w < WAVES; ++w) {                    // ascending shares of the table: the first of equal distances stays
          const float d = found_d[threadIdx.x * WAVES + w];
          if (d < bd) { bd = d; bi = found_i[threadIdx.x * WAVES + w]; }
        }
        const int which = list[1 + threadIdx.x];
        codes[which / (NT * 32) * (SPLIT ? split : 1) * (NT * 32) + which % (NT * 32)] = bi;
      }
      __syncthreads();
    }
    if (part != 0) continue;                                 // (every wave passes the same barriers: they are all above)
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    if (a.scatter_bit >= 0) {
      for (int x = lane; x < NT * 32; x += 64) {
        int o, p;
        place.item(x, o, p);
        if (o < a.rows && p < a.per_row) scatter_index(a, p, my_codes[x], bits);
      }
    } else {
      pack_items(a, place, NT * 32, pack, bits, my_codes, lane);
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  }
}

// ---- every distance on the vector ALUs ------------------------------------------------------------------------------------
//
// Short tables: a lane per vector, the table in LDS as binary32 and read with wave-uniform addresses.  Bound by the loads of W and
// by how many waves there are to wait for them (127 x 1408, v = 2, k = 16, with a base: 23 us at a lane per 8 vectors and 1024
// lanes a workgroup).
constexpr int SHORT_TABLE = 64, SHORT_THREADS = 256;

template <int V>
__global__ __launch_bounds__(SHORT_THREADS) void assign_short_kernel(Vectors first, Vectors last, Padding padding, int last_wgs, const __half *__restrict__ codebook,
                                                                     int stride, int k, int bits, int seg_len) {
  __shared__ __attribute__((aligned(16))) float table[SHORT_TABLE * V];
  __shared__ unsigned codes[SHORT_THREADS];
  clear_padding(padding);
  const bool is_last = (int)blockIdx.x < last_wgs;
  const Vectors a = is_last ? last : first;
  const long long items = items_of(a, seg_len), g0 = (long long)(is_last ? blockIdx.x : blockIdx.x - last_wgs) * SHORT_THREADS;
  const int lane = threadIdx.x & 63, wave0 = threadIdx.x & ~63;
  const Place place(a, g0 + wave0, items, seg_len);
  int o, p;
  place.item(lane, o, p);
  const bool live = o < a.rows && p < a.per_row;
  float t[V];
  if (a.B) load_vector<V, true>(a, o, p, live, t);
  else load_vector<V, false>(a, o, p, live, t);
  for (int e = threadIdx.x; e < k * V; e += SHORT_THREADS)
    table[e] = e % V < a.len ? __half2float(codebook[(long long)(e / V) * stride + e % V]) : 0.0f;
  __syncthreads();
  float best = __builtin_inff();
  unsigned arg = 0u;
#pragma unroll 4
  for (int i = 0; i < k; ++i) {
    const float d = distance<V>(t, [&](int j) -> float { return table[i * V + j]; });
    if (d < best) { best = d; arg = (unsigned)i; }
  }
  if (a.scatter_bit >= 0) {
    if (live) scatter_index(a, p, arg, bits);
    return;
  }
  codes[threadIdx.x] = live ? arg : 0u;
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  pack_items(a, place, 64, PackLane(lane, seg_len, bits), bits, codes + wave0, lane);
}

// Long vectors.  A lane owns `seg` consecutive vectors of a row, seg = 8, 16 or 32 chosen so that they fill whole dwords of
// the row's index stream (lanes never share an output dword), and takes them VB at a time against the whole table, which sits in LDS as
// binary32 and is read with wave-uniform addresses (one broadcast read feeds VB x 64 distances).  Tables larger than
// the LDS chunk are walked chunk by chunk with the running minimum kept in registers.

constexpr int AT = 1024;                 // threads per workgroup
constexpr unsigned LDS_TABLE_BYTES = 128u * 1024u;

constexpr int table_stride(int v) { return v <= 2 ? v : v <= 4 ? 4 : v <= 8 ? 8 : 16; }

template <int V, int VB>
__global__ __launch_bounds__(AT) void assign_kernel(Vectors first, Vectors last, Padding padding, int last_wgs, const __half *__restrict__ codebook, int stride, int k,
                                                    int bits, int chunk, int seg_len) {
  extern __shared__ __attribute__((aligned(16))) float table[];       // [chunk][TS]: rows padded to 16-byte reads
  constexpr int TS = table_stride(V);
  clear_padding(padding);
  const bool is_last = (int)blockIdx.x < last_wgs;
  const Vectors a = is_last ? last : first;
  const int segs = (a.per_row + seg_len - 1) / seg_len;
  const long long item = (long long)(is_last ? blockIdx.x : blockIdx.x - last_wgs) * AT + threadIdx.x;
  const bool live = item < (long long)a.rows * segs;
  const int o = live ? (int)(item / segs) : 0;
  const int seg = live ? (int)(item - (long long)o * segs) : 0;
  unsigned *row = reinterpret_cast<unsigned *>(a.idx + (long long)o * a.idx_stride);
  long long at = (long long)seg * (seg_len * bits / 32);
  unsigned long long buf = 0;
  int fill = 0;
  const int n_chunks = (k + chunk - 1) / chunk;
  auto stage = [&](int c0) {             // centroids [c0, c0 + chunk) as binary32; past k: never read
    const int n = min(chunk, k - c0) * V;
    for (int e = threadIdx.x; e < n; e += AT)
      table[(e / V) * TS + e % V] = e % V < a.len ? __half2float(codebook[(long long)(c0 + e / V) * stride + e % V]) : 0.0f;
  };
  if (n_chunks == 1) { stage(0); __syncthreads(); }
  for (int r = 0; r < seg_len / VB; ++r) {                   // every lane walks every round: the barriers below need all of them
    const int p0 = seg * seg_len + r * VB;
    float t[VB][V], best[VB];
    int arg[VB];
#pragma unroll
    for (int u = 0; u < VB; ++u) {
      best[u] = __builtin_inff(); arg[u] = 0;
      const bool on = live && p0 + u < a.per_row;
      if (a.B) load_vector<V, true>(a, o, p0 + u, on, t[u]);
      else load_vector<V, false>(a, o, p0 + u, on, t[u]);
    }
    for (int ch = 0; ch < n_chunks; ++ch) {
      if (n_chunks > 1) { __syncthreads(); stage(ch * chunk); __syncthreads(); }
      const int n = min(chunk, k - ch * chunk);
#pragma unroll 2
      for (int i = 0; i < n; ++i) {
        float c[V];
#pragma unroll
        for (int j = 0; j < V; ++j) c[j] = table[i * TS + j];
#pragma unroll
        for (int u = 0; u < VB; ++u) {
          const float d = distance<V>(t[u], [&](int j) -> float { return c[j]; });
          if (d < best[u]) { best[u] = d; arg[u] = ch * chunk + i; }
        }
      }
    }
    // append the round's indices to the lane's bit stream
#pragma unroll
    for (int u = 0; u < VB; ++u) {
      if (live && p0 + u < a.per_row) {
        if (a.scatter_bit >= 0) { scatter_index(a, p0 + u, (unsigned)arg[u], bits); continue; }
        buf |= (unsigned long long)arg[u] << fill;
        fill += bits;
        if (fill >= 32) { store_dword(a, row + at, at, (unsigned)buf); ++at; buf >>= 32; fill -= 32; }
      }
    }
  }
  if (live && fill > 0) store_dword(a, row + at, at, (unsigned)buf);              // the row's last, partly filled dword: upper bits zero
}

// vectors per segment: the fewest whose bits fill whole dwords
int segment(int bits) { return bits % 4 == 0 ? 8 : bits % 2 == 0 ? 16 : 32; }

template <int V>
int launch_plain(const Vectors &first, const Vectors &last, const Padding &padding, const __half *codebook, int k, int bits, hipStream_t s) {
  constexpr int VB = V <= 8 ? 8 : 4;       // vectors a lane holds at once: each centroid read from LDS serves VB x 64 distances
  auto kernel = assign_kernel<V, VB>;
  VQ_ALLOW_FULL_LDS(kernel);
  const int chunk = min(k, (int)(LDS_TABLE_BYTES / (table_stride(V) * sizeof(float))));
  const int seg_len = segment(bits);
  auto wgs = [&](const Vectors &a) { return (items_of(a, seg_len) / seg_len + AT - 1) / AT; };
  const long long blocks = wgs(first) + wgs(last);
  if (blocks > 0x7fffffffLL) return VQ_ERR_UNSUPPORTED;
  hipLaunchKernelGGL(kernel, dim3((unsigned)blocks), dim3(AT), (size_t)chunk * table_stride(V) * sizeof(float), s, first, last, padding, (int)wgs(last),
                     codebook, V, k, bits, chunk, seg_len);
  return hipGetLastError() == hipSuccess ? VQ_OK : VQ_ERR_HIP;
}

template <int V>
int launch_short(const Vectors &first, const Vectors &last, const Padding &padding, const __half *codebook, int k, int bits, hipStream_t s) {
  const int seg_len = segment(bits);
  const long long last_wgs = (items_of(last, seg_len) + SHORT_THREADS - 1) / SHORT_THREADS;
  const long long blocks = (items_of(first, seg_len) + SHORT_THREADS - 1) / SHORT_THREADS + last_wgs;
  if (blocks > 0x7fffffffLL) return VQ_ERR_UNSUPPORTED;
  hipLaunchKernelGGL((assign_short_kernel<V>), dim3((unsigned)blocks), dim3(SHORT_THREADS), 0, s, first, last, padding, (int)last_wgs, codebook, V, k, bits, seg_len);
  return hipGetLastError() == hipSuccess ? VQ_OK : VQ_ERR_HIP;
}

template <int V, bool BASE, int NT, bool SPLIT, bool WIDE, bool CHUNKED>
int launch_screen_nt(const Vectors &first, const Vectors &last, const Padding &padding, const __half *codebook, int k, int bits, int split, hipStream_t s) {
  auto kernel = assign_screen_kernel<V, BASE, NT, SPLIT, WIDE, CHUNKED>;
  VQ_ALLOW_FULL_LDS(kernel);
  const int seg_len = segment(bits), block_items = WAVES / split * NT * 32;
  const size_t lds = (size_t)screen_rows(k) * 32 + 2 * WAVES * sizeof(float) + WAVES * NT * 32 * sizeof(unsigned) + (SPLIT ? 3 * WAVES * 64 * sizeof(float) : 0) +
                     (k > SCREEN_ROWS ? WAVES / split * NT * 32 + 1 : 1) * sizeof(int);
  const long long blocks = (items_of(first, seg_len) + block_items - 1) / block_items;
  long long last_wgs = (items_of(last, seg_len) + block_items - 1) / block_items, wgs = blocks;
  if (blocks > 0x7fffffffLL || last_wgs > 0x7fffffffLL) return VQ_ERR_UNSUPPORTED;
  // one workgroup fits a compute unit; it keeps its table and walks the blocks (tables of several chunks are staged anew for
  // every block anyway).  The cut-off vectors' workgroups come first, the others share what is left.
  if (k <= SCREEN_ROWS && blocks + last_wgs > cu_count()) {
    last_wgs = min(last_wgs, (long long)max(1, cu_count() / 4));
    if (items_of(last, seg_len) == 0) last_wgs = 0;
    wgs = min(blocks, cu_count() - last_wgs);
  }
  hipLaunchKernelGGL(kernel, dim3((unsigned)(wgs + last_wgs)), dim3(WAVES * 64), lds, s, first, last, padding, (int)last_wgs, codebook, V, k, bits, seg_len, split);
  return hipGetLastError() == hipSuccess ? VQ_OK : VQ_ERR_HIP;
}

template <int V, bool BASE>
int launch_screen(const Vectors &first, const Vectors &last, const Padding &padding, const __half *codebook, int k, int bits, hipStream_t s) {
  const long long tiles = (items_of(first, segment(bits)) + items_of(last, segment(bits))) / 32;
  // 64 vectors of a wave share every table read, 32 where that leaves fewer waves idle in the last round (a round of the
  // smaller blocks takes about 0.6 of the time), and with less than one round of those the waves of a workgroup
  // share the table's rows until there is about one
  const long long waves = (long long)cu_count() * WAVES, rounds2 = (tiles + 2 * waves - 1) / (2 * waves), rounds1 = (tiles + waves - 1) / waves;
  if (10 * rounds2 <= 6 * rounds1)
    return k > SCREEN_ROWS    ? launch_screen_nt<V, BASE, 2, false, true, true>(first, last, padding, codebook, k, bits, 1, s)
           : k == SCREEN_ROWS ? launch_screen_nt<V, BASE, 2, false, true, false>(first, last, padding, codebook, k, bits, 1, s)
                              : launch_screen_nt<V, BASE, 2, false, false, false>(first, last, padding, codebook, k, bits, 1, s);
  int split = 1;
  while (split < WAVES && tiles * split * 2 <= waves && split * 128 < min(k, SCREEN_ROWS)) split *= 2;
  return k > SCREEN_ROWS ? launch_screen_nt<V, BASE, 1, true, false, true>(first, last, padding, codebook, k, bits, split, s)
                         : launch_screen_nt<V, BASE, 1, true, false, false>(first, last, padding, codebook, k, bits, split, s);
}

template <int V>
int launch_v(const Vectors &first, const Vectors &last, const Padding &padding, const __half *codebook, int k, int bits, hipStream_t s) {
  // (a table of one or two blocks of 32 is compared as fast as it is screened; 13: three slots for |c|^2 beside the elements)
  if (k < SHORT_TABLE) return launch_short<V>(first, last, padding, codebook, k, bits, s);
  if constexpr (V <= 13) {
    return first.B ? launch_screen<V, true>(first, last, padding, codebook, k, bits, s) : launch_screen<V, false>(first, last, padding, codebook, k, bits, s);
  } else {
    return launch_plain<V>(first, last, padding, codebook, k, bits, s);
  }
}

int launch(int v, const Vectors &first, const Vectors &last, const Padding &padding, const __half *codebook, int k, int bits, hipStream_t s) {
  switch (v) {
#define VQ_V(N) case N: return launch_v<N>(first, last, padding, codebook, k, bits, s);
    VQ_V(1) VQ_V(2) VQ_V(3) VQ_V(4) VQ_V(5) VQ_V(6) VQ_V(7) VQ_V(8) VQ_V(9) VQ_V(10) VQ_V(11) VQ_V(12) VQ_V(13) VQ_V(14) VQ_V(15) VQ_V(16)
#undef VQ_V
    default: return VQ_ERR_UNSUPPORTED;
  }
}

}  // namespace

int launch_assign(const __half *W, const __half *B, long long ld, int rows, int cols, const __half *codebook, int v, int k,
                  unsigned char *idx, long long idx_stride, bool clear, hipStream_t s) {
  const int bits = index_bits(k), full = cols / v, len = cols % v;
  const long long at = (long long)full * v, end = (long long)full * bits;
  const Vectors whole = {W, B, ld, v, 1, full ? rows : 0, full, v, idx, idx_stride, len ? end : (end + 31) / 32 * 32, -1};
  // the cut-off last vector of every row, compared over its own elements
  const Vectors last = {W + at, B ? B + at : nullptr, 0, ld, 1, len ? 1 : 0, rows, len, idx, idx_stride, 0, end};
  const int used = (int)(((long long)(full + (len ? 1 : 0)) * bits + 31) / 32);
  return launch(v, whole, last, Padding{idx, idx_stride, rows, used, clear ? (int)(idx_stride / 4) - used : 0}, codebook, k, bits, s);
}

// Vectors down the columns of W [rows][ld] (Sec. 3.1, Algorithm 1): index streams [ceil(rows / v)][idx_stride], one index per column.
int launch_assign_down(const __half *W, const __half *B, long long ld, int rows, int cols, const __half *codebook, int v, int k,
                       unsigned char *idx, long long idx_stride, bool clear, hipStream_t s) {
  const int bits = index_bits(k), full = rows / v, len = rows % v;
  const long long at = (long long)full * v * ld, end = ((long long)cols * bits + 31) / 32 * 32;
  const Vectors whole = {W, B, v * ld, 1, ld, full, cols, v, idx, idx_stride, end, -1};
  // the cut-off last block of rows: one stream of shorter vectors
  const Vectors last = {W + at, B ? B + at : nullptr, 0, 1, ld, len ? 1 : 0, cols, len, idx + (long long)full * idx_stride, idx_stride, end, -1};
  const int used = (int)(end / 32);
  return launch(v, whole, last, Padding{idx, idx_stride, full + (len ? 1 : 0), used, clear ? (int)(idx_stride / 4) - used : 0}, codebook, k, bits, s);
}

}  // namespace vq
