// vq_quantize_columns in one launch: Algorithm 1 (Sec. 3.1) with its nearest-centroid searches on the matrix cores.
#include "vq_quantize.hpp"
#include <type_traits>

namespace vq {
namespace {

// A workgroup owns up to four stack positions (P of them) and walks all columns of the matrix with them: nothing it needs comes
// from another workgroup.  Four of its eight waves search, one on each SIMD; the tables stay where they are for the whole launch: as
// operands of v_mfma_f32_16x16x32_f16 in their registers, 64 centroids a wave and group (sixteen groups of a 4096-entry table), and as
// plain entries in LDS.  The other four keep the positions' rows of the running block and of the next one, 64 columns a wave, as results of
// v_mfma_f32_4x4x1_16b_f32: four rows (broadcast from one of the sixteen blocks of operand A) by 64 columns, so that P v = 18 rows
// cost 20 (of 32x32x2 they would use 18 of 32).
//
// One column.  Every search wave holds the P vectors t, up to four elements a lane (lane 16 q + 4 n + j: vector n, the j-th quarter
// of its elements; the four rows of lanes alike), scales them by a power of two and rounds them to binary16: operand B.  Scores
// t . c - |c|^2 / 2 come from the matrix cores.  Entries of up to six elements take 8 of its 32 k slots,
// |c|^2 / 2 in two parts behind them, so a row of operand A holds four centroids and each of the 16 columns of operand B one of
// four vectors at one of the four places, zeros elsewhere: 64 centroids with four vectors at once.  Entries of up to 14
// elements take 16 slots, longer ones 32.  A lane gets the scores of four neighbouring centroids at a time and keeps the largest of these
// groups' maxima, its group's number in the lowest bits, and the second largest.  A row of lanes computes the distances of its best
// four centroids as defined, one in each lane of a quad; where anything else of the wave is within the rounding bounds of its largest
// score (in a tenth of the columns) those distances are computed too.  Scores see eleven bits of t, and their lowest six bits are the
// group's number: both are part of the bounds (loop_table), and every index is decided by distances as defined.  What the rows of all waves find meets in LDS (an atomic
// minimum of distance bits and index).  Behind the column's only barrier every search wave looks the winner up, forms the error and the
// next column's t by itself: nothing else is exchanged on the way from one column to the next.
//
// The block's running weights lag two columns behind: t of column n + 1 is the value with the errors up to column n - 2, which the
// keeping waves post while column n is searched, less the last two errors' shares, which the search waves hold.  The keeping
// waves also file E; the search waves store T, the quantized weights and the indices, one kind a wave, as they never wait for memory.
//
// Between two blocks there is little to do: the next one's columns have their errors already.  The columns beyond it take a block's errors beside the
// next block's columns: a step of eight rows of H^-1 by 128 columns a keeping wave and column, its loads a column ahead, until all columns
// have them (what is left at the end of a block, beyond 4096 columns or so, follows without a pause).
//
// What bounds it: the chain of a column.  A wave on its own issues an instruction every five clocks or so, and what counts is how many
// stand on the path between one column's t and the next (about 200 with a 4096-entry table), the LDS round trips (130 clocks, four of
// them) and the barrier, not any rate: 2300 clocks a column (of 2.35 GHz), of which the comparisons of the scores are 500.  Whatever else a SIMD
// executes adds to that, binary32 products above all: they keep the search wave from issuing for as long as they take, wherever in a column
// they stand and whatever the waves' priorities (80 instructions of 8 clocks a column: search 1910 -> 2460 clocks; without any later columns
// 4096 x 4096 would take 3.5 ms, nearly all of the 0.5 between are the products).  Eight search waves of half the table each are slower (4.8 ms against 4.6
// then): everything but the comparisons is issued twice on every SIMD.
// With the later columns' update at the end of each block, by all waves and waiting for H^-1 and W, 94 of a block's 340 thousand clocks:
// v = 6, k = 4096, 4096 x 4096 4.57 -> 4.03 ms; 3000 x 2000 1831 -> 1714 us; v = 8, k = 4096 2680 -> 2247; v = 12, k = 4096 2803 -> 2393; v = 4, k = 256
// 1348 -> 1200.  The same update as 16 x 16 x 1 products in place of 4 x 4 x 1 took as long, and so did one ahead of the kept columns' update
// in place of behind it; sums in the vector ALUs for the kept columns 2 % longer; stores of T, weights and indices by the keeping waves,
// whose loads then wait for them, 2 % longer.
typedef _Float16 half8v __attribute__((ext_vector_type(8)));
typedef _Float16 half2v __attribute__((ext_vector_type(2)));
typedef float float4v __attribute__((ext_vector_type(4)));
typedef float float2v __attribute__((ext_vector_type(2)));

constexpr int PMAX = 4;
constexpr int SEARCH = 4, KEEP = 4;      // waves
constexpr int LOOP_THREADS = (SEARCH + KEEP) * 64;
// k slots of an entry; entries side by side in an instruction's 32; registers of 8 slots a lane holds per 64 centroids.
constexpr int entry_slots(int vp) { return vp <= 6 ? 8 : vp <= 14 ? 16 : 32; }
constexpr int entries_wide(int vp) { return 32 / entry_slots(vp); }
constexpr int group_tiles(int vp) { return 4 / entries_wide(vp); }
constexpr int quarter(int vp) { return vp <= 8 ? 2 : vp <= 12 ? 3 : 4; }     // elements a lane holds of a vector
constexpr unsigned TAG = 63u;            // group, tile and place: the lowest bits of a score

struct ColumnConstants { float diag, inverse, beside, beside2; };            // of H^-1: (n, n), its reciprocal or 0, (n, n + 1), (n - 1, n + 1)

constexpr int ROWS = 36;                 // of four positions of eight or two of sixteen, and four more that whole sixteen-byte pieces take

struct LoopExchange {                    // LDS
  unsigned long long nearest[2][4][PMAX];  // [main, residual][column & 3]: smallest (distance bits, index) so far
  // by rows (vector * VP + element), in whole quarters of the last vector
  float next_w[2][ROWS];                 // the next column's weights without the last two errors
  float e[2][ROWS];
  float first_t[ROWS];                   // the weights of a block's first column
  ColumnConstants column[QB];
  float h_max[2][SEARCH + KEEP], c_bad[2][SEARCH + KEEP];
};

// An entry in LDS: its elements in order, but twelve elements in four quarters of four halfs (the last one zero).
template <int VP> constexpr int loop_entry_halfs() { return VP <= 4 ? 4 : VP <= 8 ? 8 : 16; }
template <int VP>
__device__ __forceinline__ constexpr int entry_place(int el) { return VP == 12 ? el / 3 * 4 + el % 3 : el; }

// E of a block and of the one before: [row p * VP + j][column], rows in whole operands, columns in whole steps of the update (FAR) and four more
// (sixteen-byte reads of neighbouring rows then take neighbouring banks).
constexpr int FAR = 8;
constexpr int positions_most(int vp) { return 32 / vp < PMAX ? 32 / vp : PMAX; }
constexpr int e_rows(int vp) { return (positions_most(vp) * vp + 3) / 4 * 4; }
__host__ __device__ constexpr int e_pitch(int block) { return (block + FAR - 1) / FAR * FAR + 4; }

template <int VP>
size_t loop_lds_bytes(int k, int k_res, int block) {
  return (size_t)(k + k_res) * loop_entry_halfs<VP>() * 2 + (size_t)2 * e_rows(VP) * e_pitch(block) * 4 + sizeof(LoopExchange) + 64;
}

// Centroid whose slots a lane holds in tile `tile` of group `g`, and which eight of them: row m of operand A is lane m of every
// sixteen, slots 8 q .. 8 q + 7 the q-th sixteen lanes.  Sixteen neighbours to a row's place, the waves side by side.
template <int VP>
__device__ __forceinline__ int operand_entry(int g, int tile, int lane, int wave) {
  constexpr int SW = entries_wide(VP);
  return ((g * group_tiles(VP) + tile) * SW + (lane >> 4) * SW / 4) * (SEARCH * 16) + wave * 16 + (lane & 15);
}
template <int VP>
__device__ __forceinline__ int operand_part(int lane) { return (lane >> 4) & (4 / entries_wide(VP) - 1); }

// What a slot of an entry holds: an element, the first (-1) or second (-2) part of |c|^2 / 2, or nothing (-3).
template <int VP>
__device__ __forceinline__ constexpr int slot_content(int slot) {
  if (VP == 12) return slot % 4 < 3 ? slot / 4 * 3 + slot % 4 : slot == 3 ? -1 : slot == 7 ? -2 : -3;
  return slot < VP ? slot : slot == VP ? -1 : slot == VP + 1 ? -2 : -3;
}

// |c|^2 / 2 of an entry's first `len` elements.
template <int VP>
__device__ __forceinline__ float half_norm(const __half *src, int len) {
  float q = 0.0f;
#pragma unroll
  for (int j = 0; j < VP; ++j) {
    const float c = j < len ? __half2float(src[j < len ? j : 0]) : 0.0f;
    q = __fmaf_rn(c, c, q);
  }
  return 0.5f * q;
}

// A table as matrix-core operands (groups of 64 centroids, rows past the table repeating its last entry).
template <int VP, int G>
__device__ __forceinline__ void load_operands(const __half *cb, int k, int v, int len, int f, int lane, int wave, half8v (&A)[G][group_tiles(VP)]) {
#pragma unroll
  for (int g = 0; g < G; ++g)
#pragma unroll
    for (int tile = 0; tile < group_tiles(VP); ++tile) {
      const __half *src = cb + (long long)min(operand_entry<VP>(g, tile, lane, wave), k - 1) * v;
      const float x = ldexpf(half_norm<VP>(src, len), f);
      const _Float16 n1 = (_Float16)x, n2 = (_Float16)(x - (float)n1);
      const int part = operand_part<VP>(lane);
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        _Float16 y = (_Float16)0.0f;
#pragma unroll
        for (int p = 0; p < 4 / entries_wide(VP); ++p) {
          const int what = slot_content<VP>(p * 8 + i);
          if (part == p) y = what >= 0 ? (what < len ? __builtin_bit_cast(_Float16, src[what < len ? what : 0]) : (_Float16)0.0f)
                                       : what == -1 ? n1 : what == -2 ? n2 : (_Float16)0.0f;
        }
        A[g][tile][i] = y;
      }
      asm volatile("" : "+v"(A[g][tile]) :: "memory");       // (one after the other: their loads would take all registers at once)
    }
}

// One table.  |c|^2 / 2 times 2^f stays below 2^15.  How far below the largest score of a wave (its lowest bits a tag) a nearest
// centroid's may lie, in scaled scores, with t scaled by 2^e to below 2^14:
// - what t lost to binary16, |low| |c| for each of two scores;
// - an instruction's v + 2 terms, each cut at 2^-24 of the sum of the terms' magnitudes, |t| |c| + |c|^2 / 2 (vq_assign.hip);
// - the definition's own roundings, (v + 2) 2^-24 of (|t| + |c|)^2, twice;
// - |c|^2 / 2 itself: its sum, and two binary16 parts, 2^-21 of the largest;
// - the tags: 2^-17 of either score.
// Together low_c |low| + eps0 + eps_up 2^e + eps_down 2^-e; `bad` where entries are not finite or huge: every distance decides.
struct LoopTable { int f, bad; float low_c, eps0, eps_up, eps_down; };

template <int VP>
__device__ __forceinline__ LoopTable loop_table(const float *h_max, const float *bad) {
  LoopTable t;
  float m = 0.0f, b = 0.0f;
  for (int w = 0; w < SEARCH + KEEP; ++w) { m = fmaxf(m, h_max[w]); b += bad[w]; }
  t.f = m > 0.0f ? min(14, max(-14, 15 - __builtin_amdgcn_frexp_expf(m))) : 14;
  // (operands below 2^-14 count as that)
  const float c = __builtin_amdgcn_sqrtf(2.0f * m) * 1.001f + 0x1p-12f, T = __builtin_amdgcn_sqrtf((float)VP) * 1.001f * 0x1p14f;
  constexpr float K = (VP + 3) * 0x1p-23f, TAGS = 1.01f * 0x1p-16f;
  t.low_c = 2.01f * c;
  t.eps0 = T * c * (3.0f * K + TAGS);
  t.eps_up = m * (4.0f * K + 0x1p-20f + TAGS) + K * c * c + 0x1p-37f;
  t.eps_down = K * T * T;
  // (the same in every lane: kept in scalar registers)
  auto scalar = [](float y) { return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(y))); };
  t.f = __builtin_amdgcn_readfirstlane(t.f);
  t.bad = __builtin_amdgcn_readfirstlane(b != 0.0f ? 1 : 0);
  t.low_c = scalar(t.low_c); t.eps0 = scalar(t.eps0); t.eps_up = scalar(t.eps_up); t.eps_down = scalar(t.eps_down);
  return t;
}

#define VQ_QUAD(CTRL, X) __builtin_amdgcn_update_dpp(0, (int)(X), CTRL, 0xF, 0xF, true)
template <int J>
__device__ __forceinline__ unsigned quad_lane(unsigned x) { return (unsigned)VQ_QUAD(J * 0x55, x); }     // lane J of the quad
// (maximum rather than fmaxf: no instruction to quiet its operands)
__device__ __forceinline__ float maximum(float a, float b) { return __builtin_elementwise_maximum(a, b); }
__device__ __forceinline__ float quad_max(float x) {
  x = maximum(x, __int_as_float(VQ_QUAD(0xB1, __float_as_int(x))));
  return maximum(x, __int_as_float(VQ_QUAD(0x4E, __float_as_int(x))));
}
__device__ __forceinline__ unsigned quad_max(unsigned x) {
  x = max(x, (unsigned)VQ_QUAD(0xB1, x));
  return max(x, (unsigned)VQ_QUAD(0x4E, x));
}
__device__ __forceinline__ float quad_sum(float x) {
  x += __int_as_float(VQ_QUAD(0xB1, __float_as_int(x)));
  return x + __int_as_float(VQ_QUAD(0x4E, __float_as_int(x)));
}
__device__ __forceinline__ unsigned quad_min(unsigned x) {
  x = min(x, (unsigned)VQ_QUAD(0xB1, x));
  return min(x, (unsigned)VQ_QUAD(0x4E, x));
}
#undef VQ_QUAD
// Largest of the four rows of lanes, place by place, in all of them.
__device__ __forceinline__ float rows_max(float x) {
  const auto a = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  x = maximum(__uint_as_float(a[0]), __uint_as_float(a[1]));
  const auto b = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return maximum(__uint_as_float(b[0]), __uint_as_float(b[1]));
}

// What a lane's place in operand B takes: masks of the part of its eight slots.
struct LaneMasks { unsigned part[3]; };
template <int VP>
__device__ __forceinline__ LaneMasks lane_masks(int lane) {
  constexpr int SW = entries_wide(VP);
  const bool mine = (lane >> 4) * SW / 4 == (lane & (SW - 1));
  LaneMasks m;
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    m.part[i] = mine && operand_part<VP>(lane) == i ? ~0u : 0u;
    asm volatile("" : "+v"(m.part[i]));                      // (an operand of an and, not a choice)
  }
  return m;
}

// The vectors as operand B, and what their search's bounds need.
template <int VP>
struct Posted {
  half8v B;
  float t[quarter(VP)], low[quarter(VP)];                    // (low: what the rounding to binary16 cut off)
  int e;                                                     // scaled by 2^e
  bool brute;                                                // not within binary16 so, or not a number
};

template <int VP>
__device__ __forceinline__ Posted<VP> post_vectors(const float (&t)[quarter(VP)], const LoopTable &tb, const LaneMasks &in, int lane) {
  constexpr int EPL = quarter(VP);
  Posted<VP> p;
  const int j = lane & 3;
  unsigned most = 0u;
#pragma unroll
  for (int r = 0; r < EPL; ++r) { p.t[r] = t[r]; most = max(most, __float_as_uint(t[r]) & 0x7FFFFFFFu); }
  const int e = 140 - (int)(quad_max(most) >> 23);
  p.brute = e < tb.f - 14 || tb.bad != 0;
  p.e = min(tb.f + 15, max(tb.f - 14, e));
  _Float16 hi[4] = {(_Float16)0.0f, (_Float16)0.0f, (_Float16)0.0f, (_Float16)0.0f};
#pragma unroll
  for (int r = 0; r < EPL; ++r) {
    const float scaled = ldexpf(t[r], p.e);
    hi[r] = (_Float16)scaled;
    p.low[r] = scaled - (float)hi[r];
  }
  // (the |c|^2 slots' factor: -2^(e - f))
  const unsigned one = ((unsigned)p.e << 10) + (0x8000u + (unsigned)(15 - tb.f) * 1024u);
  auto pack = [](_Float16 a, _Float16 b) {
    const half2v y = {a, b};
    return __builtin_bit_cast(unsigned, y);
  };
  const unsigned ones = pack(__builtin_bit_cast(_Float16, (unsigned short)one), __builtin_bit_cast(_Float16, (unsigned short)one));
  unsigned B[4];
  if constexpr (EPL == 2) {
    unsigned d = pack(hi[0], hi[1]);
    if constexpr (VP < 8) d = j == VP / 2 ? ones : d;
    B[0] = quad_lane<0>(d) & in.part[0]; B[1] = quad_lane<1>(d) & in.part[0];
    B[2] = quad_lane<2>(d) & in.part[0]; B[3] = quad_lane<3>(d) & in.part[0];
    if constexpr (VP == 8) B[0] |= ones & in.part[1];
  } else {
    const unsigned d0 = pack(hi[0], hi[1]);
    unsigned d1 = pack(hi[2], hi[3]);
    if constexpr (EPL == 3) d1 |= j < 2 ? ones & 0xFFFF0000u : 0u;
    B[0] = (quad_lane<0>(d0) & in.part[0]) | (quad_lane<2>(d0) & in.part[1]);
    B[1] = (quad_lane<0>(d1) & in.part[0]) | (quad_lane<2>(d1) & in.part[1]);
    B[2] = (quad_lane<1>(d0) & in.part[0]) | (quad_lane<3>(d0) & in.part[1]);
    B[3] = (quad_lane<1>(d1) & in.part[0]) | (quad_lane<3>(d1) & in.part[1]);
    if constexpr (VP == 16) B[0] |= ones & in.part[2];
  }
  const uint4v b = {B[0], B[1], B[2], B[3]};
  p.B = __builtin_bit_cast(half8v, b);
  return p;
}

// One padded table entry (EH halfs) from LDS, in whole 16-byte reads (8 bytes for the smallest entries; the compiler would narrow
// and split a read whose tail is unused).
template <int EH>
__device__ __forceinline__ void read_entry(unsigned (&dst)[EH / 2], const unsigned char *entry) {
  if constexpr (EH == 4) {
    const uint2v a = *reinterpret_cast<const uint2v *>(entry);
    dst[0] = a.x; dst[1] = a.y;
  } else {
#pragma unroll
    for (int q = 0; q < EH / 8; ++q) {
      const uint4v a = *reinterpret_cast<const uint4v *>(entry + 16 * q);
      asm volatile("" :: "v"(a.w));
      dst[4 * q] = a.x; dst[4 * q + 1] = a.y; dst[4 * q + 2] = a.z; dst[4 * q + 3] = a.w;
    }
  }
}

// Distance of a lane's vector to entry i, as defined; smallest first, then smallest index, of the four in a quad.
template <int VP>
__device__ __forceinline__ void quad_nearest(const unsigned char *entries, unsigned i, const float (&t)[VP], unsigned &d, unsigned &arg) {
  constexpr int EH = loop_entry_halfs<VP>();
  unsigned c[EH / 2];
  read_entry<EH>(c, entries + (size_t)i * (EH * 2u));
  float s = 0.0f;
#pragma unroll
  for (int el = 0; el < VP; ++el) {
    // t - c in one operation: the product c * -1 is exact
    const float diff = __fmaf_rn(half_of(c[entry_place<VP>(el) >> 1], entry_place<VP>(el) & 1), -1.0f, t[el]);
    s = __fmaf_rn(diff, diff, s);
  }
  const unsigned bits = __float_as_uint(s);
  d = quad_min(bits);
  arg = quad_min(bits == d ? i : 0xFFFFFFFFu);
}

// One search of all vectors over a wave's share of a table of `count` entries.
template <int VP, int G>
__device__ __forceinline__ void search_table(unsigned long long *nearest, const half8v (&A)[G][group_tiles(VP)], const unsigned char *entries, int count,
                                             const Posted<VP> &p, const LoopTable &tb, int lane, int wave) {
  constexpr int SW = entries_wide(VP), TILES = group_tiles(VP), EPL = quarter(VP), N = G * TILES, LEAD = N < 4 ? N : 4;
  if (wave * 16 >= count) return;
  const int place = lane & (SW - 1);
  // the instructions run LEAD groups ahead of the comparisons
  float4v acc[LEAD];
  auto scores = [&](int g) { return __builtin_amdgcn_mfma_f32_16x16x32_f16(A[g / TILES][g % TILES], p.B, float4v{0.0f, 0.0f, 0.0f, 0.0f}, 0, 0, 0); };
  auto best_of = [&](const float4v &a) { return maximum(maximum(maximum(a[0], a[1]), a[2]), a[3]); };
#pragma unroll
  for (int g = 0; g < LEAD; ++g) acc[g] = scores(g);
  __builtin_amdgcn_sched_barrier(0);
  float t[VP], low = 0.0f;
#pragma unroll
  for (int el = 0; el < VP; ++el) {
    const unsigned y = __float_as_uint(p.t[el % EPL]);
    t[el] = __uint_as_float(el / EPL == 0 ? quad_lane<0>(y) : el / EPL == 1 ? quad_lane<1>(y) : el / EPL == 2 ? quad_lane<2>(y) : quad_lane<3>(y));
  }
#pragma unroll
  for (int r = 0; r < EPL; ++r) low = __fmaf_rn(p.low[r], p.low[r], low);
  const float eps = __fmaf_rn(tb.low_c, __builtin_amdgcn_sqrtf(quad_sum(low)),
                              __fmaf_rn(tb.eps_up, ldexpf(1.0f, p.e), __fmaf_rn(tb.eps_down, ldexpf(1.0f, -p.e), tb.eps0)));
  float m1 = 0.0f, m2 = -__builtin_inff();
#pragma unroll
  for (int g = 0; g < N; ++g) {
    const float tagged = __uint_as_float((__float_as_uint(best_of(acc[g % LEAD])) & ~TAG) | (unsigned)(g * SW));
    if (g + LEAD < N) acc[g % LEAD] = scores(g + LEAD);
    if (g > 0) m2 = __builtin_amdgcn_fmed3f(m1, m2, tagged);
    m1 = g > 0 ? maximum(m1, tagged) : tagged;
    __builtin_amdgcn_sched_barrier(0);
  }
  if constexpr (SW > 1) m1 = __uint_as_float(__float_as_uint(m1) | (unsigned)place);
  const float best = quad_max(m1);
  auto index = [&](unsigned at) {                            // of the quad's four, at group * SW + place
    return min(at * (SEARCH * 16) + (wave * 16 + (lane >> 4) * 4 + (lane & 3)), (unsigned)count - 1u);
  };
  const unsigned tag = __float_as_uint(best);
  unsigned d, i;
  quad_nearest<VP>(entries, index(tag & TAG), t, d, i);
  const float bar = rows_max(best) - eps;
  const bool first = (lane & 3) == 0;
  auto file = [&] {
    __hip_atomic_fetch_min(nearest, (unsigned long long)d << 32 | i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  };
  if (first & !(best < bar)) file();
  bool more = p.brute | ((__float_as_uint(m1) != tag) & !(m1 < bar));
  if constexpr (N > 1) more |= !(m2 < bar);
  if (__builtin_expect(__builtin_amdgcn_ballot_w64(more) != 0ull, 0)) {
    // Groups of which the four distances are wanted; the scores once more, since their registers are long in other use.
    unsigned ask = 0u;
#pragma unroll
    for (int g = 0; g < N; ++g) {
      ask |= ((lane & 3) < SW) & (p.brute | !(best_of(scores(g)) < bar)) ? 1u << g : 0u;
      if (g % 4 == 3) __builtin_amdgcn_sched_barrier(0);
    }
    while (__any(ask != 0u)) {
      const unsigned next = quad_min(ask ? (unsigned)(lane & 3) << 8 | (unsigned)__builtin_ctz(ask) : 0xFFFFu);    // the quad's first: place and group
      const unsigned from = next >> 8, g = next & 0xFFu;
      const bool some = next != 0xFFFFu;
      if (some && from == (unsigned)(lane & 3)) ask &= ask - 1u;
      quad_nearest<VP>(entries, some ? index(g * SW + from) : 0u, t, d, i);
      if (some && first) file();
    }
  }
}

// The same for vectors of one or two elements: every distance, the first elements of an entry being the first slots of the operand that a
// lane holds.  In so few dimensions many entries lie within the bounds of the largest score, and the search above takes them one after
// the other.  600 columns, a last position of one row: v = 6, k = 4096 1727 -> 533 us, k = 1024 832 -> 399; v = 12, k = 4096 3080 -> 884; of two rows:
// 825 -> 533, 438 -> 400, 1497 -> 885 (whole positions alone: 502, 388, 847).  Whole positions of v = 1, k = 4096, four a workgroup 2002 ->
// 1133; of v = 2, two 933 -> 691, but four 1013 -> 1116: a vector after the other, where the search above takes four at once.
template <int VP, int G>
__device__ __forceinline__ void search_narrow(unsigned long long *nearest, const half8v (&A)[G][group_tiles(VP)], int count, const float (&t)[quarter(VP)], int P,
                                              int lane, int wave) {
  constexpr int SW = entries_wide(VP), TILES = group_tiles(VP);
  if (wave * 16 >= count) return;
  const bool holds = operand_part<VP>(lane) == 0;
  for (int n = 0; n < P; ++n) {
    const float t0 = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(t[0]), 4 * n));
    const float t1 = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(t[1]), 4 * n));
    unsigned d = ~0u, at = 0u;
#pragma unroll
    for (int i = 0; i < G * TILES; ++i) {
      const half8v &c = A[i / TILES][i % TILES];
      const float d0 = __fmaf_rn((float)c[0], -1.0f, t0), d1 = __fmaf_rn((float)c[1], -1.0f, t1);
      const unsigned bits = __float_as_uint(__fmaf_rn(d1, d1, __fmaf_rn(d0, d0, 0.0f)));
      at = bits < d ? (unsigned)i : at;
      d = min(d, bits);
    }
    const unsigned i = min((at * SW + (lane >> 4) * SW / 4) * (SEARCH * 16) + wave * 16 + (lane & 15), (unsigned)count - 1u);
    const unsigned least = wave_min_u32(holds ? d : ~0u), first = wave_min_u32(holds && d == least ? i : ~0u);
    if (lane == 0) __hip_atomic_fetch_min(nearest + n, (unsigned long long)least << 32 | first, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  }
}

// SHORT: with positions of one or two rows among them (a kernel of its own, as the second search costs the first one 4 %).
template <int VP, int G, int GR, bool SHORT>
__global__ __launch_bounds__(LOOP_THREADS) void qcol_loop_kernel(LoopArgs a) {
  constexpr int EH = loop_entry_halfs<VP>(), EPL = quarter(VP), POS = positions_most(VP), E_ROWS = e_rows(VP);
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  __half *entries = reinterpret_cast<__half *>(smem);                                          // [k + k_res][EH]
  const int pitch_e = e_pitch(a.block);
  float *E = reinterpret_cast<float *>(smem + (((size_t)(a.k + a.k_res) * EH * 2 + 15) & ~(size_t)15));   // [2][E_ROWS][pitch_e]: row p * VP + j
  LoopExchange &x = *reinterpret_cast<LoopExchange *>(E + 2 * E_ROWS * pitch_e);
  constexpr int threads = LOOP_THREADS;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const bool searching = wave < SEARCH;
  const int pos0 = blockIdx.x * a.P;
  const bool cut = pos0 >= a.whole;                                        // the workgroup of the cut-off position
  const int P = cut ? 1 : min(a.P, a.whole - pos0);
  const int first = cut ? a.whole : pos0;                                  // its first position
  const int len = cut ? a.rows - a.whole * a.v : a.v;                      // rows of a position: what its vectors are compared over
  const bool narrow = len == 1 || (len == 2 && P <= 2);                    // (see search_narrow)

  // tables: entries in LDS (elements past `len` as zeros), operands in registers
  for (int e = tid; e < (a.k + a.k_res) * EH; e += threads) {
    const int i = e / EH, slot = e % EH;
    const int j = VP == 12 ? (slot % 4 < 3 ? slot / 4 * 3 + slot % 4 : VP) : slot;
    const __half *src = i < a.k ? a.cb + (long long)i * a.v : a.cb_res + (long long)(i - a.k) * a.v;
    entries[e] = j < len ? src[j] : __float2half_rn(0.0f);
  }
  for (int e = tid; e < 2 * E_ROWS * pitch_e; e += threads) E[e] = 0.0f;
  if (tid < 8 * PMAX) (&x.nearest[0][0][0])[tid] = ~0ull;
  for (int e = tid; e < ROWS * 5; e += threads) (&x.next_w[0][0])[e] = 0.0f;                   // (and e and first_t behind them)
  LoopTable main_table, res_table;
  {
    auto post_norms = [&](int which, const __half *cb, int k) {
      float m = 0.0f;
      bool fine = true;
      for (int i = tid; i < k; i += threads) {
        const float h = half_norm<VP>(cb + (long long)i * a.v, len);
        m = fmaxf(m, h);
        fine = fine && h < 0x1p28f;                          // (false for entries that are not numbers)
      }
      for (int sft = 32; sft > 0; sft >>= 1) m = fmaxf(m, __shfl_xor(m, sft, 64));
      fine = __all(fine);
      if (lane == 0) { x.h_max[which][wave] = m; x.c_bad[which][wave] = fine ? 0.0f : 1.0f; }
    };
    post_norms(0, a.cb, a.k);
    if constexpr (GR) post_norms(1, a.cb_res, a.k_res);
    __syncthreads();
  }

  // Barriers of a block, the same ones for searching and keeping waves: its first column's weights and constants are there; one a column (two
  // with a residual table); the last column's errors are there.
  if (searching) {
    const __half *entries_res = entries + (size_t)a.k * EH;
    half8v A[G][group_tiles(VP)], AR[GR ? GR : 1][group_tiles(VP)];
    main_table = loop_table<VP>(x.h_max[0], x.c_bad[0]);
    load_operands<VP, G>(a.cb, a.k, a.v, len, main_table.f, lane, wave, A);
    if constexpr (GR) {
      res_table = loop_table<VP>(x.h_max[1], x.c_bad[1]);
      load_operands<VP, GR>(a.cb_res, a.k_res, a.v, len, res_table.f, lane, wave, AR);
    }
    // (lanes of vectors past the last repeat the first)
    const int n = ((lane >> 2) & 3) < P ? (lane >> 2) & 3 : 0, j = lane & 3;
    const int own = EPL * j < VP ? n * VP + EPL * j : 32;     // its elements' rows (past a vector: zeros)
    const LaneMasks in = lane_masks<VP>(lane);
    // an entry's elements, in the lanes that hold them of the vector that took it
    auto elements = [&](const __half *table, unsigned i, float (&q)[EPL]) {
      unsigned at = i * EH + (EPL == 2 ? 2 * j : 4 * j);
      if constexpr (VP == 4) at = i * EH + 2 * (j & 1);
      const uint2v y = EPL == 2 ? uint2v{*reinterpret_cast<const unsigned *>(table + at), 0u} : *reinterpret_cast<const uint2v *>(table + at);
#pragma unroll
      for (int r = 0; r < EPL; ++r) {
        q[r] = half_of(r < 2 ? y.x : y.y, r & 1);
        if constexpr (VP == 4) q[r] = j < 2 ? q[r] : 0.0f;
      }
    };
    // What a finished column leaves in memory: T from one wave, the quantized weights from another, the indices of either table from the other two.
    // (These waves never wait for memory.)  One row of lanes does it, for the vectors that are there; the offsets of all others are past the
    // end: a store that does nothing takes less than a branch.
    const bool files = lane < 4 * P;
    const bool files_t = wave == 1 && a.T, files_q = wave == 2;
    const int ld_mine = files_t ? (int)a.ldt : (int)a.ldw;
    const auto rows_mine = __builtin_amdgcn_make_buffer_rsrc((files_t ? a.T : a.W) + (long long)first * a.v * ld_mine, 0, P * a.v * ld_mine * 4, 0x00020000);
    const unsigned any_t = files_t ? ~0u : 0u;
    unsigned to[EPL];
#pragma unroll
    for (int r = 0; r < EPL; ++r) to[r] = (files_t || files_q) && files && EPL * j + r < len ? (unsigned)((n * a.v + EPL * j + r) * ld_mine) * 4u : 0x7FFFFFFFu;
    // indices, a stream to a lane: whole dwords of them (no other workgroup writes these streams, which were cleared beforehand)
    struct Stream { unsigned *to, bits; int filled; };
    const bool streams = files && j == 0;
    auto stream = [&](unsigned *idx, long long dwords) { return Stream{idx + (long long)(first + n) * dwords, 0u, 0}; };
    auto append = [&](Stream &st, unsigned code, int bits) {
      st.bits |= code << st.filled;
      st.filled += bits;
      if (st.filled >= 32) {
        if (streams) *st.to = st.bits;
        ++st.to;
        st.filled -= 32;
        st.bits = st.filled ? code >> (bits - st.filled) : 0u;
      }
    };
    Stream main_stream = stream(a.idx, a.idx_dwords), res_stream = GR ? stream(a.idx_res, a.idx_res_dwords) : main_stream;
    for (int s = 0; s < a.cols; s += a.block) {
      const int nb = min(a.block, a.cols - s);
      float t[EPL], e_last[EPL];
      lds_barrier();
#pragma unroll
      for (int r = 0; r < EPL; ++r) { t[r] = x.first_t[own + r]; e_last[r] = 0.0f; }
      for (int nn = 0; nn < nb; ++nn) {
        Posted<VP> p = post_vectors<VP>(t, main_table, in, lane);
        bool odd = p.brute;
        // (a t - q below 2^-80 is t, as entries are multiples of 2^-24; from there on the quotient is no subnormal number either)
        unsigned least = ~0u;
#pragma unroll
        for (int r = 0; r < EPL; ++r) least = min(least, 2u * __float_as_uint(t[r]) - 1u);     // (but zero)
        odd |= least < 2u * __float_as_uint(0x1p-80f) - 1u;
        const ColumnConstants at = x.column[nn];
        odd |= at.inverse == 0.0f;
        if (SHORT && narrow) search_narrow<VP, G>(x.nearest[0][nn & 3], A, a.k, t, P, lane, wave);
        else search_table<VP, G>(&x.nearest[0][nn & 3][n], A, smem, a.k, p, main_table, lane, wave);
        lds_barrier();
        float next[EPL], q[EPL], e[EPL];
        const unsigned code = (unsigned)x.nearest[0][nn & 3][n];
#pragma unroll
        for (int r = 0; r < EPL; ++r) next[r] = x.next_w[nn & 1][own + r];
        unsigned code_res = 0u;
        elements(entries, code, q);
        if constexpr (GR) {
          float rest[EPL], more[EPL];
#pragma unroll
          for (int r = 0; r < EPL; ++r) rest[r] = __fsub_rn(t[r], q[r]);
          p = post_vectors<VP>(rest, res_table, in, lane);
          odd |= p.brute;
          if (SHORT && narrow) search_narrow<VP, GR>(x.nearest[1][nn & 3], AR, a.k_res, rest, P, lane, wave);
          else search_table<VP, GR>(&x.nearest[1][nn & 3][n], AR, smem + (size_t)a.k * EH * 2, a.k_res, p, res_table, lane, wave);
          lds_barrier();
          code_res = (unsigned)x.nearest[1][nn & 3][n];
          elements(entries_res, code_res, more);
#pragma unroll
          for (int r = 0; r < EPL; ++r) {
            // what inference restores: the binary32 sum of the two centroids, rounded to binary16 (Sec. 3.2.2)
            float sum = __fadd_rn(q[r], more[r]);
            asm volatile("" : "+v"(sum));
            q[r] = __half2float(__float2half_rn(sum));
          }
        }
        // e = (t - q) / diag.  With the correctly rounded reciprocal, one correction of the rounded product gives the correctly rounded
        // quotient (Markstein, IBM J. Res. Dev. 34, 1990), where nothing overflows and the remainder, some 2^-47 of t - q, is a
        // binary32 number: not for numbers out of the ordinary.
#pragma unroll
        for (int r = 0; r < EPL; ++r) {
          const float diff = __fsub_rn(t[r], q[r]), about = __fmul_rn(diff, at.inverse);
          e[r] = __fmaf_rn(-__fmaf_rn(about, at.diag, -diff), at.inverse, about);
        }
        if (__builtin_expect(__builtin_amdgcn_ballot_w64(odd) != 0ull, 0)) {
#pragma unroll
          for (int r = 0; r < EPL; ++r) e[r] = __fdiv_rn(__fsub_rn(t[r], q[r]), at.diag);
        }
#pragma unroll
        for (int r = 0; r < EPL; ++r) {
          x.e[nn & 1][own + r] = e[r];                       // (every wave writes the same)
          const unsigned y = (__float_as_uint(t[r]) & any_t) | (__float_as_uint(q[r]) & ~any_t);
          __builtin_amdgcn_raw_buffer_store_b32((int)y, rows_mine, to[r], (s + nn) * 4, 0);
        }
        if (wave == 3) append(main_stream, code, a.bits);
        if constexpr (GR) { if (wave == 0) append(res_stream, code_res, a.bits_res); }
#pragma unroll
        for (int r = 0; r < EPL; ++r) {
          t[r] = __fmaf_rn(-e[r], at.beside, __fmaf_rn(-e_last[r], at.beside2, next[r]));
          e_last[r] = e[r];
        }
      }
      lds_barrier();
    }
    if (wave == 3 && streams && main_stream.filled) *main_stream.to = main_stream.bits;
    if constexpr (GR) { if (wave == 0 && streams && res_stream.filled) *res_stream.to = res_stream.bits; }
    return;
  }

  // Keeping waves: 64 columns each, two waves those of the running block, two those of the next one, and in the next block the other way round.
  // A column of the block is one row of H^-1 for them: row 4 b + i of its errors in lane 4 b + i of operand A, of which an instruction
  // (4x4x1, 16 blocks) takes block b; the row's columns in operand B, one to a lane; the lane gets back rows 4 b .. 4 b + 3 of its column.
  auto keep = [&](auto positions) {
    constexpr int NP = decltype(positions)::value, RG = (NP * VP + 3) / 4;
    const int kw = wave - SEARCH;
    const int pitch_h = (int)a.ldh * 4, pitch_w = (int)a.ldw * 4;
    const auto rows_of_W = __builtin_amdgcn_make_buffer_rsrc(a.W + (long long)first * a.v * a.ldw, 0, ((NP - 1) * a.v + len) * pitch_w, 0x00020000);
    auto row_of_W = [&](int p, int el) { return (p * a.v + min(el, len - 1)) * pitch_w; };     // (past a position's rows: its last one)
    // W[:, column] + w where a position has the row, else 0
    float4v w[RG];
    auto add_weights = [&](int col) {
      float y[RG * 4];
#pragma unroll
      for (int r = 0; r < NP * VP; ++r) y[r] = __int_as_float(__builtin_amdgcn_raw_buffer_load_b32(rows_of_W, min(col, a.cols - 1) * 4, row_of_W(r / VP, r % VP), 0));
#pragma unroll
      for (int r = 0; r < RG * 4; ++r) w[r / 4][r % 4] = r < NP * VP && r % VP < len ? y[r < NP * VP ? r : 0] + w[r / 4][r % 4] : 0.0f;
    };
    auto clear = [&] {
#pragma unroll
      for (int g = 0; g < RG; ++g) w[g] = float4v{0.0f, 0.0f, 0.0f, 0.0f};
    };
    auto post = [&](float *to) {
#pragma unroll
      for (int g = 0; g < RG; ++g) *reinterpret_cast<float4v *>(to + 4 * g) = w[g];
    };
    const int e_row = min(lane & 31, NP * VP - 1);           // operand A
    clear();
    if (kw < 2) add_weights(kw * 64 + lane);
    int parity = 0;                                          // of the block: which half of E, which waves have its columns
    for (int s = 0; s < a.cols; s += a.block, parity ^= 1) {
      const int s_end = min(s + a.block, a.cols), nb = s_end - s;
      const bool running = kw / 2 == parity;
      const int mine = (running ? s : s_end) + kw % 2 * 64 + lane;          // column
      float *E_now = E + parity * E_ROWS * pitch_e + e_row * pitch_e;
      auto hinv = [&](int row, int col) -> float { return row >= 0 && col < nb ? a.Hinv[(long long)(s + row) * a.ldh + s + col] : 0.0f; };
      const int c = tid - SEARCH * 64;
      if (c < nb) {
        ColumnConstants at;
        at.diag = hinv(c, c);
        const float size = fabsf(at.diag);
        at.inverse = size > 0x1p-40f && size < 0x1p40f ? __fdiv_rn(1.0f, at.diag) : 0.0f;
        at.beside = hinv(c, c + 1);
        at.beside2 = hinv(c - 1, c + 1);
        x.column[c] = at;
      }
      if (mine == s) post(x.first_t);
      // The update of the columns beyond this block by the block before: W[:, later] -= E * Hinv[block before, later], 128 columns a wave at a
      // time, FAR rows of H^-1 a column of the running block: row 4 b + i of E in lane 4 b + i of operand A, of which an instruction takes block b;
      // a row of H^-1 in operand B, two neighbouring columns to a lane; the lane gets back rows 4 b .. 4 b + 3 of either.
      const float *E_before = E + (parity ^ 1) * E_ROWS * pitch_e + min(lane & 31, E_ROWS - 1) * pitch_e;
      const int far_groups = s > 0 ? (a.cols - s_end + 127) / 128 : 0;
      const auto rows_before = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(a.Hinv + (long long)max(s - a.block, 0) * a.ldh), 0,
                                                                 min(a.block, a.cols) * pitch_h, 0x00020000);
      const int far_pitch = far_groups ? pitch_h : 0;        // (where there is nothing to do, the loads repeat the first row)
      int fg = kw, fk = 0;
      float4v acc[2][RG];
      float2v hv[FAR];
      float4v ev[FAR / 4];
      // (the sums of a pair that ends past the matrix are those of the last pair)
      auto far_offset = [&] { return min(s_end + fg * 128 + 2 * lane, max(a.cols - 2, 0)) * 4; };
      auto far_loads = [&] {
        const int off = far_offset();
        int row = fk * far_pitch;
#pragma unroll
        for (int u = 0; u < FAR; ++u) {
          hv[u] = __builtin_bit_cast(float2v, __builtin_amdgcn_raw_buffer_load_b64(rows_before, off, row, 0));
          row += far_pitch;
        }
#pragma unroll
        for (int u = 0; u < FAR / 4; ++u) ev[u] = *reinterpret_cast<const float4v *>(E_before + fk + 4 * u);
      };
      auto far_clear = [&] {
#pragma unroll
        for (int g = 0; g < RG; ++g) acc[0][g] = acc[1][g] = float4v{0.0f, 0.0f, 0.0f, 0.0f};
      };
      auto far_step = [&] {
#pragma unroll
        for (int u = 0; u < FAR; ++u)
#pragma unroll
          for (int half = 0; half < 2; ++half) {
#define VQ_ROWS(B) if constexpr (B < RG) acc[half][B < RG ? B : 0] = __builtin_amdgcn_mfma_f32_4x4x1f32(ev[u / 4][u % 4], hv[u][half], acc[half][B < RG ? B : 0], 4, B, 0);
            VQ_ROWS(0) VQ_ROWS(1) VQ_ROWS(2) VQ_ROWS(3) VQ_ROWS(4) VQ_ROWS(5) VQ_ROWS(6) VQ_ROWS(7)
#undef VQ_ROWS
          }
        fk += FAR;
        if (fk < a.block) return;
        const int at = s_end + fg * 128 + 2 * lane;
        if (at < a.cols) {
          // (a column has one owner, as the groups are other waves' or later turns: of the last pair moved back, which begins at another lane's column,
          // the second column alone is stored, and the first is loaded and dropped.  Branches of their own for pairs and the last column, loads and
          // stores, 1 % slower: 4096 x 4096, v = 6, k = 4096 4108 against 4027 us)
          const int off = far_offset(), to = at < a.cols - 1 ? off : 0x7FFFFFFF;
          auto each_row = [&](auto row) {
            if (len == VP) {
#pragma unroll
              for (int r = 0; r < NP * VP; ++r) row(r);
            } else {
#pragma unroll
              for (int r = 0; r < NP * VP; ++r)
                if (r % VP < len) row(r);
            }
          };
          float2v fw[NP * VP];
#pragma unroll
          for (int r = 0; r < NP * VP; ++r) fw[r] = __builtin_bit_cast(float2v, __builtin_amdgcn_raw_buffer_load_b64(rows_of_W, off, row_of_W(r / VP, r % VP), 0));
          each_row([&](int r) {
            fw[r] = float2v{fw[r].x - acc[0][r / 4][r % 4], fw[r].y - acc[1][r / 4][r % 4]};
            __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(uint2v, fw[r]), rows_of_W, to, row_of_W(r / VP, r % VP), 0);
          });
          if (at == a.cols - 1) each_row([&](int r) { __builtin_amdgcn_raw_buffer_store_b32(__float_as_int(fw[r].y), rows_of_W, at * 4, row_of_W(r / VP, r % VP), 0); });
        }
        far_clear();
        fg += KEEP; fk = 0;
      };
      far_clear();
      far_loads();                                           // (ahead of the barrier: columns 0 .. FAR - 1 of E, which has 2 FAR at least)
      constexpr int RING = 2;
      float row[RING];
      // (columns past the matrix are its last one, whose weights are not in use here)
      const auto rows_now = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(a.Hinv + (long long)s * a.ldh), 0, nb * pitch_h, 0x00020000);
      const int off_mine = min(mine, a.cols - 1) * 4;
      auto ring = [&](int nr) { return __int_as_float(__builtin_amdgcn_raw_buffer_load_b32(rows_now, off_mine, min(max(nr, 0), nb - 1) * pitch_h, 0)); };
      const float last2 = ring(nb - 2), last = ring(nb - 1);
#pragma unroll
      for (int u = 0; u < RING; ++u) row[u] = ring(u - 2);
      auto update = [&](int nn, float h) {                   // by column nn
        const float e = x.e[nn & 1][e_row];
#define VQ_ROWS(B) if constexpr (B < RG) w[B < RG ? B : 0] = __builtin_amdgcn_mfma_f32_4x4x1f32(-e, h, w[B < RG ? B : 0], 4, B, 0);
        VQ_ROWS(0) VQ_ROWS(1) VQ_ROWS(2) VQ_ROWS(3) VQ_ROWS(4) VQ_ROWS(5) VQ_ROWS(6) VQ_ROWS(7)
#undef VQ_ROWS
        if (kw == 0 && lane < NP * VP) E_now[nn] = e;
      };
      lds_barrier();
      for (int n0 = 0; n0 < nb; n0 += RING) {
#pragma unroll
        for (int u = 0; u < RING; ++u) {
          const int nn = n0 + u;
          if (nn >= nb) break;
          if (nn >= 2) update(nn - 2, row[u]);
          row[u] = ring(nn + RING - 2);
          if (mine == s + nn + 1) post(x.next_w[nn & 1]);
          if (kw == 3 && lane < 2 * PMAX) x.nearest[lane / PMAX][(nn + 1) & 3][lane % PMAX] = ~0ull;
          if constexpr (GR) lds_barrier();
          // (the loads are there in every column, so that the compiler can count what it need not wait for)
          if (fg < far_groups) far_step();
          far_loads();
          lds_barrier();
        }
      }
      while (fg < far_groups) { far_step(); far_loads(); }
      // (the next block's columns are other waves' work: their stores have to be out)
      __builtin_amdgcn_s_waitcnt(0);
      lds_barrier();
      if (kw == 3 && lane < 8 * PMAX) (&x.nearest[0][0][0])[lane] = ~0ull;       // (the next block's columns count from 0 again)
      if (nb > 1) update(nb - 2, last2);
      update(nb - 1, last);
      if (running) clear();
      else add_weights(mine);
    }
  };
  if (P == 1) keep(std::integral_constant<int, 1>{});
  if constexpr (POS >= 2) { if (P == 2) keep(std::integral_constant<int, 2>{}); }
  if constexpr (POS >= 3) { if (P == 3) keep(std::integral_constant<int, 3>{}); }
  if constexpr (POS >= 4) { if (P == 4) keep(std::integral_constant<int, 4>{}); }
}

template <int VP, int G, int GR, bool SHORT = false>
int launch_loop(LoopArgs a, hipStream_t st) {
  const int cut_rows = a.rows - a.whole * a.v, cut = cut_rows > 0;
  // (tables of up to 256 entries hold too few within the bounds: v = 6, a last position of one row 454 us, of more 351)
  if constexpr (!SHORT && (G > 1 || GR > 1))
    if ((cut && cut_rows <= 2) || a.v <= 2) return launch_loop<VP, G, GR, true>(a, st);
  auto kernel = qcol_loop_kernel<VP, G, GR, SHORT>;
  VQ_ALLOW_FULL_LDS(kernel);
  const unsigned grid = (unsigned)((a.whole + a.P - 1) / a.P + cut);
  hipLaunchKernelGGL(kernel, dim3(grid), dim3(LOOP_THREADS), loop_lds_bytes<VP>(a.k, a.k_res, a.block), st, a);
  return hipGetLastError() == hipSuccess ? VQ_OK : VQ_ERR_HIP;
}

// Groups of 64 centroids a search wave holds of each table: one up to 256 entries, four up to 1024, sixteen up to 4096.
template <int VP>
int launch_loop_vp(LoopArgs a, hipStream_t st) {
  // (whole steps of the later update, and two of them at least: its first one is read ahead of a block's first barrier, when the last two columns of
  // the block before may still be on their way into E)
  a.block = max(2 * FAR, (a.block + FAR - 1) / FAR * FAR);
  // (the block decides no more than where sums are split: where two large tables leave too little LDS for E, a smaller one)
  while (loop_lds_bytes<VP>(a.k, a.k_res, a.block) > 160 * 1024 && a.block > 64) a.block -= 16;
  if (loop_lds_bytes<VP>(a.k, a.k_res, a.block) > 160 * 1024 || a.ldh > (1 << 21) || a.ldw > (1 << 22) || a.ldt > (1 << 22)) return VQ_ERR_UNSUPPORTED;    // (a block of H^-1, the rows of a workgroup: 32-bit offsets)
  a.whole = a.rows / a.v;
  // positions per workgroup: as few as let every workgroup have a compute unit; E has 32 rows
  a.P = min(min(PMAX, 32 / VP), max(1, (a.whole + cu_count() - 2) / (cu_count() - 1)));
  const int big = max(a.k, a.k_res);
  if (a.k_res == 0) {
    if (big <= 256) return launch_loop<VP, 1, 0>(a, st);
    if (big <= 1024) return launch_loop<VP, 4, 0>(a, st);
    if constexpr (VP <= 14) { if (big <= 4096) return launch_loop<VP, 16, 0>(a, st); }
  } else {
    if (big <= 256) return launch_loop<VP, 1, 1>(a, st);
    if (big <= 1024) return launch_loop<VP, 4, 4>(a, st);
    // (longer vectors would not leave registers for the rest)
    if constexpr (VP <= 14) { if (big <= 4096 && a.k_res <= 1024) return launch_loop<VP, 16, 4>(a, st); }
    if constexpr (VP <= 6) { if (big <= 4096) return launch_loop<VP, 16, 16>(a, st); }
  }
  return VQ_ERR_UNSUPPORTED;
}

}  // namespace

int launch_quantize_loop(LoopArgs a, hipStream_t st) {
  const int v = a.v;
  return v <= 4 ? launch_loop_vp<4>(a, st) : v <= 6 ? launch_loop_vp<6>(a, st) : v <= 8 ? launch_loop_vp<8>(a, st)
       : v <= 12 ? launch_loop_vp<12>(a, st) : launch_loop_vp<16>(a, st);
}

}  // namespace vq
