// vq_quantize_columns in one launch: Algorithm 1 (Sec. 3.1) with its nearest-centroid searches on the matrix cores.
#include "vq_quantize.hpp"

namespace vq {
namespace {

// A workgroup owns up to four stack positions (P of them) and walks all columns of the matrix with them: nothing it needs comes
// from another workgroup.  The tables stay where they are for the whole launch: as operands of v_mfma_f32_16x16x32_f16 in
// registers, 64 centroids a wave and group (a wave of sixteen holds four such groups of a 4096-entry table), and as plain
// entries in LDS.
//
// One column.  The owner wave of a position posts the vector t in LDS: as binary32, and scaled by a power of two and split into
// two binary16 parts.  Every wave computes the scores t . c - |c|^2 / 2 of their centroids with all P vectors at once
// (vq_assign.hip has the same scheme and its error bounds).  Entries of up to six elements take 8 of the instruction's 32 k
// slots, |c|^2 / 2 in two parts behind them, so a row of operand A holds four centroids and each of the 16 columns of operand B
// one of four vectors at one of the four places, zeros elsewhere: 64 centroids with four vectors in two instructions, for
// the high and the low parts of t.  Entries of up to 14 elements take 16 slots, longer ones 32.  The largest score of each vector
// meets in LDS (an atomic maximum); after a barrier the lanes whose scores are within the rounding bounds of it -- as a rule one --
// compute the distances of those four centroids as defined, one each in a quad of lanes, and these meet in LDS too (an atomic
// minimum of distance bits and index).  From the index the owner forms E and the next column's t and posts that;
// while the others search it brings its tile of running weights up to date.  Three barriers a search.
//
// At the end of a block the workgroup writes its quantized columns and indices and applies E to its rows of the later columns:
// v_mfma_f32_32x32x2_f32 on 32 rows (P v of them in use) and 32 columns, the rows of H^-1 straight from memory.
//
// What bounds it: the chain of a column.  A wave on its own issues an instruction every five clocks, so what counts is how many
// stand on the path between one column's t and the next, the LDS round trips (130 clocks) and the barriers, not any rate: 3700
// clocks a column, of which the owner's part between two searches is 1100 and the search 2600.  4096 x 4096, v = 6, k = 4096, blocks
// of 128 columns: 20.9 -> 7.4 ms (of that the end of the blocks 1.5 ms); 475 x 1069: 2.5 -> 1.8 ms.
typedef _Float16 half8v __attribute__((ext_vector_type(8)));
typedef float float4v __attribute__((ext_vector_type(4)));

constexpr int PMAX = 4;
constexpr int HB = 8;                    // rows of H^-1 that are fetched together
// k slots of an entry; entries side by side in an instruction's 32; registers of 8 slots a lane holds per 64 centroids.
constexpr int entry_slots(int vp) { return vp <= 6 ? 8 : vp <= 14 ? 16 : 32; }
constexpr int entries_wide(int vp) { return 32 / entry_slots(vp); }
constexpr int group_tiles(int vp) { return 4 / entries_wide(vp); }
constexpr int E_PITCH = QB + 1;

struct LoopExchange {                  // LDS
  _Float16 operand[PMAX][2][32];       // the vectors as k slots: high and low parts
  _Float16 zeros[8];
  float t[PMAX][20];
  float eps[PMAX];                     // how far below the largest score a nearest centroid's may lie, in scaled scores
  float most[2][PMAX];                 // largest score so far
  unsigned long long nearest[2][PMAX]; // smallest (distance bits, index) so far
  float h_max[2][16], c_bad[2][16];
  float hinv[2 * HB][QB];              // rows of H^-1 inside the block, around the current column
};

template <int VP> constexpr int loop_entry_halfs() { return VP <= 4 ? 4 : VP <= 8 ? 8 : 16; }

template <int VP>
size_t loop_lds_bytes(int k, int k_res) {
  return (size_t)(k + k_res) * loop_entry_halfs<VP>() * 2 + 32 * E_PITCH * 4 + 2 * PMAX * QB * 4 + sizeof(LoopExchange) + 64;
}

// Centroid whose slots a lane holds in tile `tile` of group `g`, and which eight of them: row m of operand A is lane m of every
// sixteen, slots 8 q .. 8 q + 7 the q-th sixteen lanes.
template <int VP>
__device__ __forceinline__ int operand_entry(int g, int tile, int lane, int wave, int waves) {
  constexpr int SW = entries_wide(VP);
  return (g * waves + wave) * 64 + (tile * SW + (lane >> 4) * SW / 4) * 16 + (lane & 15);
}
template <int VP>
__device__ __forceinline__ int operand_part(int lane) { return (lane >> 4) & (4 / entries_wide(VP) - 1); }

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
__device__ __forceinline__ void load_operands(const __half *cb, int k, int v, int len, int f, int lane, int wave, int waves,
                                              half8v (&A)[G][group_tiles(VP)]) {
#pragma unroll
  for (int g = 0; g < G; ++g)
#pragma unroll
    for (int tile = 0; tile < group_tiles(VP); ++tile) {
      const __half *src = cb + (long long)min(operand_entry<VP>(g, tile, lane, wave, waves), k - 1) * v;
      const float x = ldexpf(half_norm<VP>(src, len), f);
      const _Float16 n1 = (_Float16)x, n2 = (_Float16)(x - (float)n1);
      const int part = operand_part<VP>(lane);
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const int slot = part * 8 + i;
        const _Float16 c = __builtin_bit_cast(_Float16, src[slot < len ? slot : 0]);
        A[g][tile][i] = slot < VP ? (slot < len ? c : (_Float16)0.0f) : slot == VP ? n1 : slot == VP + 1 ? n2 : (_Float16)0.0f;
      }
    }
}

// Scale of one table (|c|^2 / 2 times 2^f stays below 2^15), and the rounding bounds: with t scaled by 2^e to below 2^14, scaled
// scores are within eps0 + eps_up 2^e + eps_down 2^-e of each other's order (infinity where the table's entries are not finite or huge).
struct LoopTable { int f; float eps0, eps_up, eps_down; };

template <int VP>
__device__ __forceinline__ LoopTable loop_table(const float *h_max, const float *bad, int waves) {
  LoopTable t;
  float m = 0.0f, b = 0.0f;
  for (int w = 0; w < waves; ++w) { m = fmaxf(m, h_max[w]); b += bad[w]; }
  t.f = m > 0.0f ? min(14, max(-14, 15 - __builtin_amdgcn_frexp_expf(m))) : 14;
  // scores: two instructions whose v + 2 terms and accumulator are each cut at 2^-24 of the sum of the terms' magnitudes, |t| |c| + |c|^2 / 2
  // (vq_assign.hip), for two scores (operands below 2^-14 counted as that); |c|^2 / 2 to 2^-21 of the largest, t to 2^-20 where its
  // low part runs out of bits; the definition's own roundings: (v + 2) 2^-24 of (|t| + |c|)^2, twice
  const float c = __builtin_amdgcn_sqrtf(2.0f * m) * 1.001f + 0x1p-12f, T = __builtin_amdgcn_sqrtf((float)VP) * 1.001f * 0x1p14f;
  constexpr float D = (VP + 3) * 0x1p-23f, S = (VP + 3) * 0x1p-22f;
  t.eps0 = S * T * c + D * 2.0f * T * c + 0x1p-20f * c;
  t.eps_up = 0.5f * S * c * c + D * c * c + 0x1p-21f * m + 0x1p-37f;
  t.eps_down = D * T * T;
  if (b != 0.0f) t.eps0 = __builtin_inff();
  // (the same in every lane: kept in scalar registers)
  auto scalar = [](float y) { return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(y))); };
  t.f = __builtin_amdgcn_readfirstlane(t.f);
  t.eps0 = scalar(t.eps0); t.eps_up = scalar(t.eps_up); t.eps_down = scalar(t.eps_down);
  return t;
}

template <int N>
__device__ __forceinline__ float dpp_max(float x) {        // largest of the first N (8, 16) lanes' |x|, in those lanes
#define VQ_DPP_FMAX(CTRL) x = __uint_as_float(max(__float_as_uint(x), (unsigned)__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xF, 0xF, false)))
  x = fabsf(x);
  VQ_DPP_FMAX(0xB1);
  VQ_DPP_FMAX(0x4E);
  VQ_DPP_FMAX(0x141);
  if constexpr (N > 8) VQ_DPP_FMAX(0x140);
#undef VQ_DPP_FMAX
  return x;
}

// Lane j of the owner wave holds t_j (0 from the vector's length on): puts the vector up for the search of table `tb`.
template <int VP>
__device__ __forceinline__ void post_vector(LoopExchange &x, int p, float t, const LoopTable &tb, int lane) {
  float most = dpp_max<VP + 2 <= 8 ? 8 : 16>(t);
  if constexpr (VP + 2 > 16) most = __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(most)));
  const int e = most > 0.0f ? min(tb.f + 15, max(tb.f - 14, 14 - __builtin_amdgcn_frexp_expf(most))) : tb.f;
  const float scaled = ldexpf(t, e);
  const _Float16 hi = (_Float16)scaled, lo = (_Float16)(scaled - (float)hi);
  // (the slots behind the elements: the |c|^2 slots' factor -2^(e - f) among the high parts, zeros among the low ones)
  const _Float16 factor = __builtin_bit_cast(_Float16, (unsigned short)(0x8000u | (unsigned)(e - tb.f + 15) << 10));
  const float eps = __fmaf_rn(tb.eps_up, ldexpf(1.0f, e), __fmaf_rn(tb.eps_down, ldexpf(1.0f, -e), tb.eps0));
  if (lane < VP + 2) {
    x.operand[p][0][lane] = lane < VP ? hi : factor;
    x.operand[p][1][lane] = lo;
    x.t[p][lane] = t;
    x.eps[p] = eps;
  }
}

// One padded table entry (EH halfs) from LDS, in whole 16-byte reads (8 bytes for the smallest entries; the compiler narrows and splits
// a read whose tail is unused).  The wait stands in the same statement: this file's larger variants spill, and a register must not be
// saved while a read into it is on its way.
template <int EH>
__device__ __forceinline__ void read_entry(unsigned (&dst)[EH / 2], unsigned lds_addr) {
  if constexpr (EH == 4) {
    uint2v a;
    asm volatile("ds_read_b64 %0, %1\n\ts_waitcnt lgkmcnt(0)" : "=v"(a) : "v"(lds_addr) : "memory");
    dst[0] = a.x; dst[1] = a.y;
  } else if constexpr (EH == 8) {
    uint4v a;
    asm volatile("ds_read_b128 %0, %1\n\ts_waitcnt lgkmcnt(0)" : "=v"(a) : "v"(lds_addr) : "memory");
    dst[0] = a.x; dst[1] = a.y; dst[2] = a.z; dst[3] = a.w;
  } else {
    uint4v a, b;
    asm volatile("ds_read_b128 %0, %2\n\tds_read_b128 %1, %2 offset:16\n\ts_waitcnt lgkmcnt(0)" : "=&v"(a), "=v"(b) : "v"(lds_addr) : "memory");
    dst[0] = a.x; dst[1] = a.y; dst[2] = a.z; dst[3] = a.w;
    dst[4] = b.x; dst[5] = b.y; dst[6] = b.z; dst[7] = b.w;
  }
}

// One search of all P posted vectors over a table of `count` entries; every wave of the workgroup takes part.
template <int VP, int G>
__device__ __forceinline__ void search_table(LoopExchange &x, const half8v (&A)[G][group_tiles(VP)], unsigned lds_entries, int count, int P, int par,
                                             int lane, int wave, int waves) {
  constexpr int EH = loop_entry_halfs<VP>(), SW = entries_wide(VP), TILES = group_tiles(VP);
  // columns 4 n .. 4 n + 3 of operand B: vector n at the places 0 .. SW - 1 (and again)
  const int n = (lane >> 2) & 3, place = lane & (SW - 1);
  const bool mine = (lane >> 4) * SW / 4 == place;
  half8v B[2];
#pragma unroll
  for (int part = 0; part < 2; ++part)
    B[part] = *reinterpret_cast<const half8v *>(mine ? &x.operand[n][part][operand_part<VP>(lane) * 8] : &x.zeros[0]);
  const float eps = x.eps[n];
  float4v acc[G][TILES];
#pragma unroll
  for (int g = 0; g < G; ++g)
#pragma unroll
    for (int tile = 0; tile < TILES; ++tile)
      acc[g][tile] = __builtin_amdgcn_mfma_f32_16x16x32_f16(A[g][tile], B[0], float4v{0.0f, 0.0f, 0.0f, 0.0f}, 0, 0, 0);
#pragma unroll
  for (int g = 0; g < G; ++g)
#pragma unroll
    for (int tile = 0; tile < TILES; ++tile) acc[g][tile] = __builtin_amdgcn_mfma_f32_16x16x32_f16(A[g][tile], B[1], acc[g][tile], 0, 0, 0);
  float most = -__builtin_inff();
#pragma unroll
  for (int g = 0; g < G * TILES; ++g) {
    const float4v &a = acc[g / TILES][g % TILES];
    most = fmaxf(fmaxf(most, a[0]), a[1]);
    most = fmaxf(fmaxf(most, a[2]), a[3]);
  }
  // of the four lanes that hold one vector, then of all of them that do
  float quad = most;
  asm("s_nop 1\n\tv_max_f32_dpp %0, %0, %0 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n\ts_nop 1\n\t"
      "v_max_f32_dpp %0, %0, %0 quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf" : "+v"(quad));
  if ((lane & 3) == 0) __hip_atomic_fetch_max(&x.most[par][n], quad, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  lds_barrier();                                             // (without it most waves would take their own largest for a candidate)
  const float bar = __hip_atomic_load(&x.most[par][n], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) - eps;
  if (!__any(n < P && !(quad < bar))) return;
  // Tiles of which the four distances are wanted; the lanes of a quad compute one each, of the same four centroids.
  unsigned ask = 0u;
#pragma unroll
  for (int g = 0; g < G * TILES; ++g) {
    const float4v &a = acc[g / TILES][g % TILES];
    ask |= n < P && (lane & 3) < SW && !(fmaxf(fmaxf(a[0], a[1]), fmaxf(a[2], a[3])) < bar) ? 1u << g : 0u;
  }
  float t[VP];
#pragma unroll
  for (int j = 0; j < VP; ++j) t[j] = x.t[n][j];
  while (__any(ask != 0u)) {
    // the quad's first: place and tile
    unsigned first = ask ? (unsigned)(lane & 3) << 8 | (unsigned)__builtin_ctz(ask) : 0xFFFFu;
    first = min(first, (unsigned)__builtin_amdgcn_update_dpp(0, (int)first, 0xB1, 0xF, 0xF, false));
    first = min(first, (unsigned)__builtin_amdgcn_update_dpp(0, (int)first, 0x4E, 0xF, 0xF, false));
    if (first != 0xFFFFu) {
      const int from = (int)(first >> 8), g = (int)(first & 0xFFu);
      if (from == (lane & 3)) ask &= ask - 1u;
      const int i = min((g / TILES * waves + wave) * 64 + (g % TILES * SW + from) * 16 + (lane >> 4) * 4 + (lane & 3), count - 1);
      unsigned c[EH / 2];
      read_entry<EH>(c, lds_entries + (unsigned)i * (EH * 2u));
      float d = 0.0f;
#pragma unroll
      for (int j = 0; j < VP; ++j) {
        // t - c in one operation: the product c * -1 is exact
        const float diff = __fmaf_rn(half_of(c[j >> 1], j & 1), -1.0f, t[j]);
        d = __fmaf_rn(diff, diff, d);
      }
      __hip_atomic_fetch_min(&x.nearest[par][n], (unsigned long long)__float_as_uint(d) << 32 | (unsigned)i, __ATOMIC_RELAXED,
                             __HIP_MEMORY_SCOPE_WORKGROUP);
    }
  }
}

template <int VP, int G, int GR, int LW>
__global__ __launch_bounds__(LW * 64) void qcol_loop_kernel(LoopArgs a) {
  constexpr int EH = loop_entry_halfs<VP>();
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  __half *entries = reinterpret_cast<__half *>(smem);                                          // [k + k_res][EH]
  float *E = reinterpret_cast<float *>(smem + (((size_t)(a.k + a.k_res) * EH * 2 + 15) & ~(size_t)15));   // [32][E_PITCH]: row p * VP + j
  unsigned *codes = reinterpret_cast<unsigned *>(E + 32 * E_PITCH);                            // [2][PMAX][QB]
  LoopExchange &x = *reinterpret_cast<LoopExchange *>(codes + 2 * PMAX * QB);
  constexpr int threads = LW * 64, waves = LW;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int pos0 = blockIdx.x * a.P;
  const bool cut = pos0 >= a.whole;                                        // the workgroup of the cut-off position
  const int P = cut ? 1 : min(a.P, a.whole - pos0);
  const int first = cut ? a.whole : pos0;                                  // its first position
  const int len = cut ? a.rows - a.whole * a.v : a.v;                      // rows of a position: what its vectors are compared over
  const int mine = wave;                                                   // an owner wave's position: the first waves also own one each
  const bool owner = mine < P;

  // tables: entries in LDS (elements past `len` as zeros), operands in registers
  for (int e = tid; e < (a.k + a.k_res) * EH; e += threads) {
    const int i = e / EH, j = e % EH;
    const __half *src = i < a.k ? a.cb + (long long)i * a.v : a.cb_res + (long long)(i - a.k) * a.v;
    entries[e] = j < len ? src[j] : __float2half_rn(0.0f);
  }
  for (int e = tid; e < 32 * E_PITCH; e += threads) E[e] = 0.0f;
  for (int e = tid; e < PMAX * 2 * 32 + 8; e += threads) (&x.operand[0][0][0])[e] = (_Float16)0.0f;          // (and the zeros behind them)
  if (tid < PMAX * 20) (&x.t[0][0])[tid] = 0.0f;
  if (tid < PMAX) x.eps[tid] = 0.0f;
  if (tid < 2 * PMAX) { (&x.most[0][0])[tid] = -__builtin_inff(); (&x.nearest[0][0])[tid] = ~0ull; }
  half8v A[G][group_tiles(VP)], AR[GR ? GR : 1][group_tiles(VP)];
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
    main_table = loop_table<VP>(x.h_max[0], x.c_bad[0], waves);
    load_operands<VP, G>(a.cb, a.k, a.v, len, main_table.f, lane, wave, LW, A);
    if constexpr (GR) {
      res_table = loop_table<VP>(x.h_max[1], x.c_bad[1], waves);
      load_operands<VP, GR>(a.cb_res, a.k_res, a.v, len, res_table.f, lane, wave, LW, AR);
    }
  }
  const __half *entries_res = entries + (size_t)a.k * EH;
  const unsigned lds_entries = (unsigned)reinterpret_cast<size_t>((const __attribute__((address_space(3))) void *)smem);
  const int m0 = (first + mine) * a.v;                                     // the owner's first row
  int par = 0;

  for (int s = 0; s < a.cols; s += a.block) {
    const int s_end = min(s + a.block, a.cols), nb = s_end - s;
    {
      // the owner's tile: lane l holds columns l and l + 64
      float w[CPL][VP];
      float t = 0.0f, e = 0.0f, next_w = 0.0f;                             // lane j: element j
      // Rows of H^-1 inside the block pass through LDS, HB of them at a time: each wave holds RW of them on their way (the owners'
      // waves come last), from one eighth column to the middle of the next
      constexpr int RW = (HB + LW - 1) / LW;
      const int loader = waves - 1 - wave;
      float on_way[RW][CPL];
      auto fetch = [&](int n0) {
#pragma unroll
        for (int q = 0; q < RW; ++q)
#pragma unroll
          for (int i = 0; i < CPL; ++i) {
            const int nn = n0 + loader + q * waves, c = s + lane + 64 * i;
            on_way[q][i] = loader + q * waves < HB && nn < nb && c < s_end ? a.Hinv[(long long)(s + nn) * a.ldh + c] : 0.0f;
          }
      };
      auto land = [&](int n0) {
#pragma unroll
        for (int q = 0; q < RW; ++q)
          if (loader + q * waves < HB) {
#pragma unroll
            for (int i = 0; i < CPL; ++i) x.hinv[(n0 + loader + q * waves) & (2 * HB - 1)][lane + 64 * i] = on_way[q][i];
          }
      };
      // element j of column nn of the tile, in lane j
      auto column = [&](int nn) -> float {
        const int src = nn & 63;
        float r = 0.0f;
#pragma unroll
        for (int j = 0; j < VP; ++j) {
          const float y = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(nn >> 6 ? w[1][j] : w[0][j]), src));
          r = lane == j ? y : r;
        }
        return r;
      };
      auto take = [&](int count) -> unsigned { return min((unsigned)(x.nearest[par][mine] & 0xFFFFFFFFull), (unsigned)count - 1u); };
      auto ready = [&] {                                    // the search's slots, for the one after next
        if (lane == 0) { x.most[par][mine] = -__builtin_inff(); x.nearest[par][mine] = ~0ull; }
      };
      auto element = [&](const __half *table, unsigned i) -> float {      // of an entry, in the lane of that number
        const float y = __half2float(table[(size_t)i * EH + (lane & (EH - 1))]);
        return lane < EH ? y : 0.0f;
      };
      fetch(0);
      if (owner) {
        int lane_s = lane;
        asm volatile("" : "+v"(lane_s));                    // (see the end of the block)
#pragma unroll
        for (int i = 0; i < CPL; ++i) {
          const int c = s + lane_s + 64 * i;
#pragma unroll
          for (int j = 0; j < VP; ++j) w[i][j] = c < s_end && j < len ? a.W[(long long)(m0 + j) * a.ldw + c] : 0.0f;
        }
        t = column(0);
        post_vector<VP>(x, mine, t, main_table, lane);
      }
      land(0);
      for (int nn = 0; nn < nb; ++nn) {
        float diag = 1.0f, beside = 0.0f;
        lds_barrier();
        if ((nn & (HB - 1)) == 0) fetch(nn + HB);
        search_table<VP, G>(x, A, lds_entries, a.k, P, par, lane, wave, waves);
        if ((nn & (HB - 1)) == HB / 2) land(nn + HB / 2);
        if (owner) {
          // the last column's error reaches the tile (columns that are done may hold anything), then the next column's elements
          // are fetched from it: only this column's error is still missing from them
          if (nn > 0) {
            const float *before = x.hinv[(nn - 1) & (2 * HB - 1)];
            float h[CPL];
#pragma unroll
            for (int i = 0; i < CPL; ++i) h[i] = before[lane + 64 * i];
#pragma unroll
            for (int j = 0; j < VP; ++j) {
              const float ej = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(e), j));
#pragma unroll
              for (int i = 0; i < CPL; ++i) w[i][j] = __fmaf_rn(-ej, h[i], w[i][j]);
            }
          }
          next_w = column(min(nn + 1, QB - 1));
          diag = x.hinv[nn & (2 * HB - 1)][nn];
          beside = x.hinv[nn & (2 * HB - 1)][min(nn + 1, QB - 1)];
        }
        lds_barrier();
        float q = 0.0f;
        unsigned code = 0u, code_res = 0u;
        if (owner) {
          code = take(a.k);
          q = element(entries, code);
        }
        if constexpr (GR) {
          if (owner) { post_vector<VP>(x, mine, __fsub_rn(t, q), res_table, lane); ready(); }
          par ^= 1;
          lds_barrier();
          search_table<VP, GR>(x, AR, lds_entries + (unsigned)a.k * (EH * 2u), a.k_res, P, par, lane, wave, waves);
          lds_barrier();
          if (owner) {
            code_res = take(a.k_res);
            // what inference restores: the binary32 sum of the two centroids, rounded to binary16 (Sec. 3.2.2)
            float sum = __fadd_rn(q, element(entries_res, code_res));
            asm volatile("" : "+v"(sum));
            q = __half2float(__float2half_rn(sum));
          }
        }
        if (owner) {
          const float done = t;
          e = __fdiv_rn(__fsub_rn(t, q), diag);              // (0 in the lanes past the vector's elements)
          t = __fmaf_rn(-e, beside, next_w);
          if (nn + 1 < nb) post_vector<VP>(x, mine, t, main_table, lane);
          ready();
          if (lane < len) {
            E[(mine * VP + lane) * E_PITCH + nn] = e;
            if (a.T) a.T[(long long)(m0 + lane) * a.ldt + s + nn] = done;
          }
          if (lane == 0) { codes[mine * QB + nn] = code; codes[(PMAX + mine) * QB + nn] = code_res; }
        }
        par ^= 1;
      }
    }
    __syncthreads();

    // (what follows computes its addresses from copies of the thread's numbers that the compiler cannot see through: hoisted out
    // of the block loop they would take the registers that the columns need)
    int tid_e = tid, lane_e = lane;
    asm volatile("" : "+v"(tid_e), "+v"(lane_e));
    // the block's quantized columns and their indices (one per column: stream p, position n; the streams were cleared
    // beforehand and no other workgroup touches these)
    for (int i = tid_e; i < P * VP * QB; i += threads) {
      const int c = i & (QB - 1), r = i / QB, p = r / VP, j = r - p * VP;
      if (c >= nb || j >= len) continue;
      float q = __half2float(entries[(size_t)codes[p * QB + c] * EH + j]);
      if constexpr (GR) {
        float sum = __fadd_rn(q, __half2float(entries_res[(size_t)codes[(PMAX + p) * QB + c] * EH + j]));
        asm volatile("" : "+v"(sum));
        q = __half2float(__float2half_rn(sum));
      }
      a.W[(long long)((first + p) * a.v + j) * a.ldw + s + c] = q;
    }
    for (int i = tid_e; i < P * QB * (GR ? 2 : 1); i += threads) {
      const int c = i & (QB - 1), p = (i / QB) % P;
      const bool res = i >= P * QB;
      if (c >= nb) continue;
      const int bits = res ? a.bits_res : a.bits;
      const unsigned code = codes[((res ? PMAX : 0) + p) * QB + c];
      const unsigned long long bit = (unsigned long long)(s + c) * (unsigned)bits;
      unsigned *row = (res ? a.idx_res + (long long)(first + p) * a.idx_res_dwords : a.idx + (long long)(first + p) * a.idx_dwords) + (bit >> 5);
      const unsigned sh = (unsigned)(bit & 31u);
      atomicOr(row, code << sh);
      if (sh + bits > 32) atomicOr(row + 1, code >> (32u - sh));
    }
    // W[:, later] -= E * Hinv[block, later], a tile of 32 columns per wave (lane l gives A[l & 31][l >> 5] and B[l >> 5][l & 31]; it
    // gets back column l & 31 and, in register r, row 8 (r >> 2) + 4 (l >> 5) + (r & 3))
    const int kmax = (nb + 1) & ~1, pitch = (int)a.ldh * 4;
    const auto rows_of_block = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(a.Hinv + (long long)s * a.ldh), 0, (kmax * pitch), 0x00020000);
    for (int c0 = s_end + wave * 32; c0 < a.cols; c0 += waves * 32) {
      const int c = c0 + (lane_e & 31);
      const bool in = c < a.cols;
      const int off = (int)(((lane_e >> 5) * a.ldh + (in ? c : a.cols - 1)) * 4);
      const float *row_e = E + (lane_e & 31) * E_PITCH + (lane_e >> 5);
      float16v acc;
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[r] = 0.0f;
      constexpr int UN = LW == 4 ? 16 : 8;                   // pairs of rows on their way at once, and as many in use
      float hv[UN];
      // (past the block E has zeros, which add nothing to any row of the matrix)
      auto rows = [&](int k0, float (&y)[UN]) {
#pragma unroll
        for (int u = 0; u < UN; ++u)
          y[u] = __int_as_float(__builtin_amdgcn_raw_buffer_load_b32(rows_of_block, off, min(k0 + 2 * u, kmax - 2) * pitch, 0));
      };
      rows(0, hv);
      for (int k0 = 0; k0 < kmax; k0 += 2 * UN) {
        float ahead[UN], ev[UN];
        rows(k0 + 2 * UN, ahead);
#pragma unroll
        for (int u = 0; u < UN; ++u) ev[u] = row_e[k0 + 2 * u];
#pragma unroll
        for (int u = 0; u < UN; ++u) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(ev[u], hv[u], acc, 0, 0, 0);
#pragma unroll
        for (int u = 0; u < UN; ++u) hv[u] = ahead[u];
      }
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        if (r % 4 == 0) __builtin_amdgcn_sched_barrier(0);   // (four rows' addresses and values in registers at a time)
        const int row = 8 * (r >> 2) + 4 * (lane_e >> 5) + (r & 3), p = row / VP, j = row - p * VP;
        if (in && p < P && j < len) a.W[(long long)((first + p) * a.v + j) * a.ldw + c] -= acc[r];
      }
    }
    __syncthreads();
  }
}

template <int VP, int G, int GR, int LW>
int launch_loop(LoopArgs a, hipStream_t st) {
  auto kernel = qcol_loop_kernel<VP, G, GR, LW>;
  VQ_ALLOW_FULL_LDS(kernel);
  const int cut = a.rows - a.whole * a.v > 0;
  const unsigned grid = (unsigned)((a.whole + a.P - 1) / a.P + cut);
  hipLaunchKernelGGL(kernel, dim3(grid), dim3(LW * 64), loop_lds_bytes<VP>(a.k, a.k_res), st, a);
  return hipGetLastError() == hipSuccess ? VQ_OK : VQ_ERR_HIP;
}

// Groups of 64 centroids a wave holds: one of each table with up to 256 entries (four waves); with sixteen waves one up to 1024
// entries and four up to 4096.
template <int VP>
int launch_loop_vp(LoopArgs a, hipStream_t st) {
  if (loop_lds_bytes<VP>(a.k, a.k_res) > 160 * 1024 || a.ldh > (1 << 21)) return VQ_ERR_UNSUPPORTED;    // (a block of H^-1: 32-bit offsets)
  a.whole = a.rows / a.v;
  // positions per workgroup: as few as let every workgroup have a compute unit; E has 32 rows
  a.P = min(min(PMAX, 32 / VP), max(1, (a.whole + cu_count() - 2) / (cu_count() - 1)));
  const int big = max(a.k, a.k_res);
  if (a.k_res == 0) {
    if (big <= 256) return launch_loop<VP, 1, 0, 4>(a, st);
    if (big <= 1024) return launch_loop<VP, 1, 0, 16>(a, st);
    if constexpr (VP <= 14) { if (big <= 4096) return launch_loop<VP, 4, 0, 16>(a, st); }
  } else {
    if (big <= 256) return launch_loop<VP, 1, 1, 4>(a, st);
    if (big <= 1024) return launch_loop<VP, 1, 1, 16>(a, st);
    // (longer vectors would not leave registers for the rest)
    if constexpr (VP <= 14) { if (big <= 4096 && a.k_res <= 1024) return launch_loop<VP, 4, 1, 16>(a, st); }
    if constexpr (VP <= 6) { if (big <= 4096) return launch_loop<VP, 4, 4, 16>(a, st); }
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
