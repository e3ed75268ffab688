// vq_gemv with a workspace, one or two rows: vectors along the rows, 12-bit indices, tables of twelve-element vectors.
//
// A row's dot product is a sum over its vectors p of table[index] . x_p, and table[i] . x_p is the same number for every output row
// with that index.  So a workgroup takes eight neighbouring vector positions of one table, makes all 8 x 4096 products of entries and
// activations on the matrix cores, keeps them in LDS as binary32 numbers (128 KB), and then a row costs eight lookups of four bytes and eight
// additions, where looking the entries themselves up takes 24 bytes, as many of the activations and six dot-product instructions each.
// Lanes take rows: nothing is summed across lanes.
//
// A workgroup takes a run of pairs of such octets (24 bytes of a row's indices, two loads a lane) and a share of the rows, and leaves a
// sum a row in the workspace; gemv_products_finish_kernel adds the runs up in ascending order.  Workgroups that share lines of the index
// streams -- neighbouring runs, the same rows -- are on one XCD, behind one L2.  Outlier columns are workgroups of their own.
// Two activation rows share a lookup of eight bytes; a table of products then holds four positions.
//
// What bounds it, in clocks of a compute unit (11008 x 4096, four groups, one row, with indices and tables out of the caches: 21 thousand of
// them, 15.3 us with the second launch's and both launches' own time): 7.9 thousand until activations and the operands' 96 KB are there, 10.8 in
// the workgroups that wait for lines of the indices as well; 2.1 for storing a table of products (64 bytes a clock), twice; one a row and octet
// for the lookups (64 of four bytes take 64 clocks for a wave's eight), twice 2.2, the first time 3.6 as the index loads, a line a lane, keep
// L1's address unit busy for 4.5.
// Measured against a slot a table (vq_gemv_lds.hip), the 2.26-bit setting, the same call over and over, one / two rows: 11008 x 4096 24.0 ->
// 13.5 us, 30.5 -> 16.4; 4096 x 11008 22.6 -> 12.5, 29.1 -> 15.7; 8192 x 28672 89 -> 44, 173 -> 51; 1024 x 4096 11.0 -> 9.4, 12.0 -> 11.5.  With one
// group, one row, against vq_gemv_rows.hip: 11008 x 4096 16.1 -> 12.7, 4096 x 11008 16.6 -> 12.3, 8192 x 28672 equal.
#include <algorithm>

#include "vq_lds_tables.hpp"

namespace vq {
namespace {

using namespace lds_tables;
typedef _Float16 half8v __attribute__((ext_vector_type(8)));
typedef float float4v __attribute__((ext_vector_type(4)));
typedef float float2v __attribute__((ext_vector_type(2)));

constexpr int WAVES = 16, THREADS = WAVES * 64;
constexpr int CHUNKS = 4;                  // rows a lane takes at most
constexpr int SLOTS = 16;                  // of an operand's 32 k slots that a vector of twelve takes: two entries an instruction
constexpr int TILES = 4096 / 32 / WAVES;   // of 32 entries a wave makes the products of
constexpr unsigned UPPER = 65536u + 128u;  // two rows: the upper half of the products, half the banks further, as one instruction writes to both
constexpr unsigned PITCH = 16384u + 16u;   // one row: a position's products, four banks further than the one before for the same reason
constexpr unsigned PRODUCTS_BYTES = 131072u + 256u;
constexpr int ENTRY = 12;

struct ProductsPlan {
  int run_pairs, runs;                     // pairs of octets a workgroup takes; runs per codebook group
  int tables;                              // 1, or 2 with a residual table
  int splits, split_rows;                  // shares of the rows
  int wgs, out_wgs;                        // workgroups, and those of the outlier columns behind them
  int log_out_lanes;                       // lanes that share a row's outlier columns: 2^0 .. 2^4
  int planes;                              // sums per output row: groups x tables x runs, and one of the outlier columns
  unsigned lds;
};

constexpr unsigned whole_kb(unsigned bytes) { return (bytes + 1023u) / 1024u * 1024u; }
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

template <int B>
__global__ __launch_bounds__(THREADS) void gemv_products_kernel(Params p, ProductsPlan plan, const __half *__restrict__ x, long long ldx,
                                                                float *__restrict__ part, float *__restrict__ part_xs) {
  extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // activation of stored column c (Sec. 3.2.3), zero outside the row
  auto x_at = [&](int t, int c) {
    const int src = p.perm ? p.perm[c] : c;
    return (unsigned)src < (unsigned)p.in_features ? x[(long long)t * ldx + src] : __float2half_rn(0.0f);
  };
  float *wave_xs = reinterpret_cast<float *>(lds + PRODUCTS_BYTES);        // [B][WAVES]
  __half *xs = reinterpret_cast<__half *>(lds + PRODUCTS_BYTES + 2 * WAVES * 4);

  if ((int)blockIdx.x >= plan.wgs) {                                       // outlier columns: one to sixteen neighbouring lanes a row
    const int sub = tid & ((1 << plan.log_out_lanes) - 1), row = (((int)blockIdx.x - plan.wgs) * THREADS + tid) >> plan.log_out_lanes;
    // its rows' indices go to LDS behind the table, in whole lines: read by the lanes, each of which has a line of its own, they took longer
    // than everything else (11008 x 4096, ten vectors a row: 18.6 us against 13.6)
    const int first_row = (((int)blockIdx.x - plan.wgs) * THREADS) >> plan.log_out_lanes;
    const unsigned table_end = whole_kb((unsigned)p.k_out * 8u), bytes = (unsigned)min(THREADS >> plan.log_out_lanes, p.out_features - first_row) * (unsigned)p.stride_out;
    auto copy = [&](unsigned to, const void *from, unsigned size) {        // (not through registers; zeros up to the next KB)
      const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(from), 0, size, 0x00020000);
      for (unsigned at = (unsigned)wave * 1024u; at < size; at += WAVES * 1024u)
        __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (__attribute__((address_space(3))) void *)(lds + to + at), 16, at + (unsigned)lane * 16u, 0, 0, 0);
    };
    // (a thread's first activation is two lookups away: the first of them, the copies, the second)
    const int from_first = tid < p.n_out ? p.perm ? p.perm[tid] : tid : p.in_features;
    copy(table_end, p.idx_out + (long long)first_row * p.stride_out, bytes);
    copy(0u, p.cb_out, (unsigned)p.k_out * 8u);
    float sum_x[B], sum[B];
#pragma unroll
    for (int t = 0; t < B; ++t) {
      sum[t] = 0.0f;
      const __half first = (unsigned)from_first < (unsigned)p.in_features ? x[(long long)t * ldx + from_first] : __float2half_rn(0.0f);
      if (tid < p.n_out) xs[t * p.n_out + tid] = first;
      sum_x[t] = __half2float(first);
      for (int c = tid + THREADS; c < p.n_out; c += THREADS) {
        const __half y = x_at(t, c);
        xs[t * p.n_out + c] = y;
        sum_x[t] += __half2float(y);
      }
      sum_x[t] = wave_sum(sum_x[t]);
      if (lane == 0) wave_xs[t * WAVES + wave] = sum_x[t];
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    const unsigned char *stream = lds + table_end + min(row - first_row, p.out_features - 1 - first_row) * (int)p.stride_out;
#pragma unroll 4
    for (int c = sub; c < p.Q; c += 1 << plan.log_out_lanes) {
      const uint2v e = *reinterpret_cast<const uint2v *>(lds + min(load_index(stream, c, p.bits_out), (unsigned)p.k_out - 1u) * 8u);
#pragma unroll
      for (int t = 0; t < B; ++t) {
        const uint2v y = *reinterpret_cast<const uint2v *>(xs + t * p.n_out + c * 4);
        sum[t] = dot2(e.y, y.y, dot2(e.x, y.x, sum[t]));
      }
    }
#pragma unroll
    for (int t = 0; t < B; ++t) {
      if (plan.log_out_lanes > 0) sum[t] = dpp_add<0xB1, 0xF>(sum[t]);     // quad_perm [1,0,3,2]
      if (plan.log_out_lanes > 1) sum[t] = dpp_add<0x4E, 0xF>(sum[t]);     // quad_perm [2,3,0,1]
      if (plan.log_out_lanes > 2) sum[t] = dpp_add<0x141, 0xF>(sum[t]);    // row_half_mirror
      if (plan.log_out_lanes > 3) sum[t] = dpp_add<0x140, 0xF>(sum[t]);    // row_mirror
      if (sub == 0 && row < p.out_features) part[((long long)(plan.planes - 1) * B + t) * p.out_features + row] = sum[t];
    }
    if ((int)blockIdx.x == plan.wgs && tid < B) {
      float s = 0.0f;
      for (int w = 0; w < WAVES; ++w) s += wave_xs[tid * WAVES + w];
      part_xs[(plan.planes - 1) * 16 + tid] = s;
    }
    return;
  }

  // neighbouring runs of the same rows on one XCD (workgroups are dealt to the eight in turn)
  const int per_xcd = (plan.wgs + 7) >> 3, first_short = plan.wgs - 8 * (per_xcd - 1);     // XCDs with a workgroup more
  const int xcd = (int)blockIdx.x & 7, place = min(xcd, first_short) * per_xcd + max(xcd - first_short, 0) * (per_xcd - 1) + ((int)blockIdx.x >> 3);
  const int per_split = p.n_groups * plan.tables * plan.runs;
  const int split = place / per_split, rest = place - split * per_split;
  const int second = rest / (p.n_groups * plan.runs), run_of_all = rest - second * (p.n_groups * plan.runs);
  const int group = run_of_all / plan.runs, run = run_of_all - group * plan.runs;
  const int p_lo = group * p.Pg, p_hi = min(p.P, p_lo + p.Pg), p_first = p_lo + run * plan.run_pairs * 16;
  const int pairs = max(0, min(plan.run_pairs, (p_hi - p_first + 15) >> 4));
  const int row0 = split * plan.split_rows + wave * 64, row1 = min(p.out_features, split * plan.split_rows + plan.split_rows);

  const long long stride = second ? p.stride_res : p.stride;
  const __amdgpu_buffer_rsrc_t r_i = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t *>(second ? p.idx_res : p.idx), 0, (unsigned)((long long)p.out_features * stride), 0x00020000);
  unsigned win[CHUNKS][6];
  auto load = [&](int pair, int c) {                                       // (past a row's end: the next row's bits, or zeros)
    const int row = row0 + c * THREADS + lane;
    const unsigned at = row < row1 ? (unsigned)row * (unsigned)stride + (unsigned)((p_first >> 3) + 2 * pair) * 12u : 0xFFFFFF00u;
    const bool more = p_first + pair * 16 + 10 < p_hi;                    // (else the last indices are in the first load; the second would be the next row's line: 19.1 us)
    const uint4v a = __builtin_bit_cast(uint4v, __builtin_amdgcn_raw_buffer_load_b128(r_i, at, 0, 0));
    const uint2v b = __builtin_bit_cast(uint2v, __builtin_amdgcn_raw_buffer_load_b64(r_i, more ? at + 16u : 0xFFFFFF00u, 0, 0));
    win[c][0] = a.x; win[c][1] = a.y; win[c][2] = a.z; win[c][3] = a.w; win[c][4] = b.x; win[c][5] = b.y;
  };
  // (in the order in which they are waited for: the column of a thread's first activation, the table, the activation, the indices)
  auto column = [&](int i) {                                               // of place i of the run; the row's width: none
    const int pos = p_first + i / SLOTS, j = i % SLOTS, c = p.n_out + pos * ENTRY + j;
    return i < pairs * 16 * SLOTS && j < ENTRY && pos < p_hi ? min(c, p.in_features) : p.in_features;
  };
  const int c_first = column(tid);
  const int from_first = p.perm && c_first < p.in_features ? p.perm[c_first] : c_first;

  // the table as operand B: lane 16 q + c holds eight of the elements of entry c of the first (q = 0, 1) or second sixteen of a tile
  const int k = second ? p.k_res : p.k;
  const __half *table = second ? p.cb_res + (long long)group * p.k_res * ENTRY : p.cb + (long long)group * p.k * ENTRY;
  const __amdgpu_buffer_rsrc_t r_t = __builtin_amdgcn_make_buffer_rsrc(const_cast<__half *>(table), 0, (unsigned)(k * ENTRY * 2), 0x00020000);
  half8v entries[TILES];
  unsigned top = 0u;
#pragma unroll
  for (int i = 0; i < TILES; ++i) {
    const int e = min((wave * TILES + i) * 32 + (lane >> 5) * 16 + (lane & 15), k - 1);      // (past the table: its last entry)
    const uint4v y = __builtin_bit_cast(uint4v, __builtin_amdgcn_raw_buffer_load_b128(r_t, (unsigned)(e * ENTRY + (lane >> 4 & 1) * 8) * 2u, 0, 0));
    const unsigned both[4] = {y.x, y.y, lane >> 4 & 1 ? 0u : y.z, lane >> 4 & 1 ? 0u : y.w};
    entries[i] = __builtin_bit_cast(half8v, uint4v{both[0], both[1], both[2], both[3]});
#pragma unroll
    for (int d = 0; d < 4; ++d) top = max(top, max(both[d] & 0x7C00u, (both[d] >> 16) & 0x7C00u));
  }

  // The lines of the indices start on their way from memory to L2 here: neighbouring runs share them, so each touches a share of the
  // rows, with waves that have no activations to wait for (forty layers in turn, 11008 x 4096: 16.4 -> 15.3 us; one layer 13.5 -> 13.9).
  const int share = max(1, 5 / plan.run_pairs);
  unsigned touched[2];
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const int row = split * plan.split_rows + (tid - THREADS / 2 + u * (THREADS / 2)) * share + run % share;
    touched[u] = tid >= THREADS / 2 && row < row1 ? __builtin_amdgcn_raw_buffer_load_b32(r_i, (unsigned)row * (unsigned)stride + (unsigned)(p_first >> 3) * 12u, 0, 0) : 0u;
  }

  // activations of the run, a vector to sixteen places, zeros past it, past the group and past the row
  float sum_x[B];
  __half x_first[B];
#pragma unroll
  for (int t = 0; t < B; ++t) x_first[t] = (unsigned)from_first < (unsigned)p.in_features ? x[(long long)t * ldx + from_first] : __float2half_rn(0.0f);
#pragma unroll
  for (int t = 0; t < B; ++t) {
    __half *to = xs + t * plan.run_pairs * 16 * SLOTS;
    if (tid < pairs * 16 * SLOTS) to[tid] = x_first[t];
    sum_x[t] = __half2float(x_first[t]);
    for (int i = tid + THREADS; i < pairs * 16 * SLOTS; i += THREADS) {
      const int c = column(i);
      const __half y = c < p.in_features ? x_at(t, c) : __float2half_rn(0.0f);
      to[i] = y;
      sum_x[t] += __half2float(y);
    }
    sum_x[t] = wave_sum(sum_x[t]);
    if (lane == 0) wave_xs[t * WAVES + wave] = sum_x[t];
  }
  // entries that are no numbers: products of the two entries of a tile are then kept apart, as 0 times such an element is not 0
  const bool odd = __any(top == 0x7C00u);
  const int elements = p.in_features - p.n_out - (p.P - 1) * ENTRY;       // of the row's last vector

  float sum[CHUNKS][B];
#pragma unroll
  for (int c = 0; c < CHUNKS; ++c)
#pragma unroll
    for (int t = 0; t < B; ++t) sum[c][t] = 0.0f;

  constexpr int AT_ONCE = 8 / B;                                           // positions of a table of products
  // operand A: row m is a position (and activation row) of the first (m < 8) or second entry's eight
  const int a_plane = lane & 7, a_pos = a_plane / B, a_row = a_plane % B;
  const bool a_mine = (lane >> 3 & 1) == (lane >> 5);
  // two rows: activations times entries, a lane gets four (position, row) pairs of an entry; one row: entries times activations, four entries
  // of a position, sixteen bytes to store
  const unsigned entry_at = B == 1 ? (unsigned)a_plane * PITCH + (unsigned)((lane >> 3 & 1) * 16 + (lane >> 4) * 4) * 4u
                                   : (unsigned)((lane >> 5) * 16 + (lane & 15)) * (4u * B) + (lane >> 4 & 1 ? UPPER : 0u);
  auto multiply = [&](const half8v &a, const half8v &e) {
    const float4v zero = {0.0f, 0.0f, 0.0f, 0.0f};
    return B == 1 ? __builtin_amdgcn_mfma_f32_16x16x32_f16(e, a, zero, 0, 0, 0) : __builtin_amdgcn_mfma_f32_16x16x32_f16(a, e, zero, 0, 0, 0);
  };
  const bool first_entry = B == 1 ? (lane & 8) == 0 : lane < 32;           // which of a tile's two sixteens a lane gets products of
  for (int pair = 0; pair < pairs; ++pair) {
#pragma unroll
    for (int part_of = 0; part_of < 2 * B; ++part_of) {
      const int first = p_first + pair * 16 + part_of * AT_ONCE;
      if (first >= p_hi) break;
      lds_barrier();                                                       // (activations are there; everybody is through with the products before)
      // A lane's indices lie in a line of their own, and a load of them takes the compute unit's address unit 64 clocks: the first rows' while
      // products are made, the others' while those before them are looked up.
      if (part_of == 0) load(pair, 0);
      uint4v a = *reinterpret_cast<const uint4v *>(xs + (a_row * plan.run_pairs * 16 + pair * 16 + part_of * AT_ONCE + a_pos) * SLOTS + (lane >> 4 & 1) * 8);
      if (!a_mine) a = uint4v{0u, 0u, 0u, 0u};
      const half8v A = __builtin_bit_cast(half8v, a);
      auto keep = [&](int i, const float4v &d) {
        unsigned char *to = lds + entry_at + (unsigned)(wave * TILES + i) * (32u * 4u * B);
        if constexpr (B == 1) *reinterpret_cast<float4v *>(to) = d;
        else {
          *reinterpret_cast<float2v *>(to) = float2v{d[0], d[1]};
          *reinterpret_cast<float2v *>(to + 32768) = float2v{d[2], d[3]};
        }
      };
      if (__builtin_expect(odd, 0)) {
#pragma unroll
        for (int i = 0; i < TILES; ++i) {
          unsigned mine = lane < 32 ? ~0u : 0u;
          asm volatile("" : "+v"(mine));                                   // (here, not kept for all tiles)
          const uint4v e = __builtin_bit_cast(uint4v, entries[i]);
          const float4v d1 = multiply(A, __builtin_bit_cast(half8v, e & mine));
          const float4v d2 = multiply(A, __builtin_bit_cast(half8v, e & ~mine));
          float4v d = first_entry ? d1 : d2;
#pragma unroll
          for (int r = 0; r < 4; ++r)                                      // (whatever bits stand behind the last index: nothing)
            if (first + (B == 1 ? a_plane : ((lane >> 4 & 1) * 4 + r) / B) >= p_hi) d[r] = 0.0f;
          keep(i, d);
        }
        // of the row's last vector, what lies past the row is dropped: its products once more
        if (elements < ENTRY && first <= p.P - 1 && first + AT_ONCE >= p.P) {
#pragma unroll 1
          for (int turn = 0; turn < TILES; ++turn) {
            half8v mine;                                                   // (entry `turn` of the array, which stays in registers)
#pragma unroll
            for (int i = 0; i < TILES; ++i)
              if (i == turn) mine = entries[i];
            uint4v e = __builtin_bit_cast(uint4v, mine);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              const int left = elements - (lane >> 4 & 1) * 8 - 2 * q;     // elements of this dword that are the row's
              e[q] = left >= 2 ? e[q] : left == 1 ? e[q] & 0xFFFFu : 0u;
            }
            const unsigned low = lane < 32 ? ~0u : 0u;
            const float4v d1 = multiply(A, __builtin_bit_cast(half8v, e & low)), d2 = multiply(A, __builtin_bit_cast(half8v, e & ~low));
            const float4v d = first_entry ? d1 : d2;
            unsigned char *to = lds + entry_at + (unsigned)(wave * TILES + turn) * (32u * 4u * B);
            const int position = first + (B == 1 ? a_plane : (lane >> 4 & 1) * 2);
            if constexpr (B == 1) {
              if (position == p.P - 1) *reinterpret_cast<float4v *>(to) = d;
            } else {
              if (position == p.P - 1) *reinterpret_cast<float2v *>(to) = float2v{d[0], d[1]};
              if (position + 1 == p.P - 1) *reinterpret_cast<float2v *>(to + 32768) = float2v{d[2], d[3]};
            }
          }
        }
      } else {
#pragma unroll
        for (int i = 0; i < TILES; i += 4) {
          float4v d[4];
#pragma unroll
          for (int j = 0; j < 4; ++j) d[j] = multiply(A, entries[i + j]);
#pragma unroll
          for (int j = 0; j < 4; ++j) keep(i + j, d[j]);
        }
      }
      lds_barrier();
#pragma unroll
      for (int c = 0; c < CHUNKS; ++c) {
        if (row0 + c * THREADS >= row1) break;
        if (part_of == 0 && c + 1 < CHUNKS && row0 + (c + 1) * THREADS < row1) load(pair, c + 1);
#pragma unroll
        for (int u = 0; u < AT_ONCE; ++u) {
          const unsigned i = window_field<12, 6>(win[c], part_of * AT_ONCE + u);
          // (the kernel has no other LDS than this array, which begins at 0: addresses as numbers, constant parts in the instruction)
          if constexpr (B == 1) sum[c][0] += *(const __attribute__((address_space(3))) float *)(i * 4u + (u >= 4 ? 4 * PITCH : 0u) + (u & 3) * PITCH);
          else {
            const float2v y = *(const __attribute__((address_space(3))) float2v *)(i * 8u + (u >= 2 ? UPPER : 0u) + (u & 1) * 32768u);
            sum[c][0] += y.x; sum[c][1] += y.y;
          }
        }
      }
    }
  }
  asm volatile("" :: "v"(touched[0]), "v"(touched[1]));
  const int plane = rest;
#pragma unroll
  for (int c = 0; c < CHUNKS; ++c) {
    const int row = row0 + c * THREADS + lane;
    if (row < row1)
#pragma unroll
      for (int t = 0; t < B; ++t) part[((long long)plane * B + t) * p.out_features + row] = sum[c][t];
  }
  if (split == 0) {
    __syncthreads();
    if (tid < B) {
      float s = 0.0f;
      if (!second)
        for (int w = 0; w < WAVES; ++w) s += wave_xs[tid * WAVES + w];
      part_xs[plane * 16 + tid] = s;
    }
  }
}

// y[t][o] = fp16(scale[o] * sum of part[plane][t][o] + bias[o] * sum of part_xs[plane][t]): sixteen threads to an output, each of which adds
// neighbouring planes in ascending order, then their sums in ascending order.
constexpr int FINISH_OUTPUTS = 32, FINISH_SLICES = 16;
__global__ __launch_bounds__(FINISH_OUTPUTS * FINISH_SLICES) void gemv_products_finish_kernel(const float *__restrict__ part, const float *__restrict__ part_xs, int planes,
                                                                                              int batch, int out_features, const __half *__restrict__ scale,
                                                                                              const __half *__restrict__ bias, __half *__restrict__ y, long long ldy) {
  __shared__ float sums[FINISH_SLICES][FINISH_OUTPUTS], sums_x[FINISH_SLICES];
  const int column = threadIdx.x % FINISH_OUTPUTS, slice = threadIdx.x / FINISH_OUTPUTS, t = blockIdx.y;
  const int o = blockIdx.x * FINISH_OUTPUTS + column, at = min(o, out_features - 1);
  const int per = (planes + FINISH_SLICES - 1) / FINISH_SLICES, from = slice * per, to = min(planes, from + per);
  float sc = 1.0f, bi = 0.0f;
  if (slice == 0) { sc = scale ? __half2float(scale[at]) : 1.0f; bi = bias ? __half2float(bias[at]) : 0.0f; }
  float sum = 0.0f, xs = 0.0f;
  for (int g0 = from; g0 < to; g0 += 8) {
    float v[8], w[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int g = min(g0 + i, to - 1);
      v[i] = part[((long long)g * batch + t) * out_features + at];
      w[i] = part_xs[g * 16 + t];
    }
#pragma unroll
    for (int i = 0; i < 8; ++i)
      if (g0 + i < to) { sum += v[i]; xs += w[i]; }
  }
  sums[slice][column] = sum;
  if (column == 0) sums_x[slice] = xs;
  __syncthreads();
  if (slice == 0 && o < out_features) {
    sum = 0.0f; xs = 0.0f;
#pragma unroll
    for (int s = 0; s < FINISH_SLICES; ++s) { sum += sums[s][column]; xs += sums_x[s]; }
    y[(long long)t * ldy + o] = __float2half_rn(__fmaf_rn(sc, sum, bi * xs));
  }
}

// A share of the rows and a run of octets for every workgroup, all of them on the chip at once: the split with the least of (clocks, from the
// kernel's parts) products made, rows looked up, and sums added up behind.
bool make_products_plan(const Params &p, int batch, ProductsPlan *plan) {
  // (lanes to a row until each has sixteen of its outlier vectors, as far as an eighth of the chip does)
  plan->log_out_lanes = 0;
  while (plan->log_out_lanes < 4 && p.Q > 16 << plan->log_out_lanes && (long long)p.out_features << (plan->log_out_lanes + 1) <= (long long)cu_count() / 8 * THREADS) ++plan->log_out_lanes;
  if (p.Q && whole_kb(p.k_out * 8u) + ((size_t)(THREADS >> plan->log_out_lanes) * p.stride_out + 1023) / 1024 * 1024 > PRODUCTS_BYTES) return false;
  plan->out_wgs = p.Q ? (int)((((long long)p.out_features << plan->log_out_lanes) + THREADS - 1) / THREADS) : 0;
  const int most = cu_count() - plan->out_wgs;
  plan->tables = p.k_res ? 2 : 1;
  const int sets = p.n_groups * plan->tables, pairs = ((p.n_groups > 1 ? p.Pg : p.P) + 15) / 16;
  long long best = -1;
  for (int splits = (p.out_features + CHUNKS * THREADS - 1) / (CHUNKS * THREADS); splits * sets <= most; ++splits) {
    const int split_rows = ((p.out_features + splits - 1) / splits + 63) / 64 * 64;
    const int run_pairs = (pairs + most / (splits * sets) - 1) / (most / (splits * sets)), runs = (pairs + run_pairs - 1) / run_pairs;
    const long long clocks = run_pairs * 2 * (1700LL * batch + split_rows) + (long long)sets * runs * batch * p.out_features / 360;
    if (best < 0 || clocks < best) {
      best = clocks;
      plan->run_pairs = run_pairs; plan->runs = runs; plan->splits = splits; plan->split_rows = split_rows;
    }
    if (split_rows <= 64) break;
  }
  if (best < 0) return false;
  plan->splits = (p.out_features + plan->split_rows - 1) / plan->split_rows;
  plan->wgs = plan->splits * sets * plan->runs;
  plan->planes = sets * plan->runs + (p.Q ? 1 : 0);
  const size_t x_bytes = (size_t)batch * std::max((size_t)plan->run_pairs * 16 * SLOTS, (size_t)p.n_out) * 2;
  plan->lds = (unsigned)std::min<size_t>(PRODUCTS_BYTES + 2 * WAVES * 4 + (x_bytes + 15) / 16 * 16, 1u << 20);
  return plan->lds <= 160 * 1024;
}

size_t products_bytes(const Params &p, const ProductsPlan &plan, int batch) {
  return ((size_t)plan.planes * ((size_t)batch * (size_t)p.out_features + 16) * sizeof(float) + 255) / 256 * 256;
}

bool products_plan(const Params &p, int batch, ProductsPlan *plan) {
  if (switches().gemv || switches().groups_loop || switches().rows >= 0 || switches().products == 0) return false;
  // Two launches, each with a start of its own, want enough vectors to look up.  With codebook groups, where a table a workgroup is the
  // alternative: one row from 2^15 on (512 x 512, 22 thousand: 8.8 us without, 9.0; 256 x 2048, 43 thousand: 9.4, 9.0), two rows from 2^18 (2048 x
  // 1024, 2^17.4: 11.2, 11.3; 1024 x 4096, 2^18.4: 12.0, 11.5), with few groups of one table from 2^19 and 2^20 (four, one row, 637 x 3640: 9.0, 9.6;
  // seven, two rows, 2164 x 3903: 10.5, 12.0); with one group, where the matrix cores take several rows at the price of one, two rows never
  // (11008 x 4096: 16.2, 16.3), one row with two tables, which those look up one after the other, from 3 x 2^17 on (2048 x 2048, 350 thousand: 9.4, 9.5;
  // 4096 x 4096: 11.1, 10.2), with one from 9 x 2^19 (6399 x 1052: 6.9, 9.9; 12213 x 4395, 2^22.1: 10.0, 11.4; 5859 x 10344, 2^22.3: 14.8, 11.8).
  const long long vectors = (long long)p.out_features * p.P;
  const bool few_tables = !p.k_res && p.n_groups <= 8;
  const long long least = p.n_groups > 1 ? (batch == 1 ? few_tables ? 1 << 19 : 1 << 15 : few_tables ? 1 << 20 : 1 << 18) : p.k_res ? 3 << 17 : 9 << 19;
  if (switches().products < 0 && (vectors < least || (p.n_groups == 1 && batch > 1))) return false;
  if (p.orientation != 0 || p.v != ENTRY || p.bits != 12 || (p.k_res && p.bits_res != 12) || batch > 2 || cu_count() < 64) return false;
  if (p.n_groups > 1 && p.Pg % 8) return false;                            // (octets begin at a dword of the stream)
  if (p.Q && (p.v_out != 4 || p.k_out > 8192)) return false;
  if (p.out_features > 16384) return false;                                // (a lane would take more rows than the plan below gives it to advantage)
  if ((long long)p.out_features * p.stride >= 1LL << 31 || (p.k_res && (long long)p.out_features * p.stride_res >= 1LL << 31)) return false;
  return make_products_plan(p, batch, plan) && products_bytes(p, *plan, batch) <= VQ_GEMV_STATIC_WORKSPACE_BYTES;
}

}  // namespace

size_t gemv_products_workspace_bytes(const Params &p, int batch) {
  ProductsPlan plan;
  return products_plan(p, batch, &plan) ? products_bytes(p, plan, batch) : 0;
}

int launch_gemv_products(const Params &p, const __half *x, long long ldx, int batch, __half *y, long long ldy, void *workspace, size_t workspace_bytes, hipStream_t s) {
  ProductsPlan plan;
  if (!workspace || !products_plan(p, batch, &plan) || workspace_bytes < products_bytes(p, plan, batch)) return VQ_ERR_UNSUPPORTED;
  float *part = static_cast<float *>(workspace), *part_xs = part + (size_t)plan.planes * (size_t)batch * (size_t)p.out_features;
  const dim3 grid((unsigned)(plan.wgs + plan.out_wgs));
  if (batch == 1) {
    VQ_ALLOW_FULL_LDS(gemv_products_kernel<1>);
    hipLaunchKernelGGL(gemv_products_kernel<1>, grid, dim3(THREADS), plan.lds, s, p, plan, x, ldx, part, part_xs);
  } else {
    VQ_ALLOW_FULL_LDS(gemv_products_kernel<2>);
    hipLaunchKernelGGL(gemv_products_kernel<2>, grid, dim3(THREADS), plan.lds, s, p, plan, x, ldx, part, part_xs);
  }
  hipLaunchKernelGGL(gemv_products_finish_kernel, dim3((unsigned)((p.out_features + FINISH_OUTPUTS - 1) / FINISH_OUTPUTS), (unsigned)batch), dim3(FINISH_OUTPUTS * FINISH_SLICES), 0, s,
                     part, part_xs, plan.planes, batch, p.out_features, p.scale, p.bias, y, ldy);
  return hipGetLastError() == hipSuccess ? VQ_OK : VQ_ERR_HIP;
}

}  // namespace vq
