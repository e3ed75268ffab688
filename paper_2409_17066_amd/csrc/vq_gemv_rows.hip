// vq_gemv for up to sixteen activation rows on the matrix cores, for the settings whose tables are looked up entry by entry (v = 2,
// 4, 6, 8, 12 with 4-, 8- or 12-bit indices: one table at a time in LDS; v = 8 with 16-bit indices: a 1 MiB table read through L2),
// in both orientations.  (Decode phase: restore and multiply fused; the restored weights are never written.)
//
// v_mfma_f32_16x16x32_f16 wants of a lane eight consecutive products' weights of row (lane & 15) and the same eight activations of
// batch row (lane & 15), for four lane groups: 32 columns.  The order of the columns is free as long as both sides agree, so a
// lane simply takes eight neighbouring vectors of its row (a window: BITS bytes of indices):
//  * vectors along the row: their entries one after the other ARE 8 V weights, V operands, with no shuffling at all;
//  * vectors down the outputs: element j of the eight entries is one operand for output row V * stream + j: V products
//    of the same eight activations, after picking halves (four v_perm_b32 an operand).
// Scale and bias wait until the end, as in the other decode kernels: y = scale * sum(d x) + bias * sum(x); residual entries are a
// second pass of products over the same columns, not additions, and sum(x) is a product with ones.
//
// A workgroup of 16 waves owns RB blocks of 16 rows (one block of 16 streams), its waves take every 16th step of 32 vectors.
// Tables beyond L1 are staged one at a time; codebook groups are walked one after the other.  With a workspace the columns
// are cut into parts, one workgroup each, whose sums another kernel adds up (a group per part, where there are groups).
//
// What bounds it: the table lookups in LDS (a step reads 8 entries a lane and table), for few rows the staging of 96 KB tables.
// One launch does for any number of activation rows what the dot-product kernels did for four.
#include "vq_lds_tables.hpp"
#include <type_traits>
#include <utility>

namespace vq {

namespace {

using namespace lds_tables;

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef float float4v __attribute__((ext_vector_type(4)));

constexpr int STEP = 32;                                 // vectors (positions) of a row per step: a window of 8 for each lane group
constexpr unsigned UNIT = 256 * 4;                       // bytes of one 16 x 16 block of sums

struct RowsArgs {
  const __half *x; long long ldx; int batch;
  __half *y; long long ldy;
  float *part, *part_xs;                                 // with a workspace: [parts][batch][out_features] and [parts][16]
  int row_wgs, parts_per_group;                          // workgroups along the rows; parts_per_group = 0: no workspace
};

// 16 bytes of each lane from byte `offset` of a buffer to 1 KB of LDS at `to` (outside the template: the host pass does not take it there)
__device__ __forceinline__ void copy16(const __amdgpu_buffer_rsrc_t &from, unsigned char *to, unsigned offset) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(from, (__attribute__((address_space(3))) void *)to, 16, offset, 0, 0, 0);
}

__device__ __forceinline__ uint4v load16(const __amdgpu_buffer_rsrc_t &r, unsigned offset) { return __builtin_bit_cast(uint4v, __builtin_amdgcn_raw_buffer_load_b128(r, offset, 0, 0)); }
__device__ __forceinline__ unsigned load2(const __amdgpu_buffer_rsrc_t &r, unsigned offset) { return (unsigned)(unsigned short)__builtin_amdgcn_raw_buffer_load_b16(r, offset, 0, 0); }
template <int ND> __device__ __forceinline__ void load_dwords(unsigned (&w)[ND], __amdgpu_buffer_rsrc_t r, unsigned offset) {
  if constexpr (ND == 2) { const uint2v v = __builtin_bit_cast(uint2v, __builtin_amdgcn_raw_buffer_load_b64(r, offset, 0, 0)); w[0] = v.x; w[1] = v.y; }
  else if constexpr (ND == 4) { const uint4v v = load16(r, offset); w[0] = v.x; w[1] = v.y; w[2] = v.z; w[3] = v.w; }
  else load_window<ND>(w, r, offset);
}

template <int... I, class F> __device__ __forceinline__ void for_each(F &&f, std::integer_sequence<int, I...>) { (f(std::integral_constant<int, I>{}), ...); }
template <int N, class F> __device__ __forceinline__ void for_each(F &&f) { for_each(f, std::make_integer_sequence<int, N>{}); }

constexpr int acc_units(int v, bool down, int rb) { return down ? v : rb; }

// LOG_FOLDS: rows of operand A and columns of operand B are (stream, fold) and (batch row, fold) pairs, a block has 8 or 4 streams and their columns come in
// two or four folds, step s of a fold being step s * folds + fold of the stream.  Of a result what has the same fold on both sides counts; the folds' sums
// are added with the waves'.  For layers of few blocks and up to eight (four) batch rows, in one launch (see rows_folds).
template <int V, int BITS, bool DOWN, int RB, int RW, bool PERM, int LOG_FOLDS>
__global__ __launch_bounds__(RW * 64, 4) void gemv_rows_kernel(Params p, RowsArgs a) {
  constexpr bool GLOBAL = BITS == 16;
  constexpr int ND = BITS / 4, VD = V / 2, ED = entry_halfs(V) / 2, NU = acc_units(V, DOWN, RB);
  constexpr int NX = DOWN ? 1 : V;                       // operands of activations per step
  constexpr bool AHEAD = DOWN || V * (RB + 1) <= 15;      // whether the registers hold two steps' activations
  constexpr int EPC = V == 8 ? 1 : V == 12 ? 2 : V == 4 ? 2 : 4, HPC = EPC * V / 8;      // entries and operands of a piece of a window
  extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
  constexpr int FOLDS = 1 << LOG_FOLDS, STREAMS = 16 / FOLDS, WIDTH = STEP * FOLDS;      // (positions of a step)
  static_assert(FOLDS == 1 || RB == 1, "one block where there are few");
  const int lane = threadIdx.x & 63, slot = (lane & 15) % STREAMS, g = lane >> 4;
  const int lead = (lane & 15) / STREAMS * STEP + 8 * g;      // the lane's first position in a step
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int blk0 = (int)(blockIdx.x % (unsigned)a.row_wgs) * RB, part = (int)(blockIdx.x / (unsigned)a.row_wgs);
  const bool parts = a.parts_per_group != 0;
  const bool want_xs = p.bias && (!parts || blk0 == 0);

  float4v acc[NU], xacc = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
  for (int i = 0; i < NU; ++i) acc[i] = float4v{0.0f, 0.0f, 0.0f, 0.0f};
  int stream[RB];
#pragma unroll
  for (int i = 0; i < RB; ++i) stream[i] = min((blk0 + i) * STREAMS + slot, p.S - 1);

  // Eight activations from stored column c (even) on; past a row's end they may be the next row's, past the last one's zeros:
  // cut() clears those from `limit` on.
  const __amdgpu_buffer_rsrc_t r_x = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<__half *>(a.x), 0, (unsigned)(((long long)(a.batch - 1) * a.ldx + p.in_features + 1) * 2) & ~3u, 0x00020000);
  const unsigned x_row = (unsigned)min(slot, a.batch - 1) * (unsigned)a.ldx * 2u;      // (operand columns past the batch repeat its last row; never stored)
  const __amdgpu_buffer_rsrc_t r_p = __builtin_amdgcn_make_buffer_rsrc(const_cast<int *>(p.perm), 0, PERM ? (unsigned)p.in_features * 4u : 0u, 0x00020000);
  auto load_x = [&](int c) -> uint4v {
    if constexpr (!PERM) return load16(r_x, x_row + (unsigned)c * 2u);
    // permuted: eight lookups (columns outside the layer read zeros: their offsets lie past the buffer)
    const uint4v t0 = load16(r_p, (unsigned)c * 4u), t1 = load16(r_p, (unsigned)c * 4u + 16u);
    auto at = [&](unsigned t) { return t < (unsigned)p.in_features ? x_row + t * 2u : 0x80000000u; };
    return uint4v{load2(r_x, at(t0.x)) | load2(r_x, at(t0.y)) << 16, load2(r_x, at(t0.z)) | load2(r_x, at(t0.w)) << 16,
                  load2(r_x, at(t1.x)) | load2(r_x, at(t1.y)) << 16, load2(r_x, at(t1.z)) | load2(r_x, at(t1.w)) << 16};
  };
  auto cut = [&](uint4v v, int left) -> uint4v {         // left = limit - c
    auto keep = [&](unsigned d, int e) { return e + 1 < left ? d : e < left ? d & 0xFFFFu : 0u; };
    return uint4v{keep(v.x, 0), keep(v.y, 2), keep(v.z, 4), keep(v.w, 6)};
  };
  auto operand = [](uint4v v) { return __builtin_bit_cast(half8, v); };
  const half8 ones = {(_Float16)1, (_Float16)1, (_Float16)1, (_Float16)1, (_Float16)1, (_Float16)1, (_Float16)1, (_Float16)1};
  auto product = [](half8 w, half8 x, float4v c) { return __builtin_amdgcn_mfma_f32_16x16x32_f16(w, x, c, 0, 0, 0); };

  const int group_lo = parts ? part / a.parts_per_group : 0, group_hi = parts ? group_lo + 1 : p.n_groups;
  for (int group = group_lo; group < group_hi; ++group) {
    const int pos0 = group * p.Pg, pos_end = min(p.P, pos0 + p.Pg), steps = (pos_end - pos0 + WIDTH - 1) / WIDTH;
    int step_lo = 0, step_hi = steps;
    if (parts) {
      const int sub = part - group * a.parts_per_group;
      step_lo = (int)((long long)steps * sub / a.parts_per_group); step_hi = (int)((long long)steps * (sub + 1) / a.parts_per_group);
    }
    const bool last_steps = step_hi == steps;             // the group's ragged end is this workgroup's
    const int x_limit = DOWN ? p.n_out + pos_end : (int)min((long long)p.in_features, p.n_out + (long long)pos_end * V);
    for (int table = 0; table < (p.k_res ? 2 : 1); ++table) {
      const int k = table ? p.k_res : p.k;
      const __half *cb = (table ? p.cb_res : p.cb) + (long long)group * k * V;
      const uint8_t *idx = table ? p.idx_res : p.idx;
      const long long stride = table ? p.stride_res : p.stride;
      // (past a row's end: the next row's indices, or zeros; those vectors do not count)
      const __amdgpu_buffer_rsrc_t r_i = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t *>(idx), 0, (unsigned)((long long)p.S * stride), 0x00020000);
      auto load_window = [&](unsigned (&w)[ND], int i, int s) {
        const unsigned at = (unsigned)stream[i] * (unsigned)stride + (unsigned)((pos0 + s * WIDTH + lead) >> 3) * BITS;
        load_dwords<ND>(w, r_i, at);
      };
      auto is_last = [&](int s) {
        return pos0 + (s + 1) * WIDTH > pos_end || (!DOWN && p.n_out + (long long)(pos0 + (s + 1) * WIDTH) * V > p.in_features);
      };
      auto load_step_x = [&](auto &xw, int s) {
        const int pos = pos0 + s * WIDTH + lead;
#pragma unroll
        for (int h = 0; h < NX; ++h) xw[h] = load_x(p.n_out + (DOWN ? pos : pos * V + 8 * h));
      };
      // Loads come back in order, so what is needed first goes out first: activations (from L2) a step ahead, then the indices (from
      // HBM) of the step after; without AHEAD activations a piece ahead, the indices last.
      unsigned win[RB][ND], next[AHEAD ? RB : 1][ND];
      uint4v xw[AHEAD ? NX : 1], xn[AHEAD ? NX : 1];
      const int s0 = step_lo + wave;
      if (s0 < step_hi) {                                // (asked for before the table: the trips to memory overlap)
#pragma unroll
        for (int i = 0; i < RB; ++i) load_window(win[i], i, s0);
        if constexpr (AHEAD) load_step_x(xw, s0);
#pragma unroll
        for (int i = 0; i < (AHEAD ? RB : 0); ++i) load_window(next[i], i, s0 + RW < step_hi ? s0 + RW : s0);
      }
      if constexpr (!GLOBAL) {
        __syncthreads();
        if constexpr (entry_halfs(V) == V) {             // entries as they are in memory: copied without passing through registers
          const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(const_cast<__half *>(cb), 0, (unsigned)(k * V * 2), 0x00020000);
          for (unsigned at = (unsigned)wave * 1024u; at < (unsigned)(k * V * 2); at += RW * 1024u) copy16(r, lds + at, at + (unsigned)lane * 16u);
          asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        } else {
          for (int en = threadIdx.x; en < k; en += RW * 64) stage_entry<V>(lds, cb, en);
        }
        __syncthreads();
        if (last_steps) {                                // entry k: zeros, for the vectors past the end
          if (threadIdx.x < ED) reinterpret_cast<unsigned *>(lds)[k * ED + threadIdx.x] = 0u;
          __syncthreads();
        }
      }
      for (int s = s0; s < step_hi; s += RW) {
        unsigned far[RB][ND];
        const int s1 = s + RW < step_hi ? s + RW : s, s2 = s + 2 * RW < step_hi ? s + 2 * RW : s1;
        if constexpr (AHEAD) {
          load_step_x(xn, s1);
#pragma unroll
          for (int i = 0; i < RB; ++i) load_window(far[i], i, s2);
        }
        const int pos = pos0 + s * WIDTH + lead;
        const bool last = is_last(s);
        if (AHEAD && last)
#pragma unroll
          for (int h = 0; h < (AHEAD ? NX : 0); ++h) xw[h] = cut(xw[h], x_limit - (p.n_out + (DOWN ? pos : pos * V + 8 * h)));
        auto entry_of = [&](const unsigned (&w)[ND], int u) -> unsigned {
          unsigned i = min(window_field<BITS, ND>(w, u), (unsigned)k - 1u);
          if (last && pos + u >= pos_end) i = GLOBAL ? 0u : (unsigned)k;
          return i;
        };
        auto read = [&](unsigned (&e)[ED], unsigned i, int u) {
          if constexpr (GLOBAL) {
            const uint4v v = *reinterpret_cast<const uint4v *>(cb + (long long)i * V);
            const bool on = !last || pos + u < pos_end;
            e[0] = on ? v.x : 0u; e[1] = on ? v.y : 0u; e[2] = on ? v.z : 0u; e[3] = on ? v.w : 0u;
          } else read_entry<V>(e, lds, i);
        };
        if constexpr (DOWN) {
          unsigned ei[8];
#pragma unroll
          for (int u = 0; u < 8; ++u) ei[u] = entry_of(win[0], u);
          const half8 xo = operand(xw[0]);
          if (table == 0 && want_xs) xacc = product(ones, xo, xacc);
          // (v = 12 in three goes of four elements: all of eight entries would not fit the registers)
          constexpr int GO = V == 12 ? 2 : ED;
          for_each<ED / GO>([&](auto go) {
            constexpr int d0 = decltype(go)::value * GO;
            unsigned e[8][GO];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
              if constexpr (V == 12) {
                const uint2v v = *reinterpret_cast<const uint2v *>(lds + ei[u] * 24u + d0 * 4u);
                e[u][0] = v.x; e[u][1] = v.y;
              } else read(e[u], ei[u], u);
            }
#pragma unroll
            for (int j = 2 * d0; j < 2 * (d0 + GO) && j < V; ++j) {
              const unsigned sel = j & 1 ? 0x07060302u : 0x05040100u;      // halves j of two entries
              const int d = (j >> 1) - d0;
              uint4v w;
              w.x = __builtin_amdgcn_perm(e[1][d], e[0][d], sel);
              w.y = __builtin_amdgcn_perm(e[3][d], e[2][d], sel);
              w.z = __builtin_amdgcn_perm(e[5][d], e[4][d], sel);
              w.w = __builtin_amdgcn_perm(e[7][d], e[6][d], sel);
              acc[j] = product(operand(w), xo, acc[j]);
            }
            if constexpr (V == 12) __builtin_amdgcn_sched_barrier(0);
          });
        } else {
          uint4v xp[AHEAD ? 1 : NX];                         // (each live for two pieces)
          auto load_piece = [&](int c) {
#pragma unroll
            for (int h = c * HPC; h < (c + 1) * HPC; ++h) xp[h] = load_x(p.n_out + pos * V + 8 * h);
          };
          if constexpr (!AHEAD) load_piece(0);
          for_each<8 / EPC>([&](auto piece) {
            constexpr int c = decltype(piece)::value;
            half8 xo[HPC];
            if constexpr (AHEAD) {
#pragma unroll
              for (int h = 0; h < HPC; ++h) xo[h] = operand(xw[c * HPC + h]);
            } else {
              if constexpr (c + 1 < 8 / EPC) load_piece(c + 1);
              else
#pragma unroll
                for (int i = 0; i < RB; ++i) load_window(far[i], i, s1);
              __builtin_amdgcn_sched_barrier(0);
              if (last)
#pragma unroll
                for (int h = c * HPC; h < (c + 1) * HPC; ++h) xp[h] = cut(xp[h], x_limit - (p.n_out + pos * V + 8 * h));
#pragma unroll
              for (int h = 0; h < HPC; ++h) xo[h] = operand(xp[c * HPC + h]);
            }
            if (table == 0 && want_xs)
#pragma unroll
              for (int h = 0; h < HPC; ++h) xacc = product(ones, xo[h], xacc);
#pragma unroll
            for (int i = 0; i < RB; ++i) {
              unsigned flat[EPC * VD];
#pragma unroll
              for (int q = 0; q < EPC; ++q) {
                unsigned e[ED];
                read(e, entry_of(win[i], c * EPC + q), c * EPC + q);
#pragma unroll
                for (int d = 0; d < VD; ++d) flat[q * VD + d] = e[d];
              }
#pragma unroll
              for (int h = 0; h < HPC; ++h) acc[i] = product(operand(uint4v{flat[4 * h], flat[4 * h + 1], flat[4 * h + 2], flat[4 * h + 3]}), xo[h], acc[i]);
            }
          });
        }
#pragma unroll
        for (int i = 0; i < RB; ++i)
#pragma unroll
          for (int d = 0; d < ND; ++d) {
            if constexpr (AHEAD) { win[i][d] = next[i][d]; next[i][d] = far[i][d]; }
            else win[i][d] = far[i][d];
          }
        if constexpr (AHEAD)
#pragma unroll
          for (int h = 0; h < NX; ++h) xw[h] = xn[h];
      }
    }
  }

  // ---- outlier columns (vectors of four, a table of up to 64 K entries): looked up through the caches
  if (p.Q && (!parts || part == 0)) {
    for (int c0 = wave * WIDTH; c0 < p.n_out; c0 += RW * WIDTH) {
      const int c = c0 + lead;
      const half8 xo = operand(cut(load_x(c), p.n_out - c));
      if (want_xs) xacc = product(ones, xo, xacc);
      if constexpr (DOWN) {
        for_each<V>([&](auto element) {
          constexpr int j = decltype(element)::value;
          const int o = min(stream[0] * V + j, p.out_features - 1), so = o / 4, jo = o & 3;
          unsigned h[8];
#pragma unroll
          for (int u = 0; u < 8; ++u) {
            h[u] = 0u;
            if (c + u < p.n_out) {
              const unsigned i = min(load_index(p.idx_out + (long long)so * p.stride_out, c + u, p.bits_out), (unsigned)p.k_out - 1u);
              h[u] = __half_as_ushort(p.cb_out[i * 4u + jo]);
            }
          }
          acc[j] = product(operand(uint4v{h[0] | h[1] << 16, h[2] | h[3] << 16, h[4] | h[5] << 16, h[6] | h[7] << 16}), xo, acc[j]);
          __builtin_amdgcn_sched_barrier(0);
        });
      } else {
#pragma unroll
        for (int i = 0; i < RB; ++i) {
          uint4v w = {0u, 0u, 0u, 0u};
#pragma unroll
          for (int u = 0; u < 2; ++u) {
            const int q = (c >> 2) + u;
            if (q < p.Q) {
              const unsigned e = min(load_index(p.idx_out + (long long)stream[i] * p.stride_out, q, p.bits_out), (unsigned)p.k_out - 1u);
              const uint2v v = *reinterpret_cast<const uint2v *>(p.cb_out + e * 4u);
              if (u == 0) { w.x = v.x; w.y = v.y; } else { w.z = v.x; w.w = v.y; }
            }
          }
          acc[i] = product(operand(w), xo, acc[i]);
        }
      }
    }
  }

  // ---- the waves' sums, in wave order: [wave][unit][lane][4] in LDS, a unit for every 256 threads at a time; sum(x) first
  float *red = reinterpret_cast<float *>(lds);
  float xs = 0.0f;
  const int column = ((threadIdx.x & 255) >> 2 & 15) % STREAMS;      // the batch row of the sum that this thread adds up
  if (want_xs) {
    __syncthreads();
    if (lane < 16) red[wave * 16 + lane] = xacc[0];
    __syncthreads();
    for (int w = 0; w < RW; ++w)
#pragma unroll
      for (int f = 0; f < FOLDS; ++f) xs += red[w * 16 + f * STREAMS + column];
    if (parts && threadIdx.x < 16) {
      float sum = 0.0f;
      for (int w = 0; w < RW; ++w) sum += red[w * 16 + threadIdx.x];
      a.part_xs[part * 16 + threadIdx.x] = sum;
    }
  } else if (parts && blk0 == 0 && threadIdx.x < 16) {
    a.part_xs[part * 16 + threadIdx.x] = 0.0f;
  }
  constexpr int AT_ONCE = RW / 4;
  for_each<(NU + AT_ONCE - 1) / AT_ONCE>([&](auto round) {
    constexpr int u0 = decltype(round)::value * AT_ONCE, units = NU - u0 < AT_ONCE ? NU - u0 : AT_ONCE;
    __syncthreads();
#pragma unroll
    for (int u = 0; u < units; ++u) *reinterpret_cast<float4v *>(lds + (unsigned)(wave * units + u) * UNIT + (unsigned)lane * 16u) = acc[u0 + u];
    __syncthreads();
    const int u = threadIdx.x >> 8, e = threadIdx.x & 255;
    const bool first_fold = FOLDS == 1 || ((e >> 2 & 15) < STREAMS && 4 * (e >> 6) < STREAMS);
    if (u < units && column < a.batch && first_fold) {
      float sum = 0.0f;
#pragma unroll
      for (int w = 0; w < RW; ++w)
#pragma unroll
        for (int f = 0; f < FOLDS; ++f) sum += red[(w * units + u) * 256 + e + f * (20 * STREAMS)];      // (a fold is 5 STREAMS lanes behind the one before)
      const int row = 4 * (e >> 6) + (e & 3);              // e = 4 lane + r: result row 4 (lane >> 4) + r, column lane & 15
      const int str = (blk0 + (DOWN ? 0 : u0 + u)) * STREAMS + row, o = DOWN ? str * V + u0 + u : str;
      if (str < p.S && o < p.out_features) {
        if (parts) {
          a.part[((long long)part * a.batch + column) * p.out_features + o] = sum;
        } else {
          const float sc = p.scale ? __half2float(p.scale[o]) : 1.0f, bi = p.bias ? __half2float(p.bias[o]) : 0.0f;
          a.y[(long long)column * a.ldy + o] = __float2half_rn(__fmaf_rn(sc, sum, bi * xs));
        }
      }
    }
  });
}

// LDS of the larger table: whole pieces of 1 KB, and the entry of zeros
unsigned table_bytes(const Params &p) {
  const unsigned k = (unsigned)(p.k > p.k_res ? p.k : p.k_res), entry = (unsigned)entry_halfs(p.v) * 2u;
  return (k * entry + 1023u) / 1024u * 1024u + entry;
}

bool rows_pair(const Params &p) { return compiled_pair(p.v, p.bits, false) || (p.v == 8 && p.bits == 16); }

// Row blocks per workgroup (orientation 0: up to four) and its waves.  One round should cover the layer: sixteen waves a compute unit,
// in one workgroup, or, where there are more blocks than compute units and two tables fit, in two of eight.
struct Split { int rb, rw, wgs; };
Split rows_split(const Params &p) {
  const int blocks = (p.S + 15) / 16, cus = cu_count();
  Split t = {1, 16, blocks};
  if (blocks <= cus) return t;
  const bool two = p.bits == 16 || table_bytes(p) <= 80 * 1024;
  if (two) t.rw = 8;
  const int at_once = two ? 2 * cus : cus;
  if (p.orientation == 0) t.rb = (blocks + at_once - 1) / at_once;
  if (t.rb > 4) t.rb = 4;
  t.wgs = (blocks + t.rb - 1) / t.rb;
  return t;
}

template <int V, int BITS, bool DOWN, int RB, int RW, bool PERM = false, int LOG_FOLDS = 0>
int launch_one(const Params &p, const RowsArgs &a, hipStream_t s) {
  if constexpr (V == 12 && !PERM && LOG_FOLDS == 0) if (p.perm) return launch_one<V, BITS, DOWN, RB, RW, true>(p, a, s);
  auto kernel = gemv_rows_kernel<V, BITS, DOWN, RB, RW, PERM, LOG_FOLDS>;
  VQ_ALLOW_FULL_LDS(kernel);
  constexpr int NU = acc_units(V, DOWN, RB), AT_ONCE = RW / 4;
  const unsigned sums = RW * (NU < AT_ONCE ? NU : AT_ONCE) * UNIT;
  const unsigned table = BITS == 16 ? 0u : table_bytes(p);
  const int parts = a.parts_per_group ? a.parts_per_group * p.n_groups : 1;
  hipLaunchKernelGGL(kernel, dim3((unsigned)(a.row_wgs * parts)), dim3(RW * 64), table > sums ? table : sums, s, p, a);
  return hipGetLastError() == hipSuccess ? VQ_OK : VQ_ERR_HIP;
}

template <int V, int BITS>
int launch_pair(const Params &p, const RowsArgs &a, const Split &t, int folds, hipStream_t s) {
  if constexpr (V == 8 ? BITS == 16 : V == 4 || V == 6 ? BITS == 8 : true) {
    if (folds == 4) return p.orientation == 1 ? launch_one<V, BITS, true, 1, 16, false, 2>(p, a, s) : launch_one<V, BITS, false, 1, 16, false, 2>(p, a, s);
    if (folds == 2) return p.orientation == 1 ? launch_one<V, BITS, true, 1, 16, false, 1>(p, a, s) : launch_one<V, BITS, false, 1, 16, false, 1>(p, a, s);
  }
  constexpr bool TWO = BITS == 16 || V * (1 << BITS) * 2 < 80 * 1024;      // (pairs that never run eight waves need no such kernel)
  if (p.orientation == 1) {
    if constexpr (TWO) if (t.rw == 8) return launch_one<V, BITS, true, 1, 8>(p, a, s);
    return launch_one<V, BITS, true, 1, 16>(p, a, s);
  }
  if constexpr (TWO) if (t.rw == 8) switch (t.rb) {
    case 1: return launch_one<V, BITS, false, 1, 8>(p, a, s);
    case 2: return launch_one<V, BITS, false, 2, 8>(p, a, s);
    case 3: return launch_one<V, BITS, false, 3, 8>(p, a, s);
    default: return launch_one<V, BITS, false, 4, 8>(p, a, s);
  }
  if constexpr (V == 12) switch (t.rb) {
    case 2: return launch_one<V, BITS, false, 2, 16>(p, a, s);
    case 3: return launch_one<V, BITS, false, 3, 16>(p, a, s);
    case 4: return launch_one<V, BITS, false, 4, 16>(p, a, s);
  }
  return t.rb == 1 ? launch_one<V, BITS, false, 1, 16>(p, a, s) : VQ_ERR_UNSUPPORTED;
}

}  // namespace

// The kernel's loads of activations: rows that start on dwords, in stored order but for v = 12 (the setting that is stored permuted).
bool gemv_rows_takes(const Params &p, const __half *x, long long ldx, int batch) {
  return (!p.perm || p.v == 12) && (reinterpret_cast<uintptr_t>(x) & 3) == 0 && (batch == 1 || (ldx & 1) == 0) && batch * ldx < (1LL << 29);
}

// Layers of the compiled (v, index width) pairs whose streams and tables the kernel's loads fit: a residual table of the same index
// width, outlier vectors of four, codebook groups that start on windows, tables that fit LDS one at a time.
bool gemv_rows_applicable(const Params &p) {
  if (!rows_pair(p) || (p.k_res && p.bits_res != p.bits) || (p.Q && p.v_out != 4) || (p.n_groups > 1 && p.Pg % 8 != 0)) return false;
  if (p.n_out & 1) return false;
  const long long limit = 1LL << 31;                       // 32-bit byte offsets, with room for what lies past the ends
  if (p.S * p.stride >= limit || (p.k_res && p.S * p.stride_res >= limit)) return false;
  return p.bits == 16 || table_bytes(p) <= 160 * 1024;
}

// Parts per codebook group when there is a workspace; 0: none is wanted.  The kernel that adds the parts up costs 2 us: they have to
// save the waves more steps than that (v = 2, 640 x 2052, two steps a wave: 5.8 against 7.5 us with parts; v = 4, 256 x 19648, ten: 18
// against 10 us; v = 12, whose steps are longer, 12275 x 1728, vectors down the outputs, four: 18 against 13 us).  Codebook groups side
// by side save their tables' staging one after the other, as long as the compute units are not full without (12288 x 5760, four
// groups: 35 against 44 us).
int gemv_rows_parts(const Params &p) {
  const Split t = rows_split(p);
  const int cus = cu_count(), steps = (p.Pg + STEP - 1) / STEP, enough = p.v >= 8 ? 2 : 4;
  if (p.n_groups > 1 && (t.wgs * p.n_groups > cus + cus / 2 || p.n_groups > 256)) return 0;
  int parts = cus / (t.wgs * p.n_groups);
  if (parts > (steps + t.rw - 1) / t.rw) parts = (steps + t.rw - 1) / t.rw;
  if (p.n_groups == 1) return parts > 1 && steps > enough * t.rw ? parts : 0;
  return parts < 1 ? 1 : parts;
}

// Folds of the columns (LOG_FOLDS) that up to eight rows take in one launch; `parts`: in place of column parts.  A fold has half or a quarter of the steps
// and costs a start 0.3 or 1 us, so: not for the fewest steps, nor where the blocks are more than compute units then (two rounds: 4096 x 4096,
// v = 4, 8.1 -> 12.2 us).  Of 15 shapes (306 to 10944 columns) with each of five settings, four and eight rows, in us without and with two / four folds: vectors
// down the outputs, v = 8 / 65536, 1024 x 1024 12.9, 9.7 / 8.9, v = 12 with two tables 14.5, 12.0 / 12.3, v = 6 / 256 of 32 steps 7.5, 7.0 / 7.2, of 128 12.2, 9.5 / 9.2;
// along the rows, where operand B's loads grow with the folds, 1000 x 8000 14.0, 11.8 / 12.4, 14.9, 12.8 / 13.0, v = 4 9.3, 8.0 / 8.7, v = 2 10.3, 7.8 / 8.1,
// v = 6 eight rows 10.7, 11.0.  Parts have a second launch, but as many as there are compute units for: 4096 x 4096 down the outputs, v = 2, two parts
// 9.5, folds 7.5, v = 4, four parts 9.0, 8.1, v = 8 / 65536, eight parts 16.4, 17.9.  Settings that were not measured keep to one.
int gemv_rows_folds(const Params &p, int batch, bool parts) {
  const bool measured = p.v == 12 ? p.k_res != 0 : !p.k_res && (p.v == 8 ? p.bits == 16 : p.v == 4 || p.v == 6 ? p.bits == 8 : p.v == 2);
  if (!measured || p.n_groups > 1 || p.perm || batch > 8) return 1;
  const int steps = (p.P + STEP - 1) / STEP, blocks4 = (int)(((long long)p.S * 4 + 15) / 16);
  const bool room = blocks4 <= cu_count(), four = room && batch <= 4;
  if (((long long)p.S * 2 + 15) / 16 > cu_count()) return 1;
  constexpr int NONE = 1 << 30;
  int from2, from4, to2 = NONE, to4 = NONE;                // steps
  if (p.orientation == 1) {
    from2 = p.v >= 8 ? 10 : 17;
    from4 = p.v == 8 ? 24 : p.v == 12 ? 48 : 112;
    if (parts) {
      if (p.v >= 8) return 1;
      if (room) to2 = p.v == 2 ? 160 : p.v == 4 ? 120 : 115;      // (else there are four parts at most)
      to4 = p.v == 6 ? 200 : 350;                          // (v = 4, 1216 x 18816, 588 steps: parts 10.8, folds 13.6)
    }
  } else {
    from2 = p.v == 8 ? 12 : p.v == 12 ? 8 : p.v == 4 ? (batch > 4 ? 40 : 24) : p.v == 2 ? 14 : batch > 4 ? NONE : 18;
    from4 = p.v == 12 ? 24 : p.v == 8 ? 36 : NONE;
    if (parts) {
      if (batch > 4 || (p.v != 2 && p.v != 8)) return 1;
      if (p.v == 8) from2 = NONE;
    }
  }
  return four && steps >= from4 && steps <= to4 ? 4 : steps >= from2 && steps <= to2 ? 2 : 1;
}

size_t gemv_rows_workspace_bytes(const Params &p, int batch) {
  const size_t parts = (size_t)gemv_rows_parts(p) * (size_t)p.n_groups;
  return (parts * ((size_t)batch * (size_t)p.out_features + 16) * sizeof(float) + 255) / 256 * 256;
}

// parts_per_group = 0: y complete, in `folds` folds (0: gemv_rows_folds says).  Else the parts' sums into part [n_groups * parts_per_group][batch][out_features] and part_xs
// [..][16], for launch_groups_finish.
int launch_gemv_rows(const Params &p, const __half *x, long long ldx, int batch, __half *y, long long ldy, float *part, float *part_xs,
                     int parts_per_group, hipStream_t s, int folds) {
  const Split t = rows_split(p);
  if (!folds) folds = parts_per_group ? 1 : gemv_rows_folds(p, batch, false);
  RowsArgs a = {x, ldx, batch, y, ldy, part, part_xs, folds > 1 ? (int)(((long long)p.S * folds + 15) / 16) : t.wgs, parts_per_group};
#define VQ_PAIR(V, BITS) if (p.v == V && p.bits == BITS) return launch_pair<V, BITS>(p, a, t, folds, s);
  VQ_PAIR(2, 4) VQ_PAIR(4, 8) VQ_PAIR(6, 8) VQ_PAIR(8, 8) VQ_PAIR(4, 12) VQ_PAIR(8, 12) VQ_PAIR(12, 12) VQ_PAIR(8, 16)
#undef VQ_PAIR
  return VQ_ERR_UNSUPPORTED;
}

}  // namespace vq
