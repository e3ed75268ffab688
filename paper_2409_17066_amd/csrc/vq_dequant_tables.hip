// vq_dequant: one kernel for every setting with a compiled (v, index width) pair, both orientations, codebook groups, residual and
// outlier tables, any row alignment.  (Paper App. "Our Dequantization Implementation": the prompt phase restores the FP16 weights.)
// Arithmetic as everywhere: binary32 sum of main and residual centroid (Sec. 3.2.2), one binary32 fma with scale and bias, round to
// nearest even to binary16; the results are the same bits.
//
// Vectors along the row: a lane restores sixteen bytes of it at a time, and looks up exactly what they hold: whole vectors (v = 2, 4, 8),
// two thirds of one or two (v = 12); v = 6: one vector, twelve bytes, looked up as two dwords and one, with one store (as sixteen bytes it
// took four reads of a dword from two vectors, 11008 x 4096 with v6 + 4096 31 -> 28 us).  So a wave writes 1 KB (768 bytes) in one piece, or, where
// rows (or a codebook group's part of them) are shorter, the same of several rows.  Vectors down the outputs: a lane looks
// eight columns up and writes eight weights of each of the v rows.  The next item's indices are in flight meanwhile; along the rows they
// go to the other one of two sets of registers, so that nothing waits for the stores behind them (28 -> 26.5 us).  Tables sit in LDS
// as they are in memory, copied without passing through registers; of a residual table of 12-element vectors that does not fit beside
// the main one, the first two thirds (the others, and the 1 MiB table of 16-bit indices, are read through L2; W is then written past
// the caches, so that it does not push the table out: 11008 x 4096 with v = 12 / 4096 + 4096 38 -> 31 us, v = 8 / 65536 31 -> 28).  With
// codebook groups a workgroup serves one group.  Outlier columns (vectors of four) are extra workgroups of the same launch.
//
// W of more than 256 MiB, the memory-side cache, is written past the caches as well: 8192 x 28672 with v6 / 4096 145 -> 94 us, + 4096 162
// -> 105, v4 / 256 134 -> 94, down the outputs 114 -> 92 and 114 -> 89.  Below, what follows finds it there, and lines shared by two
// waves cost: 8192 x 8192 in four groups 29 us through the caches, 40 past them.
//
// What bounds it: writing W (6.8 TB/s on this card: 13 us for 11008 x 4096, and 3.5 of launch), with a table in memory the lookups.  v = 6
// along the rows: L1's address unit, to which a store of twelve bytes a lane is an access a lane: with two tables it is busy 34 of a compute
// unit's 47 thousand clocks, LDS with the lookups 20 (profiles/case_counters.txt).
// Measured there, along the rows / down the outputs, against the first kernels (strips and transposes in LDS, dword stores, a
// separate launch for outliers): v6 / 4096 20.3 / 17.2 us (20.4 / 18.9), + 4096 26.4 / 22 (36 / 26), + 256 and outliers 25.3 / 22
// (32 / 30), v4 and v6 / 256 18.5 / 17 (30 .. 33 / 58), v2 / 16 18 / 18 (45 / 72), v8 / 65536 30 / 30 (32 / 58),
// v12 / 4096 + 4096 30 / 22 (58 / 61), with 4 groups and outliers 38 / 34 (81 / 70), v6 with 4 groups 22 / 17 (32 / 92).
#include "vq_lds_tables.hpp"
#include <type_traits>
#include <utility>

namespace vq {

namespace {

using namespace lds_tables;

typedef unsigned uint4b __attribute__((ext_vector_type(4), aligned(2)));      // 16, 12 and 8 bytes at any half
typedef unsigned uint3b __attribute__((ext_vector_type(3), aligned(2)));
typedef unsigned uint2b __attribute__((ext_vector_type(2), aligned(2)));

constexpr int chunk_weights(int v) { return v == 6 ? 6 : 8; }      // of a row that a lane restores at a time

// Runs along the row that a wave takes at a time: two, to have enough loads and stores on their way; four left fewer, longer turns to
// share out (v6 + 4096, 11008 x 4096: 32 us at the time; 640 x 576: 4.7 instead of 4.2), and so do two of the quickest ones (v6 / 4096,
// 4096 x 4096: 11.1 us instead of 10.2; with a residual table one is slower, 28.4 instead of 26.4).
constexpr int runs_per_turn(int v, int bits, bool residual) { return v == 6 && bits == 12 && !residual ? 1 : 2; }

enum Residual { NO_RES, RES_LDS, RES_MEM, RES_SPLIT };      // where the residual table is: RES_SPLIT, its first entries in LDS, the others in memory

struct DqArgs {
  __half *W; long long ldw;
  unsigned off_res, split;           // residual table in LDS, and how many of its entries (RES_SPLIT: an entry of zeros follows)
  int wgs, segments;                 // workgroups per codebook group; runs per row (items per stream) and group
  unsigned segments_inv;             // 2^32 / segments, rounded up
  int log_lanes;                     // lanes that share a row: 2^3 .. 2^6
  int wave_step, wg_step;            // between the first items of neighbouring waves and workgroups
  int out_wgs;                       // workgroups behind those that restore the outlier columns
};

template <int... I, class F> __device__ __forceinline__ void for_each(F &&f, std::integer_sequence<int, I...>) { (f(std::integral_constant<int, I>{}), ...); }
template <int N, class F> __device__ __forceinline__ void for_each(F &&f) { for_each(f, std::make_integer_sequence<int, N>{}); }

__device__ __forceinline__ void copy16(const __amdgpu_buffer_rsrc_t &from, unsigned char *to, unsigned offset) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(from, (__attribute__((address_space(3))) void *)to, 16, offset, 0, 0, 0);
}
__device__ __forceinline__ unsigned load4(const __amdgpu_buffer_rsrc_t &r, unsigned offset) { return __builtin_amdgcn_raw_buffer_load_b32(r, offset, 0, 0); }
__device__ __forceinline__ unsigned short load2(const __amdgpu_buffer_rsrc_t &r, unsigned offset) { return (unsigned short)__builtin_amdgcn_raw_buffer_load_b16(r, offset, 0, 0); }
__device__ __forceinline__ uint2v load8(const __amdgpu_buffer_rsrc_t &r, unsigned offset) { return __builtin_bit_cast(uint2v, __builtin_amdgcn_raw_buffer_load_b64(r, offset, 0, 0)); }
__device__ __forceinline__ uint4v load16(const __amdgpu_buffer_rsrc_t &r, unsigned offset) { return __builtin_bit_cast(uint4v, __builtin_amdgcn_raw_buffer_load_b128(r, offset, 0, 0)); }

template <bool STREAM> __device__ __forceinline__ void store12(__half *to, const unsigned (&w)[3]) {
  if constexpr (STREAM) __builtin_nontemporal_store((uint3b{w[0], w[1], w[2]}), reinterpret_cast<uint3b *>(to));
  else *reinterpret_cast<uint3b *>(to) = uint3b{w[0], w[1], w[2]};
}
template <bool STREAM> __device__ __forceinline__ void store16(__half *to, const unsigned (&w)[4]) {
  if constexpr (STREAM) __builtin_nontemporal_store((uint4b{w[0], w[1], w[2], w[3]}), reinterpret_cast<uint4b *>(to));
  else *reinterpret_cast<uint4b *>(to) = uint4b{w[0], w[1], w[2], w[3]};
}

// two weights from the halves of e (and f)
template <bool ADD> __device__ __forceinline__ unsigned restore_pair(unsigned e, unsigned f, float s0, float b0, float s1, float b1) {
  float d0 = __half2float(__ushort_as_half((unsigned short)e)), d1 = __half2float(__ushort_as_half((unsigned short)(e >> 16)));
  if (ADD) {
    d0 = __fadd_rn(d0, __half2float(__ushort_as_half((unsigned short)f)));
    d1 = __fadd_rn(d1, __half2float(__ushort_as_half((unsigned short)(f >> 16))));
  }
  return (unsigned)__half_as_ushort(restore(d0, s0, b0)) | (unsigned)__half_as_ushort(restore(d1, s1, b1)) << 16;
}

// The indices of up to three neighbouring vectors or so: N BITS bits in the one dword (ONE: they never straddle) or two that hold them.
template <int N, int BITS, bool ONE> struct Run {
  unsigned lo, hi;
  __device__ __forceinline__ void load(const __amdgpu_buffer_rsrc_t &r, unsigned row, unsigned vector) {
    const unsigned at = row + (vector * BITS >> 5) * 4u;
    if constexpr (ONE) { lo = load4(r, at); hi = 0u; }
    else { const uint2v v = load8(r, at); lo = v.x; hi = v.y; }
  }
  __device__ __forceinline__ void align(unsigned vector) {
    const unsigned sh = vector * BITS & 31u;
    if constexpr (ONE) { if constexpr (N * BITS < 32) lo >>= sh; }
    else lo = __builtin_amdgcn_alignbit(hi, lo, sh);
  }
  template <int U> __device__ __forceinline__ unsigned field() const {
    static_assert((U + 1) * BITS <= 32, "indices of a chunk fit a dword");
    return U * BITS + BITS == 32 ? lo >> (U * BITS) : lo >> (U * BITS) & ((1u << BITS) - 1u);
  }
};

// entry of a [k][V] table in memory, padded to ED dwords as in LDS
template <int V, int ED> __device__ __forceinline__ void memory_entry(unsigned (&e)[ED], const __half *table, unsigned i) {
  const unsigned *src = reinterpret_cast<const unsigned *>(table) + (long long)i * (V / 2);
#pragma unroll
  for (int d = 0; d < ED; ++d) e[d] = 0u;
  if constexpr (V % 8 == 0) {
#pragma unroll
    for (int d = 0; d < V / 2; d += 4) { const uint4v a = *reinterpret_cast<const uint4v *>(src + d); e[d] = a.x; e[d + 1] = a.y; e[d + 2] = a.z; e[d + 3] = a.w; }
  } else if constexpr (V % 4 == 0) {
#pragma unroll
    for (int d = 0; d < V / 2; d += 2) { const uint2v a = *reinterpret_cast<const uint2v *>(src + d); e[d] = a.x; e[d + 1] = a.y; }
  } else {
#pragma unroll
    for (int d = 0; d < V / 2; ++d) e[d] = src[d];
  }
}

// twelve bytes of LDS at any dword (two instructions, 22 clocks for 64 lookups; an aligned read of sixteen takes 13)
__device__ __forceinline__ void read_twelve(unsigned (&e)[3], const unsigned char *at) {
  typedef unsigned uint3d __attribute__((ext_vector_type(3), aligned(4)));
  const uint3d v = *reinterpret_cast<const uint3d *>(at);
  e[0] = v.x; e[1] = v.y; e[2] = v.z;
}

// a table as it is in memory, without passing through registers (waited for by the caller)
template <int V, int NW> __device__ __forceinline__ void stage_table(unsigned char *to, const __half *cb, int k) {
  const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(const_cast<__half *>(cb), 0, (unsigned)(k * V * 2), 0x00020000);
  for (unsigned at = (threadIdx.x >> 6) * 1024u; at < (unsigned)(k * V * 2); at += NW * 1024u) {
    const unsigned base = (unsigned)__builtin_amdgcn_readfirstlane((int)at);
    copy16(r, to + base, base + (threadIdx.x & 63u) * 16u);
  }
}

__device__ __forceinline__ float lane_value(float v, int lane) { return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), lane)); }
__device__ __forceinline__ unsigned third(unsigned n) { return __umulhi(n, 0xAAAAAAABu) >> 1; }      // n / 3


template <int V, int BITS, int RBITS, int RES, bool DOWN, int NW, bool STREAM>
__global__ __launch_bounds__(NW * 64, 4) void dequant_tables_kernel(Params p, DqArgs a) {
  constexpr bool MEM = BITS == 16, ADD = RES != NO_RES;
  constexpr int ED = DOWN && V == 6 ? 3 : entry_halfs(V) / 2;
  static_assert(V != 12 || RES != RES_MEM, "of a table of 12-element vectors two thirds always fit");
  extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  auto scale_of = [&](int o) { return p.scale ? __half2float(p.scale[o]) : 1.0f; };
  auto bias_of = [&](int o) { return p.bias ? __half2float(p.bias[o]) : 0.0f; };

  if ((int)blockIdx.x >= a.wgs * p.n_groups) {           // outlier columns: a wave per row (or stream of four rows) at a time
    for (int q = ((int)blockIdx.x - a.wgs * p.n_groups) * NW + wave; q < p.S_out; q += a.out_wgs * NW) {
      for (int c = lane; c < p.Q; c += 64) {
        const unsigned i = min(load_index(p.idx_out + (long long)q * p.stride_out, c, p.bits_out), (unsigned)p.k_out - 1u);
        const uint2v e = *reinterpret_cast<const uint2v *>(p.cb_out + i * 4u);
        if constexpr (DOWN) {
#pragma unroll
          for (int j = 0; j < 4; ++j)
            if (q * 4 + j < p.out_features) {
              const unsigned d = j < 2 ? e.x : e.y;
              a.W[(long long)(q * 4 + j) * a.ldw + c] = restore(__half2float(__ushort_as_half((unsigned short)(j & 1 ? d >> 16 : d))), scale_of(q * 4 + j), bias_of(q * 4 + j));
            }
        } else {
          const float s = scale_of(q), b = bias_of(q);
          *reinterpret_cast<uint2b *>(a.W + (long long)q * a.ldw + c * 4) = uint2b{restore_pair<false>(e.x, 0u, s, b, s, b), restore_pair<false>(e.y, 0u, s, b, s, b)};
        }
      }
    }
    return;
  }

  const int group = (int)blockIdx.x / a.wgs, wg = (int)blockIdx.x - group * a.wgs;
  const __half *cb = p.cb + (long long)group * p.k * V, *cb_res = ADD ? p.cb_res + (long long)group * p.k_res * V : nullptr;
  const int p_lo = group * p.Pg, p_hi = min(p.P, p_lo + p.Pg);
  const __amdgpu_buffer_rsrc_t r_i = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t *>(p.idx), 0, (unsigned)((long long)p.S * p.stride), 0x00020000);
  const __amdgpu_buffer_rsrc_t r_r = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t *>(ADD ? p.idx_res : p.idx), 0, ADD ? (unsigned)((long long)p.S * p.stride_res) : 0u, 0x00020000);
  const unsigned k_max = (unsigned)p.k - 1u, kr_max = (unsigned)p.k_res - 1u;
  auto main_entry = [&](unsigned (&e)[ED], unsigned i) {
    if constexpr (MEM) memory_entry<V>(e, cb, i);
    else if constexpr (ED == 3) read_twelve(e, lds + i * 12u);
    else read_entry<V>(e, lds, i);
  };
  auto res_entry = [&](unsigned (&f)[ED], unsigned i) {
    if constexpr (RES == RES_MEM) memory_entry<V>(f, cb_res, i);
    else if constexpr (RES == RES_LDS && ED == 3) read_twelve(f, lds + a.off_res + i * 12u);
    else if constexpr (RES == RES_LDS) read_entry<V>(f, lds + a.off_res, i);
  };
  // RES_SPLIT: eight bytes at byte `at` of entry i; a lane finds them in LDS or in memory and zeros in the other place
  const __amdgpu_buffer_rsrc_t r_cb = __builtin_amdgcn_make_buffer_rsrc(const_cast<__half *>(ADD ? cb_res : cb), 0, ADD ? (unsigned)(p.k_res * V * 2) : 0u, 0x00020000);
  auto split_read = [&](unsigned i, unsigned at) {
    const uint2v near = *reinterpret_cast<const uint2v *>(lds + a.off_res + min(i, a.split) * (V * 2u) + at);
    const uint2v far = load8(r_cb, i < a.split ? 0x80000000u : i * (V * 2u) + at);
    return uint2v{near.x | far.x, near.y | far.y};
  };
  // (segments > 1 only with whole waves to a row: rows * segments^2 < 2^32, which the launcher sees to)
  auto by_segments = [&](unsigned n) { return a.segments == 1 ? n : __umulhi(n, a.segments_inv); };

  auto per_output = [&](const __half *values) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<__half *>(values ? values : p.cb), 0, values ? (unsigned)p.out_features * 2u : 0u, 0x00020000);
  };

  if constexpr (!DOWN) {
    // a lane's chunk: CW weights from N vectors
    constexpr int SUB = runs_per_turn(V, BITS, ADD), CW = chunk_weights(V), CD = CW / 2, N = V == 6 ? 1 : V == 12 ? 2 : 8 / V, RB_ = RBITS ? RBITS : 8;
    constexpr bool ONE = N == 1 && BITS != 12, RONE = N == 1 && RB_ != 12;      // (a group may begin at any vector)
    const unsigned lanes = 1u << a.log_lanes, rows_per_run = 64u >> a.log_lanes, row_lane = (unsigned)lane >> a.log_lanes, chunk_lane = (unsigned)lane & (lanes - 1u);
    const unsigned runs = (((unsigned)p.S + rows_per_run - 1u) >> (6 - a.log_lanes)) * (unsigned)a.segments;
    const unsigned items = (runs + SUB - 1) / SUB;
    const unsigned stride_items = (unsigned)a.wgs * NW;      // (neighbouring waves write neighbouring parts of W)
    const int weights = (int)min((long long)(p_hi - p_lo) * V, (long long)p.in_features - p.n_out - (long long)p_lo * V);      // of a row in this group
    struct Turn { Run<N, BITS, ONE> idx[SUB]; Run<N, RB_, RONE> res[ADD ? SUB : 1]; unsigned short s[SUB], b[SUB]; } even, odd;
    auto place = [&](unsigned item, int u, unsigned &o, unsigned &c) {      // the lane's row and chunk
      const unsigned run = min(item * SUB + u, runs - 1u), rb = by_segments(run);
      o = rb * rows_per_run + row_lane;
      c = (run - rb * (unsigned)a.segments) * lanes + chunk_lane;
    };
    auto first_vector = [](unsigned c) -> unsigned { return V == 6 ? c : V == 12 ? third(2u * c) : c * (8 / V); };
    // Waits go by count, and the compiler counts what every path issues: so the same loads always, also without scale or bias (zeros)
    // and behind a wave's last item (the same again); and two sets of registers in turn, because a copy would be waited for.
    const __amdgpu_buffer_rsrc_t r_s = per_output(p.scale), r_b = per_output(p.bias);
    auto load = [&](Turn &t, unsigned item) {
#pragma unroll
      for (int u = 0; u < SUB; ++u) {
        unsigned o, c;
        place(item, u, o, c);
        o = min(o, (unsigned)p.S - 1u);
        const unsigned v = (unsigned)p_lo + first_vector(c);
        t.idx[u].load(r_i, o * (unsigned)p.stride, v);       // (past a row's end: the next row's bits, or zeros; never stored)
        if constexpr (ADD) t.res[u].load(r_r, o * (unsigned)p.stride_res, v);
        t.s[u] = load2(r_s, o * 2u);
        t.b[u] = load2(r_b, o * 2u);
      }
    };
    const unsigned first = (unsigned)wave * (unsigned)a.wave_step + (unsigned)wg * (unsigned)a.wg_step;
    if (first < items) load(even, first);
    if constexpr (!MEM) {
      stage_table<V, NW>(lds, cb, p.k);
      if constexpr (RES == RES_LDS) stage_table<V, NW>(lds + a.off_res, cb_res, p.k_res);
      if constexpr (RES == RES_SPLIT) stage_table<V, NW>(lds + a.off_res, cb_res, (int)a.split);
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      __syncthreads();
      if constexpr (RES == RES_SPLIT) {
        if (threadIdx.x < V / 2) reinterpret_cast<unsigned *>(lds + a.off_res)[a.split * (V / 2) + threadIdx.x] = 0u;
        __syncthreads();
      }
    }
    // the chunk's dwords of a table
    auto chunk_of = [&](unsigned (&w)[CD], const unsigned char *table, auto &run, unsigned last, unsigned c) {
      auto get1 = [&](unsigned at) { return *reinterpret_cast<const unsigned *>(table + at); };
      if constexpr (V == 6) {
        read_twelve(w, table + min(run.template field<0>(), last) * 12u);
      } else if constexpr (V == 12) {
        const unsigned part = 2u * c - 3u * third(2u * c), e0 = min(run.template field<0>(), last) * 24u, e1 = min(run.template field<1>(), last) * 24u;
        const uint2v x = *reinterpret_cast<const uint2v *>(table + e0 + 8u * part), y = *reinterpret_cast<const uint2v *>(table + (part < 2u ? e0 + 8u * part + 8u : e1));
        w[0] = x.x; w[1] = x.y; w[2] = y.x; w[3] = y.y;
      } else if constexpr (V == 8) {
        const uint4v x = *reinterpret_cast<const uint4v *>(table + min(run.template field<0>(), last) * 16u);
        w[0] = x.x; w[1] = x.y; w[2] = x.z; w[3] = x.w;
      } else if constexpr (V == 4) {
        const uint2v x = *reinterpret_cast<const uint2v *>(table + min(run.template field<0>(), last) * 8u), y = *reinterpret_cast<const uint2v *>(table + min(run.template field<1>(), last) * 8u);
        w[0] = x.x; w[1] = x.y; w[2] = y.x; w[3] = y.y;
      } else {
        for_each<4>([&](auto q) { w[decltype(q)::value] = get1(min(run.template field<decltype(q)::value>(), last) * 4u); });
      }
    };
    auto restore_turn = [&](Turn &t, unsigned item) {
#pragma unroll
      for (int u = 0; u < SUB; ++u) {
        unsigned o, c;
        place(item, u, o, c);
        const unsigned v = (unsigned)p_lo + first_vector(c);
        const float s = p.scale ? __half2float(__ushort_as_half(t.s[u])) : 1.0f, b = __half2float(__ushort_as_half(t.b[u]));
        unsigned e[CD], f[CD], w[CD];
        t.idx[u].align(v);
        if constexpr (MEM) chunk_of(e, reinterpret_cast<const unsigned char *>(cb), t.idx[u], k_max, c);
        else chunk_of(e, lds, t.idx[u], k_max, c);
        if constexpr (ADD) {
          t.res[u].align(v);
          if constexpr (RES == RES_SPLIT) {
            const unsigned part = 2u * c - 3u * third(2u * c), i0 = min(t.res[u].template field<0>(), kr_max), i1 = min(t.res[u].template field<1>(), kr_max);
            const uint2v x = split_read(i0, 8u * part), y = split_read(part < 2u ? i0 : i1, part < 2u ? 8u * part + 8u : 0u);
            f[0] = x.x; f[1] = x.y; f[2] = y.x; f[3] = y.y;
          } else if constexpr (RES == RES_MEM) chunk_of(f, reinterpret_cast<const unsigned char *>(cb_res), t.res[u], kr_max, c);
          else chunk_of(f, lds + a.off_res, t.res[u], kr_max, c);
        }
#pragma unroll
        for (int d = 0; d < CD; ++d) w[d] = restore_pair<ADD>(e[d], ADD ? f[d] : 0u, s, b, s, b);
        const int n = o < (unsigned)p.S && item * SUB + u < runs ? weights - CW * (int)c : 0;      // weights of the chunk that exist
        __half *to = a.W + (long long)o * a.ldw + p.n_out + (long long)p_lo * V + CW * (int)c;
        if (n >= CW) {
          if constexpr (CW == 6) store12<STREAM>(to, w);
          else store16<STREAM>(to, w);
        }
        else if (n > 0) {
#pragma unroll
          for (int j = 0; j < CW; ++j)
            if (j < n) to[j] = __ushort_as_half((unsigned short)(w[j >> 1] >> (j & 1) * 16));
        }
      }
    };
    if constexpr (V == 12) {                                 // (whose lookups are the bound: in turn, 3001 x 1501 took 9.4 us instead of 9.0)
      for (unsigned item = first; item < items; item += stride_items) {
        odd = even;
        if (item + stride_items < items) load(even, item + stride_items);
        restore_turn(odd, item);
      }
    } else if (items <= stride_items) {                      // no wave has two
      if (first < items) restore_turn(even, first);
    } else {
      auto after = [&](unsigned item) { return item + stride_items < items ? item + stride_items : item; };
      for (unsigned item = first; item < items;) {
        load(odd, after(item));
        restore_turn(even, item);
        if ((item += stride_items) >= items) return;
        load(even, after(item));
        restore_turn(odd, item);
        item += stride_items;
      }
    }
  } else {
    constexpr int ND = BITS / 4, NR = ADD ? RBITS / 4 : 1, GO = V == 12 ? 2 : ED;
    const int p_base = p_lo & ~7;                            // (a group may begin anywhere: windows of eight columns do not)
    const unsigned items = (unsigned)p.S * (unsigned)a.segments, stride_items = (unsigned)a.wgs * NW;
    unsigned win[ND], next[ND], rwin[NR], rnext[NR];
    auto dwords = [](auto &w, const __amdgpu_buffer_rsrc_t &r, unsigned at) {
      constexpr int N = sizeof(w) / 4;
      if constexpr (N == 1) w[0] = load4(r, at);
      else if constexpr (N == 2) { const uint2v v = load8(r, at); w[0] = v.x; w[1] = v.y; }
      else if constexpr (N == 3) load_window<3>(w, r, at);
      else { const uint4v v = load16(r, at); w[0] = v.x; w[1] = v.y; w[2] = v.z; w[3] = v.w; }
    };
    // (the scales of the v rows: one in each of the first v lanes)
    auto load = [&](unsigned (&i)[ND], unsigned (&r)[NR], unsigned short &s, unsigned short &b, unsigned item) {
      const int q = (int)by_segments(item), pos = p_base + ((int)item - q * a.segments) * 512 + lane * 8, o = min(q * V + min(lane, V - 1), p.out_features - 1);
      s = p.scale ? __half_as_ushort(p.scale[o]) : (unsigned short)0x3C00u;
      b = p.bias ? __half_as_ushort(p.bias[o]) : (unsigned short)0;
      dwords(i, r_i, (unsigned)q * (unsigned)p.stride + (unsigned)(pos >> 3) * BITS);
      if constexpr (ADD) dwords(r, r_r, (unsigned)q * (unsigned)p.stride_res + (unsigned)(pos >> 3) * RBITS);
    };
    unsigned short scn = 0, bin = 0;
    const unsigned first = (unsigned)wave * (unsigned)a.wave_step + (unsigned)wg * (unsigned)a.wg_step;
    if (first < items) load(next, rnext, scn, bin, first);
    if constexpr (!MEM) {
      stage_table<V, NW>(lds, cb, p.k);
      if constexpr (RES == RES_LDS) stage_table<V, NW>(lds + a.off_res, cb_res, p.k_res);
      if constexpr (RES == RES_SPLIT) stage_table<V, NW>(lds + a.off_res, cb_res, (int)a.split);
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      __syncthreads();
      if constexpr (RES == RES_SPLIT) {
        if (threadIdx.x < V / 2) reinterpret_cast<unsigned *>(lds + a.off_res)[a.split * (V / 2) + threadIdx.x] = 0u;
        __syncthreads();
      }
    }
    for (unsigned item = first; item < items; item += stride_items) {
#pragma unroll
      for (int d = 0; d < ND; ++d) win[d] = next[d];
      if constexpr (ADD)
#pragma unroll
        for (int d = 0; d < NR; ++d) rwin[d] = rnext[d];
      const float sc = __half2float(__ushort_as_half(scn)), bi = __half2float(__ushort_as_half(bin));
      const int q = (int)by_segments(item), pos = p_base + ((int)item - q * a.segments) * 512 + lane * 8, n = p_hi - pos, skip = p_lo - pos;      // the window's columns of this group: [skip, n)
      if (item + stride_items < items) load(next, rnext, scn, bin, item + stride_items);
      unsigned ei[8], fi[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        ei[u] = min(window_field<BITS, ND>(win, u), k_max);
        if constexpr (ADD) fi[u] = min(window_field<RBITS ? RBITS : 8, NR>(rwin, u), kr_max);
      }
      for_each<ED / GO>([&](auto go) {
        constexpr int d0 = decltype(go)::value * GO;
        unsigned e[8][GO], f[8][GO];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          if constexpr (V == 12) {
            const uint2v m = *reinterpret_cast<const uint2v *>(lds + ei[u] * 24u + d0 * 4u);
            e[u][0] = m.x; e[u][1] = m.y;
            if constexpr (RES == RES_SPLIT) {
              const uint2v r = split_read(fi[u], d0 * 4u);
              f[u][0] = r.x; f[u][1] = r.y;
            } else if constexpr (RES == RES_LDS) {
              const uint2v r = *reinterpret_cast<const uint2v *>(lds + a.off_res + fi[u] * 24u + d0 * 4u);
              f[u][0] = r.x; f[u][1] = r.y;
            }
          } else {
            main_entry(e[u], ei[u]);
            if constexpr (ADD) res_entry(f[u], fi[u]);
          }
        }
#pragma unroll
        for (int j = 2 * d0; j < 2 * (d0 + GO) && j < V; ++j) {
          const int o = q * V + j, d = (j >> 1) - d0;
          if (o < p.out_features) {
            const float s = lane_value(sc, j), b = lane_value(bi, j);
            const unsigned sel = j & 1 ? 0x07060302u : 0x05040100u;
            unsigned w[4];
#pragma unroll
            for (int c = 0; c < 4; ++c)
              w[c] = restore_pair<ADD>(__builtin_amdgcn_perm(e[2 * c + 1][d], e[2 * c][d], sel), ADD ? __builtin_amdgcn_perm(f[2 * c + 1][d], f[2 * c][d], sel) : 0u, s, b, s, b);
            __half *to = a.W + (long long)o * a.ldw + p.n_out + pos;
            if (n >= 8 && skip <= 0) store16<STREAM>(to, w);
            else
#pragma unroll
              for (int c = 0; c < 8; ++c)
                if (c < n && c >= skip) to[c] = __ushort_as_half((unsigned short)(w[c >> 1] >> (c & 1) * 16));
          }
        }
      });
    }
  }
}

// Vectors of eight down the outputs, a 1 MiB table, and too few columns to give every wave above a run of 512 (most of the time is then
// the chain index - entry - store of one wave): a vector to a lane, a wave writes 128 bytes of each of eight rows.
__global__ __launch_bounds__(256) void dequant_down_lookup_kernel(Params p, __half *__restrict__ W, long long ldw, int wgs_per_stream) {
  const int stream = (int)blockIdx.x / wgs_per_stream, pos = ((int)blockIdx.x - stream * wgs_per_stream) * 256 + (int)threadIdx.x;
  if (pos >= p.P) return;
  const unsigned i = min((unsigned)reinterpret_cast<const unsigned short *>(p.idx + (long long)stream * p.stride)[pos], (unsigned)p.k - 1u);
  unsigned e[4];
  memory_entry<8>(e, p.cb + (long long)(pos / p.Pg) * p.k * 8, i);
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const int o = stream * 8 + j;
    if (o < p.out_features)
      W[(long long)o * ldw + pos] = restore(__half2float(__ushort_as_half((unsigned short)(e[j >> 1] >> (j & 1) * 16))), p.scale ? __half2float(p.scale[o]) : 1.0f,
                                            p.bias ? __half2float(p.bias[o]) : 0.0f);
  }
}

// Vectors of eight along the rows and a table of up to 65536 of them (1 MiB), in front of a product of many tokens: the table passes
// through LDS, a piece after the other, and every lane takes those of its sixteen vectors' entries that lie in the piece.  Two pieces of 5120
// entries: one is filled while the other is read; the workgroups start at different pieces.  A workgroup takes 16384 neighbouring
// vectors at a time, a wave 64 of them (1 KB of W).
// What bounds it: filling 1 MB of LDS a compute unit and turn, at the 11 TB/s that L2 gives all of them together: 24 us.  Entries read
// through L2 one by one bring lines of 128 bytes for sixteen: 48 us for two turns' vectors (8192 x 8192) by themselves, but behind and
// ahead of a long product, which leaves L2 without the table and the chip at its power limit, a call with new inputs is faster this way: 8192 x 8192
// at 1024 / 2048 tokens 189 -> 178 and 285 -> 276 us, 14336 x 4096 171 -> 162 and 264 -> 256, 8192 x 28672 654 -> 596 at 1024; one full turn is as good as
// two (8192 x 4096 99 -> 92 and 149 -> 142, 4096 x 8192 106 -> 103 and 155 -> 151).  At 300 tokens it is not faster (4096 x 4096 35 us through
// L2, 46), nor with turns that are not full (4096 x 11008, 5.6 M vectors, 2048 tokens: 267, 271): two of them have to be full to four fifths
// (13500 x 4096, 1024 tokens 167 -> 161), a single one to 15 / 16 (0.83 of one, 6800 x 4096 79 -> 82, 0.93, 7600 x 4096 equal, 0.96, 7900 x 4096
// 95 -> 91).  (The same call over and over, its streams in the caches, is 3 to 7 % slower.)
constexpr int MANY_TOKENS = 1024;
constexpr int PIECE = 5120, HELD = 16, PIECES_THREADS = 1024;

// Entries at bytes [from, from + PIECE * 16) of the table, which lie at `piece` in LDS, to those lanes whose byte `at` is among them; all
// lanes are active.  In one statement, the wait included: the compiler would wait for every read before the next.
__device__ __forceinline__ void read_piece(uint4v *e, const unsigned *at, unsigned from, unsigned piece) {
  unsigned t;
#define VQ_READ(E, I) "v_subrev_u32 %8, %17, %" I "\n\tv_cmpx_gt_u32 vcc, %18, %8\n\tv_add_u32 %8, %19, %8\n\tds_read_b128 %" E ", %8\n\ts_mov_b64 exec, -1\n\t"
  asm volatile(VQ_READ("0", "9") VQ_READ("1", "10") VQ_READ("2", "11") VQ_READ("3", "12") VQ_READ("4", "13") VQ_READ("5", "14") VQ_READ("6", "15") VQ_READ("7", "16")
               "s_waitcnt lgkmcnt(0)"
               : "+v"(e[0]), "+v"(e[1]), "+v"(e[2]), "+v"(e[3]), "+v"(e[4]), "+v"(e[5]), "+v"(e[6]), "+v"(e[7]), "=&v"(t)
               : "v"(at[0]), "v"(at[1]), "v"(at[2]), "v"(at[3]), "v"(at[4]), "v"(at[5]), "v"(at[6]), "v"(at[7]), "s"(from), "s"(PIECE * 16u), "s"(piece)
               : "vcc", "memory");
#undef VQ_READ
}

template <bool STREAM>
__global__ __launch_bounds__(PIECES_THREADS, 4) void dequant_pieces_kernel(Params p, __half *__restrict__ W, long long ldw, unsigned total, unsigned rows_inv) {
  extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
  constexpr unsigned BYTES = PIECE * 16u;
  const unsigned tid = threadIdx.x, lane = tid & 63u;
  const int wave = __builtin_amdgcn_readfirstlane((int)(tid >> 6));
  const unsigned lds0 = (unsigned)reinterpret_cast<size_t>((const __attribute__((address_space(3))) void *)lds);
  const unsigned P = (unsigned)p.P, n_pieces = ((unsigned)p.k + PIECE - 1) / PIECE, first_piece = blockIdx.x % n_pieces;
  const __amdgpu_buffer_rsrc_t r_cb = __builtin_amdgcn_make_buffer_rsrc(const_cast<__half *>(p.cb), 0, (unsigned)p.k * 16u, 0x00020000);
  const __amdgpu_buffer_rsrc_t r_i = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t *>(p.idx), 0, (unsigned)((long long)p.S * p.stride), 0x00020000);
  // row and position of a vector (rows_inv: 2^32 / P, rounded down; the quotient is short of one at most)
  auto place = [&](unsigned n, unsigned &o, unsigned &at) {
    o = __umulhi(n, rows_inv);
    at = n - o * P;
    if (at >= P) { ++o; at -= P; }
  };
  auto piece_of = [&](unsigned turn) { const unsigned c = first_piece + turn; return c < n_pieces ? c : c - n_pieces; };
  auto fill = [&](unsigned turn) {
    const unsigned from = piece_of(turn) * BYTES, to = (turn & 1u) * BYTES;
#pragma unroll
    for (unsigned at = 0; at < BYTES; at += PIECES_THREADS * 16u) copy16(r_cb, lds + to + at + wave * 1024u, from + at + (unsigned)wave * 1024u + lane * 16u);
  };
  static_assert(BYTES % (PIECES_THREADS * 16u) == 0, "whole rounds of all waves");
  for (unsigned base = blockIdx.x * (PIECES_THREADS * HELD); base < total; base += gridDim.x * (PIECES_THREADS * HELD)) {
    unsigned i[HELD];
    uint4v e[HELD];
#pragma unroll
    for (int u = 0; u < HELD; ++u) {
      unsigned o, at;
      place(min(base + u * PIECES_THREADS + tid, total - 1u), o, at);
      i[u] = load2(r_i, o * (unsigned)p.stride + at * 2u);
    }
    fill(0);
#pragma unroll
    for (int u = 0; u < HELD; ++u) {
      i[u] = min(i[u], (unsigned)p.k - 1u) * 16u;            // (as bytes of the table)
      e[u] = uint4v{0u, 0u, 0u, 0u};
    }
    for (unsigned turn = 0; turn < n_pieces; ++turn) {
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      __syncthreads();                                     // (the piece is in, and every wave is through with the other one)
      if (turn + 1 < n_pieces) fill(turn + 1);
      const unsigned from = piece_of(turn) * BYTES, piece = lds0 + (turn & 1u) * BYTES;
      read_piece(e, i, from, piece);
      read_piece(e + HELD / 2, i + HELD / 2, from, piece);
    }
    __syncthreads();                                       // (the next vectors' first piece goes where the last one was, or beside it)
#pragma unroll
    for (int u = 0; u < HELD; ++u) {
      const unsigned n = base + u * PIECES_THREADS + tid;
      if (n < total) {
        unsigned o, at;
        place(n, o, at);
        const float sc = p.scale ? __half2float(p.scale[o]) : 1.0f, bi = p.bias ? __half2float(p.bias[o]) : 0.0f;
        const unsigned w[4] = {restore_pair<false>(e[u].x, 0u, sc, bi, sc, bi), restore_pair<false>(e[u].y, 0u, sc, bi, sc, bi),
                               restore_pair<false>(e[u].z, 0u, sc, bi, sc, bi), restore_pair<false>(e[u].w, 0u, sc, bi, sc, bi)};
        store16<STREAM>(W + (long long)o * ldw + at * 8u, w);
      }
    }
  }
}

unsigned table_bytes(int v, int k) { return ((unsigned)k * (unsigned)v * 2u + 1023u) / 1024u * 1024u; }      // in LDS: whole pieces of 1 KB

// In front of a product W goes through the caches as long as they hold it beside the rest: v8 / 65536 at 300 tokens 4096 x 4096 43.8 -> 34.9 us,
// 11008 x 4096 102 -> 91, v12 / 4096 + 4096 2048 x 4096 28.8 -> 25.7; 8192 x 8192 at 300 tokens 141 -> 146, but at 2048 300 -> 290.  Not in front of
// a short product of very short rows: of less than 600 columns, 0.4 to 0.9 million vectors and up to 191 tokens most are slower through the
// caches, in a loop over eight layers by 4 % on average (v8 10520 x 576, 36 tokens 16.4 -> 17.7 us, v12 12312 x 576, 67 tokens 20.6 -> 23.2).  From
// there to 1216 columns such a loop takes the same either way, and a call with new inputs is faster through them by 9 % (v8 5022 x 720, 189
// tokens 14.1 -> 12.4, 6102 x 952, 44 tokens 16.0 -> 13.9, v12 5447 x 1072, 138 tokens 20.8 -> 19.0).
bool through_caches(const Params &p, int product_tokens) {
  const long long w_bytes = (long long)p.out_features * p.in_features * 2, vectors = (long long)p.S * p.P;
  if (product_tokens <= 0 || w_bytes > 192LL << 20) return false;
  if (p.in_features < 600 && product_tokens < 192 && vectors >= 3 << 17 && vectors < 7 << 17) return false;
  return w_bytes <= 96LL << 20 || product_tokens >= MANY_TOKENS;
}

template <auto KERNEL, int NW> int launch_kernel(dim3 grid, unsigned lds, hipStream_t s, const Params &p, const DqArgs &a) {
  VQ_ALLOW_FULL_LDS(KERNEL);
  hipLaunchKernelGGL(KERNEL, grid, dim3(NW * 64), lds, s, p, a);
  return VQ_OK;
}

template <int V, int BITS, int RBITS, int RES, bool DOWN>
int launch_one(const Params &p, __half *W, long long ldw, hipStream_t s, int product_tokens) {
  const long long w_bytes = (long long)p.out_features * p.in_features * 2;
  constexpr bool L2_LOOKUPS = BITS == 16 || RES == RES_MEM || RES == RES_SPLIT;
  const unsigned main = BITS == 16 ? 0u : table_bytes(V, p.k), bytes = RES == RES_SPLIT ? 160u * 1024u : main + (RES == RES_LDS ? table_bytes(V, p.k_res) : 0u);
  DqArgs a = {W, ldw, main, 0, 0, 1, 0, 6, 1, 0, 0};
  if (RES == RES_SPLIT) a.split = min((bytes - main) / (V * 2u) - 1u, (unsigned)p.k_res);
  long long items;
  if (DOWN) {
    a.segments = ((p.n_groups > 1 && p.Pg % 8 ? p.Pg + 7 : p.Pg) + 511) / 512;
    items = (long long)p.S * a.segments;
  } else {
    const long long chunks = ((long long)p.Pg * V + chunk_weights(V) - 1) / chunk_weights(V);
    while (a.log_lanes > 3 && chunks <= 1LL << (a.log_lanes - 1)) --a.log_lanes;
    a.segments = (int)((chunks + (1LL << a.log_lanes) - 1) >> a.log_lanes);
    items = (((long long)p.S + (64 >> a.log_lanes) - 1) / (64 >> a.log_lanes) * a.segments + runs_per_turn(V, BITS, RES != NO_RES) - 1) / runs_per_turn(V, BITS, RES != NO_RES);
  }
  a.segments_inv = (unsigned)(((1ULL << 32) + a.segments - 1) / a.segments);
  if (items > 0x1fffffffLL || (long long)p.S * a.segments * a.segments >= 1LL << 32) return VQ_ERR_UNSUPPORTED;
  if constexpr (DOWN && BITS == 16 && RES == NO_RES) {
    // 640 x 704: 4.0 us against 6.0; 747 x 3360 (658 runs) 6.7 against 7.7; 384 x 13888 (1344 runs) 10.6 against 8.6
    if (items < 4LL * cu_count() && !p.Q) {
      const int wgs_per_stream = (p.P + 255) / 256;
      hipLaunchKernelGGL(dequant_down_lookup_kernel, dim3((unsigned)(wgs_per_stream * p.S)), dim3(256), 0, s, p, W, ldw, wgs_per_stream);
      return hipGetLastError() == hipSuccess ? VQ_OK : VQ_ERR_HIP;
    }
  }
  if constexpr (!DOWN && V == 8 && BITS == 16 && RES == NO_RES) {
    const long long vectors = (long long)p.S * p.P, turn = (long long)PIECES_THREADS * HELD * cu_count();
    if (product_tokens >= MANY_TOKENS && p.n_groups == 1 && !p.Q && p.in_features == p.P * 8 && p.P > 1 && vectors < 1LL << 31 &&
        (vectors > turn ? vectors * 5 >= (vectors + turn - 1) / turn * turn * 4 : vectors * 16 >= turn * 15)) {      // (turns full to four fifths, a single one to 15 / 16)
      const unsigned n = (unsigned)vectors, inv = (unsigned)((1ULL << 32) / (unsigned)p.P);
      const unsigned rounds = (unsigned)((vectors + turn - 1) / turn), wg = (unsigned)((vectors + (long long)rounds * PIECES_THREADS * HELD - 1) / ((long long)rounds * PIECES_THREADS * HELD));
      auto run = [&](auto kernel) {
        VQ_ALLOW_FULL_LDS(kernel);
        hipLaunchKernelGGL(kernel, dim3(wg), dim3(PIECES_THREADS), 2u * PIECE * 16u, s, p, W, ldw, n, inv);
        return hipGetLastError() == hipSuccess ? VQ_OK : VQ_ERR_HIP;
      };
      return w_bytes > 192LL << 20 ? run(dequant_pieces_kernel<true>) : run(dequant_pieces_kernel<false>);
    }
  }
  // four workgroups of eight waves on a CU where the tables are small; else two or one of sixteen, which share them (32 x 1 KB of
  // stores in flight either way; 3 x 8 waves with a 48 KB table each spent longer staging)
  const bool small = bytes <= 40 * 1024;
  const int nw = small ? 8 : 16, slots = cu_count() * (small ? DOWN && RES != NO_RES ? 2 : 4 : bytes <= 80 * 1024 ? 2 : 1);
  long long wgs = (items + 1) / 2, most = (slots + p.n_groups - 1) / p.n_groups;
  if (wgs > most) wgs = most;
  a.wgs = (int)wgs;
  a.wg_step = nw;
  if (items <= wgs * nw) { a.wave_step = a.wgs; a.wg_step = 1; }      // no wave has two: every workgroup gets its share
  if (p.Q) a.out_wgs = (int)min((long long)(p.S_out + nw - 1) / nw, (long long)cu_count());
  const dim3 grid((unsigned)(wgs * p.n_groups + a.out_wgs));
  // past the caches: where lookups go through L2, from which W must not push the table; and where W is larger than they are
  // (down the outputs only if rows start on 64 bytes: with pieces of lines between them 8192 x 20480 took 103 us past the caches, 97 through)
  const bool through = through_caches(p, product_tokens);
  const uintptr_t starts = reinterpret_cast<uintptr_t>(W) | (uintptr_t)ldw * 2 | (uintptr_t)p.n_out * 2;
  const bool stream = (L2_LOOKUPS && !through && (starts & 15) == 0) || (w_bytes > 256LL << 20 && (!DOWN || (starts & 63) == 0));
  const int rc = small ? (stream ? launch_kernel<dequant_tables_kernel<V, BITS, RBITS, RES, DOWN, 8, true>, 8>(grid, bytes, s, p, a)
                                 : launch_kernel<dequant_tables_kernel<V, BITS, RBITS, RES, DOWN, 8, false>, 8>(grid, bytes, s, p, a))
                       : (stream ? launch_kernel<dequant_tables_kernel<V, BITS, RBITS, RES, DOWN, 16, true>, 16>(grid, bytes, s, p, a)
                                 : launch_kernel<dequant_tables_kernel<V, BITS, RBITS, RES, DOWN, 16, false>, 16>(grid, bytes, s, p, a));
  if (rc != VQ_OK) return rc;
  return hipGetLastError() == hipSuccess ? VQ_OK : VQ_ERR_HIP;
}

template <int V, int BITS, int RBITS>
int launch_pair(const Params &p, __half *W, long long ldw, hipStream_t s, int product_tokens) {
  if (!p.k_res) {
    if constexpr (RBITS == BITS) return p.orientation ? launch_one<V, BITS, 0, NO_RES, true>(p, W, ldw, s, product_tokens) : launch_one<V, BITS, 0, NO_RES, false>(p, W, ldw, s, product_tokens);
    else return VQ_ERR_UNSUPPORTED;
  }
  if constexpr (BITS == 16) {
    return p.orientation ? launch_one<V, BITS, RBITS, RES_MEM, true>(p, W, ldw, s, product_tokens) : launch_one<V, BITS, RBITS, RES_MEM, false>(p, W, ldw, s, product_tokens);
  } else {
    if (table_bytes(V, p.k) + table_bytes(V, p.k_res) <= 160 * 1024)
      return p.orientation ? launch_one<V, BITS, RBITS, RES_LDS, true>(p, W, ldw, s, product_tokens) : launch_one<V, BITS, RBITS, RES_LDS, false>(p, W, ldw, s, product_tokens);
    if constexpr (V == 12) return p.orientation ? launch_one<V, BITS, RBITS, RES_SPLIT, true>(p, W, ldw, s, product_tokens) : launch_one<V, BITS, RBITS, RES_SPLIT, false>(p, W, ldw, s, product_tokens);
    if constexpr (V == 8) return p.orientation ? launch_one<V, BITS, RBITS, RES_MEM, true>(p, W, ldw, s, product_tokens) : launch_one<V, BITS, RBITS, RES_MEM, false>(p, W, ldw, s, product_tokens);
    return VQ_ERR_UNSUPPORTED;
  }
}

}  // namespace

// Whether launch_dequant leaves W, or so many matrices of its size, in the caches for a product of so many tokens.
bool dequant_leaves_cached(const Params &p, int product_tokens, int matrices) {
  const long long w_bytes = (long long)p.out_features * p.in_features * 2 * matrices;
  const bool l2_lookups = p.bits == 16 || (p.k_res && table_bytes(p.v, p.k) + table_bytes(p.v, p.k_res) > 160 * 1024);
  return l2_lookups ? through_caches(p, product_tokens) : w_bytes <= 224LL << 20;      // (beside X, Y and the streams)
}

// The whole matrix in stored column order; VQ_ERR_UNSUPPORTED for (v, index width) pairs without a compiled kernel.
int launch_dequant_tables(const Params &p, __half *W, long long ldw, hipStream_t s, int product_tokens) {
  if (switches().dequant == 'g' || p.perm || (p.Q && p.v_out != 4)) return VQ_ERR_UNSUPPORTED;
  const long long limit = 1LL << 31;                       // 32-bit byte offsets, with room for what lies past the ends
  if (p.S * p.stride >= limit || (p.k_res && p.S * p.stride_res >= limit)) return VQ_ERR_UNSUPPORTED;
  const int rb = p.k_res ? p.bits_res : p.bits;
#define VQ_PAIR(V, BITS, RBITS) if (p.v == V && p.bits == BITS && rb == RBITS) return launch_pair<V, BITS, RBITS>(p, W, ldw, s, product_tokens);
  VQ_PAIR(2, 4, 4) VQ_PAIR(4, 8, 8) VQ_PAIR(6, 8, 8) VQ_PAIR(8, 8, 8) VQ_PAIR(4, 12, 12) VQ_PAIR(6, 12, 12) VQ_PAIR(6, 12, 8) VQ_PAIR(8, 12, 12)
  VQ_PAIR(12, 12, 12) VQ_PAIR(8, 16, 16) VQ_PAIR(8, 16, 8) VQ_PAIR(8, 8, 16)
#undef VQ_PAIR
  return VQ_ERR_UNSUPPORTED;
}

}  // namespace vq
