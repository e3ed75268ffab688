// The dense product of vq_gemm's restore-then-multiply route: Y = X * W^T with the FP16 W that vq_dequant has written to the
// caller's workspace (the paper's own prompt-phase scheme).
//
// A workgroup of four waves (2 x 2) owns 64 MB tokens x 64 NB channels, a wave 32 MB x 32 NB in blocks of
// v_mfma_f32_16x16x32_f16.  Both tiles come by asynchronous global->LDS copies, NST steps of 64 columns ahead, in 128-byte rows:
// whole cache lines (half as many L2 requests as with 64-byte rows).  The loop is pipelined by half steps: the operand reads
// of the next half step and the copies are issued between the products of the current one, and one barrier a step sits between
// its two halves.  A column count that is no multiple of 64 ends in a step whose missing chunks are fetched from past the end
// of the buffers, where copies read zeros.
//
// What bounds it: at 256 x 256 tiles the matrix cores, and their power.  2048 x 8192 x 8192 runs at 1.4 to 1.5 GHz with the
// matrix cores busy about 90% of the clocks, so energy counts: the 16x16x32 instruction in place of 32x32x16 took 219 -> 197 us at
// the same traffic (1395 TFLOP/s); before, issuing reads and copies between the products instead of ahead of them 250 -> 221 us
// (a wave that has its SIMD to itself issues nothing else meanwhile).  Deeper stages or other placements of the reads changed
// nothing.  The smaller tiles are bound by LDS traffic per product and, with few workgroups, by the latency of a step: 0.19 us for 64 x 64,
// so 16 such tiles of 8448 columns took 32 us on 16 compute units.  Then the columns are cut into parts (SPLIT), a workgroup to a tile and part,
// whose binary32 sums a second kernel adds up in their order: 704 x 8448, 64 tokens, with the restoring 38.8 -> 19.6 us.
#include "vq_gemm_tiles.hpp"
#include <algorithm>
#include <type_traits>
#include <utility>

namespace vq {

namespace {

using namespace gemm_tiles;

typedef float float4v __attribute__((ext_vector_type(4)));

struct DenseArgs {
  const __half *X; long long ldx; int tokens;
  const __half *W; long long ldw; int out_features, in_features;
  __half *Y; long long ldy;
  int gx, gy;                  // tiles along the channels and the tokens
  // CENTROIDS: W holds centroids, the residual ones in a second matrix w2 bytes behind (0: none), and y = scale * (W X) + bias * sum(X)
  unsigned w2;
  const __half *scale, *bias;
  const float *xsum;
  // SPLIT: a workgroup takes `per` steps of the columns, of which there are `parts`, and leaves its sums in partial[part][token][channel]
  float *partial;
  int parts, per;
};

constexpr int DBK = 64;                                                  // columns per step: 128-byte rows in LDS
template <int MB, int NB, int NST> constexpr unsigned dense_lds() { return NST * (MB + NB) * 64u * (DBK * 2u); }
template <int MB, int NB, int NST> constexpr int dense_workgroups() {     // per compute unit: one where the accumulators take half the registers
  return MB * NB >= 16 ? 1 : dense_lds<MB, NB, NST>() > 80 * 1024 ? 1 : dense_lds<MB, NB, NST>() > 40 * 1024 ? 2 : 4;
}

// 16 bytes of each lane, from byte `offset` of the buffer to 1 KB of LDS at `to`  (kept out of the template: the host pass does
// not accept the builtin where it has to instantiate it)
__device__ __forceinline__ void copy16(const __amdgpu_buffer_rsrc_t &from, unsigned char *to, unsigned offset) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(from, (__attribute__((address_space(3))) void *)to, 16, offset, 0, 0, 0);
}

// operand block I (blocks are 16 rows, 2 KB, apart) of the tile whose first one is at LDS byte address `at`.  The reads are issued
// from inline assembly, in program order, and waited for explicitly: left to itself the compiler gives both sets of operands the
// same registers and so has to issue a set's reads after the other set's products.
template <int I> __device__ __forceinline__ void read_block(half8 &f, unsigned at) {
  asm volatile("ds_read_b128 %0, %1 offset:%2" : "=&v"(f) : "v"(at), "n"(I * 2048) : "memory");
}

template <class F, int... I> __device__ __forceinline__ void static_for(F &&f, std::integer_sequence<int, I...>) { (f(std::integral_constant<int, I>{}), ...); }
template <int N, class F> __device__ __forceinline__ void static_for(F &&f) { static_for(f, std::make_integer_sequence<int, N>{}); }

__device__ __forceinline__ void keep_in_agprs(float4v &v) { asm volatile("" : "+a"(v)); }

template <int MB, int NB, int NST, bool CENTROIDS, bool SPLIT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(dense_workgroups<MB, NB, NST>(), dense_workgroups<MB, NB, NST>())))
void gemm_dense_kernel(DenseArgs a) {
  constexpr int TM = 64 * MB, TN = 64 * NB, PX = 2 * MB, PER = 2 * (MB + NB);      // copies of a wave and step: PX of the X tile, PER in all
  constexpr unsigned ROW = DBK * 2u, XTILE = TM * ROW, STAGE = (TM + TN) * ROW;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];   // [NST][X tile | W tile]
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = (wave >> 1) * (32 * MB), wn = (wave & 1) * (32 * NB);
  // Workgroups go round robin over the eight XCDs, each with an L2 of its own: an XCD takes a run of tiles, token tiles first,
  // whose W rows it then fetches once
  const int tiles = a.gx * a.gy * (SPLIT ? a.parts : 1), run = (tiles + 7) / 8, item = (int)(blockIdx.x & 7) * run + (int)(blockIdx.x >> 3);
  if (item >= tiles) return;
  const int part = SPLIT ? item / (a.gx * a.gy) : 0, tile = SPLIT ? item - part * (a.gx * a.gy) : item;
  const int n0 = tile / a.gy * TN, m0 = tile % a.gy * TM;
  const int wsteps = (a.in_features + DBK - 1) / DBK, first = SPLIT ? part * a.per : 0, all = CENTROIDS && a.w2 ? 2 * wsteps : wsteps, ksteps = SPLIT ? min(first + a.per, all) : all;
  // range-checked against the end of the last row: rows past the matrix read zeros
  const __amdgpu_buffer_rsrc_t r_x = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<__half *>(a.X), 0, (unsigned)(((long long)(a.tokens - 1) * a.ldx + a.in_features) * 2), 0x00020000);
  const __amdgpu_buffer_rsrc_t r_w = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<__half *>(a.W), 0, (unsigned)(((long long)(a.out_features - 1) * a.ldw + a.in_features) * 2) + (CENTROIDS ? a.w2 : 0u), 0x00020000);

  // A step's copies, 8 rows x 128 bytes each: byte offsets of the lane's 16-byte chunk at step 0.  LDS slot (r, cs) holds chunk
  // cs ^ (r / 2 mod 8): then the 16-byte chunks that a group of 16 lanes reads from consecutive rows fall into all 64 banks.
  const unsigned even = ((unsigned)lane & 7u) ^ ((unsigned)lane >> 4);      // the chunk in pieces of even number; ^ 4: odd
  unsigned from[PER];
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    const unsigned chunk = even ^ (i & 1 ? 4u : 0u);
    from[i] = i < PX ? (unsigned)(((long long)(m0 + (wave * PX + i) * 8 + (lane >> 3)) * a.ldx + chunk * 8) * 2)
                     : (unsigned)(((long long)(n0 + (wave * (PER - PX) + i - PX) * 8 + (lane >> 3)) * a.ldw + chunk * 8) * 2);
  }
  // byte offset of a step's columns; chunks past the last column, and the steps past the last one, go past the end of the
  // buffers (which end below 2 GiB: see the launcher), where copies read zeros and fetch nothing
  int steps_even = (a.in_features - (int)even * 8 + DBK - 1) / DBK, steps_odd = (a.in_features - (int)(even ^ 4u) * 8 + DBK - 1) / DBK;
  if constexpr (SPLIT) { steps_even = min(steps_even, ksteps); steps_odd = min(steps_odd, ksteps); }
  auto copy_piece = [&](int i, unsigned stage, unsigned step_even, unsigned step_odd, unsigned second) {
    unsigned char *to = smem + stage + (i < PX ? (unsigned)(wave * PX + i) * 1024u : XTILE + (unsigned)(wave * (PER - PX) + i - PX) * 1024u);
    copy16(i < PX ? r_x : r_w, to, from[i] + (i & 1 ? step_odd : step_even) + (CENTROIDS && i >= PX ? second : 0u));
  };
  // (the second matrix follows step by step, against the same columns of X; rows past the first read the second's: channels never stored)
  auto second_of = [&](int &kt) -> unsigned {
    if (!CENTROIDS || kt < wsteps) return 0u;
    kt = kt < ksteps ? kt - wsteps : 0x7fffff00;
    return a.w2;
  };
  // operand addresses: row (block base + lane & 15), whose swizzle depends on the lane only, chunk 4 h + (lane >> 4) of half h
  const unsigned lds0 = (unsigned)reinterpret_cast<size_t>((const __attribute__((address_space(3))) void *)smem);
  const unsigned half0 = lds0 + (unsigned)(lane & 15) * ROW + ((((unsigned)lane >> 4) ^ (((unsigned)lane >> 1) & 7u)) << 4), half1 = half0 ^ 64u;
  const unsigned x_base = (unsigned)wm * ROW, w_base = XTILE + (unsigned)wn * ROW;

  constexpr int AB = 2 * MB, BB = 2 * NB;      // blocks of 16 rows in the wave's tile
  float4v acc[AB][BB];
#pragma unroll
  for (int i = 0; i < AB; ++i)
#pragma unroll
    for (int c = 0; c < BB; ++c) acc[i][c] = float4v{0.0f, 0.0f, 0.0f, 0.0f};
  half8 a0[AB], b0[BB], a1[AB], b1[BB];
  auto operands_in = [&](half8 (&af)[AB], half8 (&bf)[BB]) {       // behind a wait: the values are there
#pragma unroll
    for (int i = 0; i < AB; ++i) settle(af[i]);
#pragma unroll
    for (int i = 0; i < BB; ++i) settle(bf[i]);
  };
  // The products of half a step (32 columns), with the operand reads of the next half (and, COPY, the copies of a step) issued
  // between them: a wave that has its SIMD to itself issues nothing else meanwhile, and a block of products keeps the matrix
  // core busy for 16 clocks, in which it can issue three instructions.
  auto half_step = [&](auto copies, const half8 (&af)[AB], const half8 (&bf)[BB], unsigned at, half8 (&an)[AB], half8 (&bn)[BB],
                       unsigned stage, int kt) {        // (kt: the step that is copied)
    constexpr bool COPY = decltype(copies)::value;
    constexpr int N = AB * BB, R = AB + BB;
    unsigned xa = at + x_base, wa = at + w_base;
    asm volatile("" : "+v"(xa), "+v"(wa));      // both addresses in registers of their own before the first read goes out
    const unsigned second = COPY ? second_of(kt) : 0u;
    const unsigned step_even = COPY ? (kt < steps_even ? (unsigned)kt * ROW : 0x80000000u) : 0u;
    const unsigned step_odd = COPY ? (kt < steps_odd ? (unsigned)kt * ROW : 0x80000000u) : 0u;
    static_for<N>([&](auto index) {
      constexpr int n = decltype(index)::value, i = n / BB, c = n % BB;
      acc[i][c] = __builtin_amdgcn_mfma_f32_16x16x32_f16(af[i], bf[c], acc[i][c], 0, 0, 0);
      static_for<R>([&](auto read) {
        constexpr int r = decltype(read)::value;
        if constexpr (r * N * 2 / (R * 3) == n) {
          if constexpr (r < AB) read_block<r>(an[r], xa);
          else read_block<r - AB>(bn[r - AB], wa);
        }
      });
      if constexpr (COPY) {
        static_for<PER>([&](auto piece) {
          constexpr int r = decltype(piece)::value;
          if constexpr (r * N / (PER * 2) == n) copy_piece(r, stage, step_even, step_odd, second);
        });
      }
      __builtin_amdgcn_sched_barrier(0);
    });
  };

  // Copies run NST steps ahead: step kt + NST goes to the stage that the barrier of step kt has freed.  A wave waits for its
  // own by count (PER per step), the barrier covers the others'.
  static_for<NST>([&](auto index) {
    constexpr int j = decltype(index)::value;
    int kt = first + j;
    const unsigned second = second_of(kt);
    const unsigned step_even = kt < steps_even ? (unsigned)kt * ROW : 0x80000000u, step_odd = kt < steps_odd ? (unsigned)kt * ROW : 0x80000000u;
    static_for<PER>([&](auto piece) { copy_piece(decltype(piece)::value, j * STAGE, step_even, step_odd, second); });
  });
  wait_vmem_at_most<(NST - 1) * PER>();
  step_barrier();
  {
    unsigned xa = half0 + x_base, wa = half0 + w_base;
    static_for<AB>([&](auto i) { read_block<decltype(i)::value>(a0[decltype(i)::value], xa); });
    static_for<BB>([&](auto i) { read_block<decltype(i)::value>(b0[decltype(i)::value], wa); });
  }
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  operands_in(a0, b0);
  unsigned stage = 0;
  for (int kt = first; kt < ksteps; ++kt) {
    const unsigned next = stage + STAGE == NST * STAGE ? 0u : stage + STAGE;
    half_step(std::false_type{}, a0, b0, half1 + stage, a1, b1, 0u, 0);
    // this wave's copies of step kt + 1 are in when no more are out than those of the steps after it
    wait_vmem_at_most<(NST - 2) * PER>();
    step_barrier();                                           // (waits for the operand reads above as well: they are LDS traffic)
    operands_in(a1, b1);
    // (past the last step these read a stage that nobody needs: the loop stays one straight line)
    half_step(std::true_type{}, a1, b1, half0 + next, a0, b0, stage, kt + NST);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    operands_in(a0, b0);
    stage = next;
  }
  if constexpr (MB * NB >= 16) {       // (the accumulators fill the AGPRs; left alone, the compiler moves blocks of them to VGPRs inside the loop)
#pragma unroll
    for (int i = 0; i < AB; ++i)
#pragma unroll
      for (int c = 0; c < BB; ++c) keep_in_agprs(acc[i][c]);
  }
  wait_vmem_at_most<0>();      // the copies issued past the last step write to LDS too: they end before the workgroup does

  // ---- store: a lane holds channel (lane & 15) of four tokens of block (i, c).  Range-checked 2-byte buffer stores with 32-bit
  // offsets: rows past the last token fall off the end of the buffer, channels past the last one are sent there on purpose.
  // (8-byte stores of four channels of a token, from the transposed product, were slower: 16 rows a store instead of 4.)
  if constexpr (SPLIT) {
    const __amdgpu_buffer_rsrc_t r_p = __builtin_amdgcn_make_buffer_rsrc(a.partial + (long long)part * a.tokens * a.out_features, 0,
                                                                        (unsigned)a.tokens * (unsigned)a.out_features * 4u, 0x00020000);
    const unsigned ldp4 = (unsigned)a.out_features * 4u, p_lane = (unsigned)(m0 + wm + 4 * (lane >> 4)) * ldp4 + (unsigned)(n0 + wn + (lane & 15)) * 4u;
#pragma unroll
    for (int i = 0; i < AB; ++i)
#pragma unroll
      for (int c = 0; c < BB; ++c) {
        const bool on = n0 + wn + c * 16 + (lane & 15) < a.out_features;
#pragma unroll
        for (int r = 0; r < 4; ++r)
          __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(acc[i][c][r]), r_p, on ? p_lane + (unsigned)(i * 16 + r) * ldp4 + (unsigned)(c * 64) : 0xFFFFFFF0u, 0, 0);
      }
    return;
  }
  const __amdgpu_buffer_rsrc_t r_y = __builtin_amdgcn_make_buffer_rsrc(a.Y, 0, (unsigned)(((long long)(a.tokens - 1) * a.ldy + a.out_features) * 2), 0x00020000);
  const unsigned ldy2 = (unsigned)a.ldy * 2u;
  const unsigned y_lane = (unsigned)(m0 + wm + 4 * (lane >> 4)) * ldy2 + (unsigned)(n0 + wn + (lane & 15)) * 2u;
  // (read ahead of the blocks: what the tile's channels need at once, what its tokens need one row of blocks early; one block
  // after the other took 25 us of a 256 x 256 tile (v = 6 with outlier columns, 13168 x 1216, 1382 tokens 176 -> 127 us), and all
  // sums at once crowd the accumulators out of their registers inside the steps (7760 x 8640, 1615 tokens 561 against 507))
  float scale[BB], bias[BB], xsum[4], xnext[4];
  int at = lane;                       // (addresses formed here: hoisted out of the loop over the steps they crowd the accumulators)
  asm volatile("" : "+v"(at));
  auto sums_of = [&](int i, float (&to)[4]) {
#pragma unroll
    for (int r = 0; r < 4; ++r) to[r] = a.xsum[min(m0 + wm + i * 16 + 4 * (at >> 4) + r, a.tokens - 1)];
  };
  if constexpr (CENTROIDS) {
#pragma unroll
    for (int c = 0; c < BB; ++c) {
      const int o = min(n0 + wn + c * 16 + (at & 15), a.out_features - 1);
      scale[c] = a.scale ? __half2float(a.scale[o]) : 1.0f;
      bias[c] = a.bias ? __half2float(a.bias[o]) : 0.0f;
    }
    sums_of(0, xnext);
  }
#pragma unroll
  for (int i = 0; i < AB; ++i) {
    if constexpr (CENTROIDS) {
#pragma unroll
      for (int r = 0; r < 4; ++r) xsum[r] = xnext[r];
      if (i + 1 < AB) sums_of(i + 1, xnext);
    }
#pragma unroll
    for (int c = 0; c < BB; ++c) {
      const int o = n0 + wn + c * 16 + (lane & 15);
      const bool o_on = o < a.out_features;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        float sum = acc[i][c][r];
        if constexpr (CENTROIDS) sum = __fmaf_rn(scale[c], sum, bias[c] * xsum[r]);
        const __half h = __float2half_rn(sum);
        __builtin_amdgcn_raw_buffer_store_b16((short)__half_as_ushort(h), r_y, o_on ? y_lane + (unsigned)(i * 16 + r) * ldy2 + (unsigned)(c * 32) : 0xFFFFFFF0u, 0, 0);
      }
    }
    asm volatile("" ::: "memory");
  }
}

// The parts' sums, in the order of the columns, a thread to a channel of a token.
__global__ __launch_bounds__(256) void gemm_dense_finish_kernel(DenseArgs a) {
  const int n = a.tokens * a.out_features, at = (int)blockIdx.x * 256 + (int)threadIdx.x;
  if (at >= n) return;
  float sum = 0.0f;
#pragma unroll 8
  for (int i = 0; i < a.parts; ++i) sum += a.partial[(long long)i * n + at];
  const int t = at / a.out_features;
  const int o = at - t * a.out_features;
  if (a.xsum) sum = __fmaf_rn(a.scale ? __half2float(a.scale[o]) : 1.0f, sum, (a.bias ? __half2float(a.bias[o]) : 0.0f) * a.xsum[t]);
  a.Y[t * a.ldy + o] = __float2half_rn(sum);
}

template <int MB, int NB, int NST, bool CENTROIDS, bool SPLIT = false>
int launch_tiles(DenseArgs a, hipStream_t s) {
  if constexpr (!CENTROIDS) if (a.xsum) return launch_tiles<MB, NB, NST, true, SPLIT>(a, s);
  auto kernel = gemm_dense_kernel<MB, NB, NST, CENTROIDS, SPLIT>;
  VQ_ALLOW_FULL_LDS(kernel);
  a.gx = (a.out_features + 64 * NB - 1) / (64 * NB);
  a.gy = (a.tokens + 64 * MB - 1) / (64 * MB);
  const long long tiles = (long long)a.gx * a.gy * (SPLIT ? a.parts : 1);
  if (tiles > (1 << 24)) return VQ_ERR_UNSUPPORTED;
  constexpr unsigned lds = dense_lds<MB, NB, NST>();
  hipLaunchKernelGGL(kernel, dim3((unsigned)((tiles + 7) / 8 * 8)), dim3(256), lds, s, a);
  if constexpr (SPLIT) hipLaunchKernelGGL(gemm_dense_finish_kernel, dim3((unsigned)((a.tokens * a.out_features + 255) / 256)), dim3(256), 0, s, a);
  return hipGetLastError() == hipSuccess ? VQ_OK : VQ_ERR_HIP;
}

// Tile shapes and what they cost, in microseconds at the clocks that full load leaves: a fixed part per round of workgroups, and per
// 64-column step with one or two workgroups on a compute unit.  Fitted to 60 random shapes (17 to 2048 tokens, 256 to 11008 channels,
// 512 to 11008 columns), whose times the sums below meet within 4% on average; the shapes of 64 x 192 in three stages to 192 x 192 to
// 130 others (45 to 2048 tokens, up to 28672 channels and 13824 columns).  Most products are one or two rounds of workgroups, and what a
// kind costs is how much of the last round it leaves empty: with the kinds 256 x 256, 256 x 192, 128 x 128, 64 x 192 in two
// stages, 64 x 128 and 64 x 64 alone the 130 took 2.9 % longer on average, 24 of them 3 to 37 % (1500 x 4096 x 4096: 63.6 -> 49.9 us
// in 256 tiles of 192 x 128; 900 x 8192 x 8192: 134 -> 116 in 256 of 128 x 256; 700 x 11008 x 4096: 75 -> 63 in 232 of 192 x 192;
// 200 x 11008 x 4096: 31.3 -> 29.4 in 232 of 64 x 192), and none more than 1.4 % less.  128 x 192 in two stages is not among
// them: 509 x 11008 x 4096 54.7 -> 50.9 us with W in the caches, but 3 % slower together with the restoring of W where W's memory is not.
// For the same reason 64 x 192 in three stages is not for a W past the caches, where 128 x 128, 2 % more by the sums below, is the faster one
// (v = 8 / 65536: 13016 x 7808, 169 tokens 145 -> 132 us, 7088 x 11712, 291 tokens 158 -> 141, 6768 x 10432, 395 tokens 137 -> 125; W in the caches, 40
// shapes: 4 % slower).
struct TileKind {
  int mb, nb, per_cu;
  float round, step[2];
  int (*launch)(DenseArgs, hipStream_t);
  bool later = false, cached = false;              // cached: only where W is in the caches
  int (*split)(DenseArgs, hipStream_t) = nullptr;  // the columns in parts
};
const TileKind kTiles[] = {
    {4, 4, 1, 9.9f, {1.12f, 0.0f}, launch_tiles<4, 4, 2, false>},  {2, 4, 1, 5.3f, {0.755f, 0.0f}, launch_tiles<2, 4, 3, false>, true},
    {3, 3, 1, 6.2f, {0.752f, 0.0f}, launch_tiles<3, 3, 3, false>, true}, {3, 2, 1, 5.3f, {0.545f, 0.0f}, launch_tiles<3, 2, 3, false>, true},
    {1, 3, 1, 4.0f, {0.375f, 0.0f}, launch_tiles<1, 3, 3, false>, true, true}, {4, 3, 1, 7.6f, {0.90f, 0.0f}, launch_tiles<4, 3, 2, false>},
    {2, 2, 1, 4.2f, {0.383f, 0.0f}, launch_tiles<2, 2, 3, false>, false, false, launch_tiles<2, 2, 3, false, true>}, {1, 3, 2, 2.1f, {0.478f, 0.767f}, launch_tiles<1, 3, 2, false>},
    {1, 2, 2, 2.3f, {0.273f, 0.558f}, launch_tiles<1, 2, 3, false>, false, false, launch_tiles<1, 2, 3, false, true>},
    {1, 1, 2, 1.2f, {0.190f, 0.384f}, launch_tiles<1, 1, 4, false>, false, false, launch_tiles<1, 1, 4, false, true>},
};

float tile_cost(const TileKind &t, int tokens, int out_features, int steps_of_64, int cus, int parts = 1) {
  const long long tiles = (long long)((tokens + 64 * t.mb - 1) / (64 * t.mb)) * ((out_features + 64 * t.nb - 1) / (64 * t.nb)) * parts;
  const long long most = (tiles + cus - 1) / cus, rounds = most / t.per_cu, rest = most % t.per_cu;
  const float steps = (float)((steps_of_64 + parts - 1) / parts);
  return (float)rounds * (t.round + steps * t.step[t.per_cu - 1]) + (rest ? t.round + steps * t.step[rest - 1] : 0.0f);
}

// The kind and the parts of the columns with which a product takes less than `least` us: by the same estimates, 3 us for the second launch, and the
// parts' way through the caches at 5 TB/s.  (With 1 us and more to gain: of 150 random calls of 17 to 1555 tokens 49 are cut, which takes 25 % off
// the whole vq_gemm in the geometric mean and makes none slower by more than 2 %: v = 6, 78 tokens, 624 x 10752 45.9 -> 21.8 us, 64 of
// 1024 x 4096 22.4 -> 15.5, of 4096 x 4096 32.1 -> 20.9; v = 12, 145 of 3200 x 6632 56.0 -> 43.3; 88 of 5696 x 9472 55.4 -> 55.8.  Of
// 110 with the centroids in W 44, 28 %: v = 4, 44 tokens, 632 x 7936 35.9 -> 14.2, v = 6 + 4096, 95 of 1216 x 7680 73.8 -> 47.2.  With two
// matrices 4 us and more: at 3.2 by the estimate, 81 of 2905 x 2304 took 41.5 -> 45.0.)
struct Cut {
  const TileKind *kind;
  int parts, per;
  float us;
  size_t bytes;                                    // of scratch with which the choice is this one
};
Cut cut_columns(int tokens, int out_features, int steps, size_t scratch_bytes, float least) {
  Cut best = {nullptr, 1, steps, least, 0};
  const size_t part_bytes = (size_t)tokens * (size_t)out_features * sizeof(float);
  if (part_bytes * 2 <= scratch_bytes)
    for (const TileKind &k : kTiles) {
      if (!k.split) continue;
      for (int n : {2, 3, 4, 6, 8, 12, 16, 24, 32}) {
        if (n > steps / 2 || part_bytes * (size_t)n > scratch_bytes) break;
        const int per = (steps + n - 1) / n, parts = (steps + per - 1) / per;
        const float us = tile_cost(k, tokens, out_features, steps, cu_count(), parts) + 3.0f + (float)((double)part_bytes * 2 * parts / 5e6);
        if (us < best.us) best = {&k, parts, per, us, part_bytes * (size_t)n};
      }
    }
  return best;
}

const TileKind *least_kind(int tokens, int out_features, int steps, bool cached) {
  const TileKind *best = &kTiles[sizeof(kTiles) / sizeof(kTiles[0]) - 1];
  for (const TileKind &k : kTiles)
    if ((cached || !k.cached) && tile_cost(k, tokens, out_features, steps, cu_count()) < tile_cost(*best, tokens, out_features, steps, cu_count())) best = &k;
  return best;
}
int steps_of(const Params &p, int matrices) { return (p.in_features + DBK - 1) / DBK * matrices; }
Cut cut_of(const TileKind &whole, int tokens, int out_features, int steps, int matrices, size_t scratch_bytes) {
  return cut_columns(tokens, out_features, steps, scratch_bytes, tile_cost(whole, tokens, out_features, steps, cu_count()) - (matrices > 1 ? 4.0f : 1.0f));
}

}  // namespace

bool dequant_leaves_cached(const Params &p, int product_tokens, int matrices);
bool gemm_dense_applicable(const Params &p) { return p.in_features % 8 == 0; }       // (16-byte chunks of W's rows)

// What launch_gemm_dense uses of `most` bytes of scratch for these tokens (0: the columns stay whole); with that much it makes the same choice.
// (A product that goes in several launches, of 2 GiB of X or W, has more tiles than any that is cut.)
size_t gemm_dense_scratch_bytes(const Params &p, int tokens, int matrices, size_t most) {
  if (!gemm_dense_applicable(p) || switches().dense >= 0) return 0;
  const int steps = steps_of(p, matrices);
  const Cut cut = cut_of(*least_kind(tokens, p.out_features, steps, dequant_leaves_cached(p, tokens, matrices)), tokens, p.out_features, steps, matrices, most);
  return cut.kind ? (cut.bytes + 255) / 256 * 256 : 0;
}

// The tile shape with the least estimated time, and with `scratch` (16-byte aligned, for the sums) the parts of the columns.  Switch
// dense=0 / =n: always the last one / number n of the list and whole columns, for tests.  With xsum, the
// sums of X's rows: W holds the layer's centroids (w2 bytes behind it those of the residual table), see DenseArgs.
int launch_gemm_dense(const Params &p, const __half *X, long long ldx, int tokens, __half *Y, long long ldy, const __half *Wd, long long ldw, hipStream_t s,
                      const float *xsum, unsigned w2, void *scratch, size_t scratch_bytes) {
  if (!gemm_dense_applicable(p)) return VQ_ERR_UNSUPPORTED;
  // Buffer offsets have 32 bits and the copies of missing chunks start 2 GiB up, so one launch covers at most 2 GiB of X and of W
  // and 4 GiB of Y (with room for a tile of rows past the end); more goes in several.
  const long long room = 1LL << 31, pad = 256;
  const long long most_tokens = std::min(room / (ldx * 2), (room * 2 - 4096) / (ldy * 2)) - pad, most_out = (room - w2) / (ldw * 2) - pad;
  if (most_tokens < 1 || most_out < 1) return VQ_ERR_UNSUPPORTED;
  const int force = switches().dense, matrices = w2 ? 2 : 1, steps = steps_of(p, matrices);
  const bool cached = dequant_leaves_cached(p, tokens, matrices);
  for (long long o = 0; o < p.out_features; o += most_out)
    for (long long t = 0; t < tokens; t += most_tokens) {
      const int nt = (int)std::min<long long>(most_tokens, tokens - t), no = (int)std::min<long long>(most_out, p.out_features - o);
      constexpr int kinds = sizeof(kTiles) / sizeof(kTiles[0]);
      const TileKind *best = force < 0 ? least_kind(nt, no, steps, cached) : &kTiles[force > 0 && force <= kinds ? force - 1 : kinds - 1];
      DenseArgs a = {X + t * ldx, ldx, nt, Wd + o * ldw, ldw, no, p.in_features, Y + t * ldy + o, ldy, 0, 0, w2,
                     p.scale ? p.scale + o : nullptr, p.bias ? p.bias + o : nullptr, xsum ? xsum + t : nullptr, static_cast<float *>(scratch), 1, steps};
      const Cut cut = scratch && force < 0 ? cut_of(*best, nt, no, steps, matrices, scratch_bytes) : Cut{};
      if (cut.kind) { a.parts = cut.parts; a.per = cut.per; }
      const int rc = cut.kind ? cut.kind->split(a, s) : best->launch(a, s);
      if (rc != VQ_OK) return rc;
    }
  return VQ_OK;
}

// Estimated time of launch_gemm_dense in microseconds, at least that of reading W at 4.5 TB/s (the route rules of vq_gemm compare
// it with other kernels').  For vq_gemv's kernels, which do not round W, against restoring (`against_rows`) the four later tile shapes do
// not count: that line stays where it was drawn, and with it the precision of a call (of 20000 random ones it would move one).
float gemm_dense_us(const Params &p, int tokens, bool against_rows) {
  float best = 1e30f;
  for (const TileKind &k : kTiles)
    if (!against_rows || !k.later) best = std::min(best, tile_cost(k, tokens, p.out_features, (p.in_features + DBK - 1) / DBK, cu_count()));
  return std::max(best, 3.0f + (float)((double)p.out_features * p.in_features * 2 / 4.5e6));
}

}  // namespace vq
