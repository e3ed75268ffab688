// vq_gemm fast path for v = 8 with 16-bit indices (k up to 65536: the codebook is 1 MiB and lives in
// L2 / Infinity Cache, not in LDS), no residual, no outlier columns -- the paper's v=8 / k=65536 setting
// (App. "Impact of Vector Length").  Y = X * W^T with W restored on the fly; W never touches memory.
//
// A workgroup owns BM tokens x 128 output channels and splits its waves in two roles that share the SIMDs:
//  * BM/64 "consumer" waves only issue MFMA: wave w owns token rows [64 w, 64 w + 64) and all 128 channels as
//    2 x 4 blocks of v_mfma_f32_32x32x16_f16, reading both operands from LDS;
//  * four "producer" waves keep the tiles coming: per 32-column step they gather 128 x 4 centroids
//    (16 bytes each, two per thread, issued GD steps ahead), apply scale and bias, write the FP16 W tile
//    to LDS (double buffered), and start the asynchronous global->LDS copies of the activation tile
//    XD steps ahead (XOR-swizzled 64-byte rows).
// One barrier per step.  The taller the token tile, the fewer times a centroid is gathered: each gather
// pulls a whole 128-byte line out of L2 for 16 useful bytes, which is what finally bounds this kernel.
#include "vq_gemm_tiles.hpp"
#include <cstdlib>

namespace vq {

namespace {

using namespace gemm_tiles;

// in_features % 32 == 0 here.  Wave w owns token rows [w*BM/4, (w+1)*BM/4) and all 128 channels.
template <int BM>
__global__ __launch_bounds__((BM / 64 + 4) * 64) void gemm_v8_kernel(Params p, const __half *__restrict__ X, long long ldx, int tokens,
                                                      __half *__restrict__ Y, long long ldy) {
  constexpr int NC = BM / 64;                   // consumer waves: each owns 64 token rows x 128 channels
  constexpr int MB = 2;                         // 32-row MFMA blocks per consumer wave along the tokens
  constexpr unsigned XSTAGE = BM * 64u;         // bytes per activation stage
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  unsigned char *Xs = smem;                                                        // [NSX][BM][64 bytes]
  __half *Ws = reinterpret_cast<__half *>(smem + NSX * XSTAGE);                    // [2][BN][LDT]

  const int lane = threadIdx.x & 63;
  const int wave8 = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const bool producer = wave8 >= NC;
  const int wave = producer ? wave8 - NC : wave8;             // index within the role
  const int tid = producer ? (int)threadIdx.x - NC * 64 : (int)threadIdx.x;   // thread index within the role
  const int n0 = blockIdx.x * BN, m0 = blockIdx.y * BM;
  const int ksteps = p.in_features / BK;

  // ---- this thread's share of the W tile: row w_row, vectors 2*w_half and 2*w_half + 1 of every step
  const int w_row = tid >> 1, w_half = tid & 1;
  const bool w_on = n0 + w_row < p.out_features;
  const int o_w = min(n0 + w_row, p.out_features - 1);
  const float s_w = p.scale ? __half2float(p.scale[o_w]) : 1.0f;
  const float b_w = p.bias ? __half2float(p.bias[o_w]) : 0.0f;
  // activations: range-checked against the end of the last token row, so rows >= tokens read zeros
  const __amdgpu_buffer_rsrc_t r_x = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<__half *>(X), 0, (unsigned)(((long long)(tokens - 1) * ldx + p.in_features) * 2), 0x00020000);

  // The two roles run separate loops with the same number of barriers (one after the prologue, one per step),
  // so that the accumulators of the consumers and the gather registers of the producers never live together.
  if (producer) {
    uint4v greg[GD][2];       // centroids of the steps in flight; step kt uses slot kt % GD
    struct IdxGroup { uint4v q[GD / 2]; };   // raw indices of GD consecutive steps of this row: 8 bytes per step
    const unsigned char *irow = p.idx + (long long)o_w * p.stride;     // ksteps % GD == 0: every read stays in the row
    auto load_indices = [&](int k0, IdxGroup &g) {
#pragma unroll
      for (int i = 0; i < GD / 2; ++i) async_load16(g.q[i], irow + (long long)k0 * 8 + i * 16);
    };
    auto settle_group = [&](IdxGroup &g) {
#pragma unroll
      for (int i = 0; i < GD / 2; ++i) settle(g.q[i]);
    };
    auto pick = [&](const IdxGroup &g, int j) -> unsigned {     // this thread's index pair of step k0 + j
      const uint4v &v = g.q[j >> 1];
      return (j & 1) ? (w_half ? v.w : v.z) : (w_half ? v.y : v.x);
    };
    auto issue_gather = [&](uint4v (&g)[2], unsigned pair) {
      const unsigned i0 = min(pair & 0xFFFFu, (unsigned)p.k - 1u), i1 = min(pair >> 16, (unsigned)p.k - 1u);
      async_load16(g[0], p.cb, i0 * 16u);
      async_load16(g[1], p.cb, i1 * 16u);
    };
    auto store_w = [&](int buf, uint4v (&g)[2]) {
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        settle(g[j]);
        *reinterpret_cast<uint4v *>(reinterpret_cast<unsigned char *>(Ws + buf * BN * LDT) + x_slot((unsigned)w_row, (unsigned)(w_half * 2 + j))) = restore8(g[j], s_w, b_w, w_on);
      }
    };
    // Memory operations of a producer wave, in issue order: per step two centroid gathers (for step kt+1+GD), plus
    // GD/2 index loads at the start of every group of GD steps.  They complete in order.
    // Every step and every group issues its loads, also past the end of the row (the last group and the last step are
    // loaded again and never looked at), so the counted wait below is the same on every path.
    IdxGroup nxt, far;        // raw indices of the next group and of the group after it
    load_indices(0, far);
    load_indices(min(GD, ksteps - GD), nxt);
    wait_vmem_at_most<0>();
    settle_group(far); settle_group(nxt);
#pragma unroll
    for (int j = 0; j < GD; ++j) issue_gather(greg[j], pick(far, j));        // steps 0 .. GD-1
    wait_vmem_at_most<0>();
    store_w(0, greg[0]);
    issue_gather(greg[0], pick(nxt, 0));                                     // slot 0 now carries step GD
    step_barrier();
    for (int k0 = 0; k0 < ksteps; k0 += GD) {
      load_indices(min(k0 + 2 * GD, ksteps - GD), far);                      // first used at the last step of this group
#pragma unroll
      for (int j = 0; j < GD; ++j) {
        const int kt = k0 + j;                                    // ksteps % GD == 0: kt < ksteps
        // The centroids of step kt+1 (slot (j+1) % GD) went out at the end of step kt-GD, followed by two
        // gathers in each of the GD-1 steps since (index loads not counted: with them the bound only gets safer).
        wait_vmem_at_most<2 * (GD - 1)>();
        const int sl = (j + 1) % GD;
        store_w((kt & 1) ^ 1, greg[sl]);                          // (after the last step: a tile nobody reads)
        // the wait above also covers the index loads this gather needs (they are older than those centroids)
        if (j + 1 < GD) { settle_group(nxt); issue_gather(greg[sl], pick(nxt, j + 1)); }
        else { settle_group(far); issue_gather(greg[sl], pick(far, 0)); }
        step_barrier();
      }
      nxt = far;      // the group after next becomes the next group (its loads completed before the last wait above)
    }
    wait_vmem_at_most<0>();
    return;
  }

  // ---- consumers: each wave streams its own 64 token rows through its slice of the activation stages (no other
  // wave touches them, so only the wave's own counted wait stands between a copy and its use) and multiplies
  auto copy_x = [&](int kt) {
    const unsigned stage = (unsigned)(kt % NSX) * XSTAGE;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const unsigned piece = (unsigned)(wave * 4 + i);                  // 16 rows per 1 KB piece
      const unsigned r = piece * 16u + ((unsigned)lane >> 2), cs = (unsigned)lane & 3u;   // LDS slot (r, cs) holds chunk cs ^ swz(r)
      const unsigned c = cs ^ swz(r);
      const unsigned goff = (unsigned)(((long long)(m0 + (int)r) * ldx + (long long)kt * BK + c * 8) * 2);
      __builtin_amdgcn_raw_ptr_buffer_load_lds(r_x, (__attribute__((address_space(3))) void *)(Xs + stage + piece * 1024u), 16, goff, 0, 0, 0);
    }
  };
  float16v acc[MB][4];
#pragma unroll
  for (int a = 0; a < MB; ++a)
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[a][c][r] = 0.0f;
  const int wm = wave * 64;
#pragma unroll
  for (int j = 0; j < XD; ++j)
    if (j < ksteps) copy_x(j);
  wait_vmem_at_most<0>();
  step_barrier();                                               // the W tile of step 0 is in LDS
  for (int kt = 0; kt < ksteps; ++kt) {
    const int cur = kt & 1;
    if (kt + XD < ksteps) copy_x(kt + XD);
    const unsigned char *xs = Xs + (unsigned)(kt % NSX) * XSTAGE;
#pragma unroll
    for (int ks = 0; ks < BK; ks += 16) {
      half8 af[MB], bf[4];
#pragma unroll
      for (int a = 0; a < MB; ++a)
        af[a] = *reinterpret_cast<const half8 *>(xs + x_slot((unsigned)(wm + a * 32 + (lane & 31)), (unsigned)(ks / 8 + (lane >> 5))));
#pragma unroll
      for (int c = 0; c < 4; ++c)
        bf[c] = *reinterpret_cast<const half8 *>(reinterpret_cast<const unsigned char *>(Ws + cur * BN * LDT) + x_slot((unsigned)(c * 32 + (lane & 31)), (unsigned)(ks / 8 + (lane >> 5))));
#pragma unroll
      for (int a = 0; a < MB; ++a)
#pragma unroll
        for (int c = 0; c < 4; ++c) acc[a][c] = __builtin_amdgcn_mfma_f32_32x32x16_f16(af[a], bf[c], acc[a][c], 0, 0, 0);
    }
    // this wave's rows of step kt+1 went out at step kt+1-XD; four copies per step since
    if (kt + XD < ksteps) wait_vmem_at_most<4 * (XD - 1)>(); else wait_vmem_at_most<0>();
    step_barrier();
  }

  // ---- store: lane holds channel (lane & 31) of block c and 16 token rows of block a
#pragma unroll
  for (int a = 0; a < MB; ++a)
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const int o = n0 + c * 32 + (lane & 31);
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int t = m0 + wm + a * 32 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
        if (t < tokens && o < p.out_features) Y[(long long)t * ldy + o] = __float2half_rn(acc[a][c][r]);
      }
    }
}

template <int BM>
int launch_fused(const Params &p, const __half *X, long long ldx, int tokens, __half *Y, long long ldy, hipStream_t s) {
  auto kernel = gemm_v8_kernel<BM>;
  const unsigned lds = NSX * BM * 64u + 2u * BN * LDT * 2u;
  VQ_ALLOW_FULL_LDS(kernel);
  const unsigned gx = (unsigned)((p.out_features + BN - 1) / BN), gy = (unsigned)((tokens + BM - 1) / BM);
  if (gy > 65535u) return VQ_ERR_UNSUPPORTED;
  hipLaunchKernelGGL(kernel, dim3(gx, gy), dim3((BM / 64 + 4) * 64), lds, s, p, X, ldx, tokens, Y, ldy);
  return hipGetLastError() == hipSuccess ? VQ_OK : VQ_ERR_HIP;
}

}  // namespace

bool gemm_fused_applicable(const Params &p) {
  return p.orientation == 0 && p.v == 8 && p.bits == 16 && p.k_res == 0 && p.n_out == 0 && p.n_groups == 1 && p.in_features % (GD * BK) == 0;
}

int launch_gemm_fused(const Params &p, const __half *X, long long ldx, int tokens, __half *Y, long long ldy, hipStream_t s) {
  if (((long long)(tokens - 1) * ldx + p.in_features) * 2 >= (1LL << 32)) return VQ_ERR_UNSUPPORTED;   // 32-bit buffer offsets
  return tokens > 512 ? launch_fused<512>(p, X, ldx, tokens, Y, ldy, s) : launch_fused<256>(p, X, ldx, tokens, Y, ldy, s);
}

}  // namespace vq
