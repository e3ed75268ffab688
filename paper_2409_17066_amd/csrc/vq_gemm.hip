// vq_gemm: prompt-phase product Y = X * W^T with W restored on the fly into LDS tiles that feed the
// FP16 matrix cores (paper App. "Our Dequantization Implementation", first phase, but without ever
// writing W to memory).  Accumulation in binary32, FP16 result.
#include "vq_common.hpp"
#include <cstdlib>

namespace vq {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef float float16v __attribute__((ext_vector_type(16)));

constexpr int BM = 128;        // tokens per workgroup tile
constexpr int BN = 128;        // output channels per workgroup tile
constexpr int BK = 32;         // input columns per step
constexpr int LDT = BK + 8;    // LDS row pitch in halfs: 80 bytes, so 8 consecutive rows hit 8 different 16-byte bank groups

// Restore columns [c0, c0+n) of row o into dst (LDS), zero past in_features.  Any layer shape.
__device__ __forceinline__ void restore_run_generic(const Params &p, int o, int c0, int n, float s, float b, __half *dst) {
  if (p.orientation == 1) {               // vectors down the output dimension: every column of the run is a vector of its own
    for (int t = 0; t < n; ++t) {
      const int c = c0 + t;
      if (o >= p.out_features || c >= p.in_features) { dst[t] = __float2half_rn(0.0f); continue; }
      float d;
      if (c < p.n_out) {
        const int sq = o / p.v_out;
        unsigned i = min(load_index(p.idx_out + (long long)sq * p.stride_out, c, p.bits_out), (unsigned)p.k_out - 1u);
        d = __half2float(p.cb_out[(long long)i * p.v_out + (o - sq * p.v_out)]);
      } else {
        const int pos = c - p.n_out, sp = o / p.v, j = o - sp * p.v;
        const long long group = pos / p.Pg;
        unsigned i = min(load_index(p.idx + (long long)sp * p.stride, pos, p.bits), (unsigned)p.k - 1u);
        d = __half2float(p.cb[(group * p.k + i) * p.v + j]);
        if (p.k_res) {
          unsigned r = min(load_index(p.idx_res + (long long)sp * p.stride_res, pos, p.bits_res), (unsigned)p.k_res - 1u);
          d = __fadd_rn(d, __half2float(p.cb_res[(group * p.k_res + r) * p.v + j]));
        }
      }
      dst[t] = restore(d, s, b);
    }
    return;
  }
  int c = c0;
  int j = 0, len = 0;                     // position inside / length of the current vector
  const __half *e = nullptr, *er = nullptr;
  for (int t = 0; t < n; ++t, ++c) {
    if (o >= p.out_features || c >= p.in_features) { dst[t] = __float2half_rn(0.0f); continue; }
    if (j >= len) {                       // fetch the vector that holds column c
      er = nullptr;
      if (c < p.n_out) {
        const int q = c / p.v_out;
        j = c - q * p.v_out; len = p.v_out;
        unsigned i = min(load_index(p.idx_out + (long long)o * p.stride_out, q, p.bits_out), (unsigned)p.k_out - 1u);
        e = p.cb_out + (long long)i * p.v_out;
      } else {
        const int cc = c - p.n_out;
        const int pp = cc / p.v;
        j = cc - pp * p.v; len = p.v;
        unsigned i = min(load_index(p.idx + (long long)o * p.stride, pp, p.bits), (unsigned)p.k - 1u);
        const long long group = pp / p.Pg;
        e = p.cb + (group * p.k + i) * p.v;
        if (p.k_res) {
          unsigned r = min(load_index(p.idx_res + (long long)o * p.stride_res, pp, p.bits_res), (unsigned)p.k_res - 1u);
          er = p.cb_res + (group * p.k_res + r) * p.v;
        }
      }
    }
    float d = __half2float(e[j]);
    if (er) d = __fadd_rn(d, __half2float(er[j]));
    dst[t] = restore(d, s, b);
    ++j;
    if (c + 1 == p.n_out) j = len;        // the outlier region ends: force a fetch from the main stream
  }
}

// 256 threads = 4 waves in a 2x2 arrangement; each wave owns a 64x64 block of the 128x128 tile as
// 2x2 MFMA 32x32x16 blocks.  Operand layout of v_mfma_f32_32x32x16_f16: lane l supplies row/column
// (l & 31) and the 8 consecutive k values starting at 8*(l >> 5); it receives column (l & 31) and,
// in result register r, row 8*(r >> 2) + 4*(l >> 5) + (r & 3).
__global__ __launch_bounds__(256) void gemm_tile_kernel(Params p, const __half *__restrict__ X, long long ldx, int tokens,
                                                        __half *__restrict__ Y, long long ldy) {
  __shared__ __attribute__((aligned(16))) __half Xs[BM * LDT];
  __shared__ __attribute__((aligned(16))) __half Ws[BN * LDT];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int n0 = blockIdx.x * BN, m0 = blockIdx.y * BM;
  const int wm = (wave >> 1) * 64, wn = (wave & 1) * 64;

  float16v acc[2][2];
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[a][c][r] = 0.0f;

  // W restore assignment: thread -> (row tid/2, 16 columns)
  const int w_row = tid >> 1, w_col = (tid & 1) * 16;
  const int o_w = n0 + w_row;
  const float s_w = (p.scale && o_w < p.out_features) ? __half2float(p.scale[o_w]) : 1.0f;
  const float b_w = (p.bias && o_w < p.out_features) ? __half2float(p.bias[o_w]) : 0.0f;

  for (int k0 = 0; k0 < p.in_features; k0 += BK) {
    // X tile: 128 rows x 4 chunks of 8 halfs; thread takes chunks tid and tid+256
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int chunk = tid + h * 256;
      const int row = chunk >> 2, col = (chunk & 3) * 8;
      const int t = m0 + row, c = k0 + col;
      uint4 val = make_uint4(0, 0, 0, 0);
      if (t < tokens && p.perm) {                       // permuted column order: stored column c + i meets X[t][perm[c + i]]
        __half tmp[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          const int u = c + i < p.in_features ? p.perm[c + i] : -1;
          tmp[i] = (unsigned)u < (unsigned)p.in_features ? X[(long long)t * ldx + u] : __float2half_rn(0.0f);
        }
        val = *reinterpret_cast<uint4 *>(tmp);
      } else if (t < tokens) {
        const __half *src = X + (long long)t * ldx + c;
        if (c + 8 <= p.in_features) {
          val = *reinterpret_cast<const uint4 *>(src);
        } else if (c < p.in_features) {
          __half tmp[8];
#pragma unroll
          for (int i = 0; i < 8; ++i) tmp[i] = (c + i < p.in_features) ? src[i] : __float2half_rn(0.0f);
          val = *reinterpret_cast<uint4 *>(tmp);
        }
      }
      *reinterpret_cast<uint4 *>(&Xs[row * LDT + col]) = val;
    }
    restore_run_generic(p, o_w, k0 + w_col, 16, s_w, b_w, &Ws[w_row * LDT + w_col]);
    __syncthreads();
#pragma unroll
    for (int ks = 0; ks < BK; ks += 16) {
      half8 af[2], bf[2];
#pragma unroll
      for (int a = 0; a < 2; ++a)
        af[a] = *reinterpret_cast<const half8 *>(&Xs[(wm + a * 32 + (lane & 31)) * LDT + ks + (lane >> 5) * 8]);
#pragma unroll
      for (int c = 0; c < 2; ++c)
        bf[c] = *reinterpret_cast<const half8 *>(&Ws[(wn + c * 32 + (lane & 31)) * LDT + ks + (lane >> 5) * 8]);
#pragma unroll
      for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int c = 0; c < 2; ++c)
          acc[a][c] = __builtin_amdgcn_mfma_f32_32x32x16_f16(af[a], bf[c], acc[a][c], 0, 0, 0);
    }
    __syncthreads();
  }

#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      const int o = n0 + wn + c * 32 + (lane & 31);
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int t = m0 + wm + a * 32 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
        if (t < tokens && o < p.out_features) Y[(long long)t * ldy + o] = __float2half_rn(acc[a][c][r]);
      }
    }
}

size_t gemm_workspace_bytes(const Params &, int) { return 0; }
bool gemm_dense_applicable(const Params &p);
float gemm_dense_us(const Params &p, int tokens, bool against_rows = false);
size_t gemm_dense_scratch_bytes(const Params &p, int tokens, int matrices, size_t most);

// Bytes of the FP16 weight matrix [out][in] that the two-step route below writes; 0 when that route does not apply.
// For a layer with a permuted column order (Sec. 3.2.3) the activations, gathered into stored order, come first: tokens
// rows of in_features rounded up to 8 halfs, the whole rounded up to 256 bytes; every kernel then works in stored order.
static size_t permuted_x_bytes(const Params &p, int tokens) { return ((size_t)tokens * (size_t)((p.in_features + 7) & ~7) * sizeof(__half) + 255) / 256 * 256; }

// Behind the restored matrix: the partial sums of a product whose columns are cut into parts (vq_gemm_dense.hip), the same for any number of
// tokens, so that a workspace for many serves few.  Without this part a product is not cut; 8 MiB hold what 512 tiles of 64 x 64 leave, two for
// every compute unit.  Up to 512 columns there is nothing to gain (eight steps), nor above 8192 outputs, whose tiles of 64 tokens keep half the compute
// units busy already (43 tokens, 8461 x 6912: 52.9 us whole, 53.8 in parts; 88 tokens, 5696 x 9472: 55.4 and 55.8).
static size_t restored_bytes(const Params &p) { return ((size_t)p.out_features * (size_t)p.in_features * sizeof(__half) + 255) / 256 * 256; }
static size_t dense_scratch_bytes(const Params &p) { return p.in_features > 512 && p.out_features <= 8192 ? (size_t)8 << 20 : 0; }

size_t gemm_fast_workspace_bytes(const Params &p, int tokens) {
  const size_t head = p.perm ? permuted_x_bytes(p, tokens) : 0;
  if (!gemm_dense_applicable(p)) return head;
  return head + restored_bytes(p) + dense_scratch_bytes(p);
}

bool gemm_fused_applicable(const Params &p);
bool gemv_has_lds_kernel(const Params &p, const __half *x, long long ldx);
bool gemv_rows_applicable(const Params &p);
bool gemv_rows_takes(const Params &p, const __half *x, long long ldx, int batch);
bool gemm_v6_applicable(const Params &p);
int launch_gemm_v6(const Params &p, const __half *X, long long ldx, int tokens, __half *Y, long long ldy, hipStream_t s);
int launch_gemm_fused(const Params &p, const __half *X, long long ldx, int tokens, __half *Y, long long ldy, hipStream_t s);
int launch_gemm_dense(const Params &p, const __half *X, long long ldx, int tokens, __half *Y, long long ldy, const __half *Wd,
                      long long ldw, hipStream_t s, const float *xsum = nullptr, unsigned w2 = 0, void *scratch = nullptr, size_t scratch_bytes = 0);

// Row-wise v = 6 layers have the matrix-core GEMV, whose sixteen rows cost little more than one: it still beats restoring the
// matrix for the first sixteens of tokens.  Estimates in microseconds from 130 random layers: a launch of it 5 + 1.2 per thousand
// columns and a little per million weights; restoring 5 + 0.4 per million weights (0.8 with a residual table), then the dense
// product.  10496 x 3328, 28 tokens: 18 against 38 us; 4096 + 4096 tables, 4960 x 3072, 45 tokens: 39 against 38 us.
static bool rows_beat_restoring(const Params &p, int tokens) {
  const float weights = (float)((double)p.out_features * p.in_features * 1e-6);
  const float launch = 5.0f + 1.2e-3f * (float)p.in_features + (p.k_res ? 1.5f + 0.06f * weights : 0.03f * weights) + (p.n_groups > 1 ? 8.0f : 0.0f);
  const float restore = 5.0f + (p.k_res ? 0.8f : 0.4f) * weights + (p.n_out ? 5.0f : 0.0f);
  return (float)((tokens + 15) / 16) * launch < restore + gemm_dense_us(p, tokens, true);
}

// The same for vectors down the outputs, whose matrix-core kernel takes sixteen rows at the price of one; restoring 4 and 0.3 per million weights (0.4
// with a residual table).  11008 x 4096 with a workspace, 9 / 17 / 33 tokens: 34 -> 11, 34 -> 21, 35 -> 34 us; 4096 x 11008 with residual tables 59 -> 17,
// 59 -> 33, 59 -> 51; at 65 tokens they are level or behind.
float gemv_down_rows_us(const Params &p, const __half *x, long long ldx);
static bool down_rows_beat_restoring(const Params &p, const __half *X, long long ldx, int tokens) {
  const float launch = gemv_down_rows_us(p, X, ldx), weights = (float)((double)p.out_features * p.in_features * 1e-6);
  return launch > 0.0f && (float)((tokens + 15) / 16) * launch < 4.0f + (p.k_res ? 0.4f : 0.3f) * weights + gemm_dense_us(p, tokens, true);
}

static bool v6_tiles_fill(const Params &p, int tokens) { return tokens > 128 || (long long)((p.out_features + 127) / 128) * ((tokens + 127) / 128) >= 80; }

// Whether the tile kernels would be a loss of precision: without a workspace these layers and token counts go through vq_gemv's kernels,
// which keep centroids, scale and bias apart and in binary32 where the others multiply with weights rounded to binary16.
static bool rows_hold_the_weights(const Params &p, int tokens) {
  const long long ldx = (p.in_features + 7) & ~7;
  if (p.perm || gemm_fused_applicable(p) || (gemm_v6_applicable(p) && tokens > 64 && v6_tiles_fill(p, tokens))) return false;
  if (gemv_has_fast_kernel(p, nullptr, ldx)) return tokens <= 128 || (p.orientation == 0 && p.v == 6);
  return tokens <= 32 && gemv_has_lds_kernel(p, nullptr, ldx);
}

// ---- the prompt-phase scheme with unrounded weights -------------------------------------------------------------------
// Centroids are binary16 numbers: restored without scale and bias they are exact, and y = scale * (C x + C_res x) + bias * sum(x) is what
// vq_gemv's kernels compute, with the dense product's rate.  The residual centroids are a second matrix, so that their sum with the main
// ones is never rounded.  11008 x 4096, v = 6 in four groups, 509 tokens: 489 us sixteen rows at a time, 89 us like this (restored
// and rounded: 85); vectors down the outputs, 128 tokens 146 -> 51 (43); 4096 x 4096 with a residual table and outlier columns, 509
// tokens 354 -> 71 (38).  Relative error against unrounded weights 2.1e-4, as vq_gemv's kernels; rounded 2.9e-4.
// sums[t] of X's rows (the first workgroups, a wave to a row), and zeros in the first `clear` columns of the matrix R (the others).
__global__ __launch_bounds__(256) void row_sums_kernel(const __half *__restrict__ X, long long ldx, int tokens, int columns, float *__restrict__ sums,
                                                       __half *__restrict__ R, long long ldr, int rows, int clear) {
  const int sum_wgs = (tokens + 3) / 4;
  if ((int)blockIdx.x >= sum_wgs) {
    for (int r = blockIdx.x - sum_wgs; r < rows; r += gridDim.x - sum_wgs)
      for (int c = threadIdx.x; c < clear; c += 256) R[(long long)r * ldr + c] = __float2half_rn(0.0f);
    return;
  }
  const int lane = threadIdx.x & 63, t = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (t >= tokens) return;
  const __half *row = X + (long long)t * ldx;
  float sum = 0.0f;
  for (int c = lane * 8; c < columns; c += 512) {            // (rows start on sixteen bytes; columns in multiples of eight)
    const half8 x = *reinterpret_cast<const half8 *>(row + c);
#pragma unroll
    for (int i = 0; i < 8; ++i) sum += (float)x[i];
  }
  sum = wave_sum(sum);
  if (lane == 0) sums[t] = sum;
}

static size_t centroids_workspace_bytes(const Params &p, int tokens) {
  return restored_bytes(p) * (p.k_res ? 2 : 1) + ((size_t)tokens * sizeof(float) + 255) / 256 * 256;
}

// Where this beats vq_gemv's kernels, sixteen rows at a time.  Estimates in microseconds: a launch of the row-wise v = 6 kernel 4 + 0.8 per
// thousand columns and 0.07 per million weights, twice that and 1.5 with a residual table, 5 more with codebook groups (512 x 8200: 10.5;
// 3000 x 2056: 6.4; 11008 x 4096: 10.5, four groups 15.5); of the matrix-core kernel down the outputs that kernel's own; of the others 5 and
// 0.32 per million weights, 0.5 with a residual table.
static bool centroids_beat_rows(const Params &p, int tokens) {
  const float weights = (float)((double)p.out_features * p.in_features * 1e-6), matrices = p.k_res ? 2.0f : 1.0f;
  const float v6 = 4.0f + 0.8e-3f * (float)p.in_features + (p.k_res ? 1.5f + 0.14f * weights : 0.07f * weights) + (p.n_groups > 1 ? 5.0f : 0.0f);
  const float down = gemv_down_rows_us(p, nullptr, (p.in_features + 7) & ~7);
  const float launch = p.orientation == 0 && p.v == 6 ? v6 : down > 0.0f ? down : 5.0f + (p.k_res ? 0.5f : 0.32f) * weights;
  const float restore = matrices * (6.0f + 0.33f * weights) + (p.n_out ? 5.0f : 0.0f) + 4.0f;
  return restore + matrices * gemm_dense_us(p, tokens) < (float)((tokens + 15) / 16) * launch;
}

constexpr size_t MOST_DEFAULT_WORKSPACE = (size_t)256 << 20;

// `bytes` and the sums of this product in parts behind them (vq_gemm_fast_workspace_bytes has room for any number of tokens', this one is for one
// call: 700 x 640, 200 tokens, whose product is not cut, 0.9 MB and not 9.3), or without these `bytes`, or nothing.  tokens = 0: no sums.
static size_t default_bytes(const Params &p, int tokens, int matrices, size_t bytes) {
  Params q = p;
  q.perm = nullptr;                                        // (the product runs on gathered activations)
  const size_t most = dense_scratch_bytes(p), sums = most && tokens ? gemm_dense_scratch_bytes(q, tokens, matrices, most) : 0;
  return bytes > MOST_DEFAULT_WORKSPACE ? 0 : bytes + sums <= MOST_DEFAULT_WORKSPACE ? bytes + sums : bytes;
}

static bool centroids_wanted(const Params &p, int tokens) {
  // (vq_dequant's kernel for few vectors of eight down the outputs takes no outlier columns, so it may not see such a layer without them)
  if (!gemm_dense_applicable(p) || p.perm || (p.k_res && p.bits_res == 16) || centroids_workspace_bytes(p, tokens) > MOST_DEFAULT_WORKSPACE) return false;
  if (switches().gemm != '\0') return switches().gemm == 'c';
  return rows_hold_the_weights(p, tokens) && centroids_beat_rows(p, tokens);
}

static int launch_gemm_centroids(const Params &p, const __half *X, long long ldx, int tokens, __half *Y, long long ldy, void *workspace,
                                 size_t workspace_bytes, hipStream_t s) {
  __half *C = static_cast<__half *>(workspace), *R = C + restored_bytes(p) / sizeof(__half);
  float *xsum = reinterpret_cast<float *>(static_cast<unsigned char *>(workspace) + restored_bytes(p) * (p.k_res ? 2 : 1));
  // (the residual matrix has no outlier columns of its own)
  const int clear = p.k_res ? p.n_out : 0, clear_wgs = !clear ? 0 : p.out_features < 4096 ? p.out_features : 4096;
  hipLaunchKernelGGL(row_sums_kernel, dim3((unsigned)((tokens + 3) / 4 + clear_wgs)), dim3(256), 0, s, X, ldx, tokens, p.in_features, xsum, R,
                     (long long)p.in_features, p.out_features, clear);
  Params q = p;
  q.scale = q.bias = nullptr;
  q.cb_res = nullptr; q.idx_res = nullptr; q.k_res = 0; q.stride_res = 0;
  int rc = launch_dequant(q, C, p.in_features, s, tokens);
  if (rc == VQ_OK && p.k_res) {
    // the residual table as a layer of its own, with room for outlier columns but none
    q.cb = p.cb_res; q.k = p.k_res; q.idx = p.idx_res; q.bits = p.bits_res; q.stride = p.stride_res;
    q.cb_out = nullptr; q.idx_out = nullptr; q.Q = q.S_out = 0;
    rc = launch_dequant(q, R, p.in_features, s, tokens);
  }
  if (rc != VQ_OK) return rc;
  const size_t used = centroids_workspace_bytes(p, tokens), room = std::min(workspace_bytes - used, dense_scratch_bytes(p));
  return launch_gemm_dense(p, X, ldx, tokens, Y, ldy, C, p.in_features, s, xsum, p.k_res ? (unsigned)restored_bytes(p) : 0u,
                           room ? static_cast<unsigned char *>(workspace) + used : nullptr, room);
}

// Rows of X through vq_gemv, sixteen at a time, with the workspace if it is aligned for that (vq_gemv cuts the columns into parts with it).
static int launch_gemm_rows(const Params &p, const __half *X, long long ldx, int tokens, __half *Y, long long ldy, void *workspace,
                            size_t workspace_bytes, hipStream_t s) {
  const bool lend = workspace && (reinterpret_cast<uintptr_t>(workspace) & 255) == 0;
  for (int t0 = 0; t0 < tokens; t0 += 16) {
    const int rc = launch_gemv_ws(p, X + (long long)t0 * ldx, ldx, tokens - t0 < 16 ? tokens - t0 : 16, Y + (long long)t0 * ldy, ldy,
                                  lend ? workspace : nullptr, lend ? workspace_bytes : 0, s);
    if (rc != VQ_OK) return rc;
  }
  return VQ_OK;
}

// What vq_gemm_default uses: room for W where it would be rounded in any case, else for the centroids, or what vq_gemv's kernels take;
// nothing beyond 256 MiB (W of 11008 x 11008), so that who leaves the workspace out to save memory still does
// where it counts (8192 x 28672, 448 MiB, 512 tokens: 532 us with it, 582 without).
// sums: with the room for those of a product in parts.
size_t gemm_default_workspace_bytes(const Params &p, int tokens, bool sums) {
  const int matrices = p.k_res ? 2 : 1;
  if (centroids_wanted(p, tokens)) return default_bytes(p, sums ? tokens : 0, matrices, centroids_workspace_bytes(p, tokens));
  if (!rows_hold_the_weights(p, tokens) && gemm_dense_applicable(p))
    return default_bytes(p, sums ? tokens : 0, 1, gemm_fast_workspace_bytes(p, tokens) - dense_scratch_bytes(p));
  const size_t bytes = rows_hold_the_weights(p, tokens) ? gemv_workspace_bytes(p, nullptr, (p.in_features + 7) & ~7, tokens < 16 ? tokens : 16)
                                                        : gemm_fast_workspace_bytes(p, tokens);
  return bytes <= MOST_DEFAULT_WORKSPACE ? bytes : 0;
}

int launch_gemm_default(const Params &p, const __half *X, long long ldx, int tokens, __half *Y, long long ldy, void *workspace,
                        size_t workspace_bytes, hipStream_t s) {
  if (workspace && (reinterpret_cast<uintptr_t>(workspace) & 255) == 0 && centroids_wanted(p, tokens) && workspace_bytes >= centroids_workspace_bytes(p, tokens)) {
    const int rc = launch_gemm_centroids(p, X, ldx, tokens, Y, ldy, workspace, workspace_bytes, s);
    if (rc != VQ_ERR_UNSUPPORTED) return rc;
  }
  if (rows_hold_the_weights(p, tokens) && switches().gemm == '\0') return launch_gemm_rows(p, X, ldx, tokens, Y, ldy, workspace, workspace_bytes, s);
  return launch_gemm(p, X, ldx, tokens, Y, ldy, workspace, workspace_bytes, s);
}

// Routes, in this order:
//  1. a workspace of gemm_fast_workspace_bytes() is there: vq_dequant into it, then the dense product (vq_gemm_dense.hip).  This
//     is the paper's prompt-phase scheme; on gfx950 it beats restoring on the fly at every token count measured (17 to 2048),
//     because tables are looked up once and not once for every token tile, and the restored matrix is read in full lines.
//     Any layer the library can dequantize qualifies (in_features a multiple of 8).  It leaves to vq_gemv's kernels, sixteen rows
//     at a time, what they do faster: v = 6 layers by the estimates above; layers of vq_gemv_rows.hip up to 32 tokens
//     (v = 12 with two tables, 8960 x 8192, 10 tokens: 22 against 121 us; v = 4, 8064 x 8448, 17 tokens: 34 against 73 us; level from
//     33 on), 16 with codebook groups; others up to eight.
//  2. no workspace, and a layer whose only tile kernel is the generic one: vq_gemv's kernels where that was measured faster.
//     Row-wise v = 6 layers and those of vq_gemv_rows.hip: always (512 tokens 322 against 700 us); layers with another specialised
//     kernel (orientation 1), whose cost grows faster with the rows: up to 128 tokens; layers of the LDS-table decode kernels, which
//     take four rows a launch: up to 32 (v = 12 with two tables, 16 tokens: 239 against 987 us).
//  3. v = 6 / 12-bit indices, one codebook group, no workspace, more than 64 tokens: restored on the fly from tables in LDS
//     (vq_gemm_v6.hip; up to 128 tokens only where its 128 x 128 tiles give 80 workgroups -- 8192 x 28672 at 128 tokens: 64
//     workgroups, 612 us against 515 us for eight passes of the GEMV).
//  4. v = 8 / 16-bit indices, no workspace: restored on the fly inside the MFMA kernel (vq_gemm_fused.hip), up to 32 tokens vq_gemv
//     (461 x 8448, 7 tokens: 25 against 146 us).
//  5. the generic tile kernel.
// Switch gemm=g forces 5, =f skips 1, =w takes 1 whenever a workspace is there, =6 takes 3 for every token count, =r takes
// vq_gemv's kernels, =c, for vq_gemm_default, the centroids' route wherever it can (measurement and tests).
int launch_gemm(const Params &p, const __half *X, long long ldx, int tokens, __half *Y, long long ldy,
                void *workspace, size_t workspace_bytes, hipStream_t s) {
  if (p.perm && tokens <= 65535 && workspace && workspace_bytes >= permuted_x_bytes(p, tokens) && (reinterpret_cast<uintptr_t>(workspace) & 15) == 0 &&
      switches().gemm != 'g') {
    // room for the gathered activations: from here on the layer is an unpermuted one (the rest of the workspace is its own)
    Params q = p;
    q.perm = nullptr;
    __half *Xp = static_cast<__half *>(workspace);
    const long long ldxp = (p.in_features + 7) & ~7;
    const int rc = launch_gather_cols(X, ldx, tokens, p.in_features, p.perm, Xp, ldxp, s);
    if (rc != VQ_OK) return rc;
    const size_t head = permuted_x_bytes(p, tokens);
    return launch_gemm(q, Xp, ldxp, tokens, Y, ldy, static_cast<unsigned char *>(workspace) + head, workspace_bytes - head, s);
  }
  if (p.perm) {                                            // no room: the generic tile kernel looks every activation up
    const unsigned gx = (unsigned)((p.out_features + BN - 1) / BN), gy = (unsigned)((tokens + BM - 1) / BM);
    if (gy > 65535u) return VQ_ERR_UNSUPPORTED;
    hipLaunchKernelGGL(gemm_tile_kernel, dim3(gx, gy), dim3(256), 0, s, p, X, ldx, tokens, Y, ldy);
    return hipGetLastError() == hipSuccess ? VQ_OK : VQ_ERR_HIP;
  }
  const char forced = switches().gemm;
  // (a workspace of the restored matrix alone is enough for this route)
  const size_t fast = gemm_dense_applicable(p) ? (size_t)p.out_features * (size_t)p.in_features * sizeof(__half) : 0;
  const bool have_ws = fast && workspace && workspace_bytes >= fast && (reinterpret_cast<uintptr_t>(workspace) & 15) == 0;
  if (gemm_v6_applicable(p) && (forced == '6' || (forced == '\0' && !have_ws && tokens > 64 && v6_tiles_fill(p, tokens)))) {
    const int rc = launch_gemm_v6(p, X, ldx, tokens, Y, ldy, s);
    if (rc != VQ_ERR_UNSUPPORTED) return rc;
  }
  bool rows = forced == 'r';
  if (forced == '\0') {
    const bool fast_rows = gemv_has_fast_kernel(p, X, ldx), lds_rows = gemv_has_lds_kernel(p, X, ldx);
    if (p.orientation == 0 && p.v == 6 && fast_rows) rows = !have_ws || rows_beat_restoring(p, tokens);
    else if (have_ws && p.orientation == 1 && tokens > 8 && down_rows_beat_restoring(p, X, ldx, tokens)) rows = true;
    else if (gemv_rows_applicable(p) && gemv_rows_takes(p, X, ldx, 16))
      rows = have_ws ? tokens <= (p.n_groups > 1 ? 16 : 32) : tokens <= 32 || !gemm_fused_applicable(p);
    else if (have_ws || gemm_fused_applicable(p)) rows = tokens <= (have_ws ? 8 : 16) && (fast_rows || lds_rows);
    else rows = (tokens <= 128 && fast_rows) || (tokens <= 32 && !gemm_v6_applicable(p) && lds_rows);
  }
  if (rows) return launch_gemm_rows(p, X, ldx, tokens, Y, ldy, have_ws ? workspace : nullptr, have_ws ? workspace_bytes : 0, s);
  if (forced != 'g' && forced != 'f' && have_ws) {
    __half *Wd = static_cast<__half *>(workspace);
    const size_t matrix = restored_bytes(p), room = workspace_bytes > matrix ? std::min(workspace_bytes - matrix, dense_scratch_bytes(p)) : 0;
    int rc = launch_dequant(p, Wd, p.in_features, s, tokens);
    if (rc == VQ_OK) rc = launch_gemm_dense(p, X, ldx, tokens, Y, ldy, Wd, p.in_features, s, nullptr, 0u, room ? Wd + matrix / sizeof(__half) : nullptr, room);
    if (rc != VQ_ERR_UNSUPPORTED) return rc;
  }
  if (forced != 'g' && gemm_fused_applicable(p)) {
    const int rc = launch_gemm_fused(p, X, ldx, tokens, Y, ldy, s);
    if (rc != VQ_ERR_UNSUPPORTED) return rc;
  }
  const unsigned gx = (unsigned)((p.out_features + BN - 1) / BN), gy = (unsigned)((tokens + BM - 1) / BM);
  if (gy > 65535u) return VQ_ERR_UNSUPPORTED;
  hipLaunchKernelGGL(gemm_tile_kernel, dim3(gx, gy), dim3(256), 0, s, p, X, ldx, tokens, Y, ldy);
  return hipGetLastError() == hipSuccess ? VQ_OK : VQ_ERR_HIP;
}

}  // namespace vq
