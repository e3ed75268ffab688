// vq_gemv: decode-phase fused restore + matrix-vector product for batch 1..16
// (paper App. "Our Dequantization Implementation", second phase: the FP16 weights are never written).
#include "vq_common.hpp"
#include <cstdlib>

namespace vq {

// The activation that stored column c meets (Sec. 3.2.3: the stored order of the columns may be a permutation of the
// layer's); entries outside the row count as zero.
__device__ __forceinline__ float x_at(const Params &p, const __half *xrow, int c) {
  if (!p.perm) return __half2float(xrow[c]);
  const int t = p.perm[c];
  return (unsigned)t < (unsigned)p.in_features ? __half2float(xrow[t]) : 0.0f;
}

// Any layer: one wave per output row, lanes stride over the row's vectors, tables read through the
// cache hierarchy.  Slow but complete; the specialised kernels below take the common shapes.
__global__ __launch_bounds__(256) void gemv_generic_kernel(Params p, const __half *__restrict__ x, long long ldx, int batch,
                                                           __half *__restrict__ y, long long ldy) {
  const int lane = threadIdx.x & 63;
  const int o = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (o >= p.out_features) return;
  const float s = p.scale ? __half2float(p.scale[o]) : 1.0f;
  const float b = p.bias ? __half2float(p.bias[o]) : 0.0f;
  float acc[16];
#pragma unroll
  for (int t = 0; t < 16; ++t) acc[t] = 0.0f;
  for (int slot = lane; slot < p.Q + p.P; slot += 64) {
    const __half *e, *er = nullptr;
    int c0, len;
    if (slot < p.Q) {
      unsigned i = min(load_index(p.idx_out + (long long)o * p.stride_out, slot, p.bits_out), (unsigned)p.k_out - 1u);
      e = p.cb_out + (long long)i * p.v_out;
      c0 = slot * p.v_out; len = p.v_out;
    } else {
      const int pp = slot - p.Q;
      unsigned i = min(load_index(p.idx + (long long)o * p.stride, pp, p.bits), (unsigned)p.k - 1u);
      const long long group = pp / p.Pg;
      e = p.cb + (group * p.k + i) * p.v;
      if (p.k_res) {
        unsigned r = min(load_index(p.idx_res + (long long)o * p.stride_res, pp, p.bits_res), (unsigned)p.k_res - 1u);
        er = p.cb_res + (group * p.k_res + r) * p.v;
      }
      c0 = p.n_out + pp * p.v; len = min(p.v, p.in_features - c0);
    }
    for (int j = 0; j < len; ++j) {
      float d = __half2float(e[j]);
      if (er) d = __fadd_rn(d, __half2float(er[j]));
      const float w = __half2float(restore(d, s, b));
#pragma unroll
      for (int t = 0; t < 16; ++t)
        if (t < batch) acc[t] = __fmaf_rn(w, x_at(p, x + t * ldx, c0 + j), acc[t]);
    }
  }
#pragma unroll
  for (int t = 0; t < 16; ++t) {
    if (t < batch) {
      const float r = wave_sum(acc[t]);
      if (lane == 0) y[t * ldy + o] = __float2half_rn(r);
    }
  }
}

// Orientation 1 (vectors down the output dimension; Sec. 3.1, Algorithm 1): one wave per main stream, i.e. per block of v
// output rows; lanes stride over the columns and keep one sum per row of the block; the outlier columns of each of these
// rows come from the outlier stream that holds the row.  One token at a time.  Slow but complete.
__global__ __launch_bounds__(256) void gemv_down_kernel(Params p, const __half *__restrict__ x, long long ldx, int batch,
                                                        __half *__restrict__ y, long long ldy) {
  const int lane = threadIdx.x & 63;
  const int stream = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (stream >= p.S) return;
  const int o0 = stream * p.v;
  float sc[16], bi[16];
#pragma unroll
  for (int j = 0; j < 16; ++j) {
    const bool on = j < p.v && o0 + j < p.out_features;
    sc[j] = on && p.scale ? __half2float(p.scale[o0 + j]) : 1.0f;
    bi[j] = on && p.bias ? __half2float(p.bias[o0 + j]) : 0.0f;
  }
  for (int t = 0; t < batch; ++t) {
    const __half *xt = x + (long long)t * ldx;
    float acc[16];
#pragma unroll
    for (int j = 0; j < 16; ++j) acc[j] = 0.0f;
    for (int pos = lane; pos < p.P; pos += 64) {
      unsigned i = min(load_index(p.idx + (long long)stream * p.stride, pos, p.bits), (unsigned)p.k - 1u);
      const long long group = pos / p.Pg;
      const __half *e = p.cb + (group * p.k + i) * p.v, *er = nullptr;
      if (p.k_res) {
        unsigned r = min(load_index(p.idx_res + (long long)stream * p.stride_res, pos, p.bits_res), (unsigned)p.k_res - 1u);
        er = p.cb_res + (group * p.k_res + r) * p.v;
      }
      const float xv = x_at(p, xt, p.n_out + pos);
#pragma unroll
      for (int j = 0; j < 16; ++j)
        if (j < p.v && o0 + j < p.out_features) {
          float d = __half2float(e[j]);
          if (er) d = __fadd_rn(d, __half2float(er[j]));
          acc[j] = __fmaf_rn(__half2float(restore(d, sc[j], bi[j])), xv, acc[j]);
        }
    }
#pragma unroll
    for (int j = 0; j < 16; ++j)
      if (j < p.v && o0 + j < p.out_features) {
        const int o = o0 + j, sq = p.Q ? o / p.v_out : 0, jo = p.Q ? o - sq * p.v_out : 0;
        for (int pos = lane; pos < p.Q; pos += 64) {
          unsigned i = min(load_index(p.idx_out + (long long)sq * p.stride_out, pos, p.bits_out), (unsigned)p.k_out - 1u);
          const float w = __half2float(restore(__half2float(p.cb_out[(long long)i * p.v_out + jo]), sc[j], bi[j]));
          acc[j] = __fmaf_rn(w, x_at(p, xt, pos), acc[j]);
        }
        const float r = wave_sum(acc[j]);
        if (lane == 0) y[(long long)t * ldy + o] = __float2half_rn(r);
      }
  }
}

bool gemv_fast_applicable(const Params &p, const __half *x, long long ldx);
bool gemv_res8_applicable(const Params &p, const __half *x);
bool gemv_lds_applicable(const Params &p, int batch);
int launch_gemv_lds(const Params &p, const __half *x, long long ldx, int batch, __half *y, long long ldy, hipStream_t s);
size_t gemv_lds_slots_workspace_bytes(const Params &p, int batch, bool least);
bool gemv_down_lds_applicable(const Params &p, int batch);
size_t gemv_down_lds_slots_workspace_bytes(const Params &p, int batch);
int launch_gemv_down_lds_slots(const Params &p, const __half *x, long long ldx, int batch, float *part, float *part_xs, hipStream_t s);
int launch_gemv_down_lds(const Params &p, const __half *x, long long ldx, int batch, __half *y, long long ldy, hipStream_t s);
int launch_gemv_lds_slots(const Params &p, const __half *x, long long ldx, int batch, float *part, size_t bytes, int *n_part, hipStream_t s);
int launch_gemv_res8(const Params &p, const __half *x, __half *y, hipStream_t s);
int launch_gemv_fast(const Params &p, const __half *x, long long ldx, int batch, __half *y, long long ldy, hipStream_t s);

int launch_gemv_mfma(const Params &p, const __half *x, long long ldx, int batch, __half *y, long long ldy, hipStream_t s);
bool gemv_fast_applicable_even(const Params &p);
bool gemv_down_applicable(const Params &p, const __half *x, long long ldx);
bool gemv_down_fits(const Params &p);
bool gemv_v8_wanted(const Params &p, const __half *x, long long ldx, int batch, bool workspace);
int launch_gemv_v8(const Params &p, const __half *x, long long ldx, int batch, __half *y, long long ldy, hipStream_t s);
bool gemv_v8_down_applicable(const Params &p);
int launch_gemv_v8_down(const Params &p, const __half *x, long long ldx, int batch, __half *y, long long ldy, hipStream_t s);
int launch_gemv_down(const Params &p, const __half *x, long long ldx, int batch, __half *y, long long ldy, hipStream_t s,
                     float *part = nullptr, float *part_xs = nullptr, int part_batch = 0);
int launch_groups_finish(const float *part, const float *part_xs, int n_groups, int batch, const Params &p, __half *y, long long ldy,
                         hipStream_t s);
bool gemv_down_mfma_applicable(const Params &p, const __half *x, long long ldx, int batch);
int gemv_down_mfma_parts(const Params &p);
float gemv_down_mfma_us(const Params &p, int parts, int batch, bool fold = true);
float gemv_down_streams_us(const Params &p, int batch);
int launch_gemv_down_mfma(const Params &p, const __half *x, long long ldx, int batch, __half *y, long long ldy, hipStream_t s,
                          float *part, float *part_xs, int parts);

// Switch gemv=g forces the generic kernel, =m the matrix-core kernel, =d the dot-product kernels (testing and
// measurement; unset: chosen by batch and shape).
static char forced_kernel() { return switches().gemv; }
static bool force_generic() { return forced_kernel() == 'g'; }

static bool down_mfma_wanted(const Params &p, const __half *x, long long ldx, int batch) {
  const char fk = forced_kernel();
  return fk != 'g' && fk != 'd' && gemv_down_applicable(p, x, ldx) && gemv_down_mfma_applicable(p, x, ldx, batch);
}
// What `launches` launches take at least, one after another from a host's program: 4.8, 8.4, 12 us through the torch binding.  (Not in a graph, where
// a second launch is 1.6 us: layers whose parts take less than that floor would be up to 1 us faster there with them.)
static float launched(float us, int launches) { return std::max(us, 1.3f + 3.55f * (float)launches); }
// With a workspace (column parts, one workgroup per block of 16 streams and part): from two rows on, for any batch when there are codebook
// groups (16 groups, one row: 15.5 against 17.4 us), and for one row by the estimates (4096 x 4096 8.3 against 6.7 us; 4096 x 11008 10.4
// against 11.4).
// (and for one row of a layer whose activations do not fit the other kernel's LDS beside the tables)
static bool down_mfma_parts_wanted(const Params &p, const __half *x, long long ldx, int batch) {
  return down_mfma_wanted(p, x, ldx, batch) && (batch >= 2 || p.n_groups > 1 || forced_kernel() == 'm' || !gemv_down_fits(p) ||
                                                1.06f * launched(gemv_down_mfma_us(p, gemv_down_mfma_parts(p), 1), 2) < gemv_down_streams_us(p, 1));
}
static bool down_mfma_alone_wanted(const Params &p, const __half *x, long long ldx, int batch) {
  if (!down_mfma_wanted(p, x, ldx, batch)) return false;
  if (p.n_groups > 1) {
    // groups that a workgroup walks: for one row the kernel that keeps one table in LDS at a time is the other one, which pays more for a
    // group and spreads its streams (four groups, 11008 x 4096 16.7 against 19.1 us, 4096 x 4096 16.7 / 16.0, 4096 x 11008 25.7 / 21.7; sixteen
    // 45.3 / 50.7); with an 8-bit residual table it is the generic one, which pays nothing for a group (876 x 138, 18 groups 39 / 11, 8 groups 17 / 11)
    if (batch >= 2 || forced_kernel() == 'm') return true;
    const float groups = (float)p.n_groups, vectors = (float)p.S * (float)p.P * 1e-6f, walk = gemv_down_mfma_us(p, 1, 1) - 5.0f;
    if (!gemv_down_lds_applicable(p, 1)) return 1.9f * groups + walk < 1.0f + 0.03f * (float)p.P * std::max(1.0f, 1e-3f * (float)p.S);
    return (p.k_res ? 3.1f : 1.55f) * groups + walk < (p.k_res ? 5.0f : 2.5f) * groups + (p.k_res ? 1.3f : 0.65f) * vectors;
  }
  if (batch >= 5 || forced_kernel() == 'm') return true;      // (of five rows and more a launch of four is one of two)
  const float whole = gemv_down_mfma_us(p, 1, batch, false), folded = gemv_down_mfma_us(p, 1, batch);
  // (one row of 11008 x 4096, folded 9.0 us by the clock, 8.3 by the estimate, 8.7 here)
  return (folded < whole ? 1.08f : 1.02f) * folded < gemv_down_streams_us(p, batch) || 1.02f * whole < gemv_down_streams_us(p, batch);
}
// Whether parts of the columns, which a workspace is there for, are worth the second launch, or with the activations copied in front a third one
// (4096 x 4096, two rows, parts 8.4, without 8.6; 6513 x 2176, three rows 8.7 and 8.0; 539 x 3101, sixteen copied rows 13.4 and 12.0).
static bool down_mfma_parts_pay(const Params &p, int batch, bool copied) {
  if (p.n_groups > 1 || forced_kernel() == 'm' || !gemv_down_fits(p)) return true;
  const float copy = copied ? 1.8f : 0.0f;
  const int launches = copied ? 2 : 1;
  // (more than five parts spread a layer further than four folds of the columns do)
  const int n = gemv_down_mfma_parts(p);
  const float alone = launched(gemv_down_mfma_us(p, 1, batch, n <= 5) + copy, launches);
  const float parts = launched(gemv_down_mfma_us(p, n, batch) + copy, launches + 1);
  return parts < alone && (batch > 4 || 1.06f * parts < gemv_down_streams_us(p, batch) + copy);
}

// Rows that begin off sixteen bytes, which only that kernel and the one with a table in LDS at a time take as a rule: the latter where residual tables
// of 4096 entries leave the other no room for two rows (61 x 10331, eight rows 53 against 70 us, 5602 x 11375, two 36 / 39; not 1874 x 11674, two 26.5 / 24), and several rows of a
// few hundred columns with outlier columns (13521 x 366, two 10.9 / 14.9, 4439 x 463, four 12.4 / 13.7).  Of 187 other such calls the time here is
// 0.79 of that there, one row 0.73.
static bool down_table_at_a_time(const Params &p, const __half *x, long long ldx, int batch) {
  if (!((reinterpret_cast<uintptr_t>(x) & 15) || (ldx & 7)) || batch < 2 || forced_kernel() != '\0' || !gemv_down_lds_applicable(p, 1)) return false;
  return p.k_res ? p.bits_res == 12 && p.P >= 8192 && p.P < 12288 && (batch >= 3 || p.out_features >= 4096) : p.Q && p.P < 1024;
}

// Estimated time in microseconds of up to sixteen rows on the matrix cores of that orientation with a workspace (the route rules of vq_gemm); 0 for
// layers that do not go there.  (Of 150 layers, and not the finer estimates above: that line decides how a product's weights are held, and stays.)
float gemv_down_rows_us(const Params &p, const __half *x, long long ldx) {
  if (p.orientation != 1 || !down_mfma_wanted(p, x, ldx, 16)) return 0.0f;
  const int blocks = (p.S + 15) / 16, parts = gemv_down_mfma_parts(p);
  auto us = [&](int n) { return (p.k_res ? 3.0e-3f : 1.4e-3f) * (float)p.P / (float)n * (float)((blocks * n + cu_count() - 1) / cu_count()) + (n > 1 ? 2.1f : 0.0f); };
  return 6.0f + std::min(us(1), us(parts)) + (p.k_res ? 1.0f : 0.0f) + (p.Q ? 2.0f : 0.0f) + (p.n_groups > 1 ? 3.0f : 0.0f);
}

bool gemv_rows_applicable(const Params &p);
bool gemv_rows_takes(const Params &p, const __half *x, long long ldx, int batch);
int gemv_rows_parts(const Params &p);
size_t gemv_rows_workspace_bytes(const Params &p, int batch);
int launch_gemv_rows(const Params &p, const __half *x, long long ldx, int batch, __half *y, long long ldy, float *part, float *part_xs,
                     int parts_per_group, hipStream_t s, int folds = 0);
int gemv_rows_folds(const Params &p, int batch, bool parts);
// When vq_gemv_rows.hip's kernel takes over from the ones that run four (v = 8: eight) rows a launch.  Its lookups do for any number
// of rows, but a single row needs no matrix cores: from three rows on (two tables of v = 12, 6739 x 9664, 10 rows: 174 -> 22 us;
// v = 4, 448 x 1872, 3 rows: 7.7 -> 5.5 us; 2 rows: level), and
//  * for every number of rows where two tables do not fit LDS together, which the other kernels pay for in every launch (v = 12,
//    6208 x 1856, 1 row: 11.0 -> 10.5 us; 467 x 6956, 2 rows: 20 -> 12 us) -- but not with codebook groups (1 row: 12 against 18 us);
//  * orientation 1, whose workgroups take 16 streams, i.e. 16 v rows, over all the columns: with a workspace, whose parts fill the
//    chip, from two rows on (v = 12, 12275 x 1728: 18 -> 13 us), one row of at least 16384 columns (644 x 22848: 26 -> 18 us);
//    without, from two rows on where the workgroups alone are half as many as compute units, else from five (v = 12, 717 x 5520,
//    2 rows: 18 against 37 us), and where folds of the columns take the place of parts as with one (v = 2, 206 x 3308, four rows 10.1 -> 6.3 us;
//    v = 4, 3000 x 3300, two 9.9 -> 7.2; v = 6 / 256, 245 x 2394, two 8.2 -> 7.4);
//  * v = 8 with 16-bit indices, orientation 1, whose lookups go through L2: with a workspace from five rows, or two of at least
//    4096 columns, on (768 x 7872, 5 rows: 35 -> 13 us), without from nine (5 rows: 60 us).
// Switch rows=0 / rows=1: never / wherever it can.
// Whether rows that would be taken in column parts, were there a workspace, are taken in folds of the columns, which need none.
static bool folds_spare_parts(const Params &p, int batch) { return gemv_rows_parts(p) > 0 && gemv_rows_folds(p, batch, true) > 1; }
static bool rows_wanted(const Params &p, int batch, bool workspace) {
  if (switches().rows == 0 || forced_kernel() != '\0' || !gemv_rows_applicable(p)) return false;
  if (switches().rows == 1) return true;
  if (p.orientation == 1 && p.bits == 16) return batch >= (!workspace ? 9 : p.P >= 4096 ? 2 : 5);
  if (p.n_groups > 1) return batch >= 3;
  if (p.orientation == 1) {
    if (workspace || folds_spare_parts(p, batch)) return batch >= 2 || p.P >= 16384;
    return batch >= (2 * ((p.S + 15) / 16) >= cu_count() ? 2 : 5);
  }
  if (p.v == 12) return true;
  return batch >= 3;
}

// Whether vq_gemv would run this layer on the kernels that keep one table in LDS at a time (no kernel of its own, tables that fit).
bool gemv_has_lds_kernel(const Params &p, const __half *x, long long ldx) {
  if (forced_kernel() != '\0') return false;
  if (p.orientation == 1) return !gemv_down_applicable(p, x, ldx) && !gemv_v8_down_applicable(p) && gemv_down_lds_applicable(p, 1);
  return !gemv_fast_applicable(p, x, ldx) && !gemv_v8_wanted(p, x, ldx, 16, false) && gemv_lds_applicable(p, 1);
}

// Whether vq_gemv has one of its specialised kernels for this layer and these activations (vq_gemm sends small token
// counts, and layers its own kernels do not take, through vq_gemv sixteen rows at a time).
bool gemv_has_fast_kernel(const Params &p, const __half *x, long long ldx) {
  if (forced_kernel() != '\0') return false;
  if (p.orientation == 1) return down_mfma_wanted(p, x, ldx, 16) || gemv_v8_down_applicable(p);
  return gemv_fast_applicable(p, x, ldx) || gemv_v8_wanted(p, x, ldx, 16, false);
}

// Layers without a kernel of their own whose tables fit LDS (vq_gemv_lds.hip): batch rows in launches of 4, 2 or 1, fewer
// when that many activation rows do not fit beside the tables.  VQ_ERR_UNSUPPORTED when the kernel does not take the layer.
static int gemv_through_lds_tables(const Params &p, const __half *x, long long ldx, int batch, __half *y, long long ldy, hipStream_t s) {
  const bool down = p.orientation == 1;
  if (force_generic() || !(down ? gemv_down_lds_applicable(p, 1) : gemv_lds_applicable(p, 1))) return VQ_ERR_UNSUPPORTED;
  int done = 0, g_max = 4, rc = VQ_OK;
  while (done < batch) {
    int g = batch - done >= 4 ? 4 : batch - done >= 2 ? 2 : 1;
    if (g > g_max) g = g_max;
    rc = down ? launch_gemv_down_lds(p, x + done * ldx, ldx, g, y + done * ldy, ldy, s) : launch_gemv_lds(p, x + done * ldx, ldx, g, y + done * ldy, ldy, s);
    if (rc == VQ_ERR_UNSUPPORTED && g > 1) { g_max = g / 2; continue; }
    if (rc != VQ_OK) return rc;
    done += g;
  }
  return VQ_OK;
}

int launch_gemv(const Params &p, const __half *x, long long ldx, int batch, __half *y, long long ldy, hipStream_t s) {
  if (rows_wanted(p, batch, false) && gemv_rows_takes(p, x, ldx, batch)) return launch_gemv_rows(p, x, ldx, batch, y, ldy, nullptr, nullptr, 0, s);
  if (p.perm) {
    // Permuted column order without a workspace: the dot-product kernels for v = 6 gather the activations while they stage
    // them in LDS (or load them into registers: long rows); everything else runs on the generic kernels, which look every
    // activation up.
    if (p.orientation == 0 && !force_generic()) {
      if (p.in_features >= 16384 && gemv_res8_applicable(p, x) && (ldx & 1) == 0) {
        // the long-row kernel gathers into its registers; more rows one after the other (still far ahead of the generic kernel)
        int rc = VQ_OK;
        for (int t = 0; t < batch && rc == VQ_OK; ++t) rc = launch_gemv_res8(p, x + t * ldx, y + t * ldy, s);
        if (rc != VQ_ERR_UNSUPPORTED) return rc;
      }
      if (gemv_fast_applicable(p, x, ldx) && p.n_groups == 1) {
        int done = 0, rc = VQ_OK, g_max = 4;
        while (done < batch) {
          int g = batch - done >= 4 ? 4 : batch - done >= 2 ? 2 : 1;
          if (g > g_max) g = g_max;
          rc = launch_gemv_fast(p, x + done * ldx, ldx, g, y + done * ldy, ldy, s);
          if (rc == VQ_ERR_UNSUPPORTED && g > 1) { g_max = g / 2; continue; }
          if (rc != VQ_OK) break;
          done += g;
        }
        if (rc == VQ_OK) return VQ_OK;
        if (rc != VQ_ERR_UNSUPPORTED || done != 0) return rc;
      }
    }
    {
      const int rc = gemv_through_lds_tables(p, x, ldx, batch, y, ldy, s);       // gathers the activations while it stages them
      if (rc != VQ_ERR_UNSUPPORTED) return rc;
    }
    if (p.orientation == 1) hipLaunchKernelGGL(gemv_down_kernel, dim3((unsigned)((p.S + 3) / 4)), dim3(256), 0, s, p, x, ldx, batch, y, ldy);
    else hipLaunchKernelGGL(gemv_generic_kernel, dim3((unsigned)((p.out_features + 3) / 4)), dim3(256), 0, s, p, x, ldx, batch, y, ldy);
    return hipGetLastError() == hipSuccess ? VQ_OK : VQ_ERR_HIP;
  }
  // Matrix-core kernel: one launch for any batch, at about the cost of a batch-1 launch of the dot-product
  // kernels; those are still a little faster for one row (and for two rows of a layer with few output rows
  // per compute unit), so they keep these cases.  Layers with codebook groups always go to the matrix-core kernel:
  // it is the one that swaps the tables in LDS group by group.
  if (p.orientation == 1) {
    // from three to five rows on the matrix-core kernel of this orientation is ahead (six multiply-adds per gather and row
    // bind the other one); gemv=m sends every batch there, =d none
    if (down_mfma_alone_wanted(p, x, ldx, batch)) {
      const int rc = launch_gemv_down_mfma(p, x, ldx, batch, y, ldy, s, nullptr, nullptr, 1);
      if (rc != VQ_ERR_UNSUPPORTED) return rc;
    }
    if (!force_generic() && p.n_groups == 1 && gemv_down_applicable(p, x, ldx) && !down_table_at_a_time(p, x, ldx, batch)) {
      // batch rows go in groups of 4, 2 or 1 (fewer when the rows do not fit LDS beside the tables)
      int done = 0, g_max = 4, rc = VQ_OK;
      while (done < batch) {
        int g = batch - done >= 4 ? 4 : batch - done >= 2 ? 2 : 1;
        if (g > g_max) g = g_max;
        rc = launch_gemv_down(p, x + done * ldx, ldx, g, y + done * ldy, ldy, s);
        if (rc == VQ_ERR_UNSUPPORTED && g > 1) { g_max = g / 2; continue; }
        if (rc != VQ_OK) break;
        done += g;
      }
      if (rc == VQ_OK) return VQ_OK;
      if (rc != VQ_ERR_UNSUPPORTED || done != 0) return rc;
      if (down_mfma_wanted(p, x, ldx, batch)) {   // a row too long for that kernel's LDS (28672 columns beside two 64 KB tables)
        rc = launch_gemv_down_mfma(p, x, ldx, batch, y, ldy, s, nullptr, nullptr, 1);
        if (rc != VQ_ERR_UNSUPPORTED) return rc;
      }
    }
    if (!force_generic() && gemv_v8_down_applicable(p)) {
      // 8-component vectors, tables read through L2: batch rows in launches of 4, 2 or 1
      int done = 0, rc = VQ_OK;
      while (done < batch && rc == VQ_OK) {
        const int g = batch - done >= 4 ? 4 : batch - done >= 2 ? 2 : 1;
        rc = launch_gemv_v8_down(p, x + done * ldx, ldx, g, y + done * ldy, ldy, s);
        if (rc == VQ_OK) done += g;
      }
      if (rc != VQ_ERR_UNSUPPORTED || done != 0) return rc;
    }
    {
      const int rc = gemv_through_lds_tables(p, x, ldx, batch, y, ldy, s);
      if (rc != VQ_ERR_UNSUPPORTED) return rc;
    }
    hipLaunchKernelGGL(gemv_down_kernel, dim3((unsigned)((p.S + 3) / 4)), dim3(256), 0, s, p, x, ldx, batch, y, ldy);
    return hipGetLastError() == hipSuccess ? VQ_OK : VQ_ERR_HIP;
  }
  // one activation row of a long-row layer with an 8-bit residual stream (the 8192 x 28672 layer of the 70B setting): the
  // kernel that replicates the residual table in LDS and keeps the activations out of it.  Measured against the other
  // dot-product kernel: 28672 columns 33.5 against 37.0 us; 8192 columns 16.0 against 14.7 us, hence the threshold
  // (gemv=d takes it for every layer it accepts, for the tests).
  if (batch == 1 && gemv_res8_applicable(p, x) && ((forced_kernel() == '\0' && p.in_features >= 16384) || forced_kernel() == 'd')) {
    const int rc = launch_gemv_res8(p, x, y, s);
    if (rc != VQ_ERR_UNSUPPORTED) return rc;
  }
  const bool fast = !force_generic() && gemv_fast_applicable(p, x, ldx);
  const bool many_rows = p.out_features > 16 * 256;
  // (and layers with outlier columns, whose part of the dot-product kernels is the slower one: 11008 x 4096 with 128 of
  // them, one row: 10.7 against 17.1 us; from 16384 columns on a single row is level or a little behind)
  const bool outliers_first = p.Q > 0 && (batch >= 2 || p.in_features < 16384);
  if (fast && forced_kernel() != 'd' && (batch >= 3 || (batch == 2 && many_rows) || forced_kernel() == 'm' || p.n_groups > 1 || outliers_first)) {
    const int rc = launch_gemv_mfma(p, x, ldx, batch, y, ldy, s);
    if (rc != VQ_ERR_UNSUPPORTED) return rc;
  }
  if (fast && p.n_groups == 1) {
    // batch rows go in groups of 4, 2 or 1; every group streams the indices once
    int done = 0, rc = VQ_OK;
    int g_max = 4;                      // largest group the layer's plan admits (found on the first group)
    while (done < batch) {
      int g = batch - done >= 4 ? 4 : batch - done >= 2 ? 2 : 1;
      if (g > g_max) g = g_max;
      rc = launch_gemv_fast(p, x + done * ldx, ldx, g, y + done * ldy, ldy, s);
      if (rc == VQ_ERR_UNSUPPORTED && g > 1) { g_max = g / 2; continue; }
      if (rc != VQ_OK) break;
      done += g;
    }
    if (rc == VQ_OK) return VQ_OK;
    if (rc != VQ_ERR_UNSUPPORTED || done != 0) return rc;
    if (forced_kernel() != 'd') {       // a shape the dot-product kernels do not take
      rc = launch_gemv_mfma(p, x, ldx, batch, y, ldy, s);
      if (rc != VQ_ERR_UNSUPPORTED) return rc;
    }
  }
  if (!force_generic() && gemv_v8_wanted(p, x, ldx, batch, false)) {
    // 8-component vectors, tables read through L2: batch rows in launches of 8, 4, 2 or 1
    int done = 0, rc = VQ_OK;
    while (done < batch && rc == VQ_OK) {
      const int g = batch - done >= 8 ? 8 : batch - done >= 4 ? 4 : batch - done >= 2 ? 2 : 1;
      rc = launch_gemv_v8(p, x + done * ldx, ldx, g, y + done * ldy, ldy, s);
      if (rc == VQ_OK) done += g;
    }
    if (rc != VQ_ERR_UNSUPPORTED || done != 0) return rc;
  }
  {
    const int rc = gemv_through_lds_tables(p, x, ldx, batch, y, ldy, s);
    if (rc != VQ_ERR_UNSUPPORTED) return rc;
  }
  const unsigned blocks = (unsigned)((p.out_features + 3) / 4);
  hipLaunchKernelGGL(gemv_generic_kernel, dim3(blocks), dim3(256), 0, s, p, x, ldx, batch, y, ldy);
  return hipGetLastError() == hipSuccess ? VQ_OK : VQ_ERR_HIP;
}

size_t gemv_mfma_groups_workspace_bytes(const Params &p, int batch);
int launch_gemv_mfma_groups(const Params &p, const __half *x, long long ldx, int batch, __half *y, long long ldy, void *workspace,
                            hipStream_t s);

// A workspace serves layers with codebook groups on the matrix-core kernel: one group per workgroup, then a sum over
// the groups.  groups=loop keeps every workgroup walking all groups (measurement and tests).
// Layers with a permuted column order: the activations, gathered into stored order, come first in the workspace
// (batch rows of in_features rounded up to 8 halfs, the whole rounded up to 256 bytes); the rest is what the layer needs
// without the permutation.
static size_t permuted_x_bytes(const Params &p, int rows) { return ((size_t)rows * (size_t)((p.in_features + 7) & ~7) * sizeof(__half) + 255) / 256 * 256; }
// One row of a layer that the gathering dot-product kernel takes is faster without the extra launch, as long as the row
// is short: every workgroup gathers the whole row (64 lookups a wave instruction), a gather kernel does it once.
static bool permuted_in_kernel(const Params &p, const __half *x, long long ldx, int batch) {
  return batch == 1 && p.orientation == 0 && p.n_groups == 1 && forced_kernel() != 'm' && p.in_features < 16384 && gemv_fast_applicable(p, x, ldx);
}

// Rows of an odd width start between dwords for all but the first: the kernel that wants dwords has them copied, which costs 2 us
// (v = 12, 305 x 1281, 2 rows: 10.4 us, 11.1 with the copy).  (The copy counts as workspace, and of rows beyond 2^18 columns it could ask
// for more than vq_gemv_static_workspace has, which would refuse a layer that needs none.)
// The v = 6 / 12-bit kernels want dwords at any number of rows, those along the rows an even width as well: there the copy's next column, zeros,
// counts as the layer's last (P is the same: an odd width is short of whole vectors).  3520 x 6587, 1 / 4 / 16 rows: 9.7 -> 7.9, 18.3 -> 9.2, 71 -> 11.2 us;
// down the outputs, in column parts, 4 / 16 rows 20.7 -> 10.5, 80.6 -> 12.4 (without parts 16.0, 17.5).
// Not along the rows where the kernels that keep one table in LDS at a time are as fast without the copy.  With one group (450 layers of 1024
// to 14336 outputs, 65 to 1400 columns): one and two short rows, which take them no longer than the copy (one of 12461 x 193 7.4 us, 9.3 with it, of 3589 x
// 557 5.7 / 6.2, of 735 x 1089 9.0 / 6.7; three rows and more, of any width, are two launches there: 0.2 to 0.6 of the time with the copy).  With
// codebook groups (430 layers of 256 to 14336 outputs, 300 to 28672 columns, 2 to 24 groups; there the groups are side by side either way): two rows and
// four, which they take in one launch, by the estimates below, which cost 0.7 % over the better choice where the copy always costs 12 and never 25 (two
// rows of 12996 x 2263 in 16 groups 21 / 55, of 2836 x 27149 in four 36 / 15.5, four of 2068 x 26017 in four with two tables 82 / 28); other
// numbers of rows only where outlier columns stand beside groups of few vectors (three of 9098 x 1467 in 16 groups 25 / 43, of 12378 x 437 in four
// 18.4 / 21.7).  For residual tables of 8-bit indices there is only the generic kernel without it (two of 8181 x 3129 in groups, 0.31 of its time).
static bool groups_taken_odd(const Params &p, int batch) {
  if (batch != 2 && batch != 4) return batch < 6 && p.Q && p.Pg <= 32;
  const float vectors = (float)p.out_features * (float)p.P * 1e-6f, sums = (float)p.out_features * (float)p.n_groups * 1e-4f, columns = (float)p.in_features * 1e-4f;
  const float groups = (float)p.n_groups, outliers = p.Q ? 1.0f : 0.0f;
  const float copied = p.k_res ? 10.1f + 0.95f * vectors + 1.8f * sums + 0.65f * columns + 1.5f * outliers + 0.18f * groups
                               : 9.2f + 0.5f * vectors + 0.7f * sums + 0.35f * columns + 1.5f * outliers + 0.13f * groups;
  if (batch == 2)
    return (p.k_res ? 7.7f + 2.0f * vectors + 0.4f * sums + 1.3f * columns + 0.8f * outliers + 0.25f * groups
                    : 8.3f + 0.93f * vectors + 0.2f * sums + 1.6f * columns + 0.3f * outliers + 0.06f * groups) < copied;
  return (p.k_res ? 7.6f + 3.0f * vectors + 0.5f * sums + 5.4f * columns + 1.1f * outliers + 0.26f * groups
                  : 8.6f + 1.2f * vectors + 0.4f * sums + 5.8f * columns + 0.4f * outliers) < copied;
}
static bool even_width_wanted(const Params &p, int batch) {
  if (p.orientation != 0 || !(p.in_features & 1) || !gemv_fast_applicable_even(p)) return false;
  if (p.k_res && p.bits_res == 8) return true;
  if (p.n_groups > 1) return batch >= 2 && !groups_taken_odd(p, batch);
  return batch >= 3 || p.in_features >= (batch == 2 && p.Q ? 400 : p.k_res ? 512 : batch == 2 ? 700 : 1024);
}
static size_t stored_order_workspace_bytes(const Params &p, const __half *x, long long ldx, int batch, bool least, bool copied);
static Params gathered(const Params &p, int batch) {
  Params q = p;
  q.perm = nullptr;
  if (even_width_wanted(p, batch)) ++q.in_features;
  return q;
}
// (of 2^17 vectors and more, which take longer than the copy; and not where the copy and the sums are more than vq_gemv_static_workspace has)
static bool rows_gathered(const Params &p, int batch) {
  if (!(p.in_features & 1) || p.in_features >= (1 << 18) || forced_kernel() != '\0') return false;
  if (batch >= 5 && rows_wanted(p, batch, true)) return true;
  if ((long long)p.S * p.P < 1 << 17 || !((even_width_wanted(p, batch) && (batch >= 2 || p.n_groups == 1)) || (batch >= 2 && down_mfma_wanted(p, nullptr, p.in_features + 1, batch)))) return false;
  return permuted_x_bytes(p, batch) + stored_order_workspace_bytes(gathered(p, batch), nullptr, (p.in_features + 7) & ~7, batch, false, false) <= VQ_GEMV_STATIC_WORKSPACE_BYTES;
}
// ... unless the rows can be taken as they are
static bool taken_as_they_are(const Params &p, const __half *x, long long ldx, int batch) {
  if (even_width_wanted(p, batch)) return false;
  return down_mfma_wanted(p, nullptr, p.in_features + 1, batch) ? down_mfma_wanted(p, x, ldx, batch) : gemv_rows_takes(p, x, ldx, batch);
}

size_t gemv_products_workspace_bytes(const Params &p, int batch);
int launch_gemv_products(const Params &p, const __half *x, long long ldx, int batch, __half *y, long long ldy, void *workspace, size_t workspace_bytes,
                         hipStream_t s);

// (the outlier columns are one more set of sums to add up)
static size_t down_parts_bytes(const Params &p, int batch) {
  const int parts = gemv_down_mfma_parts(p);
  return parts > 1 ? ((size_t)(parts + (p.Q ? 1 : 0)) * ((size_t)batch * (size_t)p.out_features + 16) * sizeof(float) + 255) / 256 * 256 : 0;
}
static size_t stored_order_workspace_bytes(const Params &p, const __half *x, long long ldx, int batch, bool least, bool copied) {
  if (rows_wanted(p, batch, true) && (batch == 1 || !(ldx & 1))) {
    // (0 with codebook groups that the kernel walks by itself: the slots of the kernels below are asked for instead, which run where
    // this one does not take x)
    const size_t need = gemv_rows_workspace_bytes(p, batch);
    if (need) return folds_spare_parts(p, batch) ? 0 : need;
  }
  if (p.orientation == 1 && down_mfma_parts_wanted(p, x, ldx, batch)) {   // the matrix cores: the workspace lets parts of the columns run side by side
    return gemv_down_mfma_parts(p) > 1 && down_mfma_parts_pay(p, batch, copied) ? down_parts_bytes(p, batch) : 0;
  }
  if (p.orientation == 1) {         // vectors down the output dimension: the same workspace layout, filled by that orientation's kernel
    if (p.n_groups > 1 && p.n_groups <= 256 && gemv_down_applicable(p, x, ldx))
      return ((size_t)(p.n_groups + (p.Q ? 1 : 0)) * ((size_t)batch * (size_t)p.out_features + 16) * sizeof(float) + 255) / 256 * 256;
    // (the other settings, on the kernel that keeps one table in LDS at a time: a group per workgroup)
    return gemv_down_applicable(p, x, ldx) || gemv_v8_down_applicable(p) ? 0 : gemv_down_lds_slots_workspace_bytes(p, batch);
  }
  if (!gemv_fast_applicable(p, x, ldx))       // the LDS-table kernels, when the layer gets that far: a slot per workgroup
    return gemv_v8_wanted(p, x, ldx, batch, true) ? 0 : gemv_lds_slots_workspace_bytes(p, batch, least);
  if (forced_kernel() == 'd') return 0;
  return gemv_mfma_groups_workspace_bytes(p, batch);
}

// Of a call with exactly these rows.  least: the fewest bytes that it makes use of.
static size_t workspace_bytes_of(const Params &p, const __half *x, long long ldx, int batch, bool least) {
  if (force_generic()) return 0;
  if (p.perm || rows_gathered(p, batch)) {
    if (p.perm && permuted_in_kernel(p, x, ldx, batch)) return 0;
    const Params q = gathered(p, batch);
    const size_t head = permuted_x_bytes(p, batch), rest = stored_order_workspace_bytes(q, nullptr, (p.in_features + 7) & ~7, batch, least, p.perm != nullptr);
    // (the column parts of vq_gemv_rows.hip are done without where the two together are more than vq_gemv_static_workspace has)
    return rows_wanted(q, batch, true) && head + rest > VQ_GEMV_STATIC_WORKSPACE_BYTES ? head : head + rest;
  }
  return stored_order_workspace_bytes(p, x, ldx, batch, least, false);
}

// (One and two rows of a layer with two tables a group take a slot a table, whose workspace may be larger than that of three rows, which
// another kernel takes.  What holds a slot a group of fewer rows is made to hold that, so that a loop can lend its calls the workspace of the
// largest batch.  For the same loop: down the outputs other rows may be taken in parts of the columns where these, whose folds or launch
// without parts are estimated to be as fast, are not.  They ask for what fewer rows do; v = 6 for what parts of its own would.)
static size_t other_workspace_bytes(const Params &p, const __half *x, long long ldx, int batch) {
  const size_t own = workspace_bytes_of(p, x, ldx, batch, false);
  size_t bytes = own;
  if (p.orientation == 0 && p.k_res && p.n_groups > 1)
    for (int rows = 1; rows < batch; ++rows)
      if (own >= workspace_bytes_of(p, x, ldx, rows, true)) bytes = std::max(bytes, workspace_bytes_of(p, x, ldx, rows, false));
  if (p.orientation == 1 && p.n_groups == 1) {
    const size_t copy = p.perm || rows_gathered(p, batch) ? permuted_x_bytes(p, batch) : 0;
    if (own > copy) return own;
    const Params q = copy ? gathered(p, batch) : p;
    if (down_mfma_parts_wanted(q, copy ? nullptr : x, copy ? (p.in_features + 7) & ~7 : ldx, batch)) return copy + down_parts_bytes(q, batch);
    for (int rows = 1; rows < batch; ++rows) bytes = std::max(bytes, workspace_bytes_of(p, x, ldx, rows, false));
  }
  return bytes;
}
// (one and two rows from tables of products, vq_gemv_products.hip, may take more than the other kernels do of more rows; for the same loop that is
// part of what more rows ask for)
size_t gemv_workspace_bytes(const Params &p, const __half *x, long long ldx, int batch) {
  size_t bytes = other_workspace_bytes(p, x, ldx, batch);
  for (int rows = 1; rows <= std::min(batch, 2); ++rows) bytes = std::max(bytes, gemv_products_workspace_bytes(p, rows));
  return bytes;
}

// The same for one call of exactly these rows, to which nothing is lent that its kernels leave alone (v = 12, two tables, two rows and more: tables
// of products are one row's; 11008 x 4096, 16 rows: 1.9 MB).
size_t gemv_lent_bytes(const Params &p, int batch) {
  const long long ldx = p.in_features + (p.in_features & 1);
  if (p.orientation == 1 && p.n_groups == 1) return workspace_bytes_of(p, nullptr, ldx, batch, false);
  return gemv_products_workspace_bytes(p, batch) || workspace_bytes_of(p, nullptr, ldx, batch, false) ? gemv_workspace_bytes(p, nullptr, ldx, batch) : 0;
}

// Sums of `slots` parts, groups or tables, and those of the activations, in front of a second launch that adds them up.
static size_t sums_bytes(const Params &p, size_t slots, int batch) { return slots * ((size_t)batch * (size_t)p.out_features + 16) * sizeof(float); }

static int launch_stored_order(const Params &p, const __half *x, long long ldx, int batch, __half *y, long long ldy, void *workspace,
                               size_t workspace_bytes, bool least, bool copied, hipStream_t s);
static int launch_with_workspace(const Params &p, const __half *x, long long ldx, int batch, __half *y, long long ldy, void *workspace,
                                 size_t workspace_bytes, bool least, hipStream_t s) {
  if (p.perm || (rows_gathered(p, batch) && !taken_as_they_are(p, x, ldx, batch))) {
    const size_t need = workspace_bytes_of(p, x, ldx, batch, least);
    if (!need || !workspace || workspace_bytes < need) return launch_gemv(p, x, ldx, batch, y, ldy, s);
    // gather the activations into stored order, then the layer is an unpermuted one
    const Params q = gathered(p, batch);
    __half *xp = static_cast<__half *>(workspace);
    const long long ldxp = (p.in_features + 7) & ~7;
    // (in one launch of the LDS-table kernel the workgroups gather theirs by themselves: a group's columns, in the shade of its table)
    if (p.perm && batch <= 4 && batch != 3 && p.orientation == 0 && !rows_wanted(q, batch, true) && !gemv_fast_applicable(q, xp, ldxp) && !switches().groups_loop) {
      const size_t head = permuted_x_bytes(p, batch), slot_bytes = gemv_lds_slots_workspace_bytes(q, batch, true);
      if (slot_bytes && workspace_bytes - head >= slot_bytes) {
        float *part = reinterpret_cast<float *>(static_cast<unsigned char *>(workspace) + head);
        int slots;
        const int rc = launch_gemv_lds_slots(p, x, ldx, batch, part, workspace_bytes - head, &slots, s);
        if (rc == VQ_OK) return launch_groups_finish(part, part + (size_t)slots * (size_t)batch * (size_t)p.out_features, slots, batch, p, y, ldy, s);
        if (rc != VQ_ERR_UNSUPPORTED) return rc;
      }
    }
    const int rc = launch_gather_cols(x, ldx, batch, p.in_features, p.perm, xp, ldxp, s);
    if (rc != VQ_OK) return rc;
    const size_t head = permuted_x_bytes(p, batch);
    return launch_stored_order(q, xp, ldxp, batch, y, ldy, static_cast<unsigned char *>(workspace) + head, workspace_bytes - head, false, true, s);
  }
  return launch_stored_order(p, x, ldx, batch, y, ldy, workspace, workspace_bytes, least, false, s);
}

// Activations that are taken as they are, in stored order (the caller's, or the copy of them in front of this workspace).  Every branch compares
// the workspace with what its kernels write.
static int launch_stored_order(const Params &p, const __half *x, long long ldx, int batch, __half *y, long long ldy, void *workspace,
                               size_t workspace_bytes, bool least, bool copied, hipStream_t s) {
  const size_t need = force_generic() ? 0 : stored_order_workspace_bytes(p, x, ldx, batch, least, copied);
  if (rows_wanted(p, batch, workspace != nullptr) && gemv_rows_takes(p, x, ldx, batch)) {
    const int per_group = workspace && workspace_bytes >= gemv_rows_workspace_bytes(p, batch) ? gemv_rows_parts(p) : 0, parts = per_group * p.n_groups;
    const int folds = parts ? gemv_rows_folds(p, batch, true) : 0;
    if (parts == 0 || folds > 1) return launch_gemv_rows(p, x, ldx, batch, y, ldy, nullptr, nullptr, 0, s, folds);
    float *part = static_cast<float *>(workspace), *part_xs = part + (size_t)parts * (size_t)batch * (size_t)p.out_features;
    const int rc = launch_gemv_rows(p, x, ldx, batch, nullptr, 0, part, part_xs, per_group, s);
    return rc == VQ_OK ? launch_groups_finish(part, part_xs, parts, batch, p, y, ldy, s) : rc;
  }
  if (need && workspace && workspace_bytes >= need && p.orientation == 1 && down_mfma_parts_wanted(p, x, ldx, batch)) {
    const int parts = gemv_down_mfma_parts(p), slots = parts + (p.Q ? 1 : 0);
    if (parts < 2 || workspace_bytes < sums_bytes(p, slots, batch) || !down_mfma_parts_pay(p, batch, copied)) return launch_gemv(p, x, ldx, batch, y, ldy, s);
    float *part = static_cast<float *>(workspace), *part_xs = part + (size_t)slots * (size_t)batch * (size_t)p.out_features;
    int rc = launch_gemv_down_mfma(p, x, ldx, batch, nullptr, 0, s, part, part_xs, parts);
    if (rc == VQ_OK) return launch_groups_finish(part, part_xs, slots, batch, p, y, ldy, s);
    if (rc != VQ_ERR_UNSUPPORTED) return rc;
  } else if (need && workspace && workspace_bytes >= need && p.orientation == 1 && !gemv_down_applicable(p, x, ldx)) {
    if (!switches().groups_loop && workspace_bytes >= sums_bytes(p, p.n_groups, batch)) {      // the LDS-table kernel of this orientation: a group per workgroup
      float *part = static_cast<float *>(workspace), *part_xs = part + (size_t)p.n_groups * (size_t)batch * (size_t)p.out_features;
      const int rc = launch_gemv_down_lds_slots(p, x, ldx, batch, part, part_xs, s);
      if (rc == VQ_OK) return launch_groups_finish(part, part_xs, p.n_groups, batch, p, y, ldy, s);
      if (rc != VQ_ERR_UNSUPPORTED) return rc;
    }
  } else if (need && workspace && workspace_bytes >= need && p.orientation == 1) {
    const int slots = p.n_groups + (p.Q ? 1 : 0);             // the outlier columns are one more set of sums to add up
    if (workspace_bytes < sums_bytes(p, slots, batch)) return launch_gemv(p, x, ldx, batch, y, ldy, s);
    float *part = static_cast<float *>(workspace), *part_xs = part + (size_t)slots * (size_t)batch * (size_t)p.out_features;
    int done = 0, g_max = 4, rc = VQ_OK;
    while (done < batch) {                                // batch rows in launches of 4, 2 or 1, as without groups
      int g = batch - done >= 4 ? 4 : batch - done >= 2 ? 2 : 1;
      if (g > g_max) g = g_max;
      rc = launch_gemv_down(p, x + done * ldx, ldx, g, nullptr, 0, s, part + (size_t)done * p.out_features, part_xs + done, batch);
      if (rc == VQ_ERR_UNSUPPORTED && g > 1) { g_max = g / 2; continue; }
      if (rc != VQ_OK) break;
      done += g;
    }
    if (rc == VQ_OK) return launch_groups_finish(part, part_xs, slots, batch, p, y, ldy, s);
    if (rc != VQ_ERR_UNSUPPORTED || done != 0) return rc;
  } else if (need && workspace && workspace_bytes >= need && !gemv_fast_applicable(p, x, ldx)) {
    const size_t slot_bytes = gemv_lds_slots_workspace_bytes(p, batch, true);
    if (!switches().groups_loop && slot_bytes && workspace_bytes >= slot_bytes) {
      float *part = static_cast<float *>(workspace);
      int slots;                                                   // (the outlier columns as a rule are one more)
      const int rc = launch_gemv_lds_slots(p, x, ldx, batch, part, workspace_bytes, &slots, s);
      if (rc == VQ_OK) return launch_groups_finish(part, part + (size_t)slots * (size_t)batch * (size_t)p.out_features, slots, batch, p, y, ldy, s);
      if (rc != VQ_ERR_UNSUPPORTED) return rc;
    }
  } else if (need && workspace && workspace_bytes >= std::max(need, gemv_mfma_groups_workspace_bytes(p, batch)) && !switches().groups_loop) {
    const int rc = launch_gemv_mfma_groups(p, x, ldx, batch, y, ldy, workspace, s);
    if (rc != VQ_ERR_UNSUPPORTED) return rc;
  }
  return launch_gemv(p, x, ldx, batch, y, ldy, s);
}

int launch_gemv_ws(const Params &p, const __half *x, long long ldx, int batch, __half *y, long long ldy, void *workspace,
                   size_t workspace_bytes, hipStream_t s) {
  const long long even = p.in_features + (p.in_features & 1);
  // (down the outputs what is asked for beyond the bytes of these rows is for others)
  const bool down = p.orientation == 1 && p.n_groups == 1;
  const bool enough = workspace && workspace_bytes >= (down ? workspace_bytes_of(p, nullptr, even, batch, false) : gemv_workspace_bytes(p, nullptr, even, batch));
  if (enough) {
    const int rc = launch_gemv_products(p, x, ldx, batch, y, ldy, workspace, workspace_bytes, s);
    if (rc != VQ_ERR_UNSUPPORTED) return rc;
  }
  // less than vq_gemv_workspace_bytes asks for, though not for these rows alone: vq_gemv
  if (workspace && !enough && !down && workspace_bytes >= workspace_bytes_of(p, nullptr, even, batch, false)) return launch_gemv(p, x, ldx, batch, y, ldy, s);
  // (rows of an odd width may go to other kernels than the size was asked for, which make do with what it is)
  return launch_with_workspace(p, x, ldx, batch, y, ldy, workspace, workspace_bytes, enough && !p.perm && (ldx & 1), s);
}

int launch_gemv_mfma_multi(const Params *ps, int n, const __half *x, long long ldx, int batch, __half *const *ys,
                           const long long *ldys, hipStream_t s);
int launch_gemv_fast_multi(const Params *ps, int n, const __half *x, __half *const *ys, hipStream_t s);
int launch_gemv_down_mfma_multi(const Params *ps, int n, const __half *x, long long ldx, int batch, __half *const *ys,
                                const long long *ldys, hipStream_t s);

// Several layers on the same activations: one launch of the dot-product kernel (one row) or of the matrix-core kernel
// (more rows; gemv=m: always) when all of them take it together, else (and with multi=0, for measurement and tests) one vq_gemv after the other.
int launch_gemv_multi(const Params *ps, int n, const __half *x, long long ldx, int batch, __half *const *ys, const long long *ldys,
                      hipStream_t s) {
  bool fused = n >= 2 && !switches().multi_off && forced_kernel() != 'g' && forced_kernel() != 'd';
  for (int i = 0; i < n; ++i) fused = fused && !ps[i].perm;      // permuted column orders: one layer after the other
  // layers with vectors down the output dimension: the matrix-core kernel of that orientation, any batch (a block of 16
  // streams per workgroup over all columns; the blocks of all the layers together are what fills the chip)
  bool down = fused;
  for (int i = 0; down && i < n; ++i) down = ps[i].orientation == 1 && ps[i].n_groups == 1 && down_mfma_wanted(ps[i], x, ldx, batch);
  if (down) {
    const int rc = launch_gemv_down_mfma_multi(ps, n, x, ldx, batch, ys, ldys, s);
    if (rc != VQ_ERR_UNSUPPORTED) return rc;
  }
  for (int i = 0; fused && i < n; ++i) fused = gemv_fast_applicable(ps[i], x, ldx);
  if (fused && batch == 1 && forced_kernel() != 'm') {     // a single row: the dot-product kernel is the faster body
    const int rc = launch_gemv_fast_multi(ps, n, x, ys, s);
    if (rc != VQ_ERR_UNSUPPORTED) return rc;
  }
  if (fused) {
    const int rc = launch_gemv_mfma_multi(ps, n, x, ldx, batch, ys, ldys, s);
    if (rc != VQ_ERR_UNSUPPORTED) return rc;
  }
  for (int i = 0; i < n; ++i) {
    const int rc = launch_gemv(ps[i], x, ldx, batch, ys[i], ldys[i], s);
    if (rc != VQ_OK) return rc;
  }
  return VQ_OK;
}

}  // namespace vq
