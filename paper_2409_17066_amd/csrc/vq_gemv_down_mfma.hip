// vq_gemv on the matrix cores for layers whose vectors run down the output dimension (orientation 1: the paper's own
// layout, Sec. 3.1 and Algorithm 1), v = 6, 12-bit indices, optional 12- or 8-bit residual codebook, outlier columns,
// any batch up to 16 in one launch (App. "Our Dequantization Implementation", second phase), one or more codebook groups.
//
// In this layout a gathered centroid meets ONE activation and feeds six output rows, y[6p + j] += C[I[p][n]][j] * x[n]: on the vector ALUs
// six multiply-adds per gather and token.  A lane looks up eight neighbouring columns of stream (l & 15); element j of those eight
// entries, put together with four byte permutes, is operand A of v_mfma_f32_16x16x32_f16 for output row j of sixteen streams and 32
// columns, and operand B are the token's eight activations as they lie in memory.  So a window takes six instructions (twelve with a
// residual table) and 24 (48) permutes at any number of tokens up to 16, and a lane gets row j of four streams for its token.
// (Before, operand A was the entry and operand B the activations in six places among zeros, ceil(6 batch / 16) instructions a column of entries
// and three permutes each: sixteen rows, 11008 x 4096 with column parts 18.4 -> 12.5 us, four 11.3 -> 9.9; two 4096-entry tables, without
// parts, 4096 x 11008, 93 -> 38 and 40 -> 37; a whole decoder layer, sixteen rows 89 -> 52 us, with residual tables 125 -> 70.)
//
// What bounds it: eleven of the 17 thousand clocks of 11008 x 4096 in two parts were the windows', 160 of a compute unit each, of which LDS
// takes 106 for the lookups; the rest is the start-up, tables first.  Folds of the columns (LOG_FOLDS below) in place of two to five parts spare the second
// launch: four rows 10.4 -> 9.5 us.  Without a workspace, where blocks of sixteen streams left compute units idle, 10.8 -> 9.1, 4096 x 11008 with two tables
// 37.8 -> 16.5, 8192 x 28672 48.4 -> 26.7.  Sixteen waves instead of eight (9.9 -> 10.8 us) and lookups a window ahead of the products (10.3) are slower.
//
// Work split: a workgroup of eight waves owns one block of 16 index streams (96 output rows) and one part of the
// columns; wave w takes the part's windows w, w + 8, ... of 32 columns (eight per lane: 96 index bits, three aligned
// dwords; its eight activations of its token are one 16-byte load, read straight from memory -- they are hits in L2 --
// with range-checked buffer loads).  Index words and activations run a few windows ahead in a register ring.  At the
// end the waves' 16 x 16 sums per output row of the streams meet in LDS, in the space of the tables, which are no longer needed.
// With one part the workgroup applies y = scale * sum + bias * sum(x) itself; a block of 16 streams is a coarse unit,
// though (a 4096 x 4096 layer has 43 of them for 256 compute units), so up to eight rows may take half of one or a quarter, the columns in folds, and
// where that is not enough and the caller lends a workspace the columns
// are cut into parts, every (block, part) is a workgroup, the binary32 sums go to the workspace [part][token][row] and
// the kernel that adds up codebook groups (vq_gemv_mfma.hip) adds up the parts.  Codebook groups (Sec. 3.1: ranges of
// columns with tables of their own) are parts by nature -- a part stages the tables of its group -- and are cut further
// the same way; without a workspace the workgroup of a block walks the groups one after the other, swapping the tables
// in LDS, with its sums running on.
#include "vq_common.hpp"
#include "vq_v6.hpp"

namespace vq {
namespace {

using namespace v6;

constexpr int MW = 8;            // waves per workgroup
constexpr int VPL = 8;           // columns per lane and window

typedef _Float16 half8v __attribute__((ext_vector_type(8)));
typedef float float4v __attribute__((ext_vector_type(4)));

struct DownMfmaPlan {
  int ksplit;                    // parts of the columns; grid = blocks of 16 streams x ksplit
  int sub;                       // parts per codebook group: ksplit = groups x sub
  int wpp;                       // 32-column windows per part
  int batch;
  unsigned x_bytes;              // from x[0][0] to the end of the last token's row
  float *part, *part_xs;         // workspace [part][batch][out_features], [part * 16 + token]; nullptr: one part, the kernel stores y
  // outlier columns: the workgroup's rows of them as a dense tile in LDS
  unsigned lds_o;                // [OROWS][o_pitch] dwords of weights, [16][o_pitch] of activations, [16][OROWS] sums, [16] activation sums
  int o_pitch;                   // dwords per tile row: ceil(Q / 2), made odd (rows then start in different banks)
  int o_rpw;                     // with a workspace: rows per workgroup (the rows are dealt out to all workgroups of the launch)
};

constexpr int OROWS = 96;        // rows of outlier sums a workgroup works out: its own block's, or its share of all rows (never more)

__device__ __forceinline__ float4v mfma16(uint4v a, uint4v b, float4v c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(half8v, a), __builtin_bit_cast(half8v, b), c, 0, 0, 0);
}

// WALK: the instantiation for layers with codebook groups and no workspace, whose workgroups walk all groups; the others
// take one group (or the only one) and have no loop around the start-up (with the loop in every instantiation the
// single-group ones lost up to 4 us on a 4096 x 4096 layer in 16 groups: registers held across the loop edge).
// `wg` is the workgroup's number within its layer (a launch may hold the workgroups of several layers).
// FEW: up to two tokens of a layer with a residual table: 48 permutes a window are more than those tokens are worth.  Operand A is the entry as it
// is, operand B has (token, row) pairs for columns, the activation in place j of eight for row j and zeros elsewhere, and serves both tables: 16
// instructions and 24 permutes a window (two rows, 384 x 18752 13.1 -> 12.6 us; a decoder layer's one row, 832 and 2752 wide, 33.9 -> 33.1).
// LOG_FOLDS: rows 0..15 of operand A, and columns 0..15 of operand B, are (stream or token, fold) pairs: a block has 16, 8 or 4 streams and their
// columns come in one, two or four folds, window w of a fold being window w * folds + fold of the stream.  Of a result only what has the same fold on
// both sides counts, and the folds' sums are added where the waves meet.  Up to eight (four) tokens find room beside one another, and a layer has
// twice (four times) as many blocks of half (a quarter) the windows, without a second launch to add parts of the columns up.
template <int RES_BITS, bool WALK, bool FEW, int LOG_FOLDS>
__device__ __forceinline__ void gemv_down_mfma_body(const Params &p, const DownMfmaPlan &plan, const __half *__restrict__ x, long long ldx,
                                                    __half *__restrict__ y, long long ldy, int wg) {
  typedef Layout<RES_BITS> LY;
  constexpr int RB = RES_BITS ? RES_BITS : 8;
  constexpr int NR = RES_BITS == 12 ? 3 : 2;             // dwords of a lane's residual indices
  constexpr int FOLDS = 1 << LOG_FOLDS, STREAMS = 16 / FOLDS;
  // (measured: in the few windows of a part a deeper ring only adds start-up loads; with folds, whose waves have a whole row's, two windows ahead
  // 11008 x 4096, four rows, streams in memory 9.7 -> 9.5 us, 8192 x 28672 28.0 -> 26.7, four 9.8; not beside a residual table, 698 x 1216 8.6 -> 9.0)
  constexpr int DEPTH = FOLDS > 1 && RES_BITS == 0 ? 2 : 1;
  extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
  const int lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  static_assert(!(FEW && FOLDS > 1), "FEW has other columns in operand B");
  const int n = lane & 15, g = lane >> 4;                // A: stream n of the block, column group g.  B: token n.  D: token n, streams 4g..4g+3
  const int fold = n / STREAMS;
  constexpr int PLANES = FEW ? 1 : 6;                    // sums a lane holds of its four streams
  const int token = FEW ? n / 6 : n % STREAMS;
  const int blk = wg / plan.ksplit, part_i = wg - blk * plan.ksplit;
  // A part belongs to one codebook group; without a workspace the workgroup walks all groups, one set of tables after the
  // other in LDS, and its sums simply keep running (the tables change with the column, the output rows do not).
  const int g_lo = plan.part ? part_i / plan.sub : 0, g_hi = WALK ? p.n_groups : g_lo + 1;
  const int sub_i = plan.part ? part_i - g_lo * plan.sub : 0;
  const bool need_xs = plan.part == nullptr || blk == 0;

  // ---- outlier columns (Sec. 3.2.3; any v_out and k_out; their index streams belong to blocks of v_out rows): few columns, so
  // the workgroup's rows of them are restored into a dense tile in LDS -- every (row, column) is independent: one trip to the
  // index streams, one to the table, for all of them at once -- and multiplied from there once the barrier below has passed.
  // Without a workspace the rows are the block's own and their sums wait in LDS for the end; with one, the outlier columns
  // are one more part of the workspace and every workgroup of the launch takes a share of ALL rows.
  const int o_row_lo = plan.part ? wg * plan.o_rpw : blk * (STREAMS * 6);
  const int o_rows = p.Q ? max(0, min(plan.part ? plan.o_rpw : STREAMS * 6, p.out_features - o_row_lo)) : 0;
  const int Q2 = 2 * plan.o_pitch;                       // halves per tile row
  unsigned short *o_tile = reinterpret_cast<unsigned short *>(lds + plan.lds_o);
  unsigned short *o_x = o_tile + OROWS * Q2;
  float *o_sum = reinterpret_cast<float *>(o_x + 16 * Q2), *o_xs = o_sum + 16 * OROWS;
  const unsigned st_main = (unsigned)p.stride, st_res = (unsigned)p.stride_res;
  const __amdgpu_buffer_rsrc_t r_main = make_rsrc(p.idx, (unsigned)p.S * st_main);
  const __amdgpu_buffer_rsrc_t r_res = make_rsrc(RES_BITS ? p.idx_res : p.idx, RES_BITS ? (unsigned)p.S * st_res : 0u);
  const __amdgpu_buffer_rsrc_t r_x = make_rsrc(x, plan.x_bytes);
  float4v acc[PLANES];                                   // output row j of every stream (FEW: row n % 6)
  float xs = 0.0f;
#pragma unroll
  for (int j = 0; j < PLANES; ++j) acc[j] = float4v{0.0f, 0.0f, 0.0f, 0.0f};
  // FEW: byte selectors that move the low (even column) or high (odd column) half of an activation dword into half (j & 1) of dword (j >> 1) of
  // the operand, zeros (selector byte 0x0c) everywhere else
  unsigned sel[3][2];
  if constexpr (FEW) {
    const int j = n % 6;
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      const bool mine = d == (j >> 1);
      sel[d][0] = !mine ? 0x0c0c0c0cu : (j & 1) ? 0x01000c0cu : 0x0c0c0100u;
      sel[d][1] = !mine ? 0x0c0c0c0cu : (j & 1) ? 0x03020c0cu : 0x0c0c0302u;
    }
  }

  for (int grp = g_lo; grp < g_hi; ++grp) {
    // the group's stream positions [pos_lo, pos_hi) -- pos_lo a multiple of 8, a dword boundary of the streams -- and the
    // part's windows, counted from pos_lo; a part past a short last group has none and leaves zeros
    const int pos_lo = grp * p.Pg, pos_hi = min(p.P, pos_lo + p.Pg);
    const int windows = (pos_hi - pos_lo + 32 * FOLDS - 1) / (32 * FOLDS);      // (of all folds together)
    const int w_lo = sub_i * plan.wpp, w_hi = min(windows, w_lo + plan.wpp);
    const int my_n = w_hi - w_lo > wv ? (w_hi - w_lo - wv + MW - 1) / MW : 0;  // this wave's windows: w_lo + wv + i * MW
    if (WALK && grp > g_lo) __syncthreads();             // every wave is done with the tables of the group before

    // ---- tables into LDS: 16-byte entries, zero past k (an index past k, or read beyond a stream's end, meets zeros or a
    // finite entry and a zero activation).  All their loads are asked for here, at once; they are stored after everything
    // else of the start-up has been asked for as well (a loop of load-and-store rounds costs a trip to L2 per round).
    // (The thread id is made opaque in every round, or the table addresses derived from it would stay in registers
    // through the main loop for the next group.)
    unsigned tid = threadIdx.x;
    if (WALK) asm volatile("" : "+v"(tid));
    TableStage<RES_BITS, MW * 64> tables{};
    tables.issue(p, grp, false, tid);
    if (grp == g_lo && p.Q) {
      {
        const __amdgpu_buffer_rsrc_t r_oidx = make_rsrc(p.idx_out, (unsigned)p.S_out * (unsigned)p.stride_out);
        const __amdgpu_buffer_rsrc_t r_ocb = make_rsrc(p.cb_out, (unsigned)(p.k_out * p.v_out) * 2u);
        constexpr int OU = 4;                                // entries a thread has in flight
        const int total = o_rows * Q2;
        for (int e0 = (int)threadIdx.x; e0 < total; e0 += MW * 64 * OU) {
          unsigned w0[OU], w1[OU], sh[OU], jo[OU];
          bool ok[OU];
#pragma unroll
          for (int uu = 0; uu < OU; ++uu) {
            const int e = e0 + uu * MW * 64, r = e / Q2, c = e - r * Q2;
            ok[uu] = e < total && c < p.Q;
            const int o = o_row_lo + (ok[uu] ? r : 0), sq = o / p.v_out;
            const unsigned bit = (unsigned)(ok[uu] ? c : 0) * (unsigned)p.bits_out;
            const unsigned woff = (unsigned)sq * (unsigned)p.stride_out + (bit >> 5) * 4u;
            jo[uu] = (unsigned)(o - sq * p.v_out); sh[uu] = bit & 31u;
            w0[uu] = __builtin_amdgcn_raw_buffer_load_b32(r_oidx, woff, 0, 0);
            w1[uu] = __builtin_amdgcn_raw_buffer_load_b32(r_oidx, woff + 4u, 0, 0);
          }
#pragma unroll
          for (int uu = 0; uu < OU; ++uu) {
            const unsigned i = min(__builtin_amdgcn_alignbit(w1[uu], w0[uu], sh[uu]) & ((1u << p.bits_out) - 1u), (unsigned)p.k_out - 1u);
            const unsigned short wh = (unsigned short)__builtin_amdgcn_raw_buffer_load_b16(r_ocb, (i * (unsigned)p.v_out + jo[uu]) * 2u, 0, 0);
            const int e = e0 + uu * MW * 64;
            if (e < total) o_tile[e] = ok[uu] ? wh : (unsigned short)0;
          }
        }
        for (int e = (int)threadIdx.x; e < 16 * Q2; e += MW * 64) {
          const int t = e / Q2, c = e - t * Q2;
          o_x[e] = t < plan.batch && c < p.Q ? __half_as_ushort(x[(long long)t * ldx + c]) : (unsigned short)0;
        }
      }

    }

    // byte offset of this lane's first activation of window 0; a token past the batch reads out of range, i.e. zeros
    const int col0 = p.n_out + pos_lo;                     // column of x that meets the part's window 0
    const unsigned xoff = token < plan.batch ? (unsigned)(((long long)token * ldx + col0 + 32 * fold + 8 * g) * 2) : 0x80000000u;

    // a stream past the last one reads out of range: index 0, whose products land in rows that are never stored
    const unsigned octet = (unsigned)(fold * 4 + g), stream_a = (unsigned)(blk * STREAMS + n % STREAMS);
    const unsigned srow_main = stream_a * st_main + ((unsigned)(pos_lo >> 3) + octet) * 12u;
    const unsigned srow_res = stream_a * st_res + ((unsigned)(pos_lo >> 3) + octet) * (unsigned)RB;

    // The loaders run DEPTH windows ahead of the consumer.  A slot's index words are refilled as soon as the gather
    // addresses have been formed from them; so are its activations, from a copy.
    int lw = w_lo + wv, lwx = w_lo + wv;
    auto load_idx = [&](Window<3> &wm, Window<NR> &wr) {
      const unsigned wq = (unsigned)(lw < w_hi ? lw : w_lo);                   // past the end: any window in range, never used
      lw += MW;
      load_window(wm, r_main, srow_main + wq * (4u * FOLDS) * 12u, 0u);
      if (RES_BITS == 12) load_window(wr, r_res, srow_res + wq * (4u * FOLDS) * 12u, 0u);
      if (RES_BITS == 8) load_window(wr, r_res, srow_res + wq * (4u * FOLDS) * 8u, 0u);
    };
    auto load_x = [&](uint4v &xx) {
      const unsigned wq = (unsigned)(lwx < w_hi ? lwx : w_lo);
      lwx += MW;
      xx = __builtin_amdgcn_raw_buffer_load_b128(r_x, xoff + wq * (64u * FOLDS), 0, 0);
    };

    Window<3> win[DEPTH];
    Window<NR> wres[DEPTH];
    uint4v xr[DEPTH];
#pragma unroll
    for (int d = 0; d < DEPTH; ++d) { load_idx(win[d], wres[d]); load_x(xr[d]); }
    // the table loads are older than the ring's (loads return in order): at most the ring's may still be on their way
    wait_vmem_at_most<DEPTH * (2 + (RES_BITS ? 1 : 0))>();
    tables.store(p, lds, 0u, false, tid);
    lds_barrier();                                       // the tables are in (a full barrier would also wait for the ring's loads from HBM)

    if (grp == g_lo && p.Q) {
      {                                                  // the outlier tile times the activations: a thread per (row, four tokens)
        const unsigned *wt = reinterpret_cast<const unsigned *>(o_tile), *xt = reinterpret_cast<const unsigned *>(o_x);
        const int ntg = (plan.batch + 3) >> 2;
        for (int i = (int)threadIdx.x; i < o_rows * ntg; i += MW * 64) {
          const int tg = i / o_rows, r = i - tg * o_rows;
          float a[4] = {0.0f, 0.0f, 0.0f, 0.0f};
          for (int c2 = 0; c2 < plan.o_pitch; ++c2) {
            const unsigned wd = wt[r * plan.o_pitch + c2];
#pragma unroll
            for (int tt = 0; tt < 4; ++tt) a[tt] = dot2(wd, xt[(tg * 4 + tt) * plan.o_pitch + c2], a[tt]);
          }
#pragma unroll
          for (int tt = 0; tt < 4; ++tt) {
            const int t = tg * 4 + tt;
            if (t < plan.batch) {
              if (plan.part) plan.part[((long long)plan.ksplit * plan.batch + t) * p.out_features + o_row_lo + r] = a[tt];
              else o_sum[t * OROWS + r] = a[tt];
            }
          }
        }
        if ((int)threadIdx.x < plan.batch) {                 // activation sums over the outlier columns
          float sx = 0.0f;
          for (int c2 = 0; c2 < plan.o_pitch; ++c2) sx += half_pair_sum(xt[(int)threadIdx.x * plan.o_pitch + c2]);
          if (!plan.part) o_xs[threadIdx.x] = sx;
          else if (wg == 0) plan.part_xs[plan.ksplit * 16 + (int)threadIdx.x] = sx;
        }
      }

    }

    for (int k0 = 0; k0 < my_n; k0 += DEPTH) {
#pragma unroll
      for (int d = 0; d < DEPTH; ++d) {
        const int k = k0 + d;
        if (k < my_n) {
          const int w = w_lo + wv + k * MW;
          const Window<3> cm = win[d];
          const Window<NR> cr = wres[d];
          uint4v xv = xr[d];
          load_idx(win[d], wres[d]);                     // refill the slot; the copies above are what this window uses
          load_x(xr[d]);
          uint4v e[VPL], f[RES_BITS ? VPL : 1];
#pragma unroll
          for (int u = 0; u < VPL; ++u) lds_gather16<LY::MAIN_OFF>(e[u], field_addr<12, LY::MAIN_SH>(cm, u));
          if (RES_BITS) {
#pragma unroll
            for (int u = 0; u < VPL; ++u) lds_gather16<LY::RES_OFF>(f[u], field_addr<RB, LY::RES_SH>(cr, u) + LY::RES_ADD);
          }
          if (w == windows - 1) {                          // the window that holds the end of the stream or of the group: zero what lies past it
            const int left = pos_hi - pos_lo - ((w * FOLDS + fold) * 32 + g * 8);      // of this lane's eight positions
            unsigned xd[4] = {xv.x, xv.y, xv.z, xv.w};
#pragma unroll
            for (int q = 0; q < 4; ++q) xd[q] = left >= 2 * q + 2 ? xd[q] : left == 2 * q + 1 ? xd[q] & 0xFFFFu : 0u;
            xv = uint4v{xd[0], xd[1], xd[2], xd[3]};
          }
          if (need_xs) xs = dot2(xv.x, 0x3C003C00u, dot2(xv.y, 0x3C003C00u, dot2(xv.z, 0x3C003C00u, dot2(xv.w, 0x3C003C00u, xs))));
          lds_gather_wait();
#pragma unroll
          for (int u = 0; u < VPL; ++u) { settle(e[u]); if (RES_BITS) settle(f[u]); }
          if (FOLDS > 1 && w == windows - 1) {             // (the entries too: past a stream's end a fold reads the next one's indices, whose entries need not be finite)
            const int left = pos_hi - pos_lo - ((w * FOLDS + fold) * 32 + g * 8);
#pragma unroll
            for (int u = 0; u < VPL; ++u)
              if (u >= left) { e[u] = uint4v{0u, 0u, 0u, 0u}; if (RES_BITS) f[u] = uint4v{0u, 0u, 0u, 0u}; }
          }
          if constexpr (FEW) {
#pragma unroll
            for (int u = 0; u < VPL; ++u) {
              const unsigned xd = xv[u >> 1];
              const uint4v b = {__builtin_amdgcn_perm(xd, xd, sel[0][u & 1]), __builtin_amdgcn_perm(xd, xd, sel[1][u & 1]),
                                __builtin_amdgcn_perm(xd, xd, sel[2][u & 1]), 0u};
              acc[0] = mfma16(e[u], b, acc[0]);
              if constexpr (RES_BITS != 0) acc[0] = mfma16(f[u], b, acc[0]);
            }
          } else
          // row j of the eight columns' entries, in the order of the columns: operand A against the token's activations as they are
#pragma unroll
          for (int j = 0; j < 6; ++j) {
            auto row_of = [&](const uint4v (&v)[VPL]) {
              unsigned a[4];
#pragma unroll
              for (int q = 0; q < 4; ++q) a[q] = __builtin_amdgcn_perm(v[2 * q + 1][j >> 1], v[2 * q][j >> 1], j & 1 ? 0x07060302u : 0x05040100u);
              return uint4v{a[0], a[1], a[2], a[3]};
            };
            acc[j] = mfma16(row_of(e), xv, acc[j]);
            if constexpr (RES_BITS != 0) acc[j] = mfma16(row_of(f), xv, acc[j]);
          }
        }
      }
    }

  }

  // ---- the waves meet: sums per output row of the streams, 1 KB per wave and row, in the space of the tables
  __syncthreads();
  float4v *pbuf = reinterpret_cast<float4v *>(lds);                           // [6][MW][64]
  float *xsb = reinterpret_cast<float *>(lds + 6 * MW * 1024);                // [MW][16 tokens]
#pragma unroll
  for (int j = 0; j < PLANES; ++j)
    if (FOLDS == 1 || 4 * g / STREAMS == fold) pbuf[(j * MW + wv) * 64 + lane] = acc[j];      // (of a result what has the same fold on both sides)
  if (need_xs) {                                         // (the lanes of a token meet here: read one by one their sums would take the finishing waves 0.5 us)
    xs += __shfl_xor(xs, 16, 64); xs += __shfl_xor(xs, 32, 64);
    if (FOLDS > 1) xs += __shfl_xor(xs, 8, 64);
    if (FOLDS > 2) xs += __shfl_xor(xs, 4, 64);
    if (g == 0 && fold == 0 && (!FEW || n % 6 == 0)) xsb[wv * 16 + token] = xs;
  }
  __syncthreads();
  if (wv < PLANES) {                                     // wave j finishes row j
    const int t = token, plane = wv, j = FEW ? n % 6 : wv;
    float4v s = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int w = 0; w < MW; ++w) s += pbuf[(plane * MW + w) * 64 + lane];
    if constexpr (FOLDS > 1) {                           // streams 4g.. and token n of fold f are 5 STREAMS lanes behind those of fold f - 1
      float4v one = s;
#pragma unroll
      for (int f = 1; f < FOLDS; ++f) {
#pragma unroll
        for (int r = 0; r < 4; ++r) s[r] += __shfl(one[r], (lane + f * 5 * STREAMS) & 63, 64);
      }
    }
    if (t < plan.batch && (FOLDS == 1 || (n < STREAMS && 4 * g < STREAMS))) {
      float xsum = 0.0f;
      if (need_xs) {
#pragma unroll
        for (int w = 0; w < MW; ++w) xsum += xsb[w * 16 + t];
      }
      float sv[4] = {s.x, s.y, s.z, s.w};
      if (p.Q && !plan.part) {                           // the block's own outlier sums, left in LDS before the main loop
        xsum += o_xs[t];
#pragma unroll
        for (int r = 0; r < 4; ++r) sv[r] += o_sum[t * OROWS + (4 * g + r) * 6 + j];
      }
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int stream = blk * STREAMS + 4 * g + r, o = stream * 6 + j;
        if (stream < p.S && o < p.out_features) {
          if (plan.part) {
            plan.part[((long long)part_i * plan.batch + t) * p.out_features + o] = sv[r];
          } else {
            const float sc = p.scale ? __half2float(p.scale[o]) : 1.0f, bi = p.bias ? __half2float(p.bias[o]) : 0.0f;
            y[(long long)t * ldy + o] = __float2half_rn(__fmaf_rn(sc, sv[r], bi * xsum));
          }
        }
      }
      if (plan.part && blk == 0 && g == 0 && j == 0) plan.part_xs[part_i * 16 + t] = xsum;
    }
  }
}

template <int RES_BITS, bool WALK, bool FEW, int LOG_FOLDS>
__global__ __launch_bounds__(MW * 64) void gemv_down_mfma_kernel(Params p, DownMfmaPlan plan, const __half *__restrict__ x, long long ldx,
                                                                 __half *__restrict__ y, long long ldy) {
  gemv_down_mfma_body<RES_BITS, WALK, FEW, LOG_FOLDS>(p, plan, x, ldx, y, ldy, (int)blockIdx.x);
}

// Several layers that read the same activations (the query, key and value projections of a decoder layer; its gate and up
// projections) in one launch: every workgroup belongs to one layer and runs the body above on one of its blocks of 16
// streams, over all columns.  This is where the coarse blocks stop hurting without a workspace: the blocks of all the
// layers are in flight together (three 4096 x 4096 layers: 129 workgroups instead of three times 43).
constexpr int DMULTI_MAX = 8;
struct DownMultiLayer {
  Params p;
  DownMfmaPlan plan;
  __half *y;
  long long ldy;
};
struct DownMultiArgs {
  int n;
  int first_wg[DMULTI_MAX + 1];                          // layer i owns workgroups [first_wg[i], first_wg[i + 1])
  DownMultiLayer layer[DMULTI_MAX];
};

template <int RES_BITS, bool FEW, int LOG_FOLDS>
__global__ __launch_bounds__(MW * 64) void gemv_down_mfma_multi_kernel(DownMultiArgs a, const __half *__restrict__ x, long long ldx) {
  int i = 0;
  while (i + 1 < a.n && (int)blockIdx.x >= a.first_wg[i + 1]) ++i;
  gemv_down_mfma_body<RES_BITS, false, FEW, LOG_FOLDS>(a.layer[i].p, a.layer[i].plan, x, ldx, a.layer[i].y, a.layer[i].ldy, (int)blockIdx.x - a.first_wg[i]);
}


// LDS of one layer: tables (or the meeting place of the waves, which takes their space at the end), then the outlier tile
template <int RES_BITS>
unsigned place_lds(const Params &p, DownMfmaPlan &plan) {
  unsigned lds_bytes = Layout<RES_BITS>::BYTES;
  const unsigned meet = (unsigned)(6 * MW) * 1024u + (unsigned)(MW * 16) * 4u;
  if (lds_bytes < meet) lds_bytes = meet;
  plan.lds_o = lds_bytes;
  if (p.Q) lds_bytes += (unsigned)((OROWS + 16) * plan.o_pitch + 16 * OROWS + 16) * 4u;
  return lds_bytes;
}

template <int RES_BITS, bool FEW, int LOG_FOLDS>
int launch_multi(DownMultiArgs &a, const __half *x, long long ldx, hipStream_t s) {
  auto kernel = gemv_down_mfma_multi_kernel<RES_BITS, FEW, LOG_FOLDS>;
  VQ_ALLOW_FULL_LDS(kernel);
  unsigned lds_bytes = 0;
  for (int i = 0; i < a.n; ++i) {
    const unsigned b = place_lds<RES_BITS>(a.layer[i].p, a.layer[i].plan);
    if (b > lds_bytes) lds_bytes = b;
  }
  if (lds_bytes > 160u * 1024u) return VQ_ERR_UNSUPPORTED;
  hipLaunchKernelGGL(kernel, dim3((unsigned)a.first_wg[a.n]), dim3(MW * 64), lds_bytes, s, a, x, ldx);
  return hipGetLastError() == hipSuccess ? VQ_OK : VQ_ERR_HIP;
}

template <int RES_BITS, bool WALK, bool FEW, int LOG_FOLDS>
int launch_one(const Params &p, DownMfmaPlan &plan, unsigned grid, const __half *x, long long ldx, __half *y, long long ldy,
               hipStream_t s) {
  auto kernel = gemv_down_mfma_kernel<RES_BITS, WALK, FEW, LOG_FOLDS>;
  VQ_ALLOW_FULL_LDS(kernel);
  const unsigned lds_bytes = place_lds<RES_BITS>(p, plan);
  if (lds_bytes > 160u * 1024u) return VQ_ERR_UNSUPPORTED;                  // too many outlier columns to hold beside the tables
  hipLaunchKernelGGL(kernel, dim3(grid), dim3(MW * 64), lds_bytes, s, p, plan, x, ldx, y, ldy);
  return hipGetLastError() == hipSuccess ? VQ_OK : VQ_ERR_HIP;
}

}  // namespace

// Whether the kernel above takes this layer and these buffers (the caller has checked gemv_down_applicable()).
bool gemv_down_mfma_applicable(const Params &p, const __half *x, long long ldx, int batch) {
  if (p.orientation != 1 || p.v != 6 || p.bits != 12 || p.Q > 512) return false;
  if (p.Q && (long long)p.S_out * p.stride_out >= (1LL << 31)) return false;
  if (p.n_groups > 1 && ((p.Pg & 7) || p.n_groups > 256)) return false;     // a group starts on a dword of the index streams
  if (p.k_res && p.bits_res != 12 && p.bits_res != 8) return false;
  if (batch < 1 || batch > 16) return false;
  if ((reinterpret_cast<uintptr_t>(x) & 3) || (ldx & 1) || (p.n_out & 1)) return false;      // activation loads are dword-aligned
  if (((long long)(batch - 1) * ldx + p.in_features) * 2 >= (1LL << 31)) return false;       // 32-bit buffer offsets
  const long long max_stride = p.stride > p.stride_res ? p.stride : p.stride_res;
  return (long long)p.S * max_stride < (1LL << 31);
}

// Parts the columns are cut into when a workspace is there: enough for the (block, part) workgroups to fill the chip, each
// part at least one 32-column window per wave.  1: nothing to gain from a workspace.
// Codebook groups are parts by themselves (a part has one set of tables); each is cut further on the same terms.
static int parts_per_group(const Params &p) {
  const int blocks = (p.S + 15) / 16, windows = (min(p.P, p.Pg) + 31) / 32;
  int want = cu_count() / ((blocks > 0 ? blocks : 1) * p.n_groups);
  if (want > windows / MW) want = windows / MW;
  if (want > 16) want = 16;
  if (want < 2) return 1;
  const int wpp = (windows + want - 1) / want;
  return (windows + wpp - 1) / wpp;
}
int gemv_down_mfma_parts(const Params &p) { return p.n_groups * parts_per_group(p); }

// Estimated time in microseconds of `batch` rows of a layer without codebook groups in `parts` parts, from 1560 layers (256 to 14336 outputs, 256 to
// 28672 columns, one to sixteen rows; 4 % off in the mean, sixteen rows 7): a workgroup's start and its waves' windows, as often as compute units take
// one; the second launch and its sums; the outlier columns, which a block's rows have one workgroup for, or one a part.
static float estimate_us(const Params &p, int parts, int folds, int batch) {
  const int blocks = (int)(((long long)p.S * folds + 15) / 16), windows = (p.P + 32 * folds - 1) / (32 * folds), rounds = (blocks * parts + cu_count() - 1) / cu_count();
  const int steps = ((windows + parts - 1) / parts + MW - 1) / MW;
  const bool few = p.k_res && batch <= 2 && folds == 1, long_table = p.bits_res == 12;
  const float start = (!p.k_res ? 2.5f : long_table ? (few ? 2.7f : 3.03f) : few ? 2.25f : 2.55f) + (batch > 8 ? 0.2f : 0.0f);
  const float step = !p.k_res ? 0.335f : !long_table ? 0.7f : few ? 0.715f : 0.73f, outputs = (float)p.out_features;
  // (sixteen rows, or folds of rows, that begin on one of few lines of L1 each get in one another's way; a part of them less so)
  const float pitch = parts == 1 && batch * folds > 8 && !p.k_res && p.in_features % 256 == 0 ? (folds > 1 ? 1.25f : 1.18f) : 1.0f;
  float us = start * (float)(1 + rounds) + pitch * step * (float)(rounds * steps);
  // (47 layers with each number of folds, one, four and eight rows, 2 to 4 % off: half the streams or a quarter are that many more workgroups after the
  // tables, and two tables of 4096 entries leave a compute unit no room for a second one)
  if (folds > 1) us += (folds == 2 ? 0.55f : 0.8f) + (long_table ? 2.1f * (float)(rounds - 1) : 0.0f);
  if (parts > 1) us += 0.85f + (float)parts * (0.12f + outputs * (1.7e-5f + 5.2e-6f * (float)batch));
  if (p.Q) us += 1.2f + (float)p.Q * (parts > 1 ? 0.03f + 2.2e-6f * outputs : p.k_res ? 0.06f : 0.08f);
  return us;
}

// Folds of the columns of one launch without parts.
static int folds_of(const Params &p, int batch) {
  int best = 1;
  if (p.n_groups > 1) return best;
  for (int folds = 2; folds <= 4 && batch * folds <= 16; folds *= 2)
    if (estimate_us(p, 1, folds, batch) < 0.96f * estimate_us(p, 1, best, batch)) best = folds;      // (as close as the estimates are)
  return best;
}
float gemv_down_mfma_us(const Params &p, int parts, int batch, bool fold) {
  return estimate_us(p, parts, parts == 1 && fold ? folds_of(p, batch) : 1, batch);
}

static int make_plan(const Params &p, long long ldx, int batch, float *part, float *part_xs, int parts, int folds, DownMfmaPlan &plan, long long *grid_out) {
  const int blocks = (int)(((long long)p.S * folds + 15) / 16), windows = (min(p.P, p.Pg) + 32 * folds - 1) / (32 * folds);      // windows of the widest group
  if (blocks < 1 || windows < 1) return VQ_ERR_UNSUPPORTED;
  plan.ksplit = part ? parts : 1;
  if (part && plan.ksplit % p.n_groups) return VQ_ERR_UNSUPPORTED;
  plan.sub = part ? plan.ksplit / p.n_groups : 1;      // without a workspace: one workgroup per block walks all groups and all windows
  plan.wpp = (windows + plan.sub - 1) / plan.sub;
  plan.batch = batch;
  // (a whole number of dwords: the buffer's range check drops a dword that straddles the end, and with it the last
  // column of the last row when in_features is odd; x begins at a dword and ldx is even, so that column and the half after it,
  // which need not be the caller's, are one dword and lie on one page, and the kernel masks the half like every position past the stream's end)
  plan.x_bytes = (unsigned)((((long long)(batch - 1) * ldx + p.in_features) * 2 + 3) & ~3LL);
  plan.part = part; plan.part_xs = part_xs;
  plan.o_pitch = ((p.Q + 1) / 2) | 1;
  plan.o_rpw = (int)((p.out_features + (long long)blocks * plan.ksplit - 1) / ((long long)blocks * plan.ksplit));   // <= 96: a block has 96 rows
  const long long grid = (long long)blocks * plan.ksplit;
  if (grid > 0x7FFFFFFFLL) return VQ_ERR_UNSUPPORTED;
  *grid_out = grid;
  return VQ_OK;
}

// part == nullptr: one launch that stores y (a layer with codebook groups: every workgroup walks all of them).  Else
// parts = gemv_down_mfma_parts(p) > 1 and the sums go to part[parts][batch][out_features], part_xs[parts * 16]; the caller
// adds them up.
int launch_gemv_down_mfma(const Params &p, const __half *x, long long ldx, int batch, __half *y, long long ldy, hipStream_t s,
                          float *part, float *part_xs, int parts) {
  DownMfmaPlan plan{};
  long long grid = 0;
  const int folds = part ? 1 : folds_of(p, batch), rc_plan = make_plan(p, ldx, batch, part, part_xs, parts, folds, plan, &grid);
  if (rc_plan != VQ_OK) return rc_plan;
  const int rb = p.k_res ? p.bits_res : 0;
  const bool walk = !part && p.n_groups > 1;
#define VQ_CASE(R) if (rb == R) { \
    if (folds == 4) return launch_one<R, false, false, 2>(p, plan, (unsigned)grid, x, ldx, y, ldy, s); \
    if (folds == 2) return launch_one<R, false, false, 1>(p, plan, (unsigned)grid, x, ldx, y, ldy, s); \
    return batch <= 2 && R ? (walk ? launch_one<R, true, R != 0, 0>(p, plan, (unsigned)grid, x, ldx, y, ldy, s) : launch_one<R, false, R != 0, 0>(p, plan, (unsigned)grid, x, ldx, y, ldy, s)) \
                           : (walk ? launch_one<R, true, false, 0>(p, plan, (unsigned)grid, x, ldx, y, ldy, s) : launch_one<R, false, false, 0>(p, plan, (unsigned)grid, x, ldx, y, ldy, s)); \
  }
  VQ_CASE(0) VQ_CASE(8) VQ_CASE(12)
#undef VQ_CASE
  return VQ_ERR_UNSUPPORTED;
}

// n layers (2 .. 8) of one codebook group each on the same activations in one launch, without a workspace.  VQ_ERR_UNSUPPORTED
// when they do not fit one kernel instantiation (different residual kinds, different in_features); the caller then launches
// them one by one.  The caller has checked gemv_down_mfma_applicable() for each.
int launch_gemv_down_mfma_multi(const Params *ps, int n, const __half *x, long long ldx, int batch, __half *const *ys,
                                const long long *ldys, hipStream_t s) {
  if (n < 2 || n > DMULTI_MAX) return VQ_ERR_UNSUPPORTED;
  DownMultiArgs a{};
  a.n = n;
  const int rb = ps[0].k_res ? ps[0].bits_res : 0;
  long long total = 0, streams = 0;
  for (int i = 0; i < n; ++i) streams += ps[i].S;
  Params all = ps[0];                                      // (as one layer of all their streams; beside other layers outlier columns cost what they do alone)
  all.S = (int)min(streams, 1LL << 24);
  const int folds = folds_of(all, batch);
  for (int i = 0; i < n; ++i) {
    if (ps[i].in_features != ps[0].in_features || ps[i].n_groups > 1 || (ps[i].k_res ? ps[i].bits_res : 0) != rb) return VQ_ERR_UNSUPPORTED;
    long long grid = 0;
    const int rc = make_plan(ps[i], ldx, batch, nullptr, nullptr, 1, folds, a.layer[i].plan, &grid);
    if (rc != VQ_OK) return rc;
    a.layer[i].p = ps[i]; a.layer[i].y = ys[i]; a.layer[i].ldy = ldys[i];
    a.first_wg[i] = (int)total;
    total += grid;
    if (total > 0x7FFFFFFFLL) return VQ_ERR_UNSUPPORTED;
  }
  a.first_wg[n] = (int)total;
#define VQ_CASE(R) if (rb == R) \
    return folds == 4 ? launch_multi<R, false, 2>(a, x, ldx, s) : folds == 2 ? launch_multi<R, false, 1>(a, x, ldx, s) : \
           batch <= 2 && R ? launch_multi<R, R != 0, 0>(a, x, ldx, s) : launch_multi<R, false, 0>(a, x, ldx, s);
  VQ_CASE(0) VQ_CASE(8) VQ_CASE(12)
#undef VQ_CASE
  return VQ_ERR_UNSUPPORTED;
}

}  // namespace vq
