// Internal launch interface between the FQT host layer (api.hip) and the
// kernels (quant.hip, gemm.hip, conv.hip).  Not part of the public ABI.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace fqt {

// ---- quantizer front end -------------------------------------------------

// Statistics: each block reduces one chunk of a flat tensor (rows = 1) or
// of one row, into part[row * chunks + chunk] = (min, max); min is NaN when
// the chunk holds a non-finite value.
// A per-row segment whose rows fit one block (chunks == 1) also gets the
// row ranges written directly: rmin[row] (+inf for a non-finite row, as the
// finalize combination of one NaN-flagged partial gives) and rmax[row].
struct StatsSeg {
  const float* x;
  int64_t rows, cols;
  int64_t chunk;   // columns per block
  int64_t chunks;  // blocks per row
  float2* part;
  float* rmin;     // direct per-row ranges (chunks == 1), else nullptr
  float* rmax;
};
StatsSeg stats_flat_seg(const float* x, int64_t n);
StatsSeg stats_rows_seg(const float* x, int64_t rows, int64_t cols);
// Route the row ranges of a per-row segment straight to rmin / rmax when a
// block covers a whole row.
inline void stats_direct_rows(StatsSeg& g, float* rmin, float* rmax) {
  if (g.chunks == 1) {
    g.rmin = rmin;
    g.rmax = rmax;
  }
}
__host__ __device__ inline int64_t stats_partials(const StatsSeg& g) { return g.rows * g.chunks; }
struct StatsPlan {
  StatsSeg seg[3];
  int nseg;
  int64_t block_start[4];
  int32_t* zero;  // counters cleared in the same launch (zero_n of them, 0: none)
  int64_t zero_n;
};
constexpr int64_t STATS_ZERO = 4096;  // counters per clearing block
hipError_t launch_stats(StatsPlan sp, hipStream_t s);

// One finalize block: per-tensor PTQ scale / zero (Sec. 3.3), per-row PSQ
// scale / zero (Sec. 4.1), per-row min / max of the row segment, cleared
// int32 arrays and the status word.
// per_row: 0 per tensor (PTQ), 1 per row (PSQ), 2 per-tensor range with
// per-row power-of-two steps (Sec. 4.3): s_i = s 2^e_i, shift[row] = E - e_i,
// E = min(4, 8 - bits), and s itself in tensor_scale[0].
struct ScaleOut {
  int seg;
  int bits;
  int per_row;
  float* scale;
  float* zero;
  int8_t* shift;
  float* tensor_scale;
  double* zeta;  // per_row == 2, optional: [rows] half / s_i + z_i (float64), the rows' zero-point terms
};
struct FinalizePlan {
  StatsSeg seg[3];
  int nseg;
  int row_seg;       // index of the per-row segment, -1 if none
  float* rmin;       // [rows] of the row segment
  float* rmax;
  ScaleOut out[4];
  int nout;
  int32_t* zero_i32[6];
  int64_t zero_n[6];
  int nzero;
  uint32_t* status;
};
hipError_t launch_finalize(const FinalizePlan& fp, hipStream_t s);

// Fixed-block BHQ layout, all data independent (see bhq_layout()).
struct BhqLayout {
  int64_t rows;
  int k;        // block size
  int64_t G;    // number of groups
  int64_t full; // groups of exactly k rows (first in slot order)
  int part;     // size of the one partial group after them (0: none)
  double sk_k, sk_p;        // sqrt(k), sqrt(part)
  double inv_sk_k, inv_sk_p;  // 1/sqrt(k), 1/sqrt(part) in float64 (dequantization)
  float a_k, oma_k, a_p, oma_p;  // float32(1/sqrt(size)) and float32(1 - that)
};
BhqLayout bhq_layout(int64_t rows, int k);

// Slot kind under a fixed-block layout: 0 = one-row group, 1 = full group,
// 2 = the partial group.  Groups are stored full ones first, then the
// partial one, then the one-row groups, each full / partial group starting
// at a multiple of k.
__device__ __forceinline__ int bhq_slot_kind(const BhqLayout& L, int64_t slot) {
  if (slot < L.full * L.k) return 1;
  if (L.part > 0 && slot < L.full * L.k + L.part) return 2;
  return 0;
}

// Workspace for the BHQ plan: sorted chunk keys, rank (must be zero before
// the plan runs), sigma = rows in sorted order.
size_t bhq_plan_workspace(int64_t rows);
struct BhqPlanWs {
  uint64_t* sorted;
  int32_t* rank;
  int32_t* sigma;
};
BhqPlanWs bhq_plan_carve(void* plan_ws, int64_t rows);
// fin: run this finalize step inside the first plan launch (only when the
// row ranges rmin / rmax were stored by the statistics kernel); nullptr when
// the finalize kernel already ran.
hipError_t launch_bhq_plan(const float* rmin, const float* rmax, const BhqLayout& L, int bits, void* plan_ws,
                           int32_t* perm, float* scale, float* zero, int32_t* group_off, int32_t* num_groups, const FinalizePlan* fin,
                           hipStream_t s);


// Rows in sorted order (M descending, ties by row index), for the general
// plans below; fin as for launch_bhq_plan.
hipError_t launch_bhq_sort(const float* rmin, const float* rmax, int64_t rows, void* plan_ws, int32_t* sigma,
                           const FinalizePlan* fin, hipStream_t s);

// ---- general BHQ plans: groups of any size, in slot order ----------------
// Slot record: the slot's group starts at slot `base` and has `size` slots;
// alpha = float32(1 / sqrt(size)), oma = float32(1 - alpha) (multi-row groups).
struct SlotInfo {
  int32_t base, size;
  float alpha, oma;
};
// Per sorted position r (row sigma[r]): its infinity norm M and range R
// (non-finite values read as 0, so that a plan over bad data stays a valid
// permutation), cbrt_rn(R), cbrt_rn(2 M); prefix sums P of M (float64,
// P[0] = 0, added one at a time in sorted order); the App. D objective of
// every number of groups G = 1..rows and the chosen G.
struct AppdWs {
  int32_t* sigma;
  float *Ms, *Rs, *ca, *cc;
  double* P;
  double* obj;
  int32_t* G;
};
size_t appd_workspace(int64_t rows);
AppdWs appd_carve(void* ws, int64_t rows);
// Everything of the plan after the sort: the sorted-position scalars, and
// for block_size = 0 the App. D search over G (objective into obj_out when
// given, else the workspace's), then the groups (block_size > 0: the fixed
// layout of bhq_layout).  Writes perm, scale, zero, group_off [G + 1], slot
// and num_groups (device scalar).
hipError_t launch_general_plan(const float* rmin, const float* rmax, int64_t rows, int bits, int block_size,
                               const AppdWs& w, double* obj_out, int32_t* perm, float* scale, float* zero,
                               int32_t* group_off, SlotInfo* slot, int32_t* num_groups, hipStream_t s);
// The App. D search alone (objective and chosen G), after the sort.
hipError_t launch_appd_search(const float* rmin, const float* rmax, int64_t rows, int bits, const AppdWs& w,
                              double* obj_out, int32_t* num_groups, hipStream_t s);
// Per multi-row group and column: tau = (alpha S - v_0) / (1 - alpha), S the
// group's column sum of v_p = d_p x[perm[p]] in slot order (float32),
// stored at tau[(base / 2) * cols + col] (group bases are at least 2 apart).
hipError_t launch_bhq_tau(const float* x, int64_t rows, int64_t cols, const int32_t* perm, const float* scale,
                          const SlotInfo* slot, float* tau, hipStream_t s);
// Inverse transform of the general plans' grad_X rows.  Rows of T are (block
// b, slot p) at T[(b * tstride + p) * ldt + col] (float64: the dequantized
// code row times the weights, see EPI_BHQT); per multi-row group S = sum of
// its T rows (float64, slot order), tau = (alpha S - T_0) / (1 - alpha),
// alpha = 1 / sqrt(k); out row = perm[p] * ostride + b * obstride, value
// (T_0 + (1 - alpha) tau or T_p - alpha tau) / d_p; zero where mask <= 0.
struct InverseParams {
  const double* T;
  int64_t ldt, tstride, nblk, rows, cols;
  const SlotInfo* slot;
  const int32_t* perm;
  const float* scale;
  float* out;
  int64_t ldo, ostride, obstride;
  const float* mask;
};
hipError_t launch_bhq_inverse(const InverseParams& p, hipStream_t s);

struct QuantParams {
  const float* x;
  int64_t rows, cols;
  int nt;               // the launch's inputs are read nontemporally (set at launch)
  const int32_t* perm;  // slot -> source row; nullptr = identity
  int bits;
  int stoch;
  uint64_t seed;
  uint32_t stream;
  const float* scale;  // per tensor: [1]; per row / BHQ: [rows] per slot
  const float* zero;
  int8_t* q_nat;       // [rows, cols] slot order, or nullptr (packed: [rows, cols / 2] bytes)
  int packed;          // natural codes of bits <= 4 stored two per byte (float4 rows only)
  int64_t ldn;         // row pitch of q_nat (0: cols, no padding); codes past cols are zero
  int64_t ldt;         // row pitch of q_t / q2_t (0: rows, no padding); codes past rows are zero
  int64_t pm_o;        // > 0: natural codes pixel-major, column j of row (slot) i at
                       // ((j / pm_o) rows + i) pm_o + j % pm_o (cols % pm_o == 0, pm_o % 4 == 0)
  int32_t* sum_nat;    // [rows] row sums, or nullptr
  int8_t* q_t;         // [cols, rows] slot order, or nullptr
  int32_t* sum_t;      // [cols] column sums, or nullptr
  // second, per-tensor stochastic quantizer of the same rows (Q_b1); transposed only
  int bits2;
  uint32_t stream2;
  const float* scale2;
  const float* zero2;
  int8_t* q2_t;
  int8_t* q2_n;        // natural instead: [rows, cols] in source-row order (cols % 16 == 0)
  int row2;            // q2_n: scale2 / zero2 per source row
  int32_t* sum2_t;     // [cols] column sums, or nullptr
  const int8_t* shift;   // QM_ROW: per-row left shift of the offset codes, or nullptr
  const int8_t* shift2;  // Q_b1 with per-row scale2 / zero2 / shift2 (source-row order), or nullptr
  BhqLayout L;           // BHQ: L.k = 0 selects the general plan (slot, tau)
  const SlotInfo* slot;
  const float* tau;
  // seed batch (launch_quant_seeds): nseeds roundings under keys seed + b,
  // per element [rows, cols] (slot order) the sum of the codes and of their squares
  int nseeds;
  int32_t* sum_c;
  int32_t* sum_c2;
};
enum QuantMode { QM_TENSOR = 0, QM_ROW = 1, QM_BHQ = 2 };
hipError_t launch_quant(const QuantParams& p, int mode, hipStream_t s);
// The seed batch of one quantizer (natural layout, cols % 4 == 0).
hipError_t launch_quant_seeds(const QuantParams& p, int mode, hipStream_t s);
// Two per-tensor quantizations with natural outputs only, one launch.
hipError_t launch_quant_nat_pair(QuantParams p0, QuantParams p1, hipStream_t s);
// The gradient quantizer pg (with its transposed second quantizer) and the
// per-tensor transposed quantizers px, pw in one launch.
hipError_t launch_quant_fused(const QuantParams& pg, int mode, const QuantParams& px, const QuantParams& pw,
                              hipStream_t s);

// Conv layer: X codes in pixel order, cp bytes per pixel (channels past c are
// zero codes).  cp = 4: each image row has wp pixels, the image at pad, zero
// codes around it.
struct PixelQParams {
  const float* x;  // [pixels][c]
  int64_t words;   // output words (4 bytes)
  int c, cp, w, wp, pad;
  int nt;          // as QuantParams
  int bits;
  const float* scale;
  const float* zero;
  int8_t* q;
};
constexpr int64_t PIXQ_WORDS = 1024;  // words per block
// W [o][tap][c] -> codes [c][(tap, o)], sums over o [(tap, c)]
struct ConvWQParams {
  const float* w;  // nullptr: none
  int o, taps, c;
  int bits;
  const float* scale;
  const float* zero;
  int8_t* q;
  int32_t* sum;
};
// Q_b2(G) (pixel-major natural codes) with Q_b1(G) (pg.q2_n) from one read of
// G, Q_f(X) and Q_theta(W); without pg.q_nat Q_b1 and Q_f only.
hipError_t launch_quant_conv(const QuantParams& pg, int mode, const PixelQParams& px, const ConvWQParams& pw,
                             hipStream_t s);

// ---- int8 contractions ---------------------------------------------------

enum Epilogue {
  EPI_RAW_I32 = 0,   // int32 partials [splits][M][N] (caller reduces)
  EPI_TENSOR = 1,    // per-tensor A, per-tensor B: grad_W
  EPI_ROW = 2,       // per-row A (PTQ broadcasts), per-tensor B: grad_X
  EPI_BHQ = 3,       // per-group Householder on A rows, per-tensor B: grad_X
  EPI_BHQT = 4       // general BHQ plan: one-row groups finished, other rows' T into tbuf
};

struct GemmParams {
  const int8_t* A;  // [M, K] row stride lda (bytes)
  int packedA;      // A holds codes of at most 4 bits two per byte (as the quantizer packs them), K % 16 == 0
  const int8_t* B;  // [N, K] row stride ldb
  int64_t M, N, K, lda, ldb;
  int64_t Kp;       // K with the zero codes that pad both operands' rows (0: K, no padding)
  int64_t kchunk;   // K per split (multiple of 128 when split, <= 65536)
  int splits;
  int32_t* part;    // EPI_RAW_I32 output [splits][M][N]
  // epilogue data (float64 arithmetic, float32 result)
  float* out;       // [M, N] (row index remapped through perm when given)
  int64_t ldo;
  const int32_t* perm;   // A row (slot) -> output row; nullptr = identity
  const int32_t* sumA;   // [M] sum over K of A's codes
  const int32_t* sumB;   // [N] sum over K of B's codes
  const float* scaleA;   // [1] or [M]
  const float* zeroA;
  int rowwiseA;          // scaleA / zeroA indexed per row
  int halfA;             // 2^(bitsA - 1)
  const float* scaleB;   // [1]
  const float* zeroB;
  int halfB;
  BhqLayout L;           // EPI_BHQ group structure
  int relu;              // EPI_TENSOR: store max(v, 0)
  int expA;              // EPI_TENSOR: A's step is 1 / (scaleA[0] 2^expA)
  const double* colvec;  // EPI_TENSOR: nullptr, or [N] replacing A's zero-point terms (per-row zeros of A)
  const float* mask;     // EPI_ROW / EPI_BHQ: nullptr, or [M, ldo] in output-row order; out = 0 where mask <= 0
  const SlotInfo* slot;  // EPI_BHQT: the general plan
  double* tbuf;          // EPI_BHQT: [M, ldt] T of the rows of multi-row groups
  int64_t ldt;
};
hipError_t launch_gemm(const GemmParams& p, int epi, hipStream_t s);

// Sum int32 split partials in int64; either store int64 (out64) or apply the
// per-tensor epilogue (EPI_TENSOR) into p.out.
hipError_t launch_splitk_reduce(const GemmParams& p, int64_t* out64, int epi, hipStream_t s);

// Whether a launch stores its float32 output (rows of ldo) nontemporally: rows
// in whole units of `unit` floats.  Ordinary stores that leave part of a cache
// line meet in L2 with those that fill it; nontemporal ones go out as they are,
// and a part of a line costs memory a read as well.  The unit lies where that
// outweighs the gain, nontemporal / ordinary in us:
// - STREAM_TENSOR, one float per lane (runs of 128 bytes): whole lines (forward
//   8192 x 512 -> 4096 75 / 77, -> 4095 95 / 78), and half lines up to 96 MB of
//   output, which the last-level cache still puts together (forwards of 6832 rows
//   by 512: 784 wide 34.0 / 35.4, 1360 44.4 / 46.0, 2544 60.8 / 61.9, 3568 (97
//   MB) 64.9 / 64.8, 4080 77.1 / 73.7; 8192 rows 4080 97 / 79).
// - STREAM_ROW, four floats per lane (runs of 256 bytes): half lines.  Layer
//   8192 x 1008 -> 512 97.7 / 98.4, 8192 x 1020 -> 512 104 / 99, 8192 x 4095 ->
//   128 343 / 186.
// - STREAM_CONV, the same from a conv, whose time the stores bound more: the
//   16 bytes of a lane.  56x56 b128: 3x3 80ch 264 / 282, 84ch 317 / 332, 1x1
//   104ch 310 / 324; only wide odd pitches lose (1x1 196ch 469 / 439).  Without
//   whole 16 bytes the stores are single floats: 3x3 83ch 470 / 320.
enum StreamUnit { STREAM_TENSOR = 32, STREAM_ROW = 16, STREAM_CONV = 4 };
inline bool stream_rows(const float* out, int64_t rows, int64_t ldo, StreamUnit unit) {
  const int64_t u = unit == STREAM_TENSOR && rows * ldo * 4 <= (int64_t)96 << 20 ? STREAM_ROW : unit;
  return ldo % u == 0 && (uintptr_t)out % (4 * u) == 0;
}

// Zero-point term of a contraction over samples whose A rows (samples) carry
// their own zero points: v[c] = sum_n zeta_n Xt[n, c] (zeta_n = half / s_n +
// z_n from the finalize), Xt[n, c] = dx q[c, n] + zx (q: [cols, ldq]
// transposed codes in slot order, perm slot -> row or nullptr), float64.
struct ColvecParams {
  const int8_t* q_t;
  int64_t rows, cols;
  int64_t ldq;          // row pitch of q_t, a multiple of 16
  const int32_t* perm;
  const double* zeta;   // zeta_n [rows], source-row order
  const float* scaleX;  // [1]
  const float* zeroX;   // [1]
  int halfX;
  double* part;         // scratch [colvec_splits(rows)][cols + 1]
  double* out;          // [cols]
};
int64_t colvec_splits(int64_t rows);
hipError_t launch_colvec(const ColvecParams& p, hipStream_t s);

// ---- machine probes -------------------------------------------------------
hipError_t launch_mfma_probe(int64_t blocks, int64_t iters, int32_t* sink, hipStream_t s);
hipError_t launch_copy_probe(int64_t blocks, const void* src, void* dst, int64_t n16, hipStream_t s);

// ---- 4-bit codes on 6-bit float matrix cores ---------------------------
// Packed e3m2 operands (rows of bf6_row_bytes(K) bytes, K padded to 128),
// exact int32 partials [splits][M][N] (reduce with launch_splitk_reduce).
struct Bf6Params {
  const int8_t* A;  // [M] packed rows, stride lda bytes
  const int8_t* B;  // [N] packed rows, stride ldb bytes
  int64_t M, N, Kpad, lda, ldb;
  int64_t kchunk;   // codes per split, multiple of 128, <= 131072
  int splits;
  int32_t* part;
};
int64_t bf6_row_bytes(int64_t K);
hipError_t launch_pack_e3m2(const int8_t* src, int64_t rows, int64_t K, int64_t ld, int8_t* dst, uint32_t* status,
                            hipStream_t s);
hipError_t launch_status_clear(uint32_t* status, hipStream_t s);
hipError_t launch_gemm_bf6(const Bf6Params& p, hipStream_t s);

constexpr int NUM_XCD = 8;  // accelerator dies of the GPU, each with its own L2; blocks go to them round robin

// ---- conv ----------------------------------------------------------------
struct ConvGeom {
  int n, c, h, w, o, kh, kw, stride, pad, ho, wo;
  int64_t npad;  // slots per input pixel in the grad_X rows (16, 32 or a multiple of 64)
  // X codes in pixel order: cp bytes per pixel (4 for at most 4 channels, else
  // the channels rounded up to 16); cp = 4: image rows of wp pixels with a
  // horizontal halo of zero codes
  int cp, wp;
};
// grad_W (conv_gradw.hip): Q_b1 codes [pixel][o] and X codes in pixel order,
// both in sample order; partial sums over splits of the output pixels, then the
// reduction with the zero-point terms.
// Copies of the X code sums (a power of two, at most 16), split s adding to copy
// s % copies: one for every 16 splits.  With one copy the atomics of many splits
// of few columns queue up for longer than the contraction takes (3x3 3 -> 32
// 64x64 b128, 512 splits: 22 of 36 us); every block of the reduction reads all of
// them, a few bytes beside the partial sums of as many splits.
inline int gradw_copies(int splits) {
  int c = 1;
  while (c < 16 && splits > 16 * c) c *= 2;
  return c;
}
struct ConvGradwParams {
  const int8_t* q1;
  const int8_t* xq;
  int64_t Np;         // partial-sum columns (conv_gradw_cols)
  int64_t per_split;  // pixels per split (per-sample Q_b1: 128-pixel stages, each sample's rounded up)
  int splits;
  int32_t* part;      // [splits][o][Np]
  int copies;         // of sumB
  int64_t* sumB;      // [copies][Np] parts of the X code sums over each column's valid pixels (cleared before)
  int32_t* qs;        // [ho wo][o] Q_b1 code sums over the samples (cleared before)
  int64_t* sumA;      // [tap][o] ... over the tap's valid pixels
  // per-sample Q_b1: the same in float64, weighted by 1 / s_n (the X code sums by z_n + half / s_n)
  double* partd;      // [splits][o + 2][Np], rows o and o + 1 the X code sums
  double* qsd;
  double* sumAd;
  double* zsum;       // [1] sum of z_n + half / s_n
  const float* scaleA;  // [1], or [n] per sample
  const float* zeroA;
  int halfA;
  const float* scaleB;
  const float* zeroB;
  int halfB;
  float* out;         // [o][tap][c]
};
int64_t conv_gradw_cols(const ConvGeom& g);
void conv_gradw_splits(const ConvGeom& g, bool psq, int64_t& per_split, int& splits);
hipError_t launch_conv_gradw(const ConvGradwParams& p, const ConvGeom& g, bool psq, hipStream_t s);
// Zero-point sums of grad_W, and the row sums sg [pixel][slot] of Q_b2 (sg = nullptr: none).
hipError_t launch_conv_sums(const ConvGradwParams& p, const ConvGeom& g, bool psq, const int8_t* q2, int32_t* sg,
                            hipStream_t s);
hipError_t launch_conv_gradw_reduce(const ConvGradwParams& p, const ConvGeom& g, bool psq, hipStream_t s);
// sg: row sums [output pixel][slot] of the Q_b2 codes; swq: W code sums over o
// [(tap, c)]; zero16: 16 zero bytes after q2 in the same workspace.
hipError_t launch_conv_gradx(const GemmParams& p, int epi, const ConvGeom& g, const int8_t* q2, const int8_t* zero16,
                             const int32_t* sg, const int32_t* swq, hipStream_t s);

}  // namespace fqt
