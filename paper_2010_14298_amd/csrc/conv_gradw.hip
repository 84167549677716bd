// grad_W of the conv layer on gfx950: an implicit-im2col int8 contraction over
// output pixels with both operands in their natural, channel-contiguous
// layout.
//
//   grad_W[o][(tap, ch)] = sum over pixels p of Q_b1(G)[p][o] X[p + tap][ch]
//
// The contraction index (the pixel) is the slow index of both operands, while
// a matrix-core lane wants 16 consecutive values along it.  Instead of writing
// transposed or im2col copies to memory (which took half of the layer's time:
// 426 us of 1160 us for a 3x3 stride-2 layer), a stage of 128 pixels is loaded
// into LDS as it lies in memory (direct-to-LDS loads, one 16-byte chunk of a
// pixel's channels per lane, the tap's pixel worked out per lane) and read back
// transposed (ds_read_b64_tr_b8: lanes 2r, 2r + 1 of 16 address row r of 8, lane
// c receives column c).  Padded taps load a block of zeros.  Any stride takes
// the same path.
#include <type_traits>

#include "gemm_core.h"

namespace fqt {

typedef int v2i __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(3))) v2i lds_v2i;

__device__ __attribute__((aligned(16))) int8_t gradw_zero16[16];

// Column chunk q of 16 partial-sum columns -> tap row r, byte offset of the
// chunk's first value relative to the input pixel (0, 0) of the tap row
// (packed layout: kernel columns 4 t .. 4 t + 3 of 4 channels; else one tap and
// 16 channels).
struct GradwChunk {
  int r, s, ch;
};
__device__ __forceinline__ GradwChunk gradw_chunk(const ConvGeom& g, int q) {
  if (g.cp == 4) {
    const int q4 = (g.kw + 3) / 4;
    return GradwChunk{q / q4, 4 * (q % q4), 0};
  }
  const int cc = g.cp / 16, tap = q / cc;
  return GradwChunk{tap / g.kw, tap % g.kw, 16 * (q % cc)};
}
__host__ __device__ inline int gradw_chunks(const ConvGeom& g) {
  return g.cp == 4 ? g.kh * ((g.kw + 3) / 4) : g.kh * g.kw * (g.cp / 16);
}
int64_t conv_gradw_cols(const ConvGeom& g) { return 16 * (int64_t)gradw_chunks(g); }

// Block tile BM output channels x 128 columns; 64 x 64 per wave, the wave's
// K half (64 of the stage's 128 pixels) given by wk: at one transposed read of
// 512 bytes per MFMA and wave, a 64 x 64 wave tile is what the LDS bandwidth
// feeds at the MFMA rate.  Two blocks share a CU (72 or 64 KB of LDS each), so
// that one's load waits, pixel arithmetic and epilogue overlap the other's MFMAs.
template <int BM_>
struct GradwCfg {
  static constexpr int BM = BM_, BN = 128, BK = 128;
  static constexpr int WM = BM / 64, WN = 2;
  static constexpr int WAVES = 2 * WM * WN, THREADS = 64 * WAVES;
  static constexpr int NS = BM == 64 ? 3 : 2;
  static constexpr int STAGE = (BM + BN) * BK;
  static constexpr int A_INS = BM * BK / 1024 / WAVES, B_INS = BN * BK / 1024 / WAVES;
  static constexpr int PER = A_INS + B_INS;
};

// A block walks the 128-pixel stages of its split (one range of pixels), or,
// with a per-sample Q_b1, a range of the samples' stages in order (whole samples
// or part of one); pixels past the range (sample) load zeros.
template <int BM, bool PSQ, bool LIN>
__global__ __launch_bounds__(GradwCfg<BM>::THREADS, 2) void conv_gradw_kernel(ConvGradwParams p, ConvGeom g) {
  using C = GradwCfg<BM>;
  __shared__ __attribute__((aligned(16))) int8_t lds[C::NS * C::STAGE];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wk = wave / (C::WM * C::WN), wm = (wave / C::WN) % C::WM, wn = wave % C::WN;
  const int tiles_n = (int)((p.Np + C::BN - 1) / C::BN), tiles_m = (g.o + BM - 1) / BM;
  const int T = tiles_m * tiles_n;
  int tile, split;
  {
    // every tile of a split on one XCD (blocks go to the XCDs round robin), so
    // that the tiles sharing its pixels meet in that L2
    const int L = blockIdx.x;
    if (p.splits % NUM_XCD == 0) {
      const int j = L / NUM_XCD;
      tile = j % T;
      split = L % NUM_XCD + NUM_XCD * (j / T);
    } else {
      tile = L % T;
      split = L / T;
    }
  }
  const int m0 = (tile / tiles_n) * BM, n0 = (tile % tiles_n) * C::BN;
  const int howo = g.ho * g.wo;
  // first pixel (PSQ: stage) and number of stages
  const int spn = (howo + C::BK - 1) / C::BK;  // stages per sample (PSQ)
  int64_t first = (int64_t)split * p.per_split, last = first + p.per_split;
  const int64_t total = (int64_t)g.n * (PSQ ? spn : howo);
  if (first > total) first = total;
  if (last > total) last = total;
  const int nk = PSQ ? (int)(last - first) : (int)((last - first + C::BK - 1) / C::BK);

  // ---- per-lane load state
  const int8_t* const zero16 = gradw_zero16;
  constexpr int ACPR = BM / 16;  // 16-byte chunks per A row
  const int a_slot = lane % ACPR, a_row = lane / ACPR;
  const int a_swz = BM == 64 ? (a_row >> 1) & 3 : a_row & 7;
  const int a_ch = m0 + 16 * (a_slot ^ a_swz);
  const bool aok = a_ch < g.o;
  const int b_row = lane >> 3;
  const int q = n0 / 16 + ((lane & 7) ^ b_row);
  const bool bok = q < gradw_chunks(g);
  const GradwChunk ck = gradw_chunk(g, bok ? q : 0);
  const bool packed = g.cp == 4;
  const int Wp = packed ? g.wp : g.w;
  const int sy = ck.r - g.pad, sx = packed ? 0 : ck.s - g.pad;
  const uint32_t xlim = packed ? 0xFFFFFFFFu : (uint32_t)g.w;  // packed rows carry their halo
  const int8_t* const bbase = p.xq + ck.ch;
  const uint32_t toff = (uint32_t)(sy * Wp + (packed ? ck.s : sx));  // tap displacement (modulo 2^32, as lin)
  // advance by 128 pixels: dn samples, dy rows, dx columns
  const int dn = C::BK / howo, dr = C::BK - dn * howo, dy = dr / g.wo, dx = dr - dy * g.wo;
  const int sd = g.stride, wos = g.wo * sd, hos = g.ho * sd;
  const uint32_t dl0 = (uint32_t)((dn * g.h + dy * sd) * Wp + dx * sd);
  const uint32_t dl1 = (uint32_t)(sd * Wp - wos);              // x wraps: next row
  const uint32_t dl2 = (uint32_t)(g.h * Wp - hos * Wp);        // y wraps: next sample

  const int8_t* aptr[C::A_INS];
  int aleft[C::A_INS];
  int xs[C::B_INS], ys[C::B_INS];
  uint32_t lin[C::B_INS];  // linear index of the tap's input pixel (meaningful when it exists)
  const int8_t* bptr[C::B_INS];   // LIN
  int bleft[C::B_INS];            // LIN: pixels left in the tensor; PSQ: in the sample
  const uint32_t lin_end = (uint32_t)g.n * (uint32_t)(g.h * Wp);
  // PSQ: sample and stage in it of the next stage to load, and of the next to add up
  int lsmp = PSQ ? (int)(first / spn) : 0, lst = PSQ ? (int)(first - (int64_t)lsmp * spn) : 0;
  int csmp = lsmp, cst = lst;
  // position the walk at pixel p0 of the whole tensor, `left` pixels before its end
  auto seek = [&](int64_t p0, int left) {
#pragma unroll
    for (int i = 0; i < C::A_INS; ++i) {
      const int row = (64 / ACPR) * (wave * C::A_INS + i) + a_row;
      aptr[i] = p.q1 + (p0 + row) * g.o + a_ch;
      aleft[i] = left - row;
    }
#pragma unroll
    for (int i = 0; i < C::B_INS; ++i) {
      const int64_t px = p0 + 8 * (wave * C::B_INS + i) + b_row;
      if constexpr (LIN) {
        bptr[i] = p.xq + px * g.cp + ck.ch;
        bleft[i] = (int)((int64_t)g.n * howo - px);
      } else {
        if constexpr (PSQ) bleft[i] = left - (8 * (wave * C::B_INS + i) + b_row);
        // n ho wo < 2^30 (checked at launch)
        const uint32_t smp = (uint32_t)px / (uint32_t)howo, pix = (uint32_t)px - smp * (uint32_t)howo;
        const uint32_t y = pix / (uint32_t)g.wo;
        xs[i] = (int)(pix - y * g.wo) * sd;
        ys[i] = (int)y * sd;
        lin[i] = (smp * (uint32_t)g.h + (uint32_t)ys[i]) * (uint32_t)Wp + (uint32_t)xs[i] + toff;
      }
    }
  };
  if constexpr (PSQ)
    seek((int64_t)lsmp * howo + C::BK * lst, howo - C::BK * lst);
  else
    seek(first, (int)(last - first));

  // this wave's load `i` of the next stage to load, into buffer buf
  auto load = [&](int i, int8_t* buf) __attribute__((always_inline)) {
    if (i < C::A_INS) {
      const int8_t* src = aok & (aleft[i] > 0) ? aptr[i] : zero16;
      __builtin_amdgcn_global_load_lds((gmem_void*)src, (lmem_void*)(buf + (wave * C::A_INS + i) * 1024), 16, 0, 0);
      aptr[i] += (int64_t)C::BK * g.o;
      aleft[i] -= C::BK;
    } else {
      const int j = i - C::A_INS;
      const int8_t* src;
      if constexpr (LIN) {
        src = bok & (bleft[j] > 0) ? bptr[j] : zero16;
        bptr[j] += (int64_t)C::BK * g.cp;
        bleft[j] -= C::BK;
      } else {
        // padded taps, and pixels past the last sample (whose A codes are zero)
        bool in = bok & (lin[j] < lin_end) & ((uint32_t)(ys[j] + sy) < (uint32_t)g.h) &
                        ((uint32_t)(xs[j] + sx) < xlim);  // bitwise: no branches
        if constexpr (PSQ) {  // the next sample's pixels must not join the column sums
          in = in & (bleft[j] > 0);
          bleft[j] -= C::BK;
        }
        const int8_t* at = bbase + (uint64_t)lin[j] * (uint64_t)(uint32_t)g.cp;
        src = in ? at : zero16;
        xs[j] += dx * sd;
        ys[j] += dy * sd;
        lin[j] += dl0;
        const bool wx = xs[j] >= wos;
        xs[j] -= wx ? wos : 0;
        ys[j] += wx ? sd : 0;
        lin[j] += wx ? dl1 : 0u;
        const bool wy = ys[j] >= hos;
        ys[j] -= wy ? hos : 0;
        lin[j] += wy ? dl2 : 0u;
      }
      __builtin_amdgcn_global_load_lds((gmem_void*)src,
                                       (lmem_void*)(buf + C::BM * C::BK + (wave * C::B_INS + j) * 1024), 16, 0, 0);
    }
  };
  auto loaded = [&]() {  // one stage issued (PSQ: on to the next sample after its last stage)
    if constexpr (PSQ) {
      if (++lst == spn) {
        lst = 0;
        ++lsmp;
        seek((int64_t)lsmp * howo, howo);
      }
    }
  };

  // ---- LDS read offsets.  Transposed read t of a 32-column fragment covers
  // rows 8 t .. 8 t + 7 of the lane half's 16: lane i of a 16-lane group
  // addresses 8 bytes of row i / 2, and its group's 16 columns are one chunk.
  const int rg = lane >> 4, ri = lane & 15;
  const int r_row = 64 * wk + 16 * (rg >> 1) + (ri >> 1);
  int aoff[2], boff[2];
#pragma unroll
  for (int f = 0; f < 2; ++f) {
    const int ca = 4 * wm + 2 * f + (rg & 1), cb = 4 * wn + 2 * f + (rg & 1);
    const int asw = BM == 64 ? (ri >> 2) & 3 : ri >> 1;
    aoff[f] = r_row * BM + 16 * (ca ^ asw) + 8 * (ri & 1);
    boff[f] = BM * C::BK + r_row * 128 + 16 * (cb ^ (ri >> 1)) + 8 * (ri & 1);
  }

  v16i acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[i][j] = v16i{0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
  double accd[PSQ ? 2 : 1][PSQ ? 2 : 1][PSQ ? 16 : 1];
  double wb[2] = {0.0, 0.0};
  int csum[2] = {0, 0};
  if constexpr (PSQ) {
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) accd[i][j][r] = 0.0;
  }
  const bool colsum = m0 == 0 && wm == 0;  // the column code sums, once per column tile

  auto stage = [&](const int8_t* __restrict__ cur, int8_t* __restrict__ nxt, int t) __attribute__((always_inline)) {
    const bool more = t + C::NS - 1 < nk;
    if (t + C::NS - 2 < nk)
      __builtin_amdgcn_s_waitcnt(0x3F70 | ((C::NS - 2) * C::PER));  // vmcnt: later stages may stay in flight
    else
      __builtin_amdgcn_s_waitcnt(0x3F70);                           // vmcnt(0)
    __builtin_amdgcn_s_barrier();
    auto rd8 = [&](int off) __attribute__((always_inline)) {
      return __builtin_amdgcn_ds_read_tr8_b64_v2i32((lds_v2i*)(cur + off));
    };
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) {
      v4i a[2], b[2];
#pragma unroll
      for (int f = 0; f < 2; ++f) {
        const v2i a0 = rd8(aoff[f] + 32 * kk * BM), a1 = rd8(aoff[f] + (32 * kk + 8) * BM);
        const v2i b0 = rd8(boff[f] + 32 * kk * 128), b1 = rd8(boff[f] + (32 * kk + 8) * 128);
        a[f] = v4i{a0[0], a0[1], a1[0], a1[1]};
        b[f] = v4i{b0[0], b0[1], b1[0], b1[1]};
      }
      if (colsum) {
#pragma unroll
        for (int f = 0; f < 2; ++f)
#pragma unroll
          for (int u = 0; u < 4; ++u) csum[f] = sum4_i8((uint32_t)b[f][u], csum[f]);
      }
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a[i], b[j], acc[i][j], 0, 0, 0);
          const int m = (kk * 2 + i) * 2 + j;
          if (m < C::PER && more) load(m, nxt);
        }
    }
    static_assert(C::PER <= 8, "one load slot per MFMA");
    if (more) loaded();
  };
  // PSQ: after a sample's last stage in the split its exact int32 sums join the
  // float64 ones, weighted by the sample's step 1 / s (column sums: by its zero point)
  auto flush = [&](int t) {
    if constexpr (PSQ) {
      if (++cst < spn && t + 1 < nk) return;
      cst = 0;
      const int64_t smp = csmp++;
      const double dA = 1.0 / (double)p.scaleA[smp];
      const double zA = (double)p.zeroA[smp] + (double)p.halfA * dA;
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
#pragma unroll
          for (int r = 0; r < 16; ++r) accd[i][j][r] = fma(dA, (double)acc[i][j][r], accd[i][j][r]);
          acc[i][j] = v16i{0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
        }
#pragma unroll
      for (int f = 0; f < 2; ++f) {
        wb[f] = fma(zA, (double)csum[f], wb[f]);
        csum[f] = 0;
      }
    }
  };

  int8_t* const b0 = lds;
  int8_t* const b1 = lds + C::STAGE;
  int8_t* const b2 = lds + (C::NS > 2 ? 2 : 0) * C::STAGE;
  int8_t* const bufs[3] = {b0, b1, b2};
#pragma unroll
  for (int s = 0; s < C::NS - 1; ++s)
    if (s < nk) {
#pragma unroll
      for (int i = 0; i < C::PER; ++i) load(i, bufs[s]);
      loaded();
    }
  // stage t reads buffer t % NS and fills buffer (t + NS - 1) % NS
  for (int t = 0; t < nk; t += C::NS) {
    stage(b0, C::NS == 2 ? b1 : b2, t);
    flush(t);
    if (t + 1 < nk) {
      stage(b1, b0, t + 1);
      flush(t + 1);
    }
    if (C::NS > 2 && t + 2 < nk) {
      stage(b2, b1, t + 2);
      flush(t + 2);
    }
  }
  __syncthreads();

  // ---- column sums: the two lane halves hold different pixels of a column.  A
  // split's (at most 65536 pixels) are exact in 32 bits; over the splits they
  // are added in 64, which a tensor of 2^24 pixels needs.  Per-sample sums are
  // float64: kept per split and K half, rows o and o + 1 of its partial sums,
  // and added in a fixed order.
  const int64_t prow = (int64_t)split * (PSQ ? g.o + 2 : g.o);
  if (colsum) {
#pragma unroll
    for (int f = 0; f < 2; ++f) {
      const int col = n0 + 64 * wn + 32 * f + (lane & 31);
      if constexpr (PSQ) {
        const double w = wb[f] + __shfl_xor(wb[f], 32);
        if (lane < 32 && col < p.Np) p.partd[(prow + g.o + wk) * p.Np + col] = w;
      } else {
        const int c = csum[f] + __shfl_xor(csum[f], 32);
        if (lane < 32 && col < p.Np && c != 0)
          atomicAdd(reinterpret_cast<unsigned long long*>(p.sumB) + (split & (p.copies - 1)) * p.Np + col,
                    (unsigned long long)(int64_t)c);
      }
    }
  }
  // ---- the two K halves meet in LDS; accumulator (i, j, r) of lane l holds
  // row 64 wm + 32 i + 8 (r / 4) + 4 (l / 32) + r % 4, column 64 wn + 32 j + l % 32
  const int pair = wm * C::WN + wn;
  auto each = [&](int i, auto f) __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int row = m0 + 64 * wm + 32 * i + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
        const int col = n0 + 64 * wn + 32 * j + (lane & 31);
        f(j, r, row, col);
      }
  };
  if constexpr (PSQ) {
    static_assert(C::WM * C::WN * 32 * 64 * 8 <= C::NS * C::STAGE, "one row half of each wave tile in LDS");
    double* sh = reinterpret_cast<double*>(lds) + pair * (32 * 64);
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      if (wk == 1) each(i, [&](int j, int r, int, int) { sh[(j * 16 + r) * 64 + lane] = accd[i][j][r]; });
      __syncthreads();
      if (wk == 0)
        each(i, [&](int j, int r, int row, int col) {
          if (row < g.o && col < p.Np)
            p.partd[(prow + row) * p.Np + col] = accd[i][j][r] + sh[(j * 16 + r) * 64 + lane];
        });
      __syncthreads();
    }
  } else {
    static_assert(C::WM * C::WN * 64 * 64 * 4 <= C::NS * C::STAGE, "each wave tile in LDS");
    int32_t* sh = reinterpret_cast<int32_t*>(lds) + pair * (64 * 64);
    if (wk == 1)
#pragma unroll
      for (int i = 0; i < 2; ++i) each(i, [&](int j, int r, int, int) { sh[((i * 2 + j) * 16 + r) * 64 + lane] = acc[i][j][r]; });
    __syncthreads();
    if (wk == 0)
#pragma unroll
      for (int i = 0; i < 2; ++i)
        each(i, [&](int j, int r, int row, int col) {
          if (row < g.o && col < p.Np)
            p.part[(prow + row) * p.Np + col] = acc[i][j][r] + sh[((i * 2 + j) * 16 + r) * 64 + lane];
        });
  }
}

// Valid output rows / columns of a tap offset: lo <= y < hi with 0 <= y stride - pad + r < n.
__device__ __forceinline__ void gradw_tap_range(int r, int stride, int pad, int n, int no, int& lo, int& hi) {
  const int a = pad - r;  // y stride >= a
  lo = a > 0 ? (a + stride - 1) / stride : 0;
  const int e = n + pad - r;  // y stride < e
  hi = e > 0 ? (e + stride - 1) / stride : 0;
  lo = min(lo, no);
  hi = max(lo, min(hi, no));
}

// Zero-point sums of Q_b1 per (tap, o): the column sums qs[pixel][o] over the
// tap's valid pixels (a rectangle).  A block takes one tap and 8 channels, its
// 128 pixel lanes walk the rectangle, eight loads in flight (indices past the
// end are clamped, their values dropped), and meet in LDS in a fixed order.
// Sum: the 32-bit sums over the samples add up in 64 bits.
template <typename T, typename Sum>
__device__ __forceinline__ void gradw_tapsum(const ConvGeom& g, int64_t block, const T* qs, Sum* sumA) {
  constexpr int PL = 128;
  const int ob = (g.o + 7) / 8;
  const int tap = (int)(block / ob), o0 = 8 * (int)(block % ob);
  const int c = threadIdx.x & 7, pl = threadIdx.x >> 3;
  int ylo, yhi, xlo, xhi;
  gradw_tap_range(tap / g.kw, g.stride, g.pad, g.h, g.ho, ylo, yhi);
  gradw_tap_range(tap % g.kw, g.stride, g.pad, g.w, g.wo, xlo, xhi);
  const int wx = xhi - xlo, cnt = (yhi - ylo) * wx;
  const T* q = qs + o0 + c;  // o is a multiple of 16
  Sum sum = 0;
  for (int i0 = pl; i0 < cnt; i0 += 8 * PL) {
    T v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int i = min(i0 + u * PL, cnt - 1);
      const int yy = i / wx;
      v[u] = q[((int64_t)(ylo + yy) * g.wo + xlo + (i - yy * wx)) * g.o];
    }
#pragma unroll
    for (int u = 0; u < 8; ++u)
      if (i0 + u * PL < cnt) sum += v[u];
  }
  __shared__ Sum sp[PL][8];
  sp[pl][c] = sum;
  for (int h = PL / 2; h > 0; h >>= 1) {
    __syncthreads();
    if (pl < h) sp[pl][c] += sp[pl + h][c];
  }
  if (pl == 0) sumA[(int64_t)tap * g.o + o0 + c] = sp[0][c];
}

// sum_n zA_n of a per-sample Q_b1 (zA = z + half / s), one block
__device__ __forceinline__ void gradw_zsum(const ConvGradwParams& p, int n) {
  double zs = 0.0;
  for (int i = threadIdx.x; i < n; i += blockDim.x) zs += (double)p.zeroA[i] + (double)p.halfA * (1.0 / (double)p.scaleA[i]);
  __shared__ double sw[1024];
  sw[threadIdx.x] = zs;
  for (int h = blockDim.x / 2; h > 0; h >>= 1) {
    __syncthreads();
    if ((int)threadIdx.x < h) sw[threadIdx.x] += sw[threadIdx.x + h];
  }
  if (threadIdx.x == 0) p.zsum[0] = sw[0];
}

// Row sums of Q_b2: sg[pixel][slot] = sum over the channels of the codes
// [pixel][slot][o], four lanes per row (16 bytes each step).
__device__ __forceinline__ void gradw_sg(const ConvGeom& g, int64_t block, const int8_t* q2, int32_t* sg) {
  const int64_t row = block * 256 + (threadIdx.x >> 2);
  const int64_t rows = (int64_t)g.n * g.ho * g.wo;
  const int8_t* src = q2 + (row < rows ? row : rows - 1) * g.o;
  int sum = 0;
#pragma unroll 4
  for (int o = 16 * (threadIdx.x & 3); o < g.o; o += 64) {
    const uint4 v = *reinterpret_cast<const uint4*>(src + o);
    sum = sum4_i8(v.x, sum4_i8(v.y, sum4_i8(v.z, sum4_i8(v.w, sum))));
  }
  sum += __shfl_xor(sum, 1);
  sum += __shfl_xor(sum, 2);
  if ((threadIdx.x & 3) == 0 && row < rows) sg[row] = sum;
}

// The sums both contractions need, in one launch: blocks [0, nsg) the row sums
// of Q_b2, then the tap sums of Q_b1, then (per-sample Q_b1) the zero-point sum.
template <typename T, typename Sum>
__global__ __launch_bounds__(1024) void conv_sums_kernel(ConvGeom g, ConvGradwParams p, int64_t nsg, int64_t ntap,
                                                         const int8_t* q2, int32_t* sg, const T* qs, Sum* sumA) {
  const int64_t b = blockIdx.x;
  if (b < nsg)
    gradw_sg(g, b, q2, sg);
  else if (b < nsg + ntap)
    gradw_tapsum<T, Sum>(g, b - nsg, qs, sumA);
  else
    gradw_zsum(p, g.n);
}

// qw[pixel][o] = sum over samples n of codes q1[n][pixel][o] / s_n (float64),
// four consecutive values per thread, eight samples' loads in flight.
__global__ __launch_bounds__(256) void conv_wsum_kernel(ConvGeom g, const int8_t* q1, const float* scale, double* qw) {
  const int64_t D = (int64_t)g.ho * g.wo * g.o;
  const int64_t e = 4 * ((int64_t)blockIdx.x * 256 + threadIdx.x);
  if (e >= D) return;
  double s[4] = {0.0, 0.0, 0.0, 0.0};
  for (int n0 = 0; n0 < g.n; n0 += 8) {
    uint32_t v[8];
    double d[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int n = min(n0 + u, g.n - 1);
      v[u] = *reinterpret_cast<const uint32_t*>(q1 + (int64_t)n * D + e);
      d[u] = n0 + u < g.n ? 1.0 / (double)scale[n] : 0.0;
    }
#pragma unroll
    for (int u = 0; u < 8; ++u)
#pragma unroll
      for (int k = 0; k < 4; ++k) s[k] = fma(d[u], (double)(int8_t)(v[u] >> (8 * k)), s[k]);
  }
#pragma unroll
  for (int k = 0; k < 4; ++k) qw[e + k] = s[k];
}

// The reduction over splits and the zero-point expansion, with x1 = q1 dA + zA
// on output pixels and x2 = q2 dB + zB on valid taps:
//   per tensor: dA dB acc + dA zB SA[tap][o] + zA dB SB[col] + cnt zA zB
//   per sample: dB sum_n dA_n acc_n + zB sum_n dA_n SA_n + dB sum_n zA_n SB_n
//               + zB (valid pixels per sample) sum_n zA_n
// A block takes 64 output columns and W / sl rows: sl waves per
// row, each over every sl-th split, and all W waves over the parts of the column
// sums, a batch of loads of each in flight.  The waves' sums meet in LDS and are
// added in a fixed order.  Loads waiting on each other are all there is to it,
// so sl is the least that leaves a wave one batch of eight, at most 16, and W =
// sl, at least 4.  With 64 outputs and four waves per block whatever the number
// of splits (and the column sums of a per-sample Q_b1 added by one thread each):
// 3x3 3 -> 32 64x64 b128 (512 splits) 40 us, now 8; the same per sample (128
// splits) 74, now 8; stem (256) 22, now 7; 3x3 64ch 56x56 b128 (96) 10.5, now
// 8.8; 3x3 256ch 14x14 b32 per sample (7) 17, now 10.
constexpr int GR_WAVES = 16, GR_BATCH = 8;
inline int gradw_log2_split_lanes(int splits) {
  int l = 0;
  while ((1 << l) < GR_WAVES && splits > GR_BATCH << l) ++l;
  return l;
}
template <bool PSQ>
__global__ __launch_bounds__(64 * GR_WAVES) void conv_gradw_reduce_kernel(ConvGradwParams p, ConvGeom g, int lsl) {
  using Sum = typename std::conditional<PSQ, double, int64_t>::type;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int W = blockDim.x >> 6, rows = W >> lsl, sl = 1 << lsl;
  const int taps = g.kh * g.kw, N = taps * g.c, cols = (N + 63) / 64;
  const int row0 = (int)(blockIdx.x / cols) * rows;  // o is a multiple of 16: whole runs of rows
  // output column (tap, channel) and its column cc of the partial sums
  const int col = (int)(blockIdx.x % cols) * 64 + lane;
  const int tap = min(col, N - 1) / g.c, ch = min(col, N - 1) - tap * g.c;
  const int r = tap / g.kw, s = tap - r * g.kw;
  const int64_t cc = g.cp == 4 ? 16 * (r * ((g.kw + 3) / 4) + (s >> 2)) + 4 * (s & 3) + ch : tap * g.cp + ch;
  const int64_t pitch = (int64_t)(PSQ ? g.o + 2 : g.o) * p.Np;
  typedef typename std::conditional<PSQ, double, int>::type Part;
  typedef typename std::conditional<PSQ, double, int64_t>::type Col;
  // one batch: entries e0, e0 + step, ... below n (past it: the first, dropped
  // in the sum, so that the loads issue without branches), entry e being partial
  // row r of split e, or part e of the column sums
  auto load = [&](Part (&v)[GR_BATCH], int r, int e0, int step, int n) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < GR_BATCH; ++u) {
      const int64_t i = (e0 + u * step < n ? e0 + u * step : 0) * pitch + (int64_t)r * p.Np + cc;
      if constexpr (PSQ)
        v[u] = p.partd[i];
      else
        v[u] = p.part[i];
    }
  };
  constexpr int CB = PSQ ? GR_BATCH : 4;  // at most 16 copies, at least four waves: one batch
  auto load_col = [&](Col (&v)[CB], int e0, int step, int n) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < CB; ++u) {
      const int e = e0 + u * step < n ? e0 + u * step : 0;
      if constexpr (PSQ)
        v[u] = p.partd[(e >> 1) * pitch + (int64_t)(g.o + (e & 1)) * p.Np + cc];
      else
        v[u] = p.sumB[e * p.Np + cc];
    }
  };
  auto add = [&](const auto& v, int e0, int step, int n) __attribute__((always_inline)) {
    Sum sum = 0;
#pragma unroll
    for (int u = 0; u < (int)(sizeof(v) / sizeof(v[0])); ++u) sum += e0 + u * step < n ? (Sum)v[u] : (Sum)0;
    return sum;
  };
  const int myrow = row0 + (wave >> lsl), q = wave & (sl - 1), S = p.splits;
  const int NC = PSQ ? 2 * S : p.copies;  // parts of the column sums
  Part vr[GR_BATCH];
  Col vc[CB];
  load(vr, myrow, q, sl, S);
  load_col(vc, wave, W, NC);
  // the first `rows` waves finish a row each
  const bool out = wave < rows && col < N;
  const int row = row0 + wave;
  const int64_t ia = out ? (int64_t)tap * g.o + row : 0;
  Sum SA;
  if constexpr (PSQ)
    SA = p.sumAd[ia];
  else
    SA = p.sumA[ia];
  __shared__ Sum srow[GR_WAVES][64], scol[GR_WAVES][64];
  Sum sum = add(vr, q, sl, S), SB = add(vc, wave, W, NC);
  for (int e0 = q + GR_BATCH * sl; e0 < S; e0 += GR_BATCH * sl) {
    load(vr, myrow, e0, sl, S);
    sum += add(vr, e0, sl, S);
  }
  for (int e0 = wave + CB * W; e0 < NC; e0 += CB * W) {
    load_col(vc, e0, W, NC);
    SB += add(vc, e0, W, NC);
  }
  srow[wave][lane] = sum;
  scol[wave][lane] = SB;
  __syncthreads();
  if (!out) return;
  sum = 0;
  SB = 0;
  for (int w = 0; w < sl; ++w) sum += srow[wave * sl + w][lane];
  for (int w = 0; w < W; ++w) SB += scol[w][lane];
  int ylo, yhi, xlo, xhi;
  gradw_tap_range(r, g.stride, g.pad, g.h, g.ho, ylo, yhi);
  gradw_tap_range(s, g.stride, g.pad, g.w, g.wo, xlo, xhi);
  const double cnt = (double)((yhi - ylo) * (xhi - xlo));  // valid pixels per sample
  const double dB = 1.0 / (double)p.scaleB[0];
  const double zB = (double)p.zeroB[0] + (double)p.halfB * dB;
  double v;
  if constexpr (PSQ) {
    v = dB * sum + zB * SA + dB * SB + zB * cnt * p.zsum[0];
  } else {
    const double dA = 1.0 / (double)p.scaleA[0];
    const double zA = (double)p.zeroA[0] + (double)p.halfA * dA;
    v = dA * dB * (double)sum + dA * zB * (double)SA + zA * dB * (double)SB + cnt * (double)g.n * zA * zB;
  }
  p.out[(int64_t)row * N + col] = (float)v;
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
// Pixels (stages of a per-sample Q_b1) per split: at most 512 blocks, two per
// CU, in a multiple of the XCD count of splits when there are that many; whole
// 128-pixel stages, and at most 65536 pixels per int32 sum.  A per-sample block
// holds float64 sums too: one block per CU; whole samples where there are enough
// of them, else ranges of their stages (gradw_range).
//
// A range saves a block stages, which wait for their loads one after the other,
// and adds its partial sums to the reduction: taken from two stages less on,
// where it adds at most GRADW_PART partial sums per stage less.  Layers, whole
// samples / ranges: 3x3 3 -> 32 64x64 b128 139 / 110 us, b4 83 / 42, 1x1 64 -> 64
// 28x28 b4 57 / 49, 3x3 64 -> 64 56x56 b4 113 / 82; beyond the line 3x3 64 -> 128
// 28x28 b32 98.5 / 103.5, 1x1 256 -> 128 28x28 b32 88.8 / 93.7.
constexpr int64_t GRADW_PART = 65536;
static int64_t gradw_range(int64_t n, int64_t spn, int64_t want, int64_t part) {
  for (int64_t per = (n * spn + want - 1) / want; per + 2 <= spn; ++per)
    if (((n * spn + per - 1) / per - n) * part <= (spn - per) * GRADW_PART) return per;
  return spn;
}
void conv_gradw_splits(const ConvGeom& g, bool psq, int64_t& per_split, int& splits) {
  const int64_t bm = g.o <= 64 ? 64 : 128;
  const int64_t tiles = ((g.o + bm - 1) / bm) * ((conv_gradw_cols(g) + 127) / 128);
  const int64_t howo = (int64_t)g.ho * g.wo, spn = (howo + 127) / 128;
  int64_t want = (psq ? 256 : 512) / tiles;
  if (want >= NUM_XCD) want = want / NUM_XCD * NUM_XCD;
  if (want < 1) want = 1;
  // in 128-pixel stages
  const int64_t stages = psq ? g.n * spn : (g.n * howo + 127) / 128;
  int64_t per;
  if (!psq) {
    if (want > stages) want = stages;
    per = (stages + want - 1) / want;
    if (per > 512) per = 512;
  } else if (g.n >= want) {
    per = (g.n + want - 1) / want * spn;
  } else {
    per = gradw_range(g.n, spn, want, g.o * conv_gradw_cols(g));
  }
  int64_t n = (stages + per - 1) / per;
  if (n >= NUM_XCD && n % NUM_XCD != 0) n = (n + NUM_XCD - 1) / NUM_XCD * NUM_XCD;  // trailing splits may be empty
  per_split = psq ? per : per * 128;
  splits = (int)n;
}

hipError_t launch_conv_gradw(const ConvGradwParams& p, const ConvGeom& g, bool psq, hipStream_t s) {
  const int bm = g.o <= 64 ? 64 : 128;
  const int64_t blocks = ((g.o + bm - 1) / bm) * ((p.Np + 127) / 128) * (int64_t)p.splits;
  if (blocks < 1 || blocks > 0x7FFFFFFF || (g.o & 15) != 0 || p.Np != conv_gradw_cols(g) ||
      (((uintptr_t)p.q1 | (uintptr_t)p.xq) & 15) != 0)
    return hipErrorInvalidValue;
  const dim3 grid((unsigned)blocks);
  // one tap and no stride: pixel p of the output is pixel p of the input
  const bool lin = g.kh == 1 && g.kw == 1 && g.stride == 1 && g.pad == 0 && g.cp != 4;
#define FQT_GRADW(BM)                                                                                                  \
  do {                                                                                                                 \
    const dim3 thr(GradwCfg<BM>::THREADS);                                                                             \
    if (psq)                                                                                                           \
      hipLaunchKernelGGL((conv_gradw_kernel<BM, true, false>), grid, thr, 0, s, p, g);                                 \
    else if (lin)                                                                                                      \
      hipLaunchKernelGGL((conv_gradw_kernel<BM, false, true>), grid, thr, 0, s, p, g);                                 \
    else                                                                                                               \
      hipLaunchKernelGGL((conv_gradw_kernel<BM, false, false>), grid, thr, 0, s, p, g);                                \
  } while (0)
  if (bm == 64)
    FQT_GRADW(64);
  else
    FQT_GRADW(128);
#undef FQT_GRADW
  return hipGetLastError();
}

hipError_t launch_conv_sums(const ConvGradwParams& p, const ConvGeom& g, bool psq, const int8_t* q2, int32_t* sg,
                            hipStream_t s) {
  const int64_t nsg = sg ? ((int64_t)g.n * g.ho * g.wo + 255) / 256 : 0;
  const int64_t ntap = (int64_t)g.kh * g.kw * ((g.o + 7) / 8);
  const int64_t blocks = nsg + ntap + (psq ? 1 : 0);
  if (blocks > 0x7FFFFFFF) return hipErrorInvalidValue;
  if (psq) {
    const int64_t D4 = (int64_t)g.ho * g.wo * g.o / 4;
    if ((D4 + 255) / 256 > 0x7FFFFFFF) return hipErrorInvalidValue;
    hipLaunchKernelGGL(conv_wsum_kernel, dim3((unsigned)((D4 + 255) / 256)), dim3(256), 0, s, g, p.q1, p.scaleA, p.qsd);
    hipLaunchKernelGGL((conv_sums_kernel<double, double>), dim3((unsigned)blocks), dim3(1024), 0, s, g, p, nsg, ntap, q2, sg,
                       (const double*)p.qsd, p.sumAd);
  } else {
    hipLaunchKernelGGL((conv_sums_kernel<int32_t, int64_t>), dim3((unsigned)blocks), dim3(1024), 0, s, g, p, nsg, ntap, q2, sg,
                       (const int32_t*)p.qs, p.sumA);
  }
  return hipGetLastError();
}

hipError_t launch_conv_gradw_reduce(const ConvGradwParams& p, const ConvGeom& g, bool psq, hipStream_t s) {
  const int lsl = gradw_log2_split_lanes(p.splits), sl = 1 << lsl;
  const int waves = sl > 4 ? sl : 4;
  const int64_t blocks = (int64_t)g.o * sl / waves * (((int64_t)g.kh * g.kw * g.c + 63) / 64);
  if (blocks < 1 || blocks > 0x7FFFFFFF || (g.o & 15) != 0) return hipErrorInvalidValue;
  const dim3 grid((unsigned)blocks), threads(64 * waves);
  if (psq)
    hipLaunchKernelGGL(conv_gradw_reduce_kernel<true>, grid, threads, 0, s, p, g, lsl);
  else
    hipLaunchKernelGGL(conv_gradw_reduce_kernel<false>, grid, threads, 0, s, p, g, lsl);
  return hipGetLastError();
}

}  // namespace fqt
