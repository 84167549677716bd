// Conv layer FQT backward on gfx950 (NHWC tensors, rows = samples).
//
// The conv is the linear layer Y = im2col(X) W^T (Sec. 2.1 for linear layers),
// so its backward is grad_W = Q_b1(G)^T im2col(Q_f(X)) (conv_gradw.hip) and
// grad_X = col2im(Q_b2(G) Q_theta(W)) (Sec. 2.2).  Layouts:
//
//   X codes    [pixels][c]           per-tensor PTQ, channels padded (ConvGeom)
//   Q_b1(G)    [pixels][o]           stochastic PTQ or PSQ
//   W codes    [c][(r, s, o)]        per-tensor PTQ
//   Q_b2(G)    [(y, x)][slot][o]     PTQ / PSQ / BHQ, pixel-major, slot order
//
// grad_X is an implicit-im2col
// contraction: its A rows (input pixel, slot) are gathered 16 output
// channels at a time from Q_b2(G); padded taps load zero codes and the
// epilogue subtracts nothing for them (their zero-point sums are built from
// the valid taps only).  A tile row block holds the slots of one input pixel,
// so the block Householder inverse of a group runs inside the tile.
#include "gemm_core.h"

namespace fqt {

// ---------------------------------------------------------------------------
// grad_X helpers: CT[pix_in][c] = sum of W codes over the valid taps of an
// input pixel, cnt[pix_in] = their number
// ---------------------------------------------------------------------------
// taps (r, s) whose output pixel feeds input pixel (iy, ix)
__device__ __forceinline__ bool tap_hits(const ConvGeom& g, int iy, int ix, int r, int s, int& y, int& x) {
  const int ty = iy + g.pad - r, tx = ix + g.pad - s;
  if (ty < 0 || tx < 0 || ty % g.stride || tx % g.stride) return false;
  y = ty / g.stride;
  x = tx / g.stride;
  return y < g.ho && x < g.wo;
}

// Row sums of the grad_X A rows: rs[pix][slot] = sum of S_G[pixel][slot]
// over the output pixels whose taps reach input pixel pix (slot fastest,
// so a wave reads consecutive words of each tap's S_G run).  Stride 1: the
// taps' loads go out together (missing taps read entry 0 and add nothing).
template <bool S1>
__global__ void conv_rs_kernel(ConvGeom g, const int32_t* sg, int32_t* rs) {
  const uint32_t t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= (uint32_t)g.n * (uint32_t)(g.h * g.w)) return;
  const uint32_t pix = t / (uint32_t)g.n, slot = t - pix * (uint32_t)g.n;
  const int iy = (int)(pix / (uint32_t)g.w), ix = (int)pix - iy * g.w;
  int sum = 0;
  if constexpr (S1) {
    constexpr int U = 8;  // taps per round of loads
    const int taps = g.kh * g.kw;
    for (int t0 = 0; t0 < taps; t0 += U) {
      int v[U];
      bool ok[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int tap = t0 + u;
        const int r = tap / g.kw, s = tap - r * g.kw;
        const int y = iy + g.pad - r, x = ix + g.pad - s;
        ok[u] = tap < taps && y >= 0 && y < g.ho && x >= 0 && x < g.wo;
        v[u] = sg[ok[u] ? ((int64_t)y * g.wo + x) * g.n + slot : 0];
      }
#pragma unroll
      for (int u = 0; u < U; ++u) sum += ok[u] ? v[u] : 0;
    }
  } else {
    for (int r = 0; r < g.kh; ++r)
      for (int s = 0; s < g.kw; ++s) {
        int y, x;
        if (tap_hits(g, iy, ix, r, s, y, x)) sum += sg[((int64_t)y * g.wo + x) * g.n + slot];
      }
  }
  rs[t] = sum;
}

template <bool S1>
__global__ void conv_ct_kernel(ConvGeom g, const int32_t* swq, int32_t* ct, int32_t* cnt) {
  const int64_t hw = (int64_t)g.h * g.w;
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= hw * g.c) return;
  const int64_t pix = t / g.c;
  const int c = (int)(t % g.c);
  const int iy = (int)(pix / g.w), ix = (int)(pix % g.w);
  int sum = 0, n = 0;
  if constexpr (S1) {
    constexpr int U = 8;
    const int taps = g.kh * g.kw;
    for (int t0 = 0; t0 < taps; t0 += U) {
      int v[U];
      bool ok[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int tap = t0 + u;
        const int r = tap / g.kw, s = tap - r * g.kw;
        const int y = iy + g.pad - r, x = ix + g.pad - s;
        ok[u] = tap < taps && y >= 0 && y < g.ho && x >= 0 && x < g.wo;
        v[u] = swq[ok[u] ? (int64_t)tap * g.c + c : 0];
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        sum += ok[u] ? v[u] : 0;
        n += ok[u] ? 1 : 0;
      }
    }
  } else {
    for (int r = 0; r < g.kh; ++r)
      for (int s = 0; s < g.kw; ++s) {
        int y, x;
        if (tap_hits(g, iy, ix, r, s, y, x)) {
          sum += swq[(int64_t)(r * g.kw + s) * g.c + c];
          ++n;
        }
      }
  }
  ct[t] = sum;
  if (c == 0) cnt[pix] = n;
}

// Implicit im2col rows of grad_X: row m = (input pixel m / npad, slot m % npad);
// column k = (tap k / o, channel k % o).  16-byte chunks of 16 channels.
struct ConvXLoader {
  const int8_t* q2;
  ConvGeom g;
  int64_t M, K, D;
  struct Row {
    const int8_t* base;  // this slot's gradient codes
    int iy, ix;          // input pixel
    bool ok;
  };
  // M < 2^31 (checked at launch): the row splits in 32-bit arithmetic
  __device__ __forceinline__ Row row(int64_t m) const {
    Row rw{q2, 0, 0, false};
    if (m >= M) return rw;
    const uint32_t npad = (uint32_t)g.npad;
    const uint32_t pix = (uint32_t)m / npad, slot = (uint32_t)m - pix * npad;
    if (slot >= (uint32_t)g.n) return rw;
    rw.base = q2 + (int64_t)slot * g.o;  // pixel-major codes: slot offset inside each pixel
    rw.iy = (int)(pix / (uint32_t)g.w);
    rw.ix = (int)pix - rw.iy * g.w;
    rw.ok = true;
    return rw;
  }
  struct KState {
    int o0, r, s;  // channel offset and tap of the chunk column
    bool ok;
  };
  __device__ __forceinline__ KState kstate(int64_t k) const {
    KState ks{0, 0, 0, k < K};
    const int kk = (int)k;
    const int tap = kk / g.o;
    ks.o0 = kk - tap * g.o;
    ks.r = tap / g.kw;
    ks.s = tap - ks.r * g.kw;
    return ks;
  }
  __device__ __forceinline__ Chunk16 load(const Row& rw, const KState& ks) const {
    Chunk16 c{{0u, 0u, 0u, 0u}};
    if (!rw.ok || !ks.ok) return c;
    int y, x;
    if (g.stride == 1) {
      // output pixel (iy + pad - r, ix + pad - s): no divisions
      y = rw.iy + g.pad - ks.r;
      x = rw.ix + g.pad - ks.s;
      if (y < 0 || x < 0 || y >= g.ho || x >= g.wo) return c;
    } else if (!tap_hits(g, rw.iy, rw.ix, ks.r, ks.s, y, x)) {
      return c;
    }
    const uint4 v = *reinterpret_cast<const uint4*>(rw.base + ((int64_t)y * g.wo + x) * g.n * g.o + ks.o0);
    c.w[0] = v.x;
    c.w[1] = v.y;
    c.w[2] = v.z;
    c.w[3] = v.w;
    return c;
  }
};

// Stride-1 grad_X loader with at most 32 taps.  A row maps once to the code
// offset of output pixel (iy + pad, ix + pad) of its slot and a bit mask of
// the taps (r, s) whose output pixel (iy + pad - r, ix + pad - s) exists; a
// stage maps its K offset to a tap and the offset of that tap's channels
// relative to the row's pixel.  A chunk is then a bit test and an add; a
// lane whose tap misses reads a 16-byte block of zeros instead, so no lane
// is masked off around the load.
__device__ __attribute__((aligned(16))) int8_t conv_zero16[16];

struct ConvXLoader1 {
  const int8_t* q2;
  ConvGeom g;
  int64_t M, K, D;
  struct Row {
    int64_t off;    // codes of output pixel (iy + pad, ix + pad) of this slot
    uint32_t mask;  // bit r * kw + s: that tap reaches an output pixel
  };
  __device__ __forceinline__ Row row(int64_t m) const {
    Row rw{0, 0u};
    if (m >= M) return rw;
    const uint32_t npad = (uint32_t)g.npad;
    const uint32_t pix = (uint32_t)m / npad, slot = (uint32_t)m - pix * npad;
    if (slot >= (uint32_t)g.n) return rw;
    const int iy = (int)(pix / (uint32_t)g.w), ix = (int)pix - iy * g.w;
    const int yc = iy + g.pad, xc = ix + g.pad;
    uint32_t mask = 0u;
    for (int r = 0; r < g.kh; ++r)
      for (int s = 0; s < g.kw; ++s)
        if (yc - r >= 0 && yc - r < g.ho && xc - s >= 0 && xc - s < g.wo) mask |= 1u << (r * g.kw + s);
    rw.off = (((int64_t)yc * g.wo + xc) * g.n + slot) * g.o;  // pixel-major codes
    rw.mask = mask;
    return rw;
  }
  struct KState {
    int64_t off;  // channel offset of the tap minus its pixel displacement
    int tap;      // 32 (no tap) past the end of K
  };
  __device__ __forceinline__ KState kstate(int64_t k) const {
    KState ks{0, 32};
    if (k >= K) return ks;
    const int kk = (int)k;
    const int tap = kk / g.o;
    const int o0 = kk - tap * g.o;
    const int r = tap / g.kw, s = tap - r * g.kw;
    ks.off = (int64_t)o0 - ((int64_t)r * g.wo + s) * g.n * g.o;
    ks.tap = tap;
    return ks;
  }
  __device__ __forceinline__ Chunk16 load(const Row& rw, const KState& ks) const {
    const bool hit = ks.tap < 32 && ((rw.mask >> ks.tap) & 1u);
    const int8_t* src = hit ? q2 + (rw.off + ks.off) : conv_zero16;
    const uint4 v = *reinterpret_cast<const uint4*>(src);
    return Chunk16{{v.x, v.y, v.z, v.w}};
  }
};

// B operand of the grad_X contraction: the W codes [c][(r, s, o)] (16-byte
// aligned rows, K a multiple of 16).  Rows past N are clamped to the last
// one (their columns are never stored) and chunks past K come from the zero
// block, so the K loop has no branches around its loads.
struct ConvWLoader {
  const int8_t* B;
  int64_t ldb, N, K;
  __device__ __forceinline__ Chunk16 load(int64_t r, int64_t k) const {
    const int64_t rr = r < N ? r : N - 1;
    const int8_t* src = k < K ? B + rr * ldb + k : conv_zero16;
    const uint4 v = *reinterpret_cast<const uint4*>(src);
    return Chunk16{{v.x, v.y, v.z, v.w}};
  }
};

struct ConvRowStage {
  double rterm;  // zW * (codes summed over the valid taps of the row)
  double hz;     // BHQ group row: half + c_g;  affine row: z + half / s
  double dq;     // 1 / s
  int kind;      // BHQ slot kind (0 affine)
  int orow;      // output pixel row (sample * h * w + pixel), -1 if none
};

using CfgConvX = TileCfg<128, 64, 64, 64, 64>;  // 64-code K stages, 36 KB of LDS: four blocks per CU

// The K stages of a grad_X tile: only the taps that reach one of the tile's
// input pixels (a tile's 128 rows hold the slots of at most two pixels).
// With stride 2 about a quarter of the taps reach a pixel, and pixels with
// none (odd ones of a 1 x 1 stride-2 conv) run no K loop at all.  Stage t
// at K offset 64 st[t]; past the list, K (the loaders load zeros).
constexpr int CONVX_MAXST = 512;
struct KStageList {
  const uint16_t* st;
  int64_t n, K;
  __device__ __forceinline__ int64_t k(int64_t t) const { return t < n ? 64 * (int64_t)st[t] : K; }
};

template <int EPI, int KG, class XLoader>
__global__ __launch_bounds__(256) void conv_gradx_kernel(GemmParams p, ConvGeom g, const int8_t* q2, const int32_t* rs,
                                                          const int32_t* ct, const int32_t* cnt) {
  using C = CfgConvX;
  constexpr int EP_BYTES = C::BM * C::BN * 4 + C::BM * (int)sizeof(ConvRowStage);
  constexpr int BYTES = EP_BYTES > C::OP_BYTES ? EP_BYTES : C::OP_BYTES;
  __shared__ __attribute__((aligned(16))) int8_t lds[BYTES];
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int wm = wave / C::WAVES_N, wn = wave % C::WAVES_N;
  const int64_t tiles_n = (p.N + C::BN - 1) / C::BN;
  const int64_t tiles_m = (p.M + C::BM - 1) / C::BM;
  const int64_t tile = xcd_tile(blockIdx.x, tiles_m * tiles_n);
  const int64_t m0 = (tile / tiles_n) * C::BM;
  const int64_t n0 = (tile % tiles_n) * C::BN;
  const int lrow = lane & 31;
  const int h = lane >> 5;
  const int64_t D = (int64_t)g.ho * g.wo * g.o;

  v16i acc[C::IT][C::JT];
#pragma unroll
  for (int i = 0; i < C::IT; ++i)
#pragma unroll
    for (int j = 0; j < C::JT; ++j) acc[i][j] = v16i{0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
  const XLoader aload{q2, g, p.M, p.K, D};
  const int taps = g.kh * g.kw;
  const int spt = g.o / 64;  // K stages per tap
  if (taps <= 64 && g.o % 64 == 0 && taps * spt <= CONVX_MAXST) {
    __shared__ uint16_t s_st[CONVX_MAXST];
    __shared__ int s_nst;
    if (wave == 0) {
      // lane i: does tap i reach an input pixel of this tile?
      const uint32_t npad = (uint32_t)g.npad, hw = (uint32_t)(g.h * g.w);
      const uint32_t pa = (uint32_t)m0 / npad;
      const uint32_t last = (uint32_t)((m0 + C::BM - 1 < p.M ? m0 + C::BM - 1 : p.M - 1));
      const uint32_t pb = last / npad;
      bool hit = false;
      if (lane < taps) {
        const int r = lane / g.kw, s2 = lane - (lane / g.kw) * g.kw;
        int y, x;
        for (uint32_t pix = pa; pix <= pb && pix < hw; ++pix) {
          const int iy = (int)(pix / (uint32_t)g.w), ix = (int)pix - iy * g.w;
          if (tap_hits(g, iy, ix, r, s2, y, x)) hit = true;
        }
      }
      const uint64_t mask = __ballot(hit);
      if (hit) {
        const int before = __popcll(mask & ((1ull << lane) - 1ull));
        for (int j = 0; j < spt; ++j) s_st[before * spt + j] = (uint16_t)(lane * spt + j);
      }
      if (lane == 0) s_nst = __popcll(mask) * spt;
    }
    __syncthreads();
    generic_mainloop_km<C>(p, aload, ConvWLoader{p.B, p.ldb, p.N, p.K}, lds, m0, n0, KStageList{s_st, s_nst, p.K},
                           acc);
  } else {
    generic_mainloop<C>(p, aload, ConvWLoader{p.B, p.ldb, p.N, p.K}, lds, m0, n0, 0, p.K, acc);
  }

  int32_t* sacc = reinterpret_cast<int32_t*>(lds);
  ConvRowStage* srow = reinterpret_cast<ConvRowStage*>(lds + C::BM * C::BN * 4);
  const double dW = 1.0 / (double)p.scaleB[0];
  const double zW = (double)p.zeroB[0] + (double)p.halfB * dW;
#pragma unroll
  for (int i = 0; i < C::IT; ++i)
#pragma unroll
    for (int j = 0; j < C::JT; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r)
        sacc[(wm * C::WM + i * 32 + 8 * (r >> 2) + 4 * h + (r & 3)) * C::BN + wn * C::WN + j * 32 + lrow] =
            acc[i][j][r];
  // Row terms, one thread per tile row.  M < 2^31 (checked by the launcher),
  // so the row splits into (input pixel, slot) in 32-bit arithmetic; S_G is
  // pixel-major, so the slots of one tap read consecutive words.
  if (tid < C::BM) {
    const int64_t m = m0 + tid;
    ConvRowStage q{};
    q.orow = -1;
    const uint32_t npad = (uint32_t)g.npad;
    const uint32_t pix = (uint32_t)m / npad, slot = (uint32_t)m - pix * npad;
    if (m < p.M && slot < (uint32_t)g.n) {
      const float s = p.rowwiseA ? p.scaleA[slot] : p.scaleA[0];
      const float z = p.rowwiseA ? p.zeroA[slot] : p.zeroA[0];
      q.kind = (EPI == EPI_BHQ) ? bhq_slot_kind(p.L, slot) : (EPI == EPI_BHQT ? (p.slot[slot].size > 1) : 0);
      q.rterm = zW * (double)rs[(int64_t)pix * g.n + slot];
      q.dq = 1.0 / (double)s;
      q.hz = q.kind != 0 ? (double)p.halfA + (double)z : (double)z + (double)p.halfA * q.dq;
      q.orow = (int)((p.perm ? (int64_t)p.perm[slot] : (int64_t)slot) * ((int64_t)g.h * g.w) + pix);
    }
    srow[tid] = q;
  }
  __syncthreads();
  // Wave w owns the 64 tile rows [64 w, 64 w + 64): one run, the slots of one
  // input pixel (npad % 64 == 0), so the column terms are loaded once.  Lane
  // l holds the four columns n0 + 4 (l % 16) .. +3 of row 4 i + l / 16 in
  // step i, so one step covers four rows and stores 16-byte words.  A BHQ
  // group of KG rows (KG <= 64, aligned) lies inside the run; its column sums
  // meet across the four row lanes by xor shuffles, which give every lane of
  // the group the same sum.
  constexpr int WROWS = C::BM / C::WAVES;
  static_assert(C::BN == 64 && WROWS == 64 && KG <= 64, "epilogue wave layout");
  const int r0 = wave * WROWS;
  const int cq = lane & 15, rsub = lane >> 4;
  const int64_t col = n0 + 4 * cq;
  if (col >= p.N || m0 + r0 >= p.M) return;
  const bool vec = col + 3 < p.N && (p.ldo & 3) == 0 && ((uintptr_t)p.out & 15) == 0;
  const int64_t pix = (int64_t)((uint32_t)(m0 + r0) / (uint32_t)g.npad);
  const double kz = (double)cnt[pix] * ((double)g.o * zW);
  double colterm[4];
#pragma unroll
  for (int e = 0; e < 4; ++e)
    colterm[e] = col + e < p.N ? dW * (double)ct[pix * g.c + col + e] + kz : 0.0;
  auto row_acc = [&](int row, double (&a)[4]) {
    const int4 v = *reinterpret_cast<const int4*>(&sacc[row * C::BN + 4 * cq]);
    a[0] = (double)v.x;
    a[1] = (double)v.y;
    a[2] = (double)v.z;
    a[3] = (double)v.w;
  };
  auto store = [&](int orow, const double (&v)[4]) {
    float* dst = p.out + (int64_t)orow * p.ldo + col;
    if (vec) {
      *reinterpret_cast<float4*>(dst) = make_float4((float)v[0], (float)v[1], (float)v[2], (float)v[3]);
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (col + e < p.N) dst[e] = (float)v[e];
    }
  };
  if constexpr (EPI == EPI_BHQ && KG > 1) {
    constexpr int RB = KG > 4 ? KG : 4;  // rows per block of steps
    for (int blk = r0; blk < r0 + WROWS; blk += RB) {
      double S[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll 4
      for (int i = 0; i < RB / 4; ++i) {
        const int row = blk + 4 * i + rsub;
        const ConvRowStage& q = srow[row];
        double a[4];
        row_acc(row, a);
        if (q.kind != 0) {
#pragma unroll
          for (int e = 0; e < 4; ++e) S[e] += dW * a[e] + (q.rterm + q.hz * colterm[e]);
        }
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        S[e] += __shfl_xor(S[e], 16);
        if constexpr (KG >= 4) S[e] += __shfl_xor(S[e], 32);
      }
      const int g0 = (blk + rsub) & ~(KG - 1);  // first row of this lane's group
      const ConvRowStage& q0 = srow[g0];
      if (q0.orow < 0 && q0.kind == 0) continue;
      double a0[4], tau[4];
      row_acc(g0, a0);
      const double alpha = q0.kind == 2 ? p.L.inv_sk_p : p.L.inv_sk_k;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const double T0 = dW * a0[e] + (q0.rterm + q0.hz * colterm[e]);
        tau[e] = (alpha * S[e] - T0) / (1.0 - alpha);
      }
#pragma unroll 4
      for (int i = 0; i < RB / 4; ++i) {
        const int row = blk + 4 * i + rsub;
        const ConvRowStage& q = srow[row];
        if (q.orow < 0) continue;
        double a[4], v[4];
        row_acc(row, a);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          if (q.kind != 0) {
            const double T = dW * a[e] + (q.rterm + q.hz * colterm[e]);
            const double Z = (row == g0) ? T + (1.0 - alpha) * tau[e] : T - alpha * tau[e];
            v[e] = Z * q.dq;
          } else {
            v[e] = q.dq * (dW * a[e] + q.rterm) + q.hz * colterm[e];
          }
        }
        store(q.orow, v);
      }
    }
  } else {
#pragma unroll 4
    for (int i = 0; i < WROWS / 4; ++i) {
      const int row = r0 + 4 * i + rsub;
      const ConvRowStage& q = srow[row];
      if (q.orow < 0) continue;
      double a[4], v[4];
      row_acc(row, a);
      if (EPI == EPI_BHQT && q.kind != 0) {
        // a row of a multi-row group of the general plan: its T for the inverse pass
        double* dst = p.tbuf + (m0 + row) * p.ldt + col;
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (col + e < p.N) dst[e] = dW * a[e] + (q.rterm + q.hz * colterm[e]);
        continue;
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = q.dq * (dW * a[e] + q.rterm) + q.hz * colterm[e];
      store(q.orow, v);
    }
  }
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
hipError_t launch_conv_gradx_prep(const ConvGeom& g, const int32_t* swq, const int32_t* sg, int32_t* rs, int32_t* ct,
                                  int32_t* cnt, hipStream_t s) {
  const int64_t nr = (int64_t)g.n * g.h * g.w;
  if (nr > 0x7FFFFFFF) return hipErrorInvalidValue;
  if (g.stride == 1)
    hipLaunchKernelGGL(conv_rs_kernel<true>, dim3((unsigned)((nr + 255) / 256)), dim3(256), 0, s, g, sg,
                       rs);
  else
    hipLaunchKernelGGL(conv_rs_kernel<false>, dim3((unsigned)((nr + 255) / 256)), dim3(256), 0, s, g, sg,
                       rs);
  const int64_t n2 = (int64_t)g.h * g.w * g.c;
  if (g.stride == 1)
    hipLaunchKernelGGL(conv_ct_kernel<true>, dim3((unsigned)((n2 + 255) / 256)), dim3(256), 0, s, g, swq, ct, cnt);
  else
    hipLaunchKernelGGL(conv_ct_kernel<false>, dim3((unsigned)((n2 + 255) / 256)), dim3(256), 0, s, g, swq, ct, cnt);
  return hipGetLastError();
}

template <int EPI, int KG>
static hipError_t launch_conv_gradx_t(const GemmParams& p, const ConvGeom& g, const int8_t* q2, const int32_t* rs,
                                      const int32_t* ct, const int32_t* cnt, hipStream_t s) {
  const int64_t tiles = ((p.M + CfgConvX::BM - 1) / CfgConvX::BM) * ((p.N + CfgConvX::BN - 1) / CfgConvX::BN);
  if (tiles > 0x7FFFFFFF || p.M > 0x7FFFFFFF || g.npad % 64 != 0) return hipErrorInvalidValue;
  // q2 is a workspace carve (16-byte aligned); o % 16 == 0 keeps every chunk aligned
  if (g.stride == 1 && g.kh * g.kw <= 32)
    hipLaunchKernelGGL((conv_gradx_kernel<EPI, KG, ConvXLoader1>), dim3((unsigned)tiles), dim3(CfgConvX::THREADS), 0,
                       s, p, g, q2, rs, ct, cnt);
  else
    hipLaunchKernelGGL((conv_gradx_kernel<EPI, KG, ConvXLoader>), dim3((unsigned)tiles), dim3(CfgConvX::THREADS), 0,
                       s, p, g, q2, rs, ct, cnt);
  return hipGetLastError();
}

hipError_t launch_conv_gradx(const GemmParams& p, int epi, const ConvGeom& g, const int8_t* q2, const int32_t* rs,
                             const int32_t* ct, const int32_t* cnt, hipStream_t s) {
  if (epi == EPI_ROW) return launch_conv_gradx_t<EPI_ROW, 0>(p, g, q2, rs, ct, cnt, s);
  if (epi == EPI_BHQT)
    return p.slot && p.tbuf ? launch_conv_gradx_t<EPI_BHQT, 0>(p, g, q2, rs, ct, cnt, s) : hipErrorInvalidValue;
  switch (p.L.k) {
    case 1: return launch_conv_gradx_t<EPI_BHQ, 1>(p, g, q2, rs, ct, cnt, s);
    case 2: return launch_conv_gradx_t<EPI_BHQ, 2>(p, g, q2, rs, ct, cnt, s);
    case 4: return launch_conv_gradx_t<EPI_BHQ, 4>(p, g, q2, rs, ct, cnt, s);
    case 8: return launch_conv_gradx_t<EPI_BHQ, 8>(p, g, q2, rs, ct, cnt, s);
    case 16: return launch_conv_gradx_t<EPI_BHQ, 16>(p, g, q2, rs, ct, cnt, s);
    case 32: return launch_conv_gradx_t<EPI_BHQ, 32>(p, g, q2, rs, ct, cnt, s);
    case 64: return launch_conv_gradx_t<EPI_BHQ, 64>(p, g, q2, rs, ct, cnt, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace fqt
