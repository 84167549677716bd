// Conv layer FQT backward on gfx950 (NHWC tensors, rows = samples): grad_X.
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
// grad_X row m is (input pixel m / npad, slot m % npad).  A wave owns a unit
// of 64 consecutive rows and 64 input channels, and contracts over the taps
// that reach its pixels only: its list of 16-channel chunks (valid tap, chunk)
// feeds v_mfma_i32_16x16x64_i8, whose 16-lane groups take four consecutive
// chunks.  The rows of a tap are one run of Q_b2, read straight into registers
// (a 16-row fragment has one pixel, so a tap's validity is uniform in it); the
// W codes of the block's 64 channels sit in LDS.  Waves meet only where that
// panel is (re)loaded.  The epilogue works on the accumulators in registers:
// a block Householder group (at most 64 aligned slots of one pixel) lies
// inside the unit, its column sums meet across the four lane groups.
//
// What bounds it is latency, with 8 waves per CU: the accumulators and the
// fragments ahead take up to 256 registers.  Against the 128 x 64 tiles before
// (register-staged gather through LDS, float64 epilogue through LDS, two sum
// kernels of their own): 3x3 64ch 56x56 b128 BHQ 106 -> 62 us, 3x3 s2 128ch
// 56x56 b256 BHQ 287 -> 176 us, 1x1 1024 -> 256 14x14 b256 PSQ 56 -> 49 us,
// 3x3 256ch 14x14 b32 PSQ 43 -> 42 us; with nontemporal output stores and the
// panel straight to LDS 54, 155, 42 and 31 us.  Kept back: 32 channels per wave, for
// twice the waves (spills, 174 us on the first); fragment loads three steps
// ahead (84 us); four-byte stores, one per fragment (72 us).
#include "gemm_core.h"

namespace fqt {

// One unit's scratch in LDS.  In the K loop: per valid tap the output pixel of
// each fragment (-1: none), the offset of its codes and the tap; in the epilogue the row and column data.
struct ConvXWave {
  union {
    struct {
      int4 pix[64];
      uint4 off[64];
      int tap[64];
    } k;
    struct {
      double2 ab[64];  // dq dW, dq rterm
      double e1[64];   // weight of the group's column term (dq in a multi-row group, else 0)
      double e2[64];   // weight of the column's own term (hz of a one-row group or affine row, else 0)
      int orow[64];    // output pixel row, -1: none
      int col[4][64];  // W code sums over the taps that reach each fragment's pixel
    } e;
  };
};
constexpr int CX_BN = 64;
// Channel (of the block's 64) in panel row r: fragment j of lane c then holds
// channel 4 c + j, so that a lane's four fragments are one 16-byte store.
__device__ __forceinline__ int cx_col(int r) { return 4 * (r & 15) + (r >> 4); }

struct ConvXTile {
  int per_wave;  // units per wave (1 with several panel chunks)
  int tpc, cpc;  // taps and channels per panel chunk
  uint32_t zoff; // 16 bytes of zeros, in 16-byte steps from the Q_b2 codes
  int pitch;     // bytes per panel row: an odd number of 16-byte chunks, so that 16 rows fall on distinct banks
};

// taps (r, s) whose output pixel feeds input pixel (iy, ix)
__device__ __forceinline__ bool tap_hits(const ConvGeom& g, int iy, int ix, int r, int s, int& y, int& x) {
  const int ty = iy + g.pad - r, tx = ix + g.pad - s;
  if (g.stride == 1) {
    y = ty;
    x = tx;
    return (uint32_t)ty < (uint32_t)g.ho && (uint32_t)tx < (uint32_t)g.wo;
  }
  if (g.stride == 2) {
    y = ty >> 1;
    x = tx >> 1;
    return ((ty | tx) & 1) == 0 && (uint32_t)y < (uint32_t)g.ho && (uint32_t)x < (uint32_t)g.wo;
  }
  if (ty < 0 || tx < 0 || ty % g.stride || tx % g.stride) return false;
  y = ty / g.stride;
  x = tx / g.stride;
  return y < g.ho && x < g.wo;
}

// UNI: the channels come in whole 64s, so that a step's tap and channel are the
// same in every lane: addresses are scalar plus a lane constant, and a fragment
// whose pixel the tap misses takes no MFMA.  Otherwise each lane group looks its list
// position up in LDS.
// ONE: the unit's rows share their pixel.
template <int EPI, int KE, bool UNI, bool ONE, bool NT>
__global__ __launch_bounds__(512, 2) void conv_gradx_kernel(GemmParams p, ConvGeom g, ConvXTile t, const int8_t* q2,
                                                          const int32_t* sg, const int32_t* swq) {
  extern __shared__ __attribute__((aligned(16))) int8_t cx_lds[];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int waves = blockDim.x >> 6;
  int8_t* const panel = cx_lds;
  ConvXWave& sw = *reinterpret_cast<ConvXWave*>(cx_lds + CX_BN * t.pitch + wave * (int)sizeof(ConvXWave));
  const int lg = lane >> 4, lc = lane & 15;
  const int spad = (int)g.npad, hw = g.h * g.w, taps = g.kh * g.kw;
  const uint32_t M = (uint32_t)p.M;  // < 2^31, checked at launch
  const int tiles_n = (g.c + CX_BN - 1) / CX_BN;
  const int64_t tile = xcd_tile(blockIdx.x, gridDim.x);
  const int n0 = (int)(tile % tiles_n) * CX_BN;
  const uint32_t u0 = (uint32_t)(tile / tiles_n) * (uint32_t)(waves * t.per_wave);
  constexpr bool onepix = ONE;  // the four fragments of a unit share their pixel
  const int colc = min(n0 + lane, g.c - 1);
  const double dW = 1.0 / (double)p.scaleB[0];
  const double zW = (double)p.zeroB[0] + (double)p.halfB * dW;
  // the last 16 bytes of each panel row are zero
  const int zchunk = t.pitch - 16;
  if (threadIdx.x < CX_BN) *reinterpret_cast<uint4*>(panel + threadIdx.x * t.pitch + zchunk) = make_uint4(0u, 0u, 0u, 0u);

  for (int it = 0; it < t.per_wave; ++it) {
    const uint32_t row0 = (u0 + (uint32_t)(it * waves + wave)) * 64u;  // first row of the unit
    // fragment f: its input pixel (hw: none)
    int fy[4], fx[4], fpix[4];
#pragma unroll
    for (int f = 0; f < 4; ++f) {
      const uint32_t m = row0 + 16 * (onepix ? 0 : f);
      fpix[f] = m < M ? (int)(m / (uint32_t)spad) : hw;
      fy[f] = fpix[f] / g.w;
      fx[f] = fpix[f] - fy[f] * g.w;
    }
    const int slot0 = (int)(row0 % (uint32_t)spad);  // of row 0 (spad < 64: 0)
    // slot of unit row k
    auto slot_of = [&](int k) { return onepix ? slot0 + k : k & (spad - 1); };
    // offset of this lane's row of each fragment inside an output pixel's codes
    // (16-byte steps; slots clamped: rows past n are not stored)
    const uint32_t och = (uint32_t)g.o / 16, pixoff = (uint32_t)g.n * och;
    uint32_t arow[4];
#pragma unroll
    for (int f = 0; f < 4; ++f) arow[f] = (uint32_t)min(slot_of(16 * f + lc), g.n - 1) * och;
    const int myslot = slot_of(lane), myfrag = lg;
    int mypix = fpix[0];
    if (!onepix) mypix = lg == 0 ? fpix[0] : (lg == 1 ? fpix[1] : (lg == 2 ? fpix[2] : fpix[3]));
    const bool myrow = mypix < hw && myslot < g.n;

    // this lane's row: scale, zero point, sample (used in the epilogue)
    const float row_s = p.scaleA[p.rowwiseA && myrow ? myslot : 0], row_z = p.zeroA[p.rowwiseA && myrow ? myslot : 0];
    const int row_n = myrow ? (p.perm ? p.perm[myslot] : myslot) : 0;

    const int myslot_c = min(myslot, g.n - 1);
    // UNI: byte offsets of this lane's 16 bytes in an output pixel's codes (n o
    // < 2^32, checked at launch) and in the panel
    uint32_t avo[4];
#pragma unroll
    for (int f = 0; f < 4; ++f) avo[f] = 16u * (arow[f] + (uint32_t)lg);
    const int bvo = lc * t.pitch + 16 * lg;

    v4i acc[4][4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) acc[i][j] = v4i{0, 0, 0, 0};
    int rsum = 0;                 // Q_b2 code sum of this lane's row over its taps
    int csum[4] = {0, 0, 0, 0};   // W code sum of this lane's column over each fragment's taps
    int cnt[4] = {0, 0, 0, 0};    // number of each fragment's taps

    for (int c0 = 0; c0 < g.o; c0 += t.cpc)
      for (int t0 = 0; t0 < taps; t0 += t.tpc) {
        const int nt = min(t.tpc, taps - t0), nch = min(t.cpc, g.o - c0) / 16;
        if (it == 0) {
          // the panel: 64 channels' codes of taps [t0, t0 + nt), output channels [c0, c0 + 16 nch)
          __syncthreads();
          // Straight to LDS, 64 chunks of a row per load (the last 64 overlap the
          // ones before), so that the whole panel is in flight at once: through
          // registers it took a round trip per eight rows (3x3 256ch 14x14 b32,
          // 147 KB: layer 118.2 -> 109.3 us; 3x3 s2 128ch 56x56 b256 476 -> 469).
          const int per = nt * nch;
          if (per >= 64) {
            for (int k0 = 0; k0 < per; k0 += 64) {
              const int kb = min(k0, per - 64), k = kb + lane;
              const int tp = k / nch, ch = k - tp * nch;
              const int8_t* src = p.B + (int64_t)(t0 + tp) * g.o + c0 + 16 * ch;
              for (int r = wave; r < CX_BN; r += waves)
                __builtin_amdgcn_global_load_lds((gmem_void*)(src + (int64_t)min(n0 + cx_col(r), g.c - 1) * p.ldb),
                                                 (lmem_void*)(panel + r * t.pitch + 16 * kb), 16, 0, 0);
            }
            __builtin_amdgcn_s_waitcnt(0x3F70);  // vmcnt(0)
          } else {
            // (lanes over the chunks of a row, eight rows in flight; waves is 4 or 8)
            constexpr int PR = 8;
            for (int k0 = 0; k0 < per; k0 += 64) {
              const int k = min(k0 + lane, per - 1);
              const int tp = k / nch, ch = k - tp * nch;
              const int8_t* src = p.B + (int64_t)(t0 + tp) * g.o + c0 + 16 * ch;
              for (int r0 = 0; r0 < CX_BN; r0 += PR * waves) {
                uint4 v[PR];
#pragma unroll
                for (int u = 0; u < PR; ++u)
                  v[u] = *reinterpret_cast<const uint4*>(src + (int64_t)min(n0 + cx_col(r0 + u * waves + wave), g.c - 1) * p.ldb);
#pragma unroll
                for (int u = 0; u < PR; ++u)
                  *reinterpret_cast<uint4*>(panel + (r0 + u * waves + wave) * t.pitch + 16 * k) = v[u];
              }
            }
          }
          __syncthreads();
        }
        // ---- valid taps: lane i tests tap t0 + i
        int px[4] = {-1, -1, -1, -1};
        bool any = false;
        if (lane < nt) {
          const int tp = t0 + lane, r = tp / g.kw, s = tp - r * g.kw;
#pragma unroll
          for (int f = 0; f < 4; ++f) {
            int y, x;
            if (f > 0 && onepix) {
              px[f] = px[0];
            } else if (fpix[f] < hw && tap_hits(g, fy[f], fx[f], r, s, y, x)) {
              px[f] = y * g.wo + x;
              any = true;
            }
          }
        }
        const uint64_t mask = __ballot(any);
        const int nv = __popcll(mask);
        if (!UNI && any) {
          const int at = __popcll(mask & ((1ull << lane) - 1ull));
          sw.k.pix[at] = make_int4(px[0], px[1], px[2], px[3]);
          sw.k.off[at] = make_uint4(px[0] * pixoff, px[1] * pixoff, px[2] * pixoff, px[3] * pixoff);
          sw.k.tap[at] = lane;
        }
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (UNI) {
          if (nv == 0) continue;  // the unit's pixels have no tap here
          const int stepsu = nv * (nch / 4);
          uint64_t rem = mask;
          int ch = -4, tap = 0, left = stepsu;
          int tpx[4] = {0, 0, 0, 0};  // the tap's output pixel of each fragment (-1: none)
          struct Pos {
            uint64_t ao[ONE ? 1 : 4];  // byte offset of each fragment's codes
            int bo;          // panel offset
            uint32_t vm;     // fragments that have the tap
          };
          // position of the next step to load (past the end: the last one again)
          auto next = [&](Pos& q) __attribute__((always_inline)) {
            if (left > 0) {
              ch += 4;
              if (ch == nch || left == stepsu) {
                ch = 0;
                tap = __builtin_ctzll(rem);
                rem &= rem - 1;
                tpx[0] = __builtin_amdgcn_readlane(px[0], tap);
                if (!onepix) {
#pragma unroll
                  for (int f = 1; f < 4; ++f) tpx[f] = __builtin_amdgcn_readlane(px[f], tap);
                }
              }
              --left;
            }
            q.bo = 16 * (tap * nch + ch);
            q.vm = 0xFu;
            const uint32_t cc = (uint32_t)c0 / 16 + (uint32_t)ch;
#pragma unroll
            for (int f = 0; f < (ONE ? 1 : 4); ++f) {
              const int e = tpx[f];
              if (!ONE && e < 0) q.vm &= ~(1u << f);
              q.ao[f] = 16 * (uint64_t)((!ONE && e < 0 ? 0u : (uint32_t)e * pixoff) + cc);
            }
          };
          auto aload = [&](const Pos& q, v4i (&a)[4]) __attribute__((always_inline)) {
#pragma unroll
            for (int f = 0; f < 4; ++f) a[f] = *reinterpret_cast<const v4i*>(q2 + q.ao[ONE ? 0 : f] + avo[f]);
          };
          auto bload = [&](int bo, v4i (&b)[4]) __attribute__((always_inline)) {
#pragma unroll
            for (int j = 0; j < 4; ++j) b[j] = *reinterpret_cast<const v4i*>(panel + bvo + 16 * j * t.pitch + bo);
          };
          auto mma = [&](const v4i (&a)[4], const v4i (&b)[4], uint32_t vm) __attribute__((always_inline)) {
            if constexpr (ONE) {
#pragma unroll
              for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int i = 0; i < 4; ++i)
                  acc[i][j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a[i], b[j], acc[i][j], 0, 0, 0);
            } else {
#pragma unroll
              for (int i = 0; i < 4; ++i)
                if ((vm >> i) & 1u) {
#pragma unroll
                  for (int j = 0; j < 4; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a[i], b[j], acc[i][j], 0, 0, 0);
                }
            }
          };
          v4i a0[4], a1[4], bb0[4], bb1[4];
          Pos q0, q1;
          next(q0);
          aload(q0, a0);
          next(q1);
          aload(q1, a1);
          bload(q0.bo, bb0);
          if (c0 == 0) {
            // zero-point sums over the taps: S_G of this lane's row, W sums of its column
            const int32_t* const sgl = sg + myslot_c;
            const int32_t* const swl = swq + (int64_t)t0 * g.c + colc;
            uint64_t m2 = mask;
            while (m2) {
              constexpr int U = 6;
              int va[U], vb[U];
              uint32_t vm[U];
#pragma unroll
              for (int u = 0; u < U; ++u) {
                const bool on = m2 != 0;
                const int tp = on ? __builtin_ctzll(m2) : 0;
                m2 &= m2 - 1;
                int pt = __builtin_amdgcn_readlane(px[0], tp);
                vm[u] = on && pt >= 0 ? 1u : 0u;
                if (!onepix) {
#pragma unroll
                  for (int f = 1; f < 4; ++f) {
                    const int pf = __builtin_amdgcn_readlane(px[f], tp);
                    if (on && pf >= 0) vm[u] |= 1u << f;
                    pt = myfrag == f ? pf : pt;
                  }
                }
                va[u] = on && pt >= 0 ? sgl[(int64_t)pt * g.n] : 0;
                vb[u] = on ? swl[tp * g.c] : 0;
              }
#pragma unroll
              for (int u = 0; u < U; ++u) {
                rsum += va[u];
#pragma unroll
                for (int f = 0; f < 4; ++f)
                  if (f == 0 || !onepix) {
                    csum[f] += (vm[u] >> f) & 1u ? vb[u] : 0;
                    cnt[f] += (vm[u] >> f) & 1u;
                  }
              }
            }
          }
          __builtin_amdgcn_s_waitcnt(0x3F70);  // the sums' loads are done: the loop counts its own
          for (int s = 0; s < stepsu; s += 2) {
            bload(q1.bo, bb1);
            mma(a0, bb0, q0.vm);
            next(q0);
            aload(q0, a0);
            bload(q0.bo, bb0);
            if (s + 1 < stepsu) mma(a1, bb1, q1.vm);
            next(q1);
            aload(q1, a1);
          }
        } else {
        // ---- K loop: lane group lg of step s takes list position 4 s + lg
        const int Q = nv * nch, steps = (Q + 3) / 4;
        const float inv = 1.0f / (float)nch;
        const uint32_t c16 = (uint32_t)c0 / 16;
        // this lane's 16 bytes of the four fragments' rows at its list position,
        // and the position's panel offset.  Positions past the end meet a zero
        // chunk of the panel; a fragment without the tap reads zeros.
        auto gload = [&](int s, v4i (&a)[4], int& boff) __attribute__((always_inline)) {
          const int q = 4 * s + lg;
          const bool in = q < Q;
          // q / nch: the quotient is below 64 and (q + 1/2) / nch at least 1 / (2 nch) off an integer
          const int vt = in ? (int)(((float)q + 0.5f) * inv) : 0;
          const uint32_t ch = in ? (uint32_t)(q - vt * nch) : 0u;
          boff = in ? 16 * (sw.k.tap[vt] * nch + (int)ch) : zchunk;
          uint32_t off[4];
          if (onepix) {
            const uint32_t at = sw.k.off[vt].x + c16 + ch;
#pragma unroll
            for (int f = 0; f < 4; ++f) off[f] = at + arow[f];
          } else {
            const int4 e = sw.k.pix[vt];
            const uint4 o = sw.k.off[vt];
            off[0] = e.x >= 0 ? o.x + c16 + ch + arow[0] : t.zoff;
            off[1] = e.y >= 0 ? o.y + c16 + ch + arow[1] : t.zoff;
            off[2] = e.z >= 0 ? o.z + c16 + ch + arow[2] : t.zoff;
            off[3] = e.w >= 0 ? o.w + c16 + ch + arow[3] : t.zoff;
          }
#pragma unroll
          for (int f = 0; f < 4; ++f) a[f] = *reinterpret_cast<const v4i*>(q2 + 16 * (uint64_t)off[f]);
        };
        auto compute = [&](const v4i (&a)[4], int boff) __attribute__((always_inline)) {
          v4i b[4];
#pragma unroll
          for (int j = 0; j < 4; ++j) b[j] = *reinterpret_cast<const v4i*>(panel + (16 * j + lc) * t.pitch + boff);
#pragma unroll
          for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int i = 0; i < 4; ++i) acc[i][j] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a[i], b[j], acc[i][j], 0, 0, 0);
        };
          v4i a0[4], a1[4];
          int o0, o1;
          if (nv == 0) continue;
          gload(0, a0, o0);
          gload(1, a1, o1);
        // ---- zero-point sums over the taps, four taps' loads in flight
        if (c0 == 0) {
          for (int v0 = 0; v0 < nv; v0 += 4) {
            int a[4], b[4];
            int4 e[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
              const int v = min(v0 + u, nv - 1);
              e[u] = sw.k.pix[v];
              const int pm = onepix ? e[u].x : (myfrag == 0 ? e[u].x : (myfrag == 1 ? e[u].y : (myfrag == 2 ? e[u].z : e[u].w)));
              const bool ok = myrow && pm >= 0 && v0 + u < nv;
              a[u] = ok ? sg[(int64_t)pm * g.n + myslot] : 0;
              b[u] = swq[(int64_t)(t0 + sw.k.tap[v]) * g.c + colc];
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
              rsum += a[u];
              if (v0 + u < nv) {
                csum[0] += e[u].x >= 0 ? b[u] : 0;
                cnt[0] += e[u].x >= 0;
                if (!onepix) {
                  csum[1] += e[u].y >= 0 ? b[u] : 0;
                  csum[2] += e[u].z >= 0 ? b[u] : 0;
                  csum[3] += e[u].w >= 0 ? b[u] : 0;
                  cnt[1] += e[u].y >= 0;
                  cnt[2] += e[u].z >= 0;
                  cnt[3] += e[u].w >= 0;
                }
              }
            }
          }
        }
          for (int s = 0; s < steps; s += 2) {
            compute(a0, o0);
            gload(s + 2, a0, o0);
            if (s + 1 < steps) compute(a1, o1);
            gload(s + 3, a1, o1);
          }
        }
        __builtin_amdgcn_wave_barrier();
      }

    __builtin_amdgcn_sched_barrier(0);
    // ---- epilogue: accumulator (i, j)[r] of lane l holds unit row 16 i +
    // 4 (l / 16) + r, column 4 (l % 16) + j.  With a = the integer product,
    // T = dW a + rterm + hz colterm is the row's dequantized code times the
    // weights (hz = half + c_g in a multi-row group, else z + half / s over s),
    // and the output dq T of an affine row, or dq (T - alpha tau) (first row:
    // + tau) of a group row, tau = (alpha S - T_0) / (1 - alpha): both are
    // fma(e1, group term, fma(e2, column term, fma(dq dW, a, dq rterm))).
    double dq = 0.0, hz = 0.0, rterm = 0.0;
    int kind = 0, orow = -1;
    if (myrow) {
      kind = (EPI == EPI_BHQ) ? bhq_slot_kind(p.L, myslot) : (EPI == EPI_BHQT ? (p.slot[myslot].size > 1) : 0);
      rterm = zW * (double)rsum;
      dq = 1.0 / (double)row_s;
      hz = kind != 0 ? (double)p.halfA + (double)row_z : (double)row_z + (double)p.halfA * dq;
      orow = row_n * hw + mypix;
    }
    const bool inverse = EPI == EPI_BHQ && KE > 1;
    if (EPI == EPI_BHQT && kind != 0) {
      // rows of the general plan's multi-row groups: T itself, into tbuf
      sw.e.ab[lane] = make_double2(dW, rterm);
      sw.e.e1[lane] = 0.0;
      sw.e.e2[lane] = hz;
      orow = -2;
    } else {
      sw.e.ab[lane] = make_double2(dq * dW, dq * rterm);
      sw.e.e1[lane] = inverse && kind != 0 ? dq : 0.0;
      sw.e.e2[lane] = inverse && kind != 0 ? 0.0 : hz;
    }
    sw.e.orow[lane] = orow;
#pragma unroll
    for (int f = 0; f < 4; ++f)
      if (f == 0 || !onepix) sw.e.col[f][lane] = csum[f];
    __builtin_amdgcn_wave_barrier();
    // sum of rterm over the group's rows (the lanes of an aligned run of KE)
    double rgrp = kind != 0 ? rterm : 0.0;
    if constexpr (inverse) {
#pragma unroll
      for (int h = 1; h < KE; h <<= 1) rgrp += __shfl_xor(rgrp, h);
    }
    const uint64_t multi = __ballot(kind != 0);
    const int col = n0 + 4 * lc;
    const bool vec = col + 3 < g.c && (p.ldo & 3) == 0 && ((uintptr_t)p.out & 15) == 0;
    // column terms of a fragment's pixel, and (at the first fragment of a
    // group) the group terms
    double ct[4];
    constexpr int NGF = KE == 2 ? 2 : 1;  // groups per fragment and lane
    double gp[4][NGF], tu[4][NGF];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      __builtin_amdgcn_sched_barrier(0);  // one fragment's row data in registers at a time
      if (i == 0 || !onepix) {
        const int f = i;
        const double kz = (double)cnt[f] * ((double)g.o * zW);
#pragma unroll
        for (int j = 0; j < 4; ++j) ct[j] = dW * (double)sw.e.col[f][4 * lc + j] + kz;
      }
      if constexpr (inverse) {
        constexpr int FR = KE >= 16 ? KE / 16 : 1;  // fragments per group
        if (i % FR == 0) {
#pragma unroll
          for (int q = 0; q < NGF; ++q) {
            // first row of this lane's group, and whether the group has several rows
            const int g0 = KE >= 16 ? 16 * i : (KE == 8 ? 16 * i + 8 * (lane >> 5) : 16 * i + 4 * lg + 2 * q);
            const int gk = __shfl(kind, g0);
            const double ghz = __shfl(hz, g0), grt = __shfl(rterm, g0), grs = __shfl(rgrp, g0);
            const double m = gk == 1 ? (double)p.L.k : (double)p.L.part;
            const double alpha = gk == 2 ? p.L.inv_sk_p : p.L.inv_sk_k;
            const double rom = 1.0 / (1.0 - alpha);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
              double S = 0.0;
              int a0;
              if constexpr (KE >= 4) {
#pragma unroll
                for (int ii = i; ii < i + FR; ++ii)
#pragma unroll
                  for (int r = 0; r < 4; ++r) {
                    const bool in = (multi >> (16 * ii + 4 * lg + r)) & 1ull;
                    S += in ? (double)acc[ii][j][r] : 0.0;
                  }
                if constexpr (KE >= 8) S += __shfl_xor(S, 16);
                if constexpr (KE >= 16) S += __shfl_xor(S, 32);
                a0 = acc[i][j][0];
                if constexpr (KE == 8) a0 = __shfl(a0, lane & 47);
                if constexpr (KE >= 16) a0 = __shfl(a0, lc);
              } else {
                S = (double)acc[i][j][2 * q] + (double)acc[i][j][2 * q + 1];
                a0 = acc[i][j][2 * q];
              }
              const double hc = ghz * ct[j];
              const double sum = fma(dW, S, fma(m, hc, grs));
              const double T0 = fma(dW, (double)a0, grt + hc);
              const double tau = gk != 0 ? (alpha * sum - T0) * rom : 0.0;
              gp[j][q] = gk != 0 ? fma(-alpha, tau, hc) : 0.0;
              tu[j][q] = tau;
            }
          }
        }
      }
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int row = 16 * i + 4 * lg + r;
        const int orw = sw.e.orow[row];
        if (orw == -1) continue;
        const double2 ab = sw.e.ab[row];
        const double e2 = sw.e.e2[row];
        const double e1 = inverse ? sw.e.e1[row] : 0.0;
        if (EPI == EPI_BHQT && orw == -2) {
          double* dst = p.tbuf + (int64_t)(row0 + row) * p.ldt + col;
#pragma unroll
          for (int j = 0; j < 4; ++j)
            if (col + j < g.c) dst[j] = fma(ab.x, (double)acc[i][j][r], fma(e2, ct[j], ab.y));
          continue;
        }
        float* dst = p.out + (int64_t)orw * p.ldo + col;
        float o[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          int a = acc[i][j][r];
          asm volatile("" : "+v"(a));  // convert here: 64 float64 copies kept from the group sums would not fit
          double v = fma(ab.x, (double)a, ab.y);
          v = fma(e2, ct[j], v);
          if constexpr (inverse) {
            const int q = KE == 2 ? r >> 1 : 0;
            // slot of the row in its group: KE rows aligned
            const bool first = KE == 2 ? (r & 1) == 0 : (KE == 4 ? r == 0 : ((row & (KE - 1)) == 0));
            v = fma(e1, first ? gp[j][q] + tu[j][q] : gp[j][q], v);
          }
          o[j] = (float)v;
        }
        if (vec) {
          out_store4<NT>(dst, make_float4(o[0], o[1], o[2], o[3]));
        } else {
#pragma unroll
          for (int j = 0; j < 4; ++j)
            if (col + j < g.c) out_store<NT>(dst + j, o[j]);
        }
      }
    }
    __builtin_amdgcn_wave_barrier();
  }
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
constexpr int CX_LDS = 160 * 1024;  // LDS of a CU
constexpr int CX_CUS = 256;

template <int EPI, int KE, bool NT>
static hipError_t launch_conv_gradx_nt(const GemmParams& p, const ConvGeom& g, const int8_t* q2, const int8_t* zero16,
                                       const int32_t* sg, const int32_t* swq, hipStream_t s) {
  const int taps = g.kh * g.kw;
  const int64_t M = (int64_t)g.h * g.w * g.npad;
  if (M > 0x7FFFFFFF - 64 || p.M != M || (g.npad != 16 && g.npad != 32 && g.npad % 64 != 0) || g.npad < g.n ||
      (g.o & 15) != 0)
    return hipErrorInvalidValue;
  // The panel.  Up to 68 KB it is kept whole by two blocks of 4 waves per CU, up
  // to 137 KB by one block of 8 waves, since reloading it costs a block-wide
  // barrier per chunk; larger ones go chunk by chunk, two blocks of 4 waves per
  // CU so that one computes while the other loads.
  const int64_t zb = zero16 - q2;
  if (zb < 0 || (zb & 15) != 0 || zb / 16 > 0xFFFFFFFFll || ((uintptr_t)q2 & 15) != 0) return hipErrorInvalidValue;
  ConvXTile t{};
  t.zoff = (uint32_t)(zb / 16);
  int waves;
  const int wl = (int)sizeof(ConvXWave);
  // whole 16-byte chunks and one of zeros, an odd number
  auto pitch_of = [](int64_t k) { return (int)(((k / 16 + 1) | 1) * 16); };
  const int64_t K = (int64_t)taps * g.o;
  const int64_t whole = (int64_t)CX_BN * (((K / 16 + 1) | 1) * 16);
  const int64_t tiles_n = (g.c + CX_BN - 1) / CX_BN, units = (M + 63) / 64;
  const bool small = units * tiles_n <= 4 * CX_CUS;
  t.tpc = taps;
  t.cpc = g.o;
  t.per_wave = 1;
  if (taps <= 64 && whole + 4 * wl <= CX_LDS / 2) {
    waves = 4;
  } else if (taps <= 64 && whole + 8 * wl <= CX_LDS) {
    waves = 8;
  } else if (taps <= 64 && whole + 4 * wl <= CX_LDS && small) {
    waves = 4;  // too few units to fill two blocks per CU anyway
  } else {
    waves = 4;
    const int64_t kmax = ((CX_LDS / 2 - 4 * wl) / CX_BN / 16 - 2) * 16;  // bytes per panel row
    t.cpc = (int)(g.o < kmax ? g.o : kmax / 64 * 64);
    t.tpc = (int)(kmax / t.cpc);
    if (t.tpc > 64) t.tpc = 64;
    if (t.tpc > taps) t.tpc = taps;
    t.tpc = (taps + (taps + t.tpc - 1) / t.tpc - 1) / ((taps + t.tpc - 1) / t.tpc);  // even chunks
  }
  t.pitch = pitch_of((int64_t)t.tpc * t.cpc);
  const int lds = CX_BN * t.pitch + waves * wl;
  if (t.tpc == taps && t.cpc == g.o) {
    // as many waves as the GPU holds at once (8 per CU), each taking several
    // units, so that the panel is loaded once per wave (3x3 64ch 56x56 b128:
    // 70 us with four rounds of blocks, 58 us)
    const int64_t slots = (int64_t)CX_CUS * 8;
    t.per_wave = (int)((units * tiles_n + slots - 1) / slots);
  }
  const int64_t blocks = (units + (int64_t)waves * t.per_wave - 1) / ((int64_t)waves * t.per_wave) * tiles_n;
  if (blocks > 0x7FFFFFFF || lds > CX_LDS) return hipErrorInvalidValue;
  const bool uni = g.o % 64 == 0 && t.cpc % 64 == 0 && (int64_t)g.n * g.o < ((int64_t)1 << 32);
  const bool one = g.npad >= 64;
#define FQT_GRADX(UNI, ONE)                                                                                            \
  hipLaunchKernelGGL((conv_gradx_kernel<EPI, KE, UNI, ONE, NT>), dim3((unsigned)blocks), dim3((unsigned)(64 * waves)),     \
                     (size_t)lds, s, p, g, t, q2, sg, swq)
  if constexpr (KE < 64) {
    if (uni && one)
      FQT_GRADX(true, true);
    else if (uni)
      FQT_GRADX(true, false);
    else if (one)
      FQT_GRADX(false, true);
    else
      FQT_GRADX(false, false);
  } else if (uni) {  // groups of 64 rows have one pixel
    FQT_GRADX(true, true);
  } else {
    FQT_GRADX(false, true);
  }
#undef FQT_GRADX
  return hipGetLastError();
}

template <int EPI, int KE>
static hipError_t launch_conv_gradx_t(const GemmParams& p, const ConvGeom& g, const int8_t* q2, const int8_t* zero16,
                                      const int32_t* sg, const int32_t* swq, hipStream_t s) {
  return stream_rows(p.out, p.M, p.ldo, STREAM_CONV) ? launch_conv_gradx_nt<EPI, KE, true>(p, g, q2, zero16, sg, swq, s)
                                      : launch_conv_gradx_nt<EPI, KE, false>(p, g, q2, zero16, sg, swq, s);
}

hipError_t launch_conv_gradx(const GemmParams& p, int epi, const ConvGeom& g, const int8_t* q2, const int8_t* zero16,
                             const int32_t* sg, const int32_t* swq, hipStream_t s) {
  if (epi == EPI_ROW) return launch_conv_gradx_t<EPI_ROW, 1>(p, g, q2, zero16, sg, swq, s);
  if (epi == EPI_BHQT)
    return p.slot && p.tbuf ? launch_conv_gradx_t<EPI_BHQT, 1>(p, g, q2, zero16, sg, swq, s) : hipErrorInvalidValue;
  // groups of L.k aligned slots; with fewer slots per pixel than L.k the one
  // group spans them all
  const int64_t ke = p.L.k < g.npad ? p.L.k : g.npad;
  switch (ke) {
    case 1: return launch_conv_gradx_t<EPI_ROW, 1>(p, g, q2, zero16, sg, swq, s);  // every group has one row
    case 2: return launch_conv_gradx_t<EPI_BHQ, 2>(p, g, q2, zero16, sg, swq, s);
    case 4: return launch_conv_gradx_t<EPI_BHQ, 4>(p, g, q2, zero16, sg, swq, s);
    case 8: return launch_conv_gradx_t<EPI_BHQ, 8>(p, g, q2, zero16, sg, swq, s);
    case 16: return launch_conv_gradx_t<EPI_BHQ, 16>(p, g, q2, zero16, sg, swq, s);
    case 32: return launch_conv_gradx_t<EPI_BHQ, 32>(p, g, q2, zero16, sg, swq, s);
    case 64: return launch_conv_gradx_t<EPI_BHQ, 64>(p, g, q2, zero16, sg, swq, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace fqt
