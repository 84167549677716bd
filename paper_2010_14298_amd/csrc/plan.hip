// General block Householder plans on gfx950: groups of any size in slot
// order (App. D's adaptive grouping, and fixed block sizes that are not a
// power of two up to 64), the forward transform's per-group column term, and
// the inverse transform of the input gradient.
//
//   sort        rows by infinity norm (launch_bhq_sort, quant.hip)
//   prep        per sorted position: M, R, their cube roots; prefix sums of M
//   objective   App. D, step 2: for every number of groups G the groups take
//               the G largest rows and small-row shares proportional to M_i
//               (cumulative rounding); scored by the exact |S^-1|_F^2
//   argmin      least objective, ties to fewer groups
//   build       perm, per-slot scale / zero, group offsets, slot records
//   tau         per multi-row group and column: the rank-1 term of the
//               reflection, from the column sum in slot order
//   inverse     diag(d)^-1 H of each multi-row group on the input gradient
#include <math.h>

#include "fqt_device.h"
#include "fqt_kernels.h"

namespace fqt {

// ---------------------------------------------------------------------------
// workspace
// ---------------------------------------------------------------------------
static size_t up256(size_t b) { return (b + 255) / 256 * 256; }

size_t appd_workspace(int64_t rows) {
  const size_t n = (size_t)rows;
  return up256(n * 4) + 4 * up256(n * 4) + up256((n + 1) * 8) + up256(n * 8) + 256;
}

AppdWs appd_carve(void* ws, int64_t rows) {
  const size_t n = (size_t)rows;
  char* p = static_cast<char*>(ws);
  AppdWs w{};
  w.sigma = reinterpret_cast<int32_t*>(p);
  p += up256(n * 4);
  w.Ms = reinterpret_cast<float*>(p);
  p += up256(n * 4);
  w.Rs = reinterpret_cast<float*>(p);
  p += up256(n * 4);
  w.ca = reinterpret_cast<float*>(p);
  p += up256(n * 4);
  w.cc = reinterpret_cast<float*>(p);
  p += up256(n * 4);
  w.P = reinterpret_cast<double*>(p);
  p += up256((n + 1) * 8);
  w.obj = reinterpret_cast<double*>(p);
  p += up256(n * 8);
  w.G = reinterpret_cast<int32_t*>(p);
  return w;
}

// ---------------------------------------------------------------------------
// prep: sorted-position scalars (one thread per position); the block after
// them (App. D only) forms the prefix sums of M at the same time.
// ---------------------------------------------------------------------------
__device__ __forceinline__ void appd_norms(const float* rmin, const float* rmax, int32_t row, float& M, float& R) {
  const float lo = rmin[row], hi = rmax[row];
  M = fmaxf(fabsf(lo), fabsf(hi));
  R = hi - lo;
  if (!isfinite(M)) M = 0.0f;
  if (!isfinite(R)) R = 0.0f;
}

// P[i] = P[i - 1] + M_(i), one addition at a time in sorted order: a serial
// chain of rows float64 additions.  The block stages a chunk of M in LDS (all
// loads in flight), one thread runs the chain on 16 values at a time from and
// to LDS, and the block stores the chunk's sums.  With the chain's loads and
// stores in global memory 2048 rows took 52.9 us.
constexpr int APPD_CH = 2048;
__device__ void appd_prefix(const float* rmin, const float* rmax, int64_t rows, const AppdWs& w) {
  __shared__ __attribute__((aligned(16))) float sm[APPD_CH];
  __shared__ __attribute__((aligned(16))) double sp[APPD_CH];
  const int t = threadIdx.x;
  double P = 0.0;
  if (t == 0) w.P[0] = 0.0;
  for (int64_t c0 = 0; c0 < rows; c0 += APPD_CH) {
    const int n = (int)(rows - c0 < APPD_CH ? rows - c0 : APPD_CH);
#pragma unroll
    for (int u = 0; u < APPD_CH / 256; ++u) {
      const int i = t + 256 * u;
      float M, R;
      appd_norms(rmin, rmax, w.sigma[c0 + (i < n ? i : n - 1)], M, R);
      sm[i] = i < n ? M : 0.0f;
    }
    __syncthreads();
    if (t == 0) {
      // positions past n add zero, and are not stored
      // (the next 16 are read before the chain waits for its own)
      float m[16];
#pragma unroll
      for (int u = 0; u < 16; ++u) m[u] = sm[u];
      for (int i = 0; i < n; i += 16) {
        double d[16], q[16];
#pragma unroll
        for (int u = 0; u < 16; ++u) d[u] = (double)m[u];
        const int nx = i + 16 < APPD_CH ? i + 16 : i;
#pragma unroll
        for (int u = 0; u < 16; ++u) m[u] = sm[nx + u];
#pragma unroll
        for (int u = 0; u < 16; ++u) {
          P = P + d[u];
          q[u] = P;
        }
#pragma unroll
        for (int u = 0; u < 16; ++u) sp[i + u] = q[u];
      }
    }
    __syncthreads();
    for (int i = t; i < n; i += 256) w.P[c0 + i + 1] = sp[i];
    __syncthreads();
  }
}

__global__ __launch_bounds__(256) void appd_prep_kernel(const float* rmin, const float* rmax, int64_t rows, AppdWs w,
                                                        int64_t nprep) {
  if ((int64_t)blockIdx.x >= nprep) {
    appd_prefix(rmin, rmax, rows, w);
    return;
  }
  const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= rows) return;
  float M, R;
  appd_norms(rmin, rmax, w.sigma[r], M, R);
  w.Ms[r] = M;
  w.Rs[r] = R;
  w.ca[r] = cbrt_rn(R);
  w.cc[r] = cbrt_rn(2.0f * M);
}

// First j groups' share of the small rows for G groups (App. D, step 2):
// floor((N - G) P_j / P_G + 1/2) in float64 (product, quotient, sum), with
// c_0 = 0 and c_G = N - G; P_j replaced by j when P_G = 0.
__device__ __forceinline__ int64_t appd_cum(const double* P, int64_t N, int64_t G, int64_t j) {
  const int64_t small = N - G;
  if (j <= 0) return 0;
  if (j >= G) return small;
  const double S = P[G];
  const double q = S > 0.0 ? ((double)small * P[j]) / S : (double)(small * j) / (double)G;
  const int64_t c = (int32_t)floor(q + 0.5);  // at most N - G < 2^31
  return c < small ? c : small;
}

// The term of group i (0-based) of the G-group plan: a one-row group's PSQ
// scale, or the Householder pair of App. C.4.
__device__ __forceinline__ double appd_term(const AppdWs& w, int64_t G, int64_t i, int64_t c0, int64_t c1, int B) {
  const int64_t n = c1 - c0;
  if (n == 0) {
    const float s = scale_from_range(w.Rs[i], B);
    return group_term(s, s, 1);
  }
  const int64_t f = G + c0;  // sorted position of the group's first small row
  float s1, s2;
  group_scales(w.Rs[i], 2.0f * w.Ms[f], w.ca[i], w.cc[f], n + 1, sqrt((double)(n + 1)), B, s1, s2);
  return group_term(s1, s2, n + 1);
}

// One block per G (the largest first): four waves compute a round of terms, 63
// each (lane l holds c_i of group i and takes c_(i+1) from lane l + 1; the last
// lane's group is the next wave's first), into one of two LDS buffers, while the
// fifth adds the previous round's to the total one at a time in group order
// (float64; every lane reads them as broadcasts and runs the same chain).  The
// latency of the largest G's terms and chain bounds the kernel: with one wave
// per G, terms and chain by turns, 2048 rows took 54 us (2048 x 1024 -> 1024
// layer with adaptive groups: 183.6 -> 158.0 us, with the prefix sums' reads
// ahead of the chain).  Terms past G are zero, and adding +0 to a total that is
// never -0 changes nothing.
constexpr int OBJ_WAVES = 4, OBJ_TERMS = 63 * OBJ_WAVES;
__global__ __launch_bounds__(64 * (OBJ_WAVES + 1)) void appd_objective_kernel(int64_t rows, int B, AppdWs w,
                                                                              double* obj) {
  __shared__ __attribute__((aligned(16))) double sterm[2][OBJ_TERMS];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  for (int64_t id = blockIdx.x; id < rows; id += gridDim.x) {
    const int64_t G = rows - id;
    const int64_t rounds = (G + OBJ_TERMS - 1) / OBJ_TERMS;
    double total = 0.0;
    for (int64_t k = 0; k <= rounds; ++k) {
      if (wave < OBJ_WAVES) {
        const int64_t i = k * OBJ_TERMS + 63 * wave + lane;
        if (k < rounds && i - lane < G) {
          const int c0 = (int)appd_cum(w.P, rows, G, i < G ? i : G);
          const int c1 = __shfl_down(c0, 1);
          if (lane < 63) sterm[k & 1][63 * wave + lane] = i < G ? appd_term(w, G, i, c0, c1, B) : 0.0;
        } else if (lane < 63) {
          sterm[k & 1][63 * wave + lane] = 0.0;
        }
      } else if (k > 0) {
        const double* q = sterm[(k - 1) & 1];
        for (int l0 = 0; l0 < OBJ_TERMS; l0 += 84) {
#pragma unroll
          for (int l = 0; l < 84; ++l) total = total + q[l0 + l];
        }
      }
      __syncthreads();
    }
    if (wave == OBJ_WAVES && lane == 0) obj[G - 1] = total;
  }
}
static_assert(OBJ_TERMS % 84 == 0, "whole runs of the chain");

// Least objective over G = 1..rows, ties to the smaller G (one block).
__global__ __launch_bounds__(1024) void appd_argmin_kernel(int64_t rows, const double* obj, int32_t* G_out) {
  __shared__ double sv[1024];
  __shared__ int64_t sg[1024];
  const int t = threadIdx.x;
  double best = 0.0;
  int64_t bg = -1;
  for (int64_t g = t; g < rows; g += 1024) {
    const double v = obj[g];
    if (bg < 0 || v < best) {
      best = v;
      bg = g;
    }
  }
  sv[t] = best;
  sg[t] = bg;
  __syncthreads();
  for (int h = 512; h > 0; h >>= 1) {
    if (t < h) {
      const double v = sv[t + h];
      const int64_t g = sg[t + h];
      if (g >= 0 && (sg[t] < 0 || v < sv[t] || (v == sv[t] && g < sg[t]))) {
        sv[t] = v;
        sg[t] = g;
      }
    }
    __syncthreads();
  }
  if (t == 0) *G_out = (int32_t)(sg[0] + 1);
}

// One wave per group g of the chosen plan (App. D: G from the device; fixed
// block size k: G = ceil(rows / k) and c_g = min(N - G, g (k - 1))).
__global__ __launch_bounds__(256) void plan_build_kernel(const float* rmin, int64_t rows, int B, int k, AppdWs w,
                                                         const int32_t* Gdev, int32_t* perm, float* scale,
                                                         float* zero, int32_t* group_off, SlotInfo* slot,
                                                         int32_t* num_groups) {
  const int lane = threadIdx.x & 63;
  const int64_t g = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  int64_t G = k > 0 ? (rows + k - 1) / k : (int64_t)*Gdev;
  G = G < 1 ? 1 : (G > rows ? rows : G);  // the search writes 1..rows; kept in range regardless
  if (g >= G) return;
  const int64_t small = rows - G;
  int64_t c0, c1;
  if (k > 0) {
    c0 = min(small, g * (int64_t)(k - 1));
    c1 = min(small, (g + 1) * (int64_t)(k - 1));
  } else {
    c0 = appd_cum(w.P, rows, G, g);
    c1 = appd_cum(w.P, rows, G, g + 1);
  }
  const int64_t n = c1 - c0, base = g + c0, size = n + 1;
  if (lane == 0) {
    group_off[g] = (int32_t)base;
    if (g == G - 1) {
      group_off[G] = (int32_t)rows;
      if (num_groups) *num_groups = (int32_t)G;
    }
  }
  const int32_t big = w.sigma[g];
  const float mn0 = rmin[big];
  if (n == 0) {
    if (lane == 0) {
      perm[base] = big;
      scale[base] = scale_from_range(w.Rs[g], B);
      zero[base] = mn0;
      slot[base] = SlotInfo{(int32_t)base, 1, 0.0f, 0.0f};
    }
    return;
  }
  const int64_t f = G + c0;
  const float lam2 = 2.0f * w.Ms[f];
  const double sk = sqrt((double)size);
  float s1, s2;
  group_scales(w.Rs[g], lam2, w.ca[g], w.cc[f], size, sk, B, s1, s2);
  const float alpha = (float)(1.0 / sk);
  const float oma = 1.0f - alpha;
  const double t1 = ((double)alpha * (double)s1) * (double)mn0;
  const double t2 = ((0.5 * (double)lam2) * (double)s2) * sk;
  const float cg = (float)(t1 - t2);
  const SlotInfo si{(int32_t)base, (int32_t)size, alpha, oma};
  for (int64_t j = lane; j < size; j += 64) {
    perm[base + j] = j == 0 ? big : w.sigma[f + j - 1];
    scale[base + j] = j == 0 ? s1 : s2;
    zero[base + j] = cg;
    slot[base + j] = si;
  }
}

static hipError_t launch_prep(const float* rmin, const float* rmax, int64_t rows, const AppdWs& w, bool prefix,
                              hipStream_t s) {
  const int64_t nprep = (rows + 255) / 256;
  hipLaunchKernelGGL(appd_prep_kernel, dim3((unsigned)(nprep + (prefix ? 1 : 0))), dim3(256), 0, s, rmin, rmax, rows, w,
                     nprep);
  return hipGetLastError();
}

hipError_t launch_appd_search(const float* rmin, const float* rmax, int64_t rows, int bits, const AppdWs& w,
                              double* obj_out, int32_t* num_groups, hipStream_t s) {
  if (rows < 1 || rows > 0x7FFFFFFF) return hipErrorInvalidValue;
  hipError_t e = launch_prep(rmin, rmax, rows, w, true, s);
  if (e != hipSuccess) return e;
  const int B = (1 << bits) - 1;
  double* obj = obj_out ? obj_out : w.obj;
  hipLaunchKernelGGL(appd_objective_kernel, dim3((unsigned)(rows < (1 << 20) ? rows : 1 << 20)), dim3(64 * (OBJ_WAVES + 1)), 0, s, rows, B, w, obj);
  hipLaunchKernelGGL(appd_argmin_kernel, dim3(1), dim3(1024), 0, s, rows, obj, num_groups ? num_groups : w.G);
  return hipGetLastError();
}

hipError_t launch_general_plan(const float* rmin, const float* rmax, int64_t rows, int bits, int block_size,
                               const AppdWs& w, double* obj_out, int32_t* perm, float* scale, float* zero,
                               int32_t* group_off, SlotInfo* slot, int32_t* num_groups, hipStream_t s) {
  if (rows < 1 || rows > 0x7FFFFFFF || block_size < 0) return hipErrorInvalidValue;
  hipError_t e;
  if (block_size == 0) {
    e = launch_appd_search(rmin, rmax, rows, bits, w, obj_out, w.G, s);
  } else {
    e = launch_prep(rmin, rmax, rows, w, false, s);
  }
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(plan_build_kernel, dim3((unsigned)((rows + 3) / 4)), dim3(256), 0, s, rmin, rows,
                     (1 << bits) - 1, block_size, w, w.G, perm, scale, zero, group_off, slot, num_groups);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// tau and inverse share their split: a block takes 64 columns (one per lane)
// and the multi-row groups whose first slot lies in its chunk of 64 slots.
// Groups of at most GW_ROWS rows go to one wave each; the rows of a larger
// group are spread over the block's waves.  With one thread per column
// walking every row of its chunk's groups, an adaptive plan of 2048 x 1024
// (128 blocks, groups of hundreds of rows) took 33 us (tau) and 76 us
// (inverse).
// ---------------------------------------------------------------------------
constexpr int GW_WAVES = 8;
constexpr int GW_ROWS = 64;

// Bit b: a group of at least two rows starts at slot s0 + b of the chunk;
// size: the lane's slot record (lane b holds slot s0 + b).
__device__ __forceinline__ uint64_t chunk_groups(const SlotInfo* slot, int64_t s0, int64_t rows, SlotInfo& si) {
  const int lane = threadIdx.x & 63;
  const int64_t sb = s0 + lane;
  si = slot[sb < rows ? sb : rows - 1];
  return __ballot(sb < rows && si.base == sb && si.size >= 2);
}

// A group's column sum S of v_p = d_p x[perm[p]] adds its rows one at a time
// in slot order (float32); in a large group the waves load and scale 64 rows
// at a time into LDS, from where the first wave adds them in order.
__global__ __launch_bounds__(64 * GW_WAVES) void bhq_tau_kernel(const float* x, int64_t rows, int64_t cols,
                                                                const int32_t* perm, const float* scale,
                                                                const SlotInfo* slot, float* tau) {
  __shared__ float sv[2][64][64];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t col = (int64_t)blockIdx.x * 64 + lane;
  const int64_t cc = col < cols ? col : cols - 1;  // clamped: loads stay inside x, the store is skipped
  const int64_t s0 = (int64_t)blockIdx.y * 64;
  SlotInfo lsi;
  const uint64_t groups = chunk_groups(slot, s0, rows, lsi);
  int k = 0;
  for (uint64_t m = groups; m; m &= m - 1) {
    const int b = __ffsll((unsigned long long)m) - 1;
    const int size = __builtin_amdgcn_readlane(lsi.size, b);
    const float alpha = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, lsi.alpha), b));
    const float oma = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, lsi.oma), b));
    const int64_t sb = s0 + b;
    float S = 0.0f, v0 = 0.0f;
    if (size <= GW_ROWS) {
      if (k++ % GW_WAVES != wave) continue;
      // the group's rows and scales, lane p holding slot p; eight loads in flight
      const int64_t sp = sb + (lane < size ? lane : 0);
      const int32_t lrow = perm[sp];
      const float ld = scale[sp];
      constexpr int U = 8;
      for (int p = 0; p < size; p += U) {
        float v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const int q = p + u < size ? p + u : size - 1;
          const float d = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, ld), q));
          v[u] = d * x[(int64_t)__builtin_amdgcn_readlane(lrow, q) * cols + cc];
        }
        if (p == 0) v0 = v[0];
#pragma unroll
        for (int u = 0; u < U; ++u)
          if (p + u < size) S = S + v[u];
      }
    } else {
      const int nch = (size + 63) / 64;
      auto fill = [&](int c) {
        constexpr int RW = 64 / GW_WAVES;  // rows per wave
        const int64_t base = sb + 64 * (int64_t)c + wave * RW;
        const int left = size - 64 * c - wave * RW;  // rows of this wave in the chunk (may be <= 0)
        const int64_t sp = base + ((lane & (RW - 1)) < left ? (lane & (RW - 1)) : 0);
        const int64_t sq = sp < sb + size ? sp : sb;
        const int32_t lrow = perm[sq];
        const float ld = scale[sq];
#pragma unroll
        for (int r = 0; r < RW; ++r) {
          const float d = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, ld), r));
          sv[c & 1][wave * RW + r][lane] = d * x[(int64_t)__builtin_amdgcn_readlane(lrow, r) * cols + cc];
        }
      };
      fill(0);
      for (int c = 0; c < nch; ++c) {
        __syncthreads();  // chunk c is in LDS, and chunk c - 1 has been added
        if (c + 1 < nch) fill(c + 1);
        if (wave == 0) {
          const int n = size - 64 * c < 64 ? size - 64 * c : 64;
          if (c == 0) v0 = sv[0][0][lane];
          if (n == 64) {
#pragma unroll
            for (int r = 0; r < 64; ++r) S = S + sv[c & 1][r][lane];
          } else {
            for (int r = 0; r < n; ++r) S = S + sv[c & 1][r][lane];
          }
        }
      }
      __syncthreads();  // the next group's first fill reuses the buffers
      if (wave != 0) continue;
    }
    const float mm = alpha * S - v0;
    if (col < cols) tau[(sb >> 1) * cols + col] = __fdiv_rn(mm, oma);
  }
}

hipError_t launch_bhq_tau(const float* x, int64_t rows, int64_t cols, const int32_t* perm, const float* scale,
                          const SlotInfo* slot, float* tau, hipStream_t s) {
  const int64_t cb = (cols + 63) / 64, rb = (rows + 63) / 64;
  if (cb > 0x7FFFFFFF || rb > 65535) return hipErrorInvalidValue;
  hipLaunchKernelGGL(bhq_tau_kernel, dim3((unsigned)cb, (unsigned)rb), dim3(64 * GW_WAVES), 0, s, x, rows, cols, perm, scale,
                     slot, tau);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// inverse: the split of bhq_tau_kernel, for row block b.  S adds the rows of
// a large group wave by wave (float64), each wave's rows in slot order.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(64 * GW_WAVES) void bhq_inverse_kernel(InverseParams p) {
  __shared__ double ss[GW_WAVES][64];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t col = (int64_t)blockIdx.x * 64 + lane;
  const int64_t cc = col < p.cols ? col : p.cols - 1;
  const int64_t s0 = (int64_t)blockIdx.y * 64;
  const int64_t b = blockIdx.z;
  const double* T = p.T + (b * p.tstride) * p.ldt + cc;
  SlotInfo lsi;
  const uint64_t groups = chunk_groups(p.slot, s0, p.rows, lsi);
  int k = 0;
  for (uint64_t m = groups; m; m &= m - 1) {
    const int bit = __ffsll((unsigned long long)m) - 1;
    const int size = __builtin_amdgcn_readlane(lsi.size, bit);
    const int64_t sb = s0 + bit;
    const bool one = size <= GW_ROWS;  // one wave's group, else the block's
    if (one && k++ % GW_WAVES != wave) continue;
    const int w0 = one ? 0 : wave, step = one ? 1 : GW_WAVES;
    constexpr int U = 8;
    double S = 0.0;
    for (int q = w0; q < size; q += U * step) {
      double v[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int r = q + u * step;
        v[u] = T[(sb + (r < size ? r : 0)) * p.ldt];
      }
#pragma unroll
      for (int u = 0; u < U; ++u) S = S + (q + u * step < size ? v[u] : 0.0);
    }
    if (!one) {
      __syncthreads();  // the sums of the previous group have been read
      ss[wave][lane] = S;
      __syncthreads();
      S = 0.0;
#pragma unroll
      for (int w = 0; w < GW_WAVES; ++w) S = S + ss[w][lane];
    }
    const double T0 = T[sb * p.ldt];
    const double alpha = 1.0 / sqrt((double)size);
    const double tau = (alpha * S - T0) / (1.0 - alpha);
    const double up0 = (1.0 - alpha) * tau, dn = alpha * tau;
    for (int q = w0; q < size; q += U * step) {
      double v[U];
      float d[U];
      int32_t row[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int64_t r = sb + (q + u * step < size ? q + u * step : 0);
        v[u] = T[r * p.ldt];
        d[u] = p.scale[r];
        row[u] = p.perm[r];
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int r = q + u * step;
        if (r >= size || col >= p.cols) continue;
        const float f = (float)((r == 0 ? v[u] + up0 : v[u] - dn) / (double)d[u]);
        const int64_t o = ((int64_t)row[u] * p.ostride + b * p.obstride) * p.ldo + col;
        p.out[o] = (p.mask && !(p.mask[o] > 0.0f)) ? 0.0f : f;
      }
    }
  }
}

hipError_t launch_bhq_inverse(const InverseParams& p, hipStream_t s) {
  const int64_t cb = (p.cols + 63) / 64, rb = (p.rows + 63) / 64;
  if (cb > 0x7FFFFFFF || rb > 65535 || p.nblk > 65535 || p.nblk < 1) return hipErrorInvalidValue;
  hipLaunchKernelGGL(bhq_inverse_kernel, dim3((unsigned)cb, (unsigned)rb, (unsigned)p.nblk), dim3(64 * GW_WAVES), 0, s, p);
  return hipGetLastError();
}

}  // namespace fqt
