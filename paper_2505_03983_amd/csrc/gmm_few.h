// Mixture denoiser for calls whose rows are few against the mixture (a handful of chains, or a mixture that is itself
// small): posterior means on the fp32 matrix pipe straight from global memory, any d and C.
//
// What bounds such a call is latency: the mixture (a megabyte or so, in the caches after the first round) has to pass
// the matrix cores once, and one row per wavefront leaves it to a single CU (C dependent loads of d floats: 830 us a
// call at d = 300, C = 1000, 114 rows).  Two launches spread it over the chip instead:
//   logits   workgroup = 16 MI rows x 64 components, a wavefront per 16 components;
//   combine  workgroup = 16 MI rows x 16 coordinates, C split over its wavefronts, partial sums added through LDS
//            in wavefront order.
// v_mfma_f32_16x16x4_f32 takes one float of A and B per lane (row lane % 16, k lane / 16).  Which four k a step holds
// is free as long as A and B agree, so a lane fetches four consecutive floats of its row -- 16 k per row and load of
// 64 contiguous bytes -- and feeds them to four steps: 16-byte loads, no LDS staging, no transposition.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "gmm_cert.h"

namespace asd {

typedef float v4f_m __attribute__((ext_vector_type(4)));   // accumulator of v_mfma_f32_16x16x4_f32

struct FewArgs {
  const int32_t* n_dev;         // rows of the whole call
  int base, n_max;              // this launch's first row of them, and how many it takes at most; the row pointers start there
  int d, C, dp, cp;             // dp, cp: d and C rounded up to 4, the pitches of means_p and of means_t and logits
  const float* in_base;
  const int64_t* in_off;
  float* out_base;
  const int64_t* out_off;
  const int32_t* tau;
  const float4* coef_tau;       // kappa, gamma, c_x', c_m'
  const float* means_p;         // [C][dp], zero-padded
  const float* means_t;         // [d][cp], zero-padded
  const float* musq;
  const float* log_w;
  float* logits;                // [n_max][cp], base-2 units; -inf behind C
  float* pmax;                  // [n_max][np]
  int np;
};

__device__ __forceinline__ v4f_m mfma_4k(float4 a, float4 b, v4f_m acc) {
  acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a.x, b.x, acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a.y, b.y, acc, 0, 0, 0);
  acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a.z, b.z, acc, 0, 0, 0);
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a.w, b.w, acc, 0, 0, 0);
}

// A wavefront owns 16 MI rows x 16 NJ columns.  (The k loops below have the same trip count in every lane -- the matrix
// instruction takes the registers of all 64, whatever the execution mask says -- and lanes past the end feed zeros.)
template <int MI_, int NJ_, int U_>
struct FewTile {
  static constexpr int MI = MI_, NJ = NJ_, U = U_, ROWS = 16 * MI, COLS = 16 * NJ;
  static constexpr int GROUP = 4 * COLS;   // components of a logits workgroup = columns behind one partial row maximum
};

// KS: wavefronts that share a tile's k (each takes a contiguous part; partial products added in order through LDS).
// VX: d % 4 == 0 (rows of x are read 16 bytes at a time).
template <class T, int KS, bool VX>
__global__ __launch_bounds__(256 * KS) void gmm_few_logits_kernel(FewArgs p) {
  constexpr int MI = T::MI, NJ = T::NJ;
  const int n = min(*p.n_dev - p.base, p.n_max);
  const int row0 = blockIdx.x * T::ROWS;
  if (row0 >= n) return;
  const int lane = threadIdx.x & 63, i = lane & 15, g = lane >> 4;
  const int wave = (threadIdx.x >> 6) & 3, ks = threadIdx.x >> 8;
  const int col0 = blockIdx.y * T::GROUP + wave * T::COLS + i;
  const float* b[NJ];
  const float* a[MI];
#pragma unroll
  for (int u = 0; u < NJ; ++u) b[u] = p.means_p + (int64_t)min(col0 + 16 * u, p.C - 1) * p.dp;
#pragma unroll
  for (int t = 0; t < MI; ++t) a[t] = p.in_base + p.in_off[min(row0 + 16 * t + i, n - 1)];
  v4f_m acc[MI][NJ];
#pragma unroll
  for (int t = 0; t < MI; ++t)
#pragma unroll
    for (int u = 0; u < NJ; ++u) acc[t][u] = (v4f_m){0.f, 0.f, 0.f, 0.f};
  const int steps = (p.dp + 15) / 16, per = (steps + KS - 1) / KS;
  const int s_end = min(steps, (ks + 1) * per);
  // U steps' loads in flight ahead of their products (steps past the end: zeros against whatever lies at the row's start)
  for (int s0 = ks * per; s0 < s_end; s0 += T::U) {
    float4 bv[T::U][NJ], av[T::U][MI];
#pragma unroll
    for (int v = 0; v < T::U; ++v) {
      const int k = 16 * (s0 + v) + 4 * g;
      const bool kok = s0 + v < s_end && k < p.dp;
      const int kc = kok ? k : 0;
#pragma unroll
      for (int u = 0; u < NJ; ++u) bv[v][u] = *reinterpret_cast<const float4*>(b[u] + kc);
#pragma unroll
      for (int t = 0; t < MI; ++t) {
        float4 x;
        if constexpr (VX) {
          x = *reinterpret_cast<const float4*>(a[t] + kc);
        } else {   // kc < d; the other three may lie behind the row
          x.x = a[t][kc];
          x.y = kc + 1 < p.d ? a[t][kc + 1] : 0.f;
          x.z = kc + 2 < p.d ? a[t][kc + 2] : 0.f;
          x.w = kc + 3 < p.d ? a[t][kc + 3] : 0.f;
        }
        av[v][t] = kok ? x : make_float4(0.f, 0.f, 0.f, 0.f);
      }
    }
#pragma unroll
    for (int v = 0; v < T::U; ++v)
#pragma unroll
      for (int t = 0; t < MI; ++t)
#pragma unroll
        for (int u = 0; u < NJ; ++u) acc[t][u] = mfma_4k(av[v][t], bv[v][u], acc[t][u]);
  }
  if constexpr (KS > 1) {
    static_assert(MI * NJ == 1, "k shared among wavefronts: small tiles only");
    __shared__ v4f_m s_acc[KS - 1][4][64];
    if (ks > 0) s_acc[ks - 1][wave][lane] = acc[0][0];
    __syncthreads();
    if (ks == 0)
#pragma unroll
      for (int z = 0; z < KS - 1; ++z) acc[0][0] += s_acc[z][wave][lane];
  }
  __shared__ float s_max[4][T::ROWS];
  if (ks == 0) {
    float bias[NJ], q[NJ];
#pragma unroll
    for (int u = 0; u < NJ; ++u) {
      const int c = min(col0 + 16 * u, p.C - 1);
      bias[u] = kCertLog2e * p.log_w[c];
      q[u] = p.musq[c];
    }
#pragma unroll
    for (int t = 0; t < MI; ++t)
#pragma unroll
      for (int r = 0; r < 4; ++r) {   // element r of a lane: row 4 g + r, column i
        const int m = row0 + 16 * t + 4 * g + r;
        const float4 cf = p.coef_tau[p.tau[min(m, n - 1)]];
        float mx = -INFINITY;
#pragma unroll
        for (int u = 0; u < NJ; ++u) {
          const int col = col0 + 16 * u;
          const float l = col < p.C ? fmaf(kCertLog2e * cf.x, acc[t][u][r], fmaf(-kCertLog2e * cf.y, q[u], bias[u])) : -INFINITY;
          if (m < n && col < p.cp) p.logits[(int64_t)m * p.cp + col] = l;
          mx = fmaxf(mx, l);
        }
#pragma unroll
        for (int o = 8; o > 0; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o, 64));
        if (i == 0) s_max[wave][16 * t + 4 * g + r] = mx;
      }
  }
  __syncthreads();
  if (threadIdx.x < T::ROWS && row0 + (int)threadIdx.x < n)
    p.pmax[(int64_t)(row0 + threadIdx.x) * p.np + blockIdx.y] =
        fmaxf(fmaxf(s_max[0][threadIdx.x], s_max[1][threadIdx.x]), fmaxf(s_max[2][threadIdx.x], s_max[3][threadIdx.x]));
}

template <class T, int WAVES>
__global__ __launch_bounds__(64 * WAVES) void gmm_few_combine_kernel(FewArgs p) {
  constexpr int MI = T::MI, NJ = T::NJ;
  const int n = min(*p.n_dev - p.base, p.n_max);
  const int row0 = blockIdx.x * T::ROWS;
  if (row0 >= n) return;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, i = lane & 15, g = lane >> 4;
  const int j0 = blockIdx.y * T::COLS;
  const float* b[NJ];
  const float* a[MI];
  float mx[MI], sum[MI];
  v4f_m acc[MI][NJ];
#pragma unroll
  for (int u = 0; u < NJ; ++u) b[u] = p.means_t + (int64_t)min(j0 + 16 * u + i, p.d - 1) * p.cp;
#pragma unroll
  for (int t = 0; t < MI; ++t) {
    const int64_t m = min(row0 + 16 * t + i, n - 1);
    a[t] = p.logits + m * p.cp;
    sum[t] = 0.f;
    float v = -INFINITY;
    for (int e = g; e < p.np; e += 4) v = fmaxf(v, p.pmax[m * p.np + e]);
    v = fmaxf(v, __shfl_xor(v, 16, 64));
    mx[t] = fmaxf(v, __shfl_xor(v, 32, 64));
#pragma unroll
    for (int u = 0; u < NJ; ++u) acc[t][u] = (v4f_m){0.f, 0.f, 0.f, 0.f};
  }
  const int steps = (p.cp + 15) / 16, per = (steps + WAVES - 1) / WAVES;
  const int s_end = min(steps, (wave + 1) * per);
  for (int s0 = wave * per; s0 < s_end; s0 += T::U) {
    float4 bv[T::U][NJ], av[T::U][MI];
#pragma unroll
    for (int v = 0; v < T::U; ++v) {
      const int k = 16 * (s0 + v) + 4 * g;
      const bool kok = s0 + v < s_end && k < p.cp;
      const int kc = kok ? k : 0;
#pragma unroll
      for (int u = 0; u < NJ; ++u) bv[v][u] = *reinterpret_cast<const float4*>(b[u] + kc);
#pragma unroll
      for (int t = 0; t < MI; ++t) {
        const float4 l = *reinterpret_cast<const float4*>(a[t] + kc);
        av[v][t] = kok ? l : make_float4(-INFINITY, -INFINITY, -INFINITY, -INFINITY);
      }
    }
#pragma unroll
    for (int v = 0; v < T::U; ++v)
#pragma unroll
      for (int t = 0; t < MI; ++t) {
        const float4 l = av[v][t];
        float4 w;   // weights below 2^-40 of the row's largest are zero by definition (gmm_cert.h)
        w.x = l.x - mx[t] < -kCertZeroGap ? 0.f : __builtin_amdgcn_exp2f(l.x - mx[t]);
        w.y = l.y - mx[t] < -kCertZeroGap ? 0.f : __builtin_amdgcn_exp2f(l.y - mx[t]);
        w.z = l.z - mx[t] < -kCertZeroGap ? 0.f : __builtin_amdgcn_exp2f(l.z - mx[t]);
        w.w = l.w - mx[t] < -kCertZeroGap ? 0.f : __builtin_amdgcn_exp2f(l.w - mx[t]);
        sum[t] += (w.x + w.y) + (w.z + w.w);
#pragma unroll
        for (int u = 0; u < NJ; ++u) acc[t][u] = mfma_4k(w, bv[v][u], acc[t][u]);
      }
  }
  extern __shared__ float few_lds[];   // [WAVES][ROWS][COLS + 1] partial tiles, [WAVES][ROWS] partial row sums
  float* s_sum = few_lds + WAVES * T::ROWS * (T::COLS + 1);
  float* mine = few_lds + wave * T::ROWS * (T::COLS + 1);
#pragma unroll
  for (int t = 0; t < MI; ++t) {
#pragma unroll
    for (int u = 0; u < NJ; ++u)
#pragma unroll
      for (int r = 0; r < 4; ++r) mine[(16 * t + 4 * g + r) * (T::COLS + 1) + 16 * u + i] = acc[t][u][r];
    float v = sum[t];
    v += __shfl_xor(v, 16, 64);
    v += __shfl_xor(v, 32, 64);
    if (g == 0) s_sum[wave * T::ROWS + 16 * t + i] = v;
  }
  __syncthreads();
  for (int e = threadIdx.x; e < T::ROWS * T::COLS; e += 64 * WAVES) {
    const int r = e / T::COLS, c = e % T::COLS, m = row0 + r, j = j0 + c;
    if (m >= n || j >= p.d) continue;
    float v = 0.f, s = 0.f;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) {
      v += few_lds[(w * T::ROWS + r) * (T::COLS + 1) + c];
      s += s_sum[w * T::ROWS + r];
    }
    const float4 cf = p.coef_tau[p.tau[m]];
    p.out_base[p.out_off[m] + j] = fmaf(cf.z, p.in_base[p.in_off[m] + j], cf.w * (v / s));
  }
}

template <class T, int KS>
inline void launch_few_logits(const FewArgs& p, hipStream_t st) {
  const dim3 grid((unsigned)((p.n_max + T::ROWS - 1) / T::ROWS), (unsigned)p.np);
  if (p.d % 4 == 0)
    hipLaunchKernelGGL((gmm_few_logits_kernel<T, KS, true>), grid, dim3(256 * KS), 0, st, p);
  else
    hipLaunchKernelGGL((gmm_few_logits_kernel<T, KS, false>), grid, dim3(256 * KS), 0, st, p);
}
template <class T, int WAVES>
inline void launch_few_combine(const FewArgs& p, hipStream_t st) {
  const dim3 grid((unsigned)((p.n_max + T::ROWS - 1) / T::ROWS), (unsigned)((p.d + T::COLS - 1) / T::COLS));
  constexpr size_t lds = sizeof(float) * WAVES * T::ROWS * (T::COLS + 2);
  hipLaunchKernelGGL((gmm_few_combine_kernel<T, WAVES>), grid, dim3(64 * WAVES), lds, st, p);
}

// Rows whose logits the scratch holds at a time: 256 MB of them.  A call of more rows goes through it in parts, each of which
// leaves the chip half idle at its end (d 2, C 1000, 60000 rows: 162 us in one part, 230 in four).
inline int few_scratch_rows(int64_t rows, int C) {
  const int64_t cap = ((int64_t)256 << 20) / ((int64_t)sizeof(float) * (((C + 3) & ~3) + (C + 63) / 64));
  return (int)(rows < cap ? rows : cap / 32 * 32 > 32 ? cap / 32 * 32 : 32);
}

// Tile: 32 x 32 per wavefront (twice the products per byte) once that still gives every CU a workgroup -- d 128, C 1024:
// 1000 rows 25 us against 32 with 16 x 16, 200 rows 27 against 16 -- else 16 x 16.  Wavefronts that share a k loop: as
// many as leave each about four steps of 16 k.  (The rows of the whole call decide: all its parts add in one order.)
typedef FewTile<1, 1, 4> FewSmall;
typedef FewTile<2, 2, 2> FewLarge;
inline bool few_large_tiles(int64_t rows, int C) {
  return (rows + FewLarge::ROWS - 1) / FewLarge::ROWS * ((C + FewLarge::GROUP - 1) / FewLarge::GROUP) >= 256;
}
// scratch_rows: rows that logits and pmax have room for.
inline hipError_t launch_gmm_few(FewArgs p, int scratch_rows, hipStream_t st) {
  typedef FewSmall Small;
  typedef FewLarge Large;
  const int rows = p.n_max;
  const bool large = few_large_tiles(rows, p.C);
  p.np = large ? (p.C + Large::GROUP - 1) / Large::GROUP : (p.C + Small::GROUP - 1) / Small::GROUP;
  for (p.base = 0; p.base < rows; p.base += scratch_rows) {
    p.n_max = rows - p.base < scratch_rows ? rows - p.base : scratch_rows;
    if (large) {
      launch_few_logits<Large, 1>(p, st);
      if (p.C <= 1024) launch_few_combine<Large, 4>(p, st);
      else launch_few_combine<Large, 8>(p, st);
    } else {
      if (p.d > 256) launch_few_logits<Small, 4>(p, st);
      else if (p.d > 96) launch_few_logits<Small, 2>(p, st);
      else launch_few_logits<Small, 1>(p, st);
      if (p.C <= 128) launch_few_combine<Small, 4>(p, st);
      else if (p.C <= 512) launch_few_combine<Small, 8>(p, st);
      else launch_few_combine<Small, 16>(p, st);
    }
    p.in_off += scratch_rows;
    p.out_off += scratch_rows;
    p.tau += scratch_rows;
  }
  return hipGetLastError();
}

}  // namespace asd
