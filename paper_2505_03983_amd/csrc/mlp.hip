// Residual-MLP denoiser (stand-in for the paper's trained networks; the
// diffusion-policy and image-shaped workloads):
//   in  = [ bf16(x) ; temb[tau] ]                    (d + E)
//   h   = W_in in + b_in
//   h  += SiLU( W_l bf16(h) + b_l )                  l = 0..n_blocks-1
//   out = W_out bf16(h) + b_out,  D = clamp(out, -clip, clip)   interpreted as E[x_0 | x]
// Every matrix product takes bf16 inputs and accumulates in fp32 on the matrix
// cores; bias, SiLU and the residual stream are fp32 and are fused into the
// GEMM epilogues, which also emit the bf16 copy of h the next product reads.
//
// Activation precision (act_terms).  1: an activation enters a product as one bf16 number, bf16(h) above.
// 2: as the sum of two, hi = bf16(h), lo = bf16(h - hi) -- 16 significant bits -- held as two planes of the
// same matrix; the GEMM multiplies the weights with both planes into one accumulator.  Why it exists: a
// random-weight residual network amplifies the 2^-9 relative rounding of one-term activations to ~2e-3 of
// its output scale, whatever the accumulation order, so two correct implementations of the one-term
// network differ by that much (0.03-0.05 on outputs clipped to [-1, 1] when the unclipped scale is ~17);
// with two terms the same figure is ~4e-6 of the output scale.
#include "common.h"
#include "gemm_bf16.h"
#include "gemm_bf16_few.h"
#include "gemm_bf16_slab.h"

namespace asd {

// Tile shapes: output rows x columns, slabs per stage, stages, wavefronts, planes of A.  With two planes a slab of the
// largest tile is 32 KB, so its stages are single slabs.  The small ones read fragments a stage ahead.
template <int PL>
struct MlpTiles {
  typedef SlabCfg<128, 256, 3 - PL, PL == 2 ? 4 : 3, 2, 4, PL> T128x256;
  typedef SlabCfg<128, 128, 2, PL == 2 ? 3 : 4, 2, 4, PL> T128x128;
  typedef SlabCfg<64, 128, 2, PL == 2 ? 4 : 5, 2, 2, PL> T64x128;
  typedef SlabCfg<64, 64, 2, PL == 2 ? 6 : 8, 2, 2, PL, true> T64x64;
  typedef SlabCfg<32, 64, 2, PL == 2 ? 6 : 8, 1, 2, PL, true> T32x64;
};
// Which one: the least rounds x time of a tile, a tile taking f + k per 64 of K (a workgroup has its CU to itself;
// microseconds, fitted to K = 1024 and 4096 with two planes, 960 and 1536 with one, from a single tile to eight rounds of
// them).  rounds is ceil(tiles / CUs) up to two; past that the CUs no longer finish together, and a started round costs
// less than a whole one.  Measured, two planes, 4096 x 4096 weights (128 x 128 tiles throughout, before the slab layout: 160 us
// at 1984 rows and 63 at 456): 1984 rows 128 / 148 / 157 / - / -, 456 rows 79 / 55 / 39 / 56 / -, 200 rows - / 51 / 38 / 28 / 42;
// 2632 x 2632, 6746 rows 190 / 205 / 255 / 295 / -; 1024 x 1024: 3840 rows 32 / 27 / 31 / - / -, 960 rows 26 / 18 / 12 / 11 / 16, 120
// rows - / 17 / 13 / 9 / 8.  Of 300 networks of 16..3072 inputs and widths of 64..4096 on 1..8192 rows, six run more than 7%
// longer than on the one tile that suits them best, one more than 5% longer than on 128 x 128 tiles throughout.
struct TileCost {
  int bm, bn;
  float f, k;
  float least;   // of the widest tile, whose 128 KB of results alone take this long: K up to 450 (64-wide layers, 5659 rows, one
                 // plane: 9.0 a layer, 6.7 on 128 x 128, 6.1 on 64 x 128)
};
constexpr TileCost kTileCost[2][5] = {
    {{128, 256, 1.f, 1.05f, 9.f}, {128, 128, 3.f, 0.75f, 0.f}, {64, 128, 3.f, 0.45f, 0.f}, {64, 64, 3.5f, 0.33f, 0.f}, {32, 64, 4.f, 0.2f, 0.f}},
    {{128, 256, 0.f, 2.0f, 10.5f}, {128, 128, 3.f, 1.1f, 0.f}, {64, 128, 3.5f, 0.6f, 0.f}, {64, 64, 4.7f, 0.365f, 0.f}, {32, 64, 4.5f, 0.26f, 0.f}}};
static int pick_tile(int planes, int n, int N, int K, float* time = nullptr) {
  int best = 0;
  float best_t = INFINITY;
  for (int i = 0; i < 5; ++i) {
    const TileCost& c = kTileCost[planes - 1][i];
    const int64_t tiles = ceil_div(n, c.bm) * ceil_div(N, c.bn);
    float rounds = (float)ceil_div(tiles, 256);
    if (rounds > 2.f) rounds = 0.4f * rounds + 0.6f * (float)tiles / 256.f;
    const float t = rounds * std::max(c.least, c.f + c.k * (float)K / 64.f);
    if (t < best_t) {
      best_t = t;
      best = i;
    }
  }
  if (time) *time = best_t;
  return best;
}

constexpr int kMaxSplits = 8;

struct SplitScratch {
  float* part = nullptr;   // [kMaxSplits][rows][max N] fp32 partial tiles
  int rows = 0;            // rows the scratch was sized for (one per chain)
};

template <int PL, int CALL, class Epi>
static hipError_t mlp_gemm_tile(int tile, const int* n_dev, int n, int N, int K, SlabMat A, SlabMat Wt, Epi e, hipStream_t st) {
  typedef MlpTiles<PL> T;
  switch (tile) {
    case 0: return launch_gemm_bf16_slab<typename T::T128x256, CALL>(n_dev, n, N, K, A, Wt, e, st);
    case 1: return launch_gemm_bf16_slab<typename T::T128x128, CALL>(n_dev, n, N, K, A, Wt, e, st);
    case 2: return launch_gemm_bf16_slab<typename T::T64x128, CALL>(n_dev, n, N, K, A, Wt, e, st);
    case 3: return launch_gemm_bf16_slab<typename T::T64x64, CALL>(n_dev, n, N, K, A, Wt, e, st);
    default: return launch_gemm_bf16_slab<typename T::T32x64, CALL>(n_dev, n, N, K, A, Wt, e, st);
  }
}

// The kernel for few rows (gemm_bf16_few.h), where one of its tiles gives every workgroup a CU to itself: 0 is 16 x 32, 1 is
// 32 x 32, -1 neither.  Measured, microseconds a layer, this / the tiles above, 1, 32, 64, 128, 256 rows: 1024 x 1024, two
// planes, 5.1 5.2 5.7 6.0 7.9 / 7.3 8.0 8.6 8.9 9.2, one plane 4.0 4.2 4.3 4.6 5.9 / 6.5 7.2 7.4 7.6 8.0; 1536 x 1536, one
// plane, 128 rows (192 workgroups) 7.1 / 9.6, 256 rows (384) 11.2 / 9.8.  A product that is split over K below reads each
// weight once per 64 rows there and once per 32 here: 4096 x 4096, 24 rows 13.7 / 19.6, 64 rows 18.0 / 19.9 from the Infinity
// Cache, but slower from HBM, where a network of that size lies; it takes the smaller tile only.
static int pick_few_tile(int n, int N, int splits) {
  if (ceil_div(n, 16) * ceil_div(N, 32) <= 256) return 0;
  return splits == 1 && ceil_div(n, 32) * ceil_div(N, 32) <= 256 ? 1 : -1;
}
template <int PL, class Epi>
static hipError_t mlp_gemm_few(int tile, const int* n_dev, int n, int N, int K, SlabMat A, SlabMat Wt, Epi e, hipStream_t st,
                               int splits) {
  return tile == 0 ? launch_gemm_bf16_few<FewRowsCfg<1, 2, 16, PL>>(n_dev, n, N, K, A, Wt, e, st, splits)
                   : launch_gemm_bf16_few<FewRowsCfg<2, 2, 8, PL>>(n_dev, n, N, K, A, Wt, e, st, splits);
}

static bool large_matrix(int N, int Kp) { return (int64_t)N * Kp * 2 >= (8 << 20); }   // takes several microseconds to stream
// Workgroups that share the K of a draft call's tile: see mlp_gemm_planes.
static int draft_splits(int n, int N, int Kp) {
  const int64_t tiles = ceil_div(n, 64) * ceil_div(N, 64);
  int splits = 1;
  while (large_matrix(N, Kp) && splits < kMaxSplits && tiles * splits < 256 && (Kp / 64) % (2 * splits) == 0) splits *= 2;
  return splits;
}

// likely: rows to expect (n is the most there can be)
template <int PL, class Epi>
static hipError_t mlp_gemm_planes(int call, const int* n_dev, int n, int likely, int N, int K, SlabMat A, SlabMat Wt, Epi e,
                                  hipStream_t st, const SplitScratch& sc) {
  const int Kp = slab_count(K) * 32;
  // One row per chain against a large matrix: a stream of the weights, K split over workgroups.  64 x 64 tiles and a K split
  // that gives every CU a workgroup keep ~14 MB of it in flight, which is what HBM latency asks for; only a large matrix
  // repays the second launch.  (The split is a matter of the sizes alone, and the kernel for few rows adds its parts up
  // the same way: the bits do not depend on which of them runs.)
  typedef typename MlpTiles<PL>::T64x64 T;
  const int splits = call == 0 && n <= sc.rows ? draft_splits(n, N, Kp) : 1;
  const int few = pick_few_tile(n, N, splits);
  if (few >= 0) return mlp_gemm_few<PL>(few, n_dev, n, N, K, A, Wt, e, st, splits);
  if (call == 0) {
    if (splits > 1) return launch_gemm_bf16_slab<T, 0>(n_dev, n, N, K, A, Wt, e, st, splits, sc.part);
    return mlp_gemm_tile<PL, 0>(pick_tile(PL, n, N, Kp), n_dev, n, N, K, A, Wt, e, st);
  }
  return mlp_gemm_tile<PL, 1>(pick_tile(PL, likely, N, Kp), n_dev, n, N, K, A, Wt, e, st);
}

template <class Epi>
static hipError_t mlp_gemm(const RowPlan& rows, int N, int K, SlabMat A, SlabMat Wt, Epi e, hipStream_t st,
                           const SplitScratch& sc) {
  const int likely = rows.likely > 0 ? std::min(rows.likely, rows.n) : rows.n;
  return A.plane > 0 ? mlp_gemm_planes<2>(rows.call, rows.n_dev, rows.n, likely, N, K, A, Wt, e, st, sc)
                     : mlp_gemm_planes<1>(rows.call, rows.n_dev, rows.n, likely, N, K, A, Wt, e, st, sc);
}

// A product of `rows` rows, where the call could bring `most`, in microseconds, by the figures at pick_tile and pick_few_tile; one
// that is split over K streams its weights at 2.4 TB/s and adds its parts in 5 us.
static double product_cost(int planes, int call, int rows, int most, int N, int K) {
  const int Kp = slab_count(K) * 32, splits = call == 0 ? draft_splits(rows, N, Kp) : 1;
  const int few = pick_few_tile(most, N, splits);
  if (few >= 0) return (few == 0 ? 1.5 : 2.0) + (planes == 2 ? 3.6 : 2.5) * (few == 0 ? 1.0 : 1.6) * Kp / 1024.0;
  if (splits > 1) return 2e-6 * N * Kp / 2.4 + 5.0;
  float t;
  (void)pick_tile(planes, rows, N, Kp, &t);
  return t;
}

struct MlpState {
  int width = 0, n_blocks = 0, E = 0, in_dim = 0;
  uint16_t* wp_in = nullptr;     // copies of the caller's weights in slab layout (gemm_bf16_slab.h)
  uint16_t* wp_blk = nullptr;
  uint16_t* wp_out = nullptr;
  float out_clip = 0.f;
  float2* eps_coef = nullptr;    // [n_tau] (1/sqrt(abar), sqrt(1-abar)/sqrt(abar)) when the network predicts the noise
  const uint16_t* w_in = nullptr;
  const uint16_t* w_blk = nullptr;
  const uint16_t* w_out = nullptr;
  const float* b_in = nullptr;
  const float* b_blk = nullptr;
  const float* b_out = nullptr;
  const uint16_t* temb = nullptr;
  int act_terms = 1;          // bf16 terms an activation enters a product with (1 or 2)
  // activations in slab layout, act_terms planes each, the planes of a matrix in_plane / h_plane elements apart
  int64_t rows_pad = 0;       // rows they are laid out with
  uint16_t* in_bf = nullptr;  // [act_terms][slabs of d + E][rows_pad][32]
  float* h = nullptr;         // [rows_max, width]
  uint16_t* hb[2] = {nullptr, nullptr};   // [act_terms][slabs of width][rows_pad][32] each
  int64_t in_plane = 0, h_plane = 0;      // 0 when act_terms == 1
  SplitScratch split;
};


// in_bf[n] = [ bf16(x_n) ; temb[tau_n] ], eight elements per thread; in_plane > 0: the lo terms of x (zero for
// the time embedding, which is bf16 data) go to the second plane
__global__ void mlp_pack_kernel(const int* __restrict__ n_dev, int n_rows, int d, int E, const float* __restrict__ in_base,
                                const int64_t* __restrict__ in_off, const int32_t* __restrict__ tau,
                                const uint16_t* __restrict__ temb, uint16_t* __restrict__ in_bf, int64_t in_slab,
                                int64_t in_plane) {
  const int n = blockIdx.x;
  const int q = blockIdx.y * blockDim.x + threadIdx.x;  // group of 8 elements
  const int in_dim = d + E;
  if (q * 8 >= in_dim || n >= min(*n_dev, n_rows)) return;
  uint4 o, l = make_uint4(0u, 0u, 0u, 0u);
  if (q * 8 < d) {
    const float* x = in_base + in_off[n] + q * 8;
    const float4 lo = *reinterpret_cast<const float4*>(x);
    const float4 hi = *reinterpret_cast<const float4*>(x + 4);
    const float v[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
    uint16_t h[8], r[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      h[k] = f32_to_bf16_rne(v[k]);
      r[k] = bf16_lo(v[k], h[k]);
    }
    o = make_uint4((uint32_t)h[0] | ((uint32_t)h[1] << 16), (uint32_t)h[2] | ((uint32_t)h[3] << 16),
                   (uint32_t)h[4] | ((uint32_t)h[5] << 16), (uint32_t)h[6] | ((uint32_t)h[7] << 16));
    l = make_uint4((uint32_t)r[0] | ((uint32_t)r[1] << 16), (uint32_t)r[2] | ((uint32_t)r[3] << 16),
                   (uint32_t)r[4] | ((uint32_t)r[5] << 16), (uint32_t)r[6] | ((uint32_t)r[7] << 16));
  } else {
    o = *reinterpret_cast<const uint4*>(temb + (int64_t)tau[n] * E + (q * 8 - d));
  }
  uint16_t* dst = in_bf + (q >> 2) * in_slab + (int64_t)n * 32 + (q & 3) * 8;
  *reinterpret_cast<uint4*>(dst) = o;
  if (in_plane) *reinterpret_cast<uint4*>(dst + in_plane) = l;
}

// The caller's weights [rows, K] (row-major bf16) in slab layout: eight elements per thread, zeros in the padding.  (K is a
// multiple of 8; the array itself may start at any element of a larger one.)
__global__ __launch_bounds__(256) void mlp_pack_weights_kernel(int rows, int K, int64_t rows_pad, int nslabs,
                                                               const uint16_t* __restrict__ w, uint16_t* __restrict__ out) {
  const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;   // chunk: slab, row, quarter
  if (t >= rows_pad * nslabs * 4) return;
  const int64_t row = (t >> 2) % rows_pad;
  const int k = (int)((t >> 2) / rows_pad) * 32 + (int)(t & 3) * 8;
  uint4 v = make_uint4(0u, 0u, 0u, 0u);
  if (row < rows && k < K) {
    const uint16_t* p = w + row * K + k;
    if (((uintptr_t)w & 15) == 0) {
      v = *reinterpret_cast<const uint4*>(p);
    } else {
      v.x = p[0] | (uint32_t)p[1] << 16;
      v.y = p[2] | (uint32_t)p[3] << 16;
      v.z = p[4] | (uint32_t)p[5] << 16;
      v.w = p[6] | (uint32_t)p[7] << 16;
    }
  }
  *reinterpret_cast<uint4*>(out + t * 8) = v;
}

// SiLU with the hardware exp2 and reciprocal: relative error ~1e-6, inside what the re-rounding of the
// activations leaves of the value (2^-9 with one bf16 term, 2^-17 with two).
__device__ __forceinline__ float silu(float z) {
  return z * __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(-1.4426950408889634f * z));
}

__device__ __forceinline__ float4 load_bias4(const float* bias, int n) {
  return bias ? *reinterpret_cast<const float4*>(bias + n) : make_float4(0.f, 0.f, 0.f, 0.f);
}

struct InEpi {  // h = acc + b; hb = bf16 terms of h
  float* h;
  uint16_t* hb;
  const float* bias;
  int64_t ld, slab;  // pitch of h (fp32), elements of a slab of hb (bf16)
  int64_t lo_plane; // > 0: offset of hb's second plane (two-term activations)
  static constexpr bool kLoads = false, kAux = false;
  // four consecutive columns n..n+3 (n % 4 == 0) of row m
  __device__ __forceinline__ float4 load4(int, int) const { return make_float4(0.f, 0.f, 0.f, 0.f); }
  __device__ __forceinline__ float4 column4(int n) const { return load_bias4(bias, n); }
  __device__ __forceinline__ void store4(int m, int n, float4 a, float4, float4 b) const {
    const float4 v = make_float4(a.x + b.x, a.y + b.y, a.z + b.z, a.w + b.w);
    *reinterpret_cast<float4*>(h + (int64_t)m * ld + n) = v;
    store_act4(hb + (n >> 5) * slab + (int64_t)m * 32 + (n & 31), lo_plane, v);
  }
};

struct BlockEpi {  // h += SiLU(acc + b); hb_next = bf16 terms of h
  float* h;
  uint16_t* hb_next;
  const float* bias;
  int64_t ld, slab;
  int64_t lo_plane;
  static constexpr bool kLoads = true, kAux = false;
  __device__ __forceinline__ float4 load4(int m, int n) const {
    return *reinterpret_cast<const float4*>(h + (int64_t)m * ld + n);
  }
  __device__ __forceinline__ float4 column4(int n) const { return load_bias4(bias, n); }
  __device__ __forceinline__ void store4(int m, int n, float4 a, float4 p, float4 b) const {
    float* hp = h + (int64_t)m * ld + n;
    const float4 v = make_float4(p.x + silu(a.x + b.x), p.y + silu(a.y + b.y), p.z + silu(a.z + b.z),
                                 p.w + silu(a.w + b.w));
    *reinterpret_cast<float4*>(hp) = v;
    store_act4(hb_next + (n >> 5) * slab + (int64_t)m * 32 + (n & 31), lo_plane, v);
  }
};

// The output layer's acc + b as x_0: converted where the network estimates the noise (x the row evaluated), and clipped.
__device__ __forceinline__ float4 from_noise(float4 v, float2 ec, float4 x) {
  return make_float4(fmaf(x.x, ec.x, -v.x * ec.y), fmaf(x.y, ec.x, -v.y * ec.y), fmaf(x.z, ec.x, -v.z * ec.y),
                     fmaf(x.w, ec.x, -v.w * ec.y));
}
__device__ __forceinline__ float4 clipped(float4 v, float clip) {
  if (clip > 0.f) {
    v.x = fminf(fmaxf(v.x, -clip), clip);
    v.y = fminf(fmaxf(v.y, -clip), clip);
    v.z = fminf(fmaxf(v.z, -clip), clip);
    v.w = fminf(fmaxf(v.w, -clip), clip);
  }
  return v;
}

struct OutEpi {  // out[out_off[m] + n] = acc + b, as x_0 (or converted from a noise estimate), clipped
  float* out_base;
  const int64_t* out_off;
  const float* bias;
  float clip;  // 0: none
  // noise-predicting networks: x_0 = x / sqrt(abar) - out * sqrt(1 - abar) / sqrt(abar), x = the row evaluated
  const float2* eps_coef;  // NULL: the network predicts x_0
  const int32_t* tau;
  const float* in_base;
  const int64_t* in_off;
  static constexpr bool kLoads = false, kAux = false;
  __device__ __forceinline__ float4 load4(int, int) const { return make_float4(0.f, 0.f, 0.f, 0.f); }
  __device__ __forceinline__ float4 column4(int n) const { return load_bias4(bias, n); }
  __device__ __forceinline__ void store4(int m, int n, float4 a, float4, float4 b) const {
    float4 v = make_float4(a.x + b.x, a.y + b.y, a.z + b.z, a.w + b.w);
    if (eps_coef) v = from_noise(v, eps_coef[tau[m]], *reinterpret_cast<const float4*>(in_base + in_off[m] + n));
    *reinterpret_cast<float4*>(out_base + out_off[m] + n) = clipped(v, clip);
  }
};

// The output layer of a sequential step (row m: chain m, at step i): takes the step with the value it has just formed, and
// packs the row for the next one.  As a kernel of its own the step was 4 us of a policy step's 38.  Same expressions as
// seq_step_kernel's, same bits.
struct SeqEpi {
  float* traj;   // the chains' row i, (K + 1) d apart; row i + 1 behind it
  int64_t chain_stride;
  const float* bias;
  float clip;
  const float2* eps_coef;   // NULL: the network predicts x_0
  const int32_t* tau;       // step -> time index
  const float* c_x;
  const float* c_0;
  const float* sigma;
  const Key* key;
  int i, d;
  PackOut pack;             // in_bf NULL: the last step
  int64_t* row_counts;      // row total for the profiler, or NULL
  static constexpr bool kLoads = true, kAux = true;
  __device__ __forceinline__ float4 load4(int m, int n) const {
    return *reinterpret_cast<const float4*>(traj + m * chain_stride + n);
  }
  __device__ __forceinline__ float4 column4(int n) const { return load_bias4(bias, n); }
  __device__ __forceinline__ float4 aux4(int m, int n) const { return normal4(*key, (uint32_t)m, (uint32_t)(i + 1), (uint32_t)n >> 2); }
  __device__ __forceinline__ void store4(int m, int n, float4 a, float4 y, float4 b) const { store4(m, n, a, y, b, aux4(m, n)); }
  __device__ __forceinline__ void store4(int m, int n, float4 a, float4 y, float4 b, float4 xi) const {
    float4 g = make_float4(a.x + b.x, a.y + b.y, a.z + b.z, a.w + b.w);
    if (eps_coef) g = from_noise(g, eps_coef[tau[i]], y);
    g = clipped(g, clip);
    const float cx = c_x[i], c0 = c_0[i], sg = sigma[i];
    y.x = fmaf(sg, xi.x, fmaf(cx, y.x, c0 * g.x));
    y.y = fmaf(sg, xi.y, fmaf(cx, y.y, c0 * g.y));
    y.z = fmaf(sg, xi.z, fmaf(cx, y.z, c0 * g.z));
    y.w = fmaf(sg, xi.w, fmaf(cx, y.w, c0 * g.w));
    *reinterpret_cast<float4*>(traj + m * chain_stride + d + n) = y;
    if (!pack.in_bf) return;
    store_act4(pack.in_bf + (n >> 5) * pack.slab + (int64_t)m * 32 + (n & 31), pack.plane, y);
    const uint16_t* te = pack.temb + (int64_t)tau[i + 1] * pack.E;
    for (int e = n; e < pack.E; e += d) {   // four numbers of the embedding to four columns of the row
      const int k = d + e;
      uint16_t* dst = pack.in_bf + (k >> 5) * pack.slab + (int64_t)m * 32 + (k & 31);
      *reinterpret_cast<uint2*>(dst) = *reinterpret_cast<const uint2*>(te + e);
      if (pack.plane) *reinterpret_cast<uint2*>(dst + pack.plane) = make_uint2(0u, 0u);
    }
    if (row_counts && n == 0) atomicAdd((unsigned long long*)row_counts, 1ull);
  }
};

asd_status mlp_create(asd_ctx* ctx, const asd_denoiser& den) {
  MlpState* s = new (std::nothrow) MlpState();
  if (!s) return ASD_ENOMEM;
  ctx->mlp = s;
  s->width = den.width;
  s->n_blocks = den.n_blocks;
  s->E = den.temb_dim;
  s->out_clip = den.out_clip;
  s->act_terms = den.act_terms;
  if (den.predict_eps) {
    std::vector<float2> ec((size_t)ctx->n_tau);
    for (int t = 0; t < ctx->n_tau; ++t) {
      const double ab = den.abar[t];
      ec[t] = make_float2((float)(1.0 / sqrt(ab)), (float)(sqrt(1.0 - ab) / sqrt(ab)));
    }
    ASD_HIP(hipMalloc(&s->eps_coef, sizeof(float2) * ec.size()));
    ASD_HIP(hipMemcpy(s->eps_coef, ec.data(), sizeof(float2) * ec.size(), hipMemcpyHostToDevice));
  }
  s->in_dim = ctx->d + den.temb_dim;
  s->w_in = (const uint16_t*)den.w_in;
  s->w_blk = (const uint16_t*)den.w_blk;
  s->w_out = (const uint16_t*)den.w_out;
  s->b_in = den.b_in;
  s->b_blk = den.b_blk;
  s->b_out = den.b_out;
  s->temb = (const uint16_t*)den.temb;
  const size_t rows = (size_t)ctx->n_rows_max;
  ctx->model_macs_per_row = (double)s->in_dim * s->width + (double)s->n_blocks * s->width * s->width +
                            (double)s->width * ctx->d;
  const int64_t Wd = s->width, dd = ctx->d;
  const size_t planes = (size_t)s->act_terms;
  s->rows_pad = slab_rows((int64_t)rows);
  const size_t in_elems = slab_elems((int64_t)rows, s->in_dim), h_elems = slab_elems((int64_t)rows, s->width);
  if (planes > 1) {
    s->in_plane = (int64_t)in_elems;
    s->h_plane = (int64_t)h_elems;
  }
  ASD_HIP(hipMalloc(&s->in_bf, sizeof(uint16_t) * planes * in_elems));
  ASD_HIP(hipMalloc(&s->h, sizeof(float) * rows * s->width));
  ASD_HIP(hipMalloc(&s->hb[0], sizeof(uint16_t) * planes * h_elems));
  ASD_HIP(hipMalloc(&s->hb[1], sizeof(uint16_t) * planes * h_elems));
  ASD_HIP(hipMemset(s->in_bf, 0, sizeof(uint16_t) * planes * in_elems));
  ASD_HIP(hipMemset(s->hb[0], 0, sizeof(uint16_t) * planes * h_elems));
  ASD_HIP(hipMemset(s->hb[1], 0, sizeof(uint16_t) * planes * h_elems));
  // the weights in slab layout (one-time; the caller's arrays are not read again)
  auto pack = [](uint16_t* dst, const uint16_t* src, int64_t n, int K) -> hipError_t {
    const int64_t chunks = (int64_t)slab_elems(n, K) / 8;
    hipLaunchKernelGGL(mlp_pack_weights_kernel, dim3((unsigned)ceil_div(chunks, 256)), dim3(256), 0, 0, (int)n, K,
                       slab_rows(n), slab_count(K), src, dst);
    return hipGetLastError();
  };
  ASD_HIP(hipMalloc(&s->wp_in, sizeof(uint16_t) * slab_elems(Wd, s->in_dim)));
  ASD_HIP(hipMalloc(&s->wp_out, sizeof(uint16_t) * slab_elems(dd, s->width)));
  ASD_HIP(pack(s->wp_in, s->w_in, Wd, s->in_dim));
  ASD_HIP(pack(s->wp_out, s->w_out, dd, s->width));
  if (s->n_blocks) {
    const size_t blk = slab_elems(Wd, s->width);
    ASD_HIP(hipMalloc(&s->wp_blk, sizeof(uint16_t) * s->n_blocks * blk));
    for (int l = 0; l < s->n_blocks; ++l) ASD_HIP(pack(s->wp_blk + l * blk, s->w_blk + (size_t)l * Wd * Wd, Wd, s->width));
  }
  {
    const size_t max_n = (size_t)std::max(Wd, dd);
    s->split.rows = ctx->B;
    ASD_HIP(hipMalloc(&s->split.part, sizeof(float) * kMaxSplits * (size_t)ctx->B * max_n));
  }
  ASD_HIP(hipDeviceSynchronize());
  return ASD_OK;
}

void mlp_destroy(asd_ctx* ctx) {
  MlpState* s = ctx->mlp;
  if (!s) return;
  (void)hipFree(s->in_bf);
  (void)hipFree(s->h);
  (void)hipFree(s->hb[0]);
  (void)hipFree(s->hb[1]);
  (void)hipFree(s->wp_in);
  (void)hipFree(s->wp_blk);
  (void)hipFree(s->wp_out);
  (void)hipFree(s->eps_coef);
  (void)hipFree(s->split.part);
  delete s;
  ctx->mlp = nullptr;
}

PackOut mlp_pack_out(const asd_ctx* ctx) {
  const MlpState* s = ctx->mlp;
  return PackOut{s->in_bf, s->rows_pad * 32, s->in_plane, s->temb, s->E, ctx->d};
}

double mlp_call_cost(const asd_ctx* ctx, int call, int rows, int most) {
  const MlpState* s = ctx->mlp;
  const int p = s->act_terms, W = s->width;
  return product_cost(p, call, rows, most, W, s->in_dim) + s->n_blocks * product_cost(p, call, rows, most, W, W) +
         product_cost(p, call, rows, most, ctx->d, W);
}

uint32_t mlp_verify_tiles(const asd_ctx* ctx, int likely, int most) {
  const MlpState* s = ctx->mlp;
  const int shapes[3][2] = {{s->width, s->in_dim}, {s->width, s->width}, {ctx->d, s->width}};
  uint32_t tiles = 0;
  for (const auto& p : shapes) {   // (as mlp_gemm_planes picks them)
    const int few = pick_few_tile(most, p[0], 1);
    tiles = 8 * tiles + (few >= 0 ? 5 + few : pick_tile(s->act_terms, likely, p[0], slab_count(p[1]) * 32));
  }
  return tiles;
}

asd_status mlp_eval(asd_ctx* ctx, const RowPlan& rows, hipStream_t st) {
  MlpState* s = ctx->mlp;
  const int n = rows.n, d = ctx->d, W = s->width;
  if (!rows.packed) {
    ProfScope ps(ctx, ASD_PROF_MLP_PACK, rows.call, st);
    const int groups = s->in_dim / 8;
    const int threads = groups >= 256 ? 256 : 64;
    dim3 grid((unsigned)n, (unsigned)ceil_div(groups, threads));
    hipLaunchKernelGGL(mlp_pack_kernel, grid, dim3(threads), 0, st, rows.n_dev, n, d, s->E, rows.in_base, rows.in_off,
                       rows.tau, s->temb, s->in_bf, s->rows_pad * 32, s->in_plane);
    ASD_HIP(hipGetLastError());
  }
  const int64_t slab = s->rows_pad * 32, w_rows = slab_rows(W);
  const SlabMat in{s->in_bf, s->rows_pad, s->in_plane};
  SlabMat h[2] = {{s->hb[0], s->rows_pad, s->h_plane}, {s->hb[1], s->rows_pad, s->h_plane}};
  {
    ProfScope ps(ctx, ASD_PROF_MLP_GEMM_IN, rows.call, st);
    ASD_HIP(mlp_gemm(rows, W, s->in_dim, in, SlabMat{s->wp_in, w_rows, 0},
                     InEpi{s->h, s->hb[0], s->b_in, W, slab, s->h_plane}, st, s->split));
  }
  int cur = 0;
  const size_t blk = slab_elems(W, W);
  for (int l = 0; l < s->n_blocks; ++l) {
    ProfScope ps(ctx, ASD_PROF_MLP_GEMM_BLK, rows.call, st);
    const BlockEpi e{s->h, s->hb[cur ^ 1], s->b_blk ? s->b_blk + (size_t)l * W : nullptr, W, slab, s->h_plane};
    ASD_HIP(mlp_gemm(rows, W, W, h[cur], SlabMat{s->wp_blk + l * blk, w_rows, 0}, e, st, s->split));
    cur ^= 1;
  }
  {
    ProfScope ps(ctx, ASD_PROF_MLP_GEMM_OUT, rows.call, st);
    if (rows.seq_step >= 0) {
      const bool more = rows.seq_step + 1 < ctx->K;
      const SeqEpi e{const_cast<float*>(rows.in_base) + (int64_t)rows.seq_step * d, (int64_t)(ctx->K + 1) * d, s->b_out, s->out_clip,
                     s->eps_coef, ctx->tau, ctx->c_x, ctx->c_0, ctx->sigma, ctx->key_dev, rows.seq_step, d,
                     more ? mlp_pack_out(ctx) : PackOut{}, more && prof_counting(ctx) ? ctx->row_counts : nullptr};
      ASD_HIP(mlp_gemm(rows, d, W, h[cur], SlabMat{s->wp_out, slab_rows(d), 0}, e, st, s->split));
      return ASD_OK;
    }
    const OutEpi e{rows.out_base, rows.out_off, s->b_out, s->out_clip, s->eps_coef, rows.tau, rows.in_base, rows.in_off};
    ASD_HIP(mlp_gemm(rows, d, W, h[cur], SlabMat{s->wp_out, slab_rows(d), 0}, e, st, s->split));
  }
  return ASD_OK;
}

}  // namespace asd
