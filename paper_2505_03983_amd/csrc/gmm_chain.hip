// Chain-resident ASD sampler for Gaussian-mixture denoisers that fit in LDS.
//
// For small shapes a round of ASD is a handful of microsecond kernels and the
// sample is bound by launches, not by arithmetic.  Chains never interact, so here
// one workgroup runs the *whole* of Alg. 1 for one chain in a single launch:
// the mixture, the schedule, the window of proposal samples, the model values
// and the noise of the window live in LDS, and the only HBM traffic inside the
// loop is the trajectory rows the round produces.  Per round (notation of
// Alg. 1, x0-prediction form):
//   A. x0a = D(y_a, tau_a): the logits of a tile of 16 components per wavefront, then a wavefront per
//      part of the weighted sum over components;
//   B. the parts put together and the draft: yhat_{i+1} = c_x yhat_i + c_0 x0a + sigma xi_{i+1},
//      a thread per coordinate walks the window; the wavefronts without a coordinate meanwhile make
//      xi and log u of later steps from the counter (noise is kept in a ring of up to two windows);
//   C. verify: x0_i = D(yhat_i, tau_i), i = a+1..b-1, all rows at once, and Alg. 3's accept test, a
//      wavefront per slot (it adds the parts of its row and reduces <D,xi>, |D|^2);
//   D. Alg. 2 as ballot + trailing ones, reflection of the first rejected row, the rows the chain
//      keeps to the trajectory, advance.
// The denoiser is two small matrix products around a softmax, done by the whole
// workgroup; the verify rows go through the matrix cores 16 at a time (a window
// of L <= 17 is one tile; the single row of x0a stays on the vector ALUs): v_mfma_f32_16x16x4_f32
// takes a 16 x 4 and a 4 x 16 operand straight from LDS.  Where every wavefront has at most one tile of logits
// (16 components x 16 rows) they stay in registers until the rows' maxima are known.  The formulas and the counters
// are those of the stand-alone kernels, so the same parity bars apply.  Every wavefront leaves the loop when its
// chain reaches K, which takes at most K rounds.
//
// What bounds it: one workgroup is all a chain has, so a round is the sum of its stages.  At d 64, C 256, L 16, K 1000 it is
// 23 800 cycles: 4 200 for A, 5 000 for B (the walk of one wavefront through the window, an LDS round trip and two dependent
// products a step), 13 200 for C and 1 300 for D.  In C the four wavefronts of a SIMD share its issue slots and its matrix
// core: the two products are 2 050 cycles of fp32 MFMA each, and every vector instruction that all of them execute is another
// 16.  Noise made ahead, logits that stay in registers, the accept test merged with the sum of the parts, loops whose LDS reads
// are in flight together (a read in a loop of unknown length costs its 130 cycles each time) and addresses made from sums
// instead of products took a sample from 1063 to 828 us, (2, 256, 16) at K 200 from 229 to 165, (16, 64, 64) from 299 to 233,
// (4, 256, 64) from 343 to 281, (30, 100, 6) from 403 to 265; not a bit of a sample changed.
//
// Mixtures of a few numbers have a kernel of their own, a wavefront per chain (gmm_wave_sample_kernel, below).
#include "common.h"
#include "device_util.h"
#include "gmm_state.h"

namespace asd {

// Where a launch leaves its largest round count: (launch id, rounds) packed, so that the maximum needs no reset between
// samples, and a count of the chains that have reported; the last of them hands the result to the host (a copy behind the
// kernel was 4 us of the sample).
struct RoundsOut {
  unsigned long long* state;   // DEV [2]: the maximum; chains reported, over all launches of the context
  uint32_t* host;              // the result, in pinned host memory
  uint32_t launch_id;
  __device__ __forceinline__ void report(int R, int chains) const {
    atomicMax(state, ((unsigned long long)launch_id << 32) | (unsigned)R);
    __threadfence();
    if ((atomicAdd(state + 1, 1ull) + 1ull) % (unsigned)chains == 0) {
      __threadfence();
      const unsigned long long m = __hip_atomic_load(state, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      __hip_atomic_store(host, (uint32_t)m, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
    }
  }
};

namespace {

typedef float v4f_c __attribute__((ext_vector_type(4)));

// LDS layout, in floats.  Rows that feed the matrix cores (mixture, proposal samples, softmax
// weights) are padded to a multiple of 16 plus 4: a 16-byte operand read by 16 lanes from 16
// consecutive rows then falls into 16 different bank groups.
struct ChainLayout {
  int d16, dp, C16, cp, nblk, tr, ring;
  size_t m, q, lw, ps, part, yh, x0, xi, sch, total;
};

constexpr int kChainSplits = 4;  // most ways the component sum of a tile is split over wavefronts

__host__ __device__ inline ChainLayout chain_layout(int C, int d, int L, int K, int ring) {
  ChainLayout l;
  l.d16 = (d + 15) & ~15;
  l.dp = l.d16 + 4;
  l.C16 = (C + 15) & ~15;
  l.cp = l.C16 + 4;
  l.nblk = (d + 3) >> 2;
  l.tr = 16 * ((((L > 1) ? L - 1 : 1) + 15) / 16);  // rows of softmax scratch: whole tiles of 16
  l.ring = ring;                             // steps the noise ring holds: the window's, or those and as many more
  l.m = 0;                                   // [C16][dp] means, rows past C and columns past d zero
  l.q = l.m + (size_t)l.C16 * l.dp;          // [C16] |mu|^2
  l.lw = l.q + l.C16;                        // [C16] log w
  l.ps = l.lw + l.C16;                       // [tr][cp] logits, then softmax weights
  l.part = l.ps + (size_t)l.tr * l.cp;       // [max(16, splits * tr)][dp] partial sums over components
  l.yh = l.part + (size_t)(kChainSplits * l.tr > 16 ? kChainSplits * l.tr : 16) * l.dp;  // [L+1][dp] yhat_a (= y_a) .. yhat_b
  l.x0 = l.yh + (size_t)(L + 1) * l.dp;      // [L][dp] model value at yhat_{a+s}
  l.xi = l.x0 + (size_t)L * l.dp;            // [ring][dp] xi_{i+1} of step i in row i % ring
  l.sch = l.xi + (size_t)ring * l.dp;        // [K][8] (c_x, c_0, sigma, -, kappa, gamma, cx, cm) of step i
  l.total = l.sch + (size_t)K * 8;
  return l;
}

// Workgroup barrier that orders LDS traffic only.  __syncthreads() also waits for this wavefront's
// global stores to be acknowledged (a microsecond each round for the trajectory rows, which nobody
// in the workgroup reads back from memory).
__device__ __forceinline__ void lds_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

__device__ __forceinline__ float4 lds4(const float* row, int blk) {
  return *reinterpret_cast<const float4*>(row + 4 * blk);
}

// Softmax weights of the drafted rows 1 .. n of yh into ps, and their rows' scales, where there are more tiles of (16 rows x 16
// components) than wavefronts: a pass over the logits, then a wavefront per row.  (Every thread must call; a barrier
// inside and one at the end.)
//
// v_mfma_f32_16x16x4_f32: A is 16 x 4 (lane l holds A[l % 16][l / 16]), B is 4 x 16 (lane l holds
// B[l / 16][l % 16]), D is 16 x 16 (lane l, register r holds D[4 (l / 16) + r][l % 16]).  A lane reads
// four consecutive k of its row at once (16 bytes) and feeds them to four MFMAs; since both operands
// do the same, the pairing of the elements is exact.  Rows past the last one repeat it (computed, never stored).
__device__ __forceinline__ void softmax_tiles(int n, int T, int a, const ChainLayout& l, int C, const float* m_l,
                                              const float* q_l, const float* lw_l, float* ps, const float* yh,
                                              const float4* sch, float* s_sc, int wave, int nw, int lane) {
  const int dp = l.dp, cp = l.cp;
  const int li = lane & 15, kq = lane >> 4;
  constexpr float kLog2e = 1.4426950408889634f;
  {
    const int NT = l.C16 >> 4;
    for (int item = wave; item < T * NT; item += nw) {
      int t = 0, nt = item;
      for (; nt >= NT; nt -= NT) ++t;
      const float* xa = yh + (size_t)(1 + min(16 * t + li, n - 1)) * dp + 4 * kq;
      const float* mb = m_l + (size_t)(16 * nt + li) * dp + 4 * kq;
      v4f_c acc = {0.f, 0.f, 0.f, 0.f};
      for (int s = 0; s < l.d16; s += 16) {
        const float4 av = *reinterpret_cast<const float4*>(xa + s);
        const float4 bv = *reinterpret_cast<const float4*>(mb + s);
        acc = __builtin_amdgcn_mfma_f32_16x16x4f32(av.x, bv.x, acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_16x16x4f32(av.y, bv.y, acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_16x16x4f32(av.z, bv.z, acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_16x16x4f32(av.w, bv.w, acc, 0, 0, 0);
      }
      const int comp = 16 * nt + li;
      const float qk = q_l[comp], lwk = lw_l[comp];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int row = 16 * t + 4 * kq + r;
        if (row < n) {
          const float4 cf = sch[2 * (a + 1 + row) + 1];
          ps[(size_t)row * cp + comp] = kLog2e * fmaf(cf.x, acc[r], fmaf(-cf.y, qk, lwk));
        }
      }
    }
  }
  lds_barrier();
  for (int row = wave; row < n; row += nw) {
    float* pr = ps + (size_t)row * cp;
    float mx = -INFINITY;
    for (int k = lane; k < C; k += 64) mx = fmaxf(mx, pr[k]);
    mx = wave_max(mx);
    float sum = 0.f;
    for (int k = lane; k < l.C16; k += 64) {
      // components past C weigh nothing, nor do weights below 2^-kCertZeroGap of the largest (gmm_cert.h)
      const float p = (k < C && !(pr[k] - mx < -kCertZeroGap)) ? __builtin_amdgcn_exp2f(pr[k] - mx) : 0.f;
      pr[k] = p;
      sum += p;
    }
    sum = wave_sum(sum);
    if (lane == 0) s_sc[row] = sch[2 * (a + 1 + row) + 1].w / sum;
  }
  lds_barrier();
}

template <int MASK>
__device__ __forceinline__ float dpp(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), MASK, 0xf, 0xf, true));
}
// Sum and maximum over groups of n (1, 2, 4, 8, 16) neighbouring lanes, in every lane (the steps of wave_sum).
__device__ __forceinline__ float group_sum(float v, int n) {
  if (n > 1) v += dpp<0xB1>(v);
  if (n > 2) v += dpp<0x4E>(v);
  if (n > 4) v += dpp<0x141>(v);
  if (n > 8) v += dpp<0x140>(v);
  return v;
}
__device__ __forceinline__ float group_max(float v, int n) {
  if (n > 1) v = fmaxf(v, dpp<0xB1>(v));
  if (n > 2) v = fmaxf(v, dpp<0x4E>(v));
  if (n > 4) v = fmaxf(v, dpp<0x141>(v));
  if (n > 8) v = fmaxf(v, dpp<0x140>(v));
  return v;
}
__device__ __forceinline__ float lane_value(float v, int lane) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), lane));
}
// Sums and maxima of a value over the four quarters of a wavefront that hold the same lane % 16, in every lane.
__device__ __forceinline__ float quarters_sum(float v) {   // (0 + 1) + (2 + 3)
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  const float u = __uint_as_float(r[0]) + __uint_as_float(r[1]);
  const auto h = __builtin_amdgcn_permlane32_swap(__float_as_uint(u), __float_as_uint(u), false, false);
  return __uint_as_float(h[0]) + __uint_as_float(h[1]);
}
__device__ __forceinline__ float quarters_max(float v) {
  const auto h = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  const float u = fmaxf(__uint_as_float(h[0]), __uint_as_float(h[1]));
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(u), __float_as_uint(u), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float zero_cut_exp2(float x) {   // 2^x, 0 below the zero cut (gmm_cert.h)
  return x < -kCertZeroGap ? 0.f : __builtin_amdgcn_exp2f(x);
}

// Float offset of a lane's row in an array of rows of `pitch`, as a value of its own: the compiler would carry the product into
// every address derived from it (a 32-bit product takes a SIMD as long as four additions).
__device__ __forceinline__ int row_offset(int row, int pitch) {
  int o = __mul24(row, pitch);
  asm("" : "+v"(o));
  return o;
}

// What a lane adds up of n values of a row: numbers lane, lane + 64, ... in order.  (Every lane reads, four values at a time: a
// loop as long as a lane has values would wait for each.)
__device__ __forceinline__ float lane_part(const float* row, int n, int lane) {
  float sum = 0.f;
  for (int k0 = 0; k0 < n; k0 += 256) {
    float v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) v[u] = row[min(k0 + 64 * u + lane, n - 1)];
#pragma unroll
    for (int u = 0; u < 4; ++u) sum += k0 + 64 * u + lane < n ? v[u] : 0.f;
  }
  return sum;
}

// A logit in base-2 units (for the hardware exp2), rounded before anything is taken from it, whether it stays in a register or
// passes through LDS.
__device__ __forceinline__ float logit2(float c, float dot, float q, float musq, float logw) {
#pragma clang fp contract(off)
  constexpr float kLog2e = 1.4426950408889634f;
  return kLog2e * fmaf(c, dot, fmaf(-q, musq, logw));
}

}  // namespace

// NW wavefronts; sums over components in PARTS parts
template <int NW, int PARTS>
__global__ __launch_bounds__(64 * NW) void gmm_chain_sample_kernel(
    int K, int L, int d, int C, Key key, const float* __restrict__ c_x,
    const float* __restrict__ c_0, const float* __restrict__ sigma, const int32_t* __restrict__ tau,
    const float4* __restrict__ coef_tau, const float* __restrict__ means, const float* __restrict__ musq,
    const float* __restrict__ log_w, const float* __restrict__ y0, float* __restrict__ traj,
    int32_t* __restrict__ rounds, RoundsOut out, int adaptive, int ring) {
  extern __shared__ __attribute__((aligned(16))) float lds[];
  __shared__ float s_logu[128], s_dot[64], s_vv[64], s_sc[64], s_m[16];
  __shared__ int s_bit[64];

  const int c = blockIdx.x;
  constexpr int nw = NW, parts = PARTS, nthreads = 64 * NW;
  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int li = lane & 15, kq = lane >> 4;
  const ChainLayout l = chain_layout(C, d, L, K, ring);
  const int dp = l.dp, nblk = l.nblk;
  const bool vec = (d & 3) == 0;
  float* m_l = lds + l.m;
  float* q_l = lds + l.q;
  float* lw_l = lds + l.lw;
  float* ps = lds + l.ps;
  float* part = lds + l.part;
  float* yh = lds + l.yh;
  float* x0 = lds + l.x0;
  float* xi_l = lds + l.xi;
  // The schedule and the denoiser's per-step coefficients: a round would otherwise start with a chain
  // of dependent global loads (tau_a, then its coefficients) and reload the tables step by step.
  const float4* sch = reinterpret_cast<const float4*>(lds + l.sch);
  for (int i = tid; i < K; i += nthreads) {
    float4* e = reinterpret_cast<float4*>(lds + l.sch) + 2 * i;
    e[0] = make_float4(c_x[i], c_0[i], sigma[i], 0.f);
    e[1] = coef_tau[tau[i]];
  }
  for (int t = tid; t < l.C16 * dp; t += nthreads) {
    const int k = t / dp, j = t - k * dp;
    m_l[t] = (k < C && j < d) ? means[(int64_t)k * d + j] : 0.f;
  }
  for (int t = tid; t < l.C16; t += nthreads) {
    q_l[t] = (t < C) ? musq[t] : 0.f;
    lw_l[t] = (t < C) ? log_w[t] : 0.f;
  }
  // everything between the softmax scratch and the schedule starts as zero: the padding of the rows is
  // multiplied (by zero mixture entries) on the matrix cores and must be finite
  for (size_t t = l.ps + tid; t < l.sch; t += nthreads) lds[t] = 0.f;
  lds_barrier();
  {  // y_0 (Alg. 1: given, or drawn from N(0, I))
    float* row0 = traj + (int64_t)c * (K + 1) * d;
    for (int blk = tid; blk < nblk; blk += nthreads) {
      const float4 v = y0 ? load4(y0 + (int64_t)c * d, blk, d, vec) : normal4(key, (uint32_t)c, 0u, (uint32_t)blk);
      store4(row0, blk, d, vec, v);
      *reinterpret_cast<float4*>(yh + 4 * blk) = v;
    }
  }
  // Noise and log u of steps first .. last - 1 into the ring, by wavefronts w0 .. nw - 1: a lane per block of a step's coordinates,
  // several steps a wavefront where they are few.  (at: ring row of step `from`)
  int bshift = 0;
  while (bshift < 6 && (1 << bshift) < nblk) ++bshift;
  auto make_noise = [&](int w0, int first, int last, int from, int at) {
    const int per = 64 >> bshift, sub = lane >> bshift;
    for (int i0 = first + (wave - w0) * per; i0 < last; i0 += (nw - w0) * per) {
      const int i = i0 + sub;
      if (i >= last) continue;
      int row = at + i - from;
      if (row >= ring) row -= ring;
      for (int blk = lane & ((1 << bshift) - 1); blk < nblk; blk += 64)
        *reinterpret_cast<float4*>(xi_l + (size_t)row * dp + 4 * blk) = normal4(key, (uint32_t)c, (uint32_t)(i + 1), (uint32_t)blk);
      if ((lane & ((1 << bshift) - 1)) == 0) s_logu[row] = logf(uniform1(key, (uint32_t)c, (uint32_t)(i + 1)));
    }
  };
  // wavefronts whose threads hold a coordinate each (all, if there are more coordinates than threads); the others of
  // them make the noise of later steps while those draft
  const int ncw = min(nw, (l.d16 + 63) >> 6);
  lds_barrier();
  // what a wavefront reads of the mixture twice a round: its tile of components for the logits of y_a and of the window (64
  // coordinates of component li)
  int tw = 0, nt = wave;   // tile of rows and of components (an integer division is some hundred cycles)
  for (; nt >= l.C16 >> 4; nt -= l.C16 >> 4) ++tw;
  const float* mtile = m_l + (size_t)(16 * nt + li) * dp + 4 * kq;
  float4 mrow[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) mrow[i] = 16 * i < l.d16 ? *reinterpret_cast<const float4*>(mtile + 16 * i) : make_float4(0.f, 0.f, 0.f, 0.f);
  const float4 qv = lds4(q_l, 4 * nt + kq), wv = lds4(lw_l, 4 * nt + kq);
  const float qc = q_l[16 * nt + li], wc = lw_l[16 * nt + li];

  int a = 0, R = 0;
  int at = 0;          // ring row of step a
  int made = 0;        // steps whose noise has been made
  int wstate = 4 * L;  // window controller (device_util.h); without it every window is L
  const ChainLayout l_all = l;
  while (a < K) {
    // Sizes the compiler may not know to be the same each round: every address of a round is a sum and a product of these, and
    // kept across rounds they are far more than there are registers.
    ChainLayout l = l_all;
    asm volatile("" : "+s"(l.d16), "+s"(l.dp), "+s"(l.C16), "+s"(l.cp), "+s"(l.tr), "+s"(l.nblk));
    const int dp = l.dp, cp = l.cp, nblk = l.nblk, NT = l.C16 >> 4;
    const int w = min(adaptive ? window_of(wstate, L) : L, K - a);
    const float4 cf0 = sch[2 * a + 1];
    // A. what the window still lacks of its noise, and the model at y_a: a tile of 16 components per wavefront, then a
    // wavefront per part of the sum over components
    if (made < a + w) {
      make_noise(0, made, a + w, a, at);
      made = a + w;
    }
    {
      float mrun = -INFINITY;
      for (int t = wave; t < NT; t += nw) {
        // lane: component li of the tile, every fourth block of coordinates (16 lanes then read 16 bank groups)
        const int comp = 16 * t + li;
        const float* mk = m_l + row_offset(comp, dp);
        float4 xv[4];
        float dot = 0.f;
#pragma unroll
        for (int i = 0; i < 4; ++i) xv[i] = lds4(yh, min(4 * i, (l.d16 >> 2) - 4) + kq);
        if (t == wave) {
#pragma unroll
          for (int i = 0; i < 4; ++i)
            dot = fmaf(xv[i].x, mrow[i].x, fmaf(xv[i].y, mrow[i].y, fmaf(xv[i].z, mrow[i].z, fmaf(xv[i].w, mrow[i].w, dot))));
        }
#pragma unroll 4
        for (int b = (t == wave ? 16 : 0) + kq; b < l.d16 >> 2; b += 4) {
          const float4 x = lds4(yh, b), mv = lds4(mk, b);
          dot = fmaf(x.x, mv.x, fmaf(x.y, mv.y, fmaf(x.z, mv.z, fmaf(x.w, mv.w, dot))));
        }
        dot = quarters_sum(dot);
        const float lg = comp < C ? (t == wave ? logit2(cf0.x, dot, cf0.y, qc, wc) : logit2(cf0.x, dot, cf0.y, q_l[comp], lw_l[comp])) : -INFINITY;
        if (kq == 0) ps[comp] = lg;
        mrun = fmaxf(mrun, lg);
      }
      mrun = group_max(mrun, 16);
      if (lane == 0) s_m[wave] = mrun;
    }
    lds_barrier();
    if (wave < parts) {
      // part g takes the component quads g, g + parts, ..., four of them at a time: lane i has the weight of number i % 4 of quad i / 4
      for (int j0 = 0; j0 < l.d16; j0 += 64) {   // (every lane stays in: weights are read from lanes without a coordinate too)
        const int j = min(j0 + lane, l.d16 - 1);
        float a0 = 0.f, a1 = 0.f, a2 = 0.f, a3 = 0.f;
        for (int q0 = wave; 4 * q0 < l.C16; q0 += 4 * parts) {
          const int comp = 4 * (q0 + parts * (li >> 2)) + (li & 3);
          const float lg = ps[min(comp, l.C16 - 1)], sm = s_m[min(li, nw - 1)];
          float v[16];
#pragma unroll
          for (int i = 0; i < 16; ++i) v[i] = m_l[(min(4 * (q0 + parts * (i >> 2)), l.C16 - 4) + (i & 3)) * dp + j];
          __builtin_amdgcn_sched_barrier(0);
          float p = zero_cut_exp2(lg - group_max(sm, 16));
          p = comp < l.C16 ? p : 0.f;
          if (j0 == 0 && lane < 16 && comp < l.C16) ps[cp + comp] = p;   // (for their sum)
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            a0 = fmaf(lane_value(p, 4 * u), v[4 * u], a0);
            a1 = fmaf(lane_value(p, 4 * u + 1), v[4 * u + 1], a1);
            a2 = fmaf(lane_value(p, 4 * u + 2), v[4 * u + 2], a2);
            a3 = fmaf(lane_value(p, 4 * u + 3), v[4 * u + 3], a3);
          }
        }
        if (j0 + lane < l.d16) part[wave * dp + j] = (a0 + a1) + (a2 + a3);
      }
    }
    lds_barrier();
    // B. the parts put together, and the draft (proposal loop of Alg. 1): a thread per coordinate
    if (wave < ncw) {
      __builtin_amdgcn_s_setprio(3);   // (the wavefronts that make noise share its SIMD)
      const float sum = wave_sum(lane_part(ps + cp, l.C16, lane));
      const float sc = cf0.w / sum;
      for (int j0 = 64 * wave; j0 < l.d16; j0 += 64 * ncw) {
        const int j = min(j0 + lane, l.d16 - 1);
        const bool mine = j0 + lane < l.d16;
        float pt[parts];
#pragma unroll
        for (int g = 0; g < parts; ++g) pt[g] = part[g * dp + j];
        float acc = pt[0];
#pragma unroll
        for (int g = 1; g < parts; ++g) acc += pt[g];
        float y = yh[j];
        const float g0 = j < d ? fmaf(cf0.z, y, sc * acc) : 0.f;
        if (mine) x0[j] = g0;
        float* yo = yh + dp + j;
        struct Step {
          float4 tab;
          float xi;
        };
        auto fetch = [&](int k) {
          const int kk = min(k, w - 1);
          int r = at + kk;
          if (r >= ring) r -= ring;
          return Step{sch[2 * (a + kk)], xi_l[r * dp + j]};
        };
        auto step = [&](int k, const Step& q) {
          y = fmaf(q.tab.z, q.xi, fmaf(q.tab.x, y, q.tab.y * g0));
          if (mine) yo[k * dp] = y;
        };
        Step now[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) now[u] = fetch(u);
        int k0 = 0;
        for (; k0 + 4 <= w; k0 += 4) {   // the next four are on their way
          Step nx[4];
#pragma unroll
          for (int u = 0; u < 4; ++u) nx[u] = fetch(k0 + 4 + u);
#pragma unroll
          for (int u = 0; u < 4; ++u) step(k0 + u, now[u]);
#pragma unroll
          for (int u = 0; u < 4; ++u) now[u] = nx[u];
        }
#pragma unroll
        for (int u = 0; u < 3; ++u)
          if (k0 + u < w) step(k0 + u, now[u]);
      }
      __builtin_amdgcn_s_setprio(0);
    } else if (made < min(K, a + ring)) {
      make_noise(ncw, made, min(K, a + ring), a, at);
    }
    if (ncw < nw) made = max(made, min(K, a + ring));
    lds_barrier();
    // C. verify (target-mean model values at the drafted points; slot 0 reuses x0a) and Alg. 3's test, a wavefront per slot
    const int n = w - 1, T = (n + 15) >> 4;
    if (n > 0) {
      const bool direct = T * NT <= nw;
      int KS = 1;
      if (direct) {
        // logits^T = M X^T: a wavefront per tile of 16 components x 16 rows.  A lane ends up with four components of one
        // row, keeps them, and the softmax weights go to LDS once the rows' maxima are known.
        float lg[4];
        const int row = 16 * tw + li;
        if (wave < T * NT) {
          const int rc = min(row, n - 1);
          const float* xa = yh + row_offset(1 + rc, dp) + 4 * kq;
          const float4 cf = sch[2 * (a + 1 + rc) + 1];
          float4 xv[4];
#pragma unroll
          for (int i = 0; i < 4; ++i) xv[i] = *reinterpret_cast<const float4*>(xa + min(16 * i, l.d16 - 16));
          v4f_c acc = {0.f, 0.f, 0.f, 0.f};
          auto product = [&](const float4& m, const float4& x) {
            acc = __builtin_amdgcn_mfma_f32_16x16x4f32(m.x, x.x, acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_16x16x4f32(m.y, x.y, acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_16x16x4f32(m.z, x.z, acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_16x16x4f32(m.w, x.w, acc, 0, 0, 0);
          };
#pragma unroll
          for (int i = 0; i < 4; ++i)
            if (16 * i < l.d16) product(mrow[i], xv[i]);
#pragma unroll 4
          for (int s = 64; s < l.d16; s += 16)
            product(*reinterpret_cast<const float4*>(mtile + s), *reinterpret_cast<const float4*>(xa + s));
          const float qa[4] = {qv.x, qv.y, qv.z, qv.w}, wa[4] = {wv.x, wv.y, wv.z, wv.w};
          float mx = -INFINITY;
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            lg[r] = 16 * nt + 4 * kq + r < C ? logit2(cf.x, acc[r], cf.y, qa[r], wa[r]) : -INFINITY;
            mx = fmaxf(mx, lg[r]);
          }
          mx = quarters_max(mx);
          if (kq == 0) part[wave * 16 + li] = mx;   // (the partial sums' place: they come later)
        }
        lds_barrier();
        if (wave < T * NT) {
          float mx = -INFINITY;
          for (int q0 = 0; q0 < NT; q0 += 8) {
            float v[8];
#pragma unroll
            for (int q = 0; q < 8; ++q) v[q] = part[(tw * NT + min(q0 + q, NT - 1)) * 16 + li];
#pragma unroll
            for (int q = 0; q < 8; ++q) mx = fmaxf(mx, v[q]);
          }
          float4 p;
          p.x = zero_cut_exp2(lg[0] - mx);
          p.y = zero_cut_exp2(lg[1] - mx);
          p.z = zero_cut_exp2(lg[2] - mx);
          p.w = zero_cut_exp2(lg[3] - mx);
          *reinterpret_cast<float4*>(ps + row_offset(row, cp) + 16 * nt + 4 * kq) = p;
        }
        lds_barrier();
      } else {
        softmax_tiles(n, T, a, l, C, m_l, q_l, lw_l, ps, yh, sch, s_sc, wave, nw, lane);
      }
      {
        // out = P M: the sum over components of a (16 rows x 16 coordinates) tile is cut into KS pieces so that every wavefront
        // has one; the pieces land in LDS and are added in order
        const int CT = l.d16 >> 4;
        int lks = 0;
        while ((2 << lks) <= kChainSplits && (T * CT << lks) * 2 <= parts && (NT & ((2 << lks) - 1)) == 0) ++lks;
        KS = 1 << lks;
        const int steps = NT >> lks;
        for (int item = wave; item < T * CT * KS; item += nw) {
          const int ks = item & (KS - 1);
          int t = 0, ct = item >> lks;
          for (; ct >= CT; ct -= CT) ++t;
          const float* pa = ps + row_offset(min(16 * t + li, n - 1), cp) + 4 * kq + 16 * ks * steps;
          const float* mb = m_l + row_offset(4 * kq, dp) + 16 * ks * steps * dp + 16 * ct + li;
          v4f_c acc = {0.f, 0.f, 0.f, 0.f};
          // four steps at a time: their operands are requested together and held ahead of the products
          auto some = [&](int s0, auto count) {
            float4 av[count];
            float b[count][4];
#pragma unroll
            for (int s = 0; s < count; ++s) {
              av[s] = *reinterpret_cast<const float4*>(pa + 16 * (s0 + s));
#pragma unroll
              for (int e = 0; e < 4; ++e, mb += dp) b[s][e] = *mb;
              mb += 12 * dp;
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int s = 0; s < count; ++s) {
              acc = __builtin_amdgcn_mfma_f32_16x16x4f32(av[s].x, b[s][0], acc, 0, 0, 0);
              acc = __builtin_amdgcn_mfma_f32_16x16x4f32(av[s].y, b[s][1], acc, 0, 0, 0);
              acc = __builtin_amdgcn_mfma_f32_16x16x4f32(av[s].z, b[s][2], acc, 0, 0, 0);
              acc = __builtin_amdgcn_mfma_f32_16x16x4f32(av[s].w, b[s][3], acc, 0, 0, 0);
            }
          };
          int s0 = 0;
          for (; s0 + 4 <= steps; s0 += 4) some(s0, std::integral_constant<int, 4>{});
          for (; s0 < steps; ++s0) some(s0, std::integral_constant<int, 1>{});
          float* o = part + row_offset(16 * t + 4 * kq, dp) + ks * l.tr * dp + 16 * ct + li;   // (rows past the last one too)
#pragma unroll
          for (int r = 0; r < 4; ++r, o += dp) *o = acc[r];
        }
      }
      if (direct)
        for (int r = wave; r < n; r += nw) {
          const float sum = wave_sum(lane_part(ps + r * cp, l.C16, lane));
          if (lane == 0) s_sc[r] = sch[2 * (a + 1 + r) + 1].w / sum;
        }
      lds_barrier();
      for (int k = 1 + wave; k < w; k += nw) {
        const float4 cf = sch[2 * (a + k) + 1], tab = sch[2 * (a + k)];
        int xr = at + k;
        if (xr >= ring) xr -= ring;
        float dot = 0.f, vv = 0.f;
        const float sck = s_sc[k - 1];
        for (int blk = lane; blk < nblk; blk += 64) {
          float4 pt[kChainSplits];
#pragma unroll
          for (int ks = 0; ks < kChainSplits; ++ks) pt[ks] = lds4(part + (min(ks, KS - 1) * l.tr + k - 1) * dp, blk);
          const float4 y = lds4(yh + k * dp, blk), ga = lds4(x0, blk), xi = lds4(xi_l + xr * dp, blk);
          float4 sum = pt[0], v;
#pragma unroll
          for (int ks = 1; ks < kChainSplits; ++ks) {
            sum.x += ks < KS ? pt[ks].x : 0.f;
            sum.y += ks < KS ? pt[ks].y : 0.f;
            sum.z += ks < KS ? pt[ks].z : 0.f;
            sum.w += ks < KS ? pt[ks].w : 0.f;
          }
          v.x = fmaf(cf.z, y.x, sck * sum.x);
          v.y = 4 * blk + 1 < d ? fmaf(cf.z, y.y, sck * sum.y) : 0.f;
          v.z = 4 * blk + 2 < d ? fmaf(cf.z, y.z, sck * sum.z) : 0.f;
          v.w = 4 * blk + 3 < d ? fmaf(cf.z, y.w, sck * sum.w) : 0.f;
          *reinterpret_cast<float4*>(x0 + k * dp + 4 * blk) = v;
          const float dx = ga.x - v.x, dy = ga.y - v.y, dz = ga.z - v.z, dw = ga.w - v.w;
          dot = fmaf(dx, xi.x, dot);
          dot = fmaf(dy, xi.y, dot);
          dot = fmaf(dz, xi.z, dot);
          dot = fmaf(dw, xi.w, dot);
          vv = fmaf(dx, dx, vv);
          vv = fmaf(dy, dy, vv);
          vv = fmaf(dz, dz, vv);
          vv = fmaf(dw, dw, vv);
        }
        dot = wave_sum(dot);
        vv = wave_sum(vv);
        if (lane == 0) {
          int bit = 0;  // sigma == 0 rejects
          if (tab.z > 0.f) {
            const float vxi = tab.y * dot;
            const float v2 = tab.y * tab.y * vv;
            bit = (s_logu[xr] <= -(vxi / tab.z + v2 / (2.0f * tab.z * tab.z))) ? 1 : 0;
          }
          s_bit[k] = bit;
          s_dot[k] = dot;
          s_vv[k] = vv;
        }
      }
      lds_barrier();
    }
    // Alg. 2: accepted prefix = trailing ones of the ballot (slot 0 is accepted by construction), by every wavefront
    const unsigned long long inv = ~__ballot((lane >= 1 && lane < w) ? s_bit[lane] : 1);
    const int n_acc = min(inv ? (__ffsll((long long)inv) - 1) : 64, w);
    // reject branch of Alg. 3 (reflection) and the advance rule of Alg. 1.  The rows the chain keeps go to the trajectory, one
    // to a wavefront; y_{a_next} becomes row 0 of the proposal samples
    const int src = n_acc < w ? n_acc + 1 : w;
    float* rows = traj + ((int64_t)c * (K + 1) + a) * d;
    for (int k = nw - wave; k < src; k += nw)   // (the first wavefronts have the last row to do)
      for (int j = lane; j < d; j += 64) rows[(int64_t)k * d + j] = yh[k * dp + j];
    if (wave < ncw) {
      float coef = 0.f;
      if (n_acc < w) {
        const float4 tab = sch[2 * (a + n_acc)];
        const float dot = s_dot[n_acc], vv = s_vv[n_acc];
        coef = (vv > 0.f) ? (tab.y + 2.0f * tab.z * dot / vv) : 0.f;
      }
      for (int j = tid; j < l.d16; j += 64 * ncw) {
        float y = yh[src * dp + j];
        if (n_acc < w) y = fmaf(-(x0[j] - x0[n_acc * dp + j]), coef, y);
        if (j < d) rows[(int64_t)src * d + j] = y;
        yh[j] = y;
      }
    }
    wstate = window_next(wstate, w, n_acc);
    at += src;
    if (at >= ring) at -= ring;
    a += src;
    ++R;
    lds_barrier();
  }
  if (tid == 0) {
    if (rounds) rounds[c] = R;
    out.report(R, gridDim.x);
  }
}

// ----------------------------------------------------------------------------
// Mixtures of a few numbers: a chain is one wavefront, and nothing in its loop is shared.
//
// What bounds the kernel above on such a shape is its stages, each an LDS round trip and a barrier of mostly idle
// wavefronts (9 us a round at d 2, C 4, L 8, of which the arithmetic is a few hundred cycles).  Here a slot of
// the window is a lane -- G = 64 / (slots, rounded up to a power of two) lanes, which share its components -- so the model
// value of every slot, its accept test and the scan over the slots are register arithmetic, and the only barrier is the
// one behind the set-up.  The noise of a chain depends on its steps only: the set-up generates it, and log u, for all K
// steps with every thread of the workgroup (four wavefronts at least; those without a chain then leave).  A round is
//   x0a by every slot's lanes alike; the draft by a lane per coordinate; the verify call, a slot per lane; the test; one
//   ballot; the reflection by the lanes of the coordinates, which keep y_a in a register; the rows the chain keeps go to
//   the trajectory (those behind the first rejection would be written again by the next round).
// A lane's first component, and often its only one, stays in registers, the walk's operands are asked for ahead of x0a, and no
// value is picked from a row by an index (which the compiler makes a trip through scratch memory of).
// Measured, microseconds a sample with its launch and the wait for it, a workgroup (as it was then) / a wavefront a chain / without
// those trips, (d, C, L, K, chains): (2, 4, 8, 100, 8) 138 / 53 / 47, K = 1000 922 / 269 / 230; (4, 16, 16, 200, 64) 217 / 96 / 88;
// (12, 16, 10, 200, 8) 237 / 160 / 149; (2, 4, 8, 100, 20000) 1878 / 785 / 624.
// LDS operations of a wavefront complete in order; wave_lds_fence keeps the compiler to it.
// ----------------------------------------------------------------------------
namespace {

constexpr int kWaveBlocks = 4;   // d <= 16

struct WaveLayout {
  int dq, lanes, per_lane;     // floats of a padded row; lanes a slot's components are shared by; components a lane has
  size_t m, ql, sch, chain;    // offsets in floats; first chain's part
  size_t xi, logu, yh, ps, chain_floats;   // offsets within a chain's part; its size
};

__host__ __device__ inline WaveLayout wave_layout(int C, int d, int L, int K) {
  WaveLayout l;
  l.dq = (d + 3) & ~3;
  int slots = 4;
  while (slots < L) slots *= 2;
  l.lanes = 64 / slots;
  l.per_lane = (C + l.lanes - 1) / l.lanes;
  l.m = 0;                                  // [C][dq] means, columns past d zero
  l.sch = l.m + (size_t)C * l.dq;           // [K][8] (c_x, c_0, sigma, -, kappa, gamma, cx, cm) of step i
  l.ql = l.sch + (size_t)K * 8;             // [C][2] |mu|^2, log w
  l.chain = l.ql + (((size_t)C * 2 + 3) & ~(size_t)3);
  l.xi = 0;                                 // [K][dq] xi_{i+1}, columns past d zero
  l.yh = l.xi + (size_t)K * l.dq;           // [L+1][dq] yhat_a (= y_a) .. yhat_b
  l.ps = l.yh + (size_t)(L + 1) * l.dq;     // [per_lane][64] logits
  l.logu = l.ps + (size_t)l.per_lane * 64;  // [K] log u_{i+1}
  l.chain_floats = l.logu + (((size_t)K + 3) & ~(size_t)3);
  return l;
}

__device__ __forceinline__ void wave_lds_fence() { asm volatile("" ::: "memory"); }

// component e (0 .. 4 DB - 1, a lane's own) of a row in registers.  (The compiler makes an indexed read of scratch memory of these
// selections unless each is a value of its own: a store and a load through the caches, a few hundred cycles.)
template <int DB>
__device__ __forceinline__ float pick(const float (&v)[4 * DB], int e) {
  float r = v[0];
#pragma unroll
  for (int j = 1; j < 4 * DB; ++j) {
    r = e == j ? v[j] : r;
    asm("" : "+v"(r));
  }
  return r;
}

}  // namespace

// DB: blocks of four coordinates in a row.  Chains blockIdx.x cpw .. + cpw - 1, a wavefront each; blockDim.x is a multiple of
// 64 and at least 64 cpw.
template <int DB>
__global__ __launch_bounds__(512) void gmm_wave_sample_kernel(
    int B, int K, int L, int d, int C, int cpw, Key key, const float* __restrict__ c_x, const float* __restrict__ c_0,
    const float* __restrict__ sigma, const int32_t* __restrict__ tau, const float4* __restrict__ coef_tau,
    const float* __restrict__ means, const float* __restrict__ musq, const float* __restrict__ log_w,
    const float* __restrict__ y0, float* __restrict__ traj, int32_t* __restrict__ rounds, RoundsOut rout, int adaptive) {
  constexpr int DQ = 4 * DB;
  extern __shared__ __attribute__((aligned(16))) float lds[];
  const WaveLayout l = wave_layout(C, d, L, K);
  const int tid = threadIdx.x, nthreads = blockDim.x;
  const int c0 = blockIdx.x * cpw, chains = min(cpw, B - c0);
  for (int i = tid; i < K; i += nthreads) {
    float4* e = reinterpret_cast<float4*>(lds + l.sch) + 2 * i;
    e[0] = make_float4(c_x[i], c_0[i], sigma[i], 0.f);
    e[1] = coef_tau[tau[i]];
  }
  for (int t = tid; t < C * DQ; t += nthreads) {
    const int k = t / DQ, j = t % DQ;
    lds[l.m + t] = j < d ? means[(int64_t)k * d + j] : 0.f;
  }
  for (int k = tid; k < C; k += nthreads) {
    lds[l.ql + 2 * k] = musq[k];
    lds[l.ql + 2 * k + 1] = log_w[k];
  }
  for (int cc = 0; cc < chains; ++cc) {
    float* mine = lds + l.chain + cc * l.chain_floats;
    for (int t = tid; t < K * DB; t += nthreads) {
      const int i = t / DB, blk = t % DB;
      float4 v = normal4(key, (uint32_t)(c0 + cc), (uint32_t)(i + 1), (uint32_t)blk);
      if (4 * blk + 1 >= d) v.y = 0.f;
      if (4 * blk + 2 >= d) v.z = 0.f;
      if (4 * blk + 3 >= d) v.w = 0.f;
      *reinterpret_cast<float4*>(mine + l.xi + 4 * t) = v;
    }
    for (int i = tid; i < K; i += nthreads) mine[l.logu + i] = logf(uniform1(key, (uint32_t)(c0 + cc), (uint32_t)(i + 1)));
  }
  __syncthreads();
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  if (wave >= chains) return;

  const int c = c0 + wave;
  float* mine = lds + l.chain + wave * l.chain_floats;
  const float* m_l = lds + l.m;
  const float* xi_l = mine + l.xi;
  const float* logu = mine + l.logu;
  float* yh = mine + l.yh;
  float* ps = mine + l.ps + lane;
  const float2* ql = reinterpret_cast<const float2*>(lds + l.ql);
  const float4* sch = reinterpret_cast<const float4*>(lds + l.sch);
  const int gshift = __builtin_ctz((unsigned)l.lanes), G = 1 << gshift, slot = lane >> gshift, part = lane & (G - 1);

  // the lane's first component, and often its only one, stays in registers
  float m0[DQ];
#pragma unroll
  for (int b = 0; b < DB; ++b) {
    const float4 t = *reinterpret_cast<const float4*>(m_l + min(part, C - 1) * DQ + 4 * b);
    m0[4 * b] = t.x;
    m0[4 * b + 1] = t.y;
    m0[4 * b + 2] = t.z;
    m0[4 * b + 3] = t.w;
  }
  const float2 ql0 = ql[min(part, C - 1)];

  // D(x, .) with the step's coefficients cf, in every lane of the slot
  auto model = [&](const float (&x)[DQ], float4 cf, float (&out)[DQ]) {
    float dot0 = 0.f;
#pragma unroll
    for (int b = 0; b < DB; ++b)
      dot0 = fmaf(x[4 * b], m0[4 * b], fmaf(x[4 * b + 1], m0[4 * b + 1], fmaf(x[4 * b + 2], m0[4 * b + 2], fmaf(x[4 * b + 3], m0[4 * b + 3], dot0))));
    const float lg0 = part < C ? logit2(cf.x, dot0, cf.y, ql0.x, ql0.y) : -INFINITY;
    float mx = lg0;
    int j = 1;
    for (int k = part + G; k < C; k += G, ++j) {
      float dot = 0.f;
#pragma unroll
      for (int b = 0; b < DB; ++b) {
        const float4 mv = *reinterpret_cast<const float4*>(m_l + k * DQ + 4 * b);
        dot = fmaf(x[4 * b], mv.x, fmaf(x[4 * b + 1], mv.y, fmaf(x[4 * b + 2], mv.z, fmaf(x[4 * b + 3], mv.w, dot))));
      }
      const float2 q = ql[k];
      const float lg = logit2(cf.x, dot, cf.y, q.x, q.y);
      ps[64 * j] = lg;
      mx = fmaxf(mx, lg);
    }
    mx = group_max(mx, G);
    const float p0 = zero_cut_exp2(lg0 - mx);
    float sum = p0, acc[DQ];
#pragma unroll
    for (int e = 0; e < DQ; ++e) acc[e] = p0 * m0[e];
    j = 1;
    for (int k = part + G; k < C; k += G, ++j) {
      const float p = zero_cut_exp2(ps[64 * j] - mx);
      sum += p;
#pragma unroll
      for (int b = 0; b < DB; ++b) {
        const float4 mv = *reinterpret_cast<const float4*>(m_l + k * DQ + 4 * b);
        acc[4 * b] = fmaf(p, mv.x, acc[4 * b]);
        acc[4 * b + 1] = fmaf(p, mv.y, acc[4 * b + 1]);
        acc[4 * b + 2] = fmaf(p, mv.z, acc[4 * b + 2]);
        acc[4 * b + 3] = fmaf(p, mv.w, acc[4 * b + 3]);
      }
    }
    const float sc = cf.w / group_sum(sum, G);
#pragma unroll
    for (int e = 0; e < DQ; ++e) out[e] = e < d ? fmaf(cf.z, x[e], sc * group_sum(acc[e], G)) : 0.f;
  };
  auto row = [&](const float* p, float (&v)[DQ]) {
#pragma unroll
    for (int b = 0; b < DB; ++b) {
      const float4 t = *reinterpret_cast<const float4*>(p + 4 * b);
      v[4 * b] = t.x;
      v[4 * b + 1] = t.y;
      v[4 * b + 2] = t.z;
      v[4 * b + 3] = t.w;
    }
  };

  float* out_row = traj + (int64_t)c * (K + 1) * d;
  // lane e < DQ: coordinate e of y_a (0 past d)
  float y = 0.f;
  if (lane < d) {
    if (y0) {
      y = y0[(int64_t)c * d + lane];
    } else {
      const float4 v = normal4(key, (uint32_t)c, 0u, (uint32_t)(lane >> 2));
      y = (lane & 3) == 0 ? v.x : (lane & 3) == 1 ? v.y : (lane & 3) == 2 ? v.z : v.w;
    }
    out_row[lane] = y;
  }
  const int e = min(lane, DQ - 1);
  int a = 0, R = 0;
  int wstate = 4 * L;
  while (a < K) {
    const int w = min(adaptive ? window_of(wstate, L) : L, K - a);
    if (lane < DQ) yh[lane] = y;
    wave_lds_fence();
    float x[DQ], ga[DQ], gk[DQ];
    struct Step {
      float4 sc;
      float xi;
    };
    auto fetch = [&](int k) {
      const int i = a + min(k, w - 1);
      return Step{sch[2 * i], xi_l[i * DQ + e]};
    };
    Step now[4];   // (asked for ahead of the model value)
#pragma unroll
    for (int u = 0; u < 4; ++u) now[u] = fetch(u);
    row(yh, x);
    model(x, sch[2 * a + 1], ga);
    // draft: the lanes of the coordinates walk the window, operands of four steps at a time
    float v = y;
    const float g = pick<DB>(ga, e);
    auto step = [&](int k, const Step& q) {
      v = fmaf(q.sc.z, q.xi, fmaf(q.sc.x, v, q.sc.y * g));
      if (lane < DQ) yh[(k + 1) * DQ + lane] = v;
    };
    int k0 = 0;
    for (; k0 + 4 <= w; k0 += 4) {   // the next four are on their way
      Step nx[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) nx[u] = fetch(k0 + 4 + u);
#pragma unroll
      for (int u = 0; u < 4; ++u) step(k0 + u, now[u]);
#pragma unroll
      for (int u = 0; u < 4; ++u) now[u] = nx[u];
    }
#pragma unroll
    for (int u = 0; u < 3; ++u)
      if (k0 + u < w) step(k0 + u, now[u]);
    wave_lds_fence();
    // verify and test: slot 0 is accepted by construction, sigma == 0 rejects
    const int s = min(slot, w - 1), i = a + s;
    float dot = 0.f, vv = 0.f;
    bool bit = true;
    if (w > 1) {
      row(yh + s * DQ, x);
      model(x, sch[2 * i + 1], gk);
      float xi[DQ];
      row(xi_l + i * DQ, xi);
#pragma unroll
      for (int j = 0; j < DQ; ++j) {
        const float D = ga[j] - gk[j];
        dot = fmaf(D, xi[j], dot);
        vv = fmaf(D, D, vv);
      }
      const float4 sc = sch[2 * i];
      if (slot >= 1 && slot < w) {
        bit = false;
        if (sc.z > 0.f) {
          const float vxi = sc.y * dot, v2 = sc.y * sc.y * vv;
          bit = logu[i] <= -(vxi / sc.z + v2 / (2.0f * sc.z * sc.z));
        }
      }
    }
    const unsigned long long rejected = __ballot(!bit);
    const int lr = rejected ? __ffsll((long long)rejected) - 1 : 64;   // first lane of the first rejected slot
    const int n_acc = rejected ? lr >> gshift : w;
    int keep = w;   // rows y_{a+1} .. y_{a+keep} are final
    if (n_acc < w) {
      const float4 sc = sch[2 * (a + n_acc)];
      const float dr = lane_value(dot, lr), vr = lane_value(vv, lr);
      const float coef = (vr > 0.f) ? (sc.y + 2.0f * sc.z * dr / vr) : 0.f;
      float gr[DQ];
#pragma unroll
      for (int j = 0; j < DQ; ++j) gr[j] = lane_value(gk[j], lr);
      keep = n_acc + 1;
      y = fmaf(-(g - pick<DB>(gr, e)), coef, yh[keep * DQ + e]);
      if (lane < DQ) yh[keep * DQ + lane] = y;
    } else {
      y = v;
    }
    wave_lds_fence();
    float* dst = out_row + (int64_t)(a + 1) * d;
    for (int t = lane; t < keep * DQ; t += 64) {
      const int r = t / DQ, j = t % DQ;
      if (j < d) dst[(int64_t)r * d + j] = yh[DQ + t];
    }
    wave_lds_fence();
    wstate = window_next(wstate, w, n_acc);
    a += keep;
    ++R;
  }
  if (lane == 0) {
    if (rounds) rounds[c] = R;
    rout.report(R, B);
  }
}

namespace {

// Wavefronts per workgroup: enough for the tiles of the logits pass, within 4..16, and eight where the draft, a thread per coordinate,
// would leave no more than two of four to make the noise (microseconds a sample of K 200, 4 / 8 wavefronts: (300, 4, 8) 561 / 441,
// (240, 16, 8) 443 / 359, (200, 8, 4) 503 / 432, (128, 16, 16) 304 / 250, (128, 60, 4) 401 / 370).  Chains that share a CU take
// each other's slots instead: with more than 256 of them eight only where a row has more coordinates than four have threads ((100, 20,
// 12), 600 chains: 570 / 676; (300, 30, 4) at K 100, 300 chains: 766 / 659).  And the parts that sums over components are cut
// into, which are a wavefront's each but keep to fewer where the tiles are few (results do not depend on the wavefronts).
inline int chain_items(const asd_ctx* ctx) {
  const ChainLayout l = chain_layout(ctx->gmm->C, ctx->d, ctx->L, ctx->K, ctx->L);
  return (l.C16 / 16) * (l.tr / 16);
}
inline int chain_waves(int items, int d, int chains) {
  return items > 8 ? 16 : (items > 4 || d > (chains > 256 ? 240 : 100) ? 8 : 4);
}
inline int chain_parts(int items) { return items >= 16 ? 16 : (items >= 8 ? 8 : 4); }
// ring: steps the noise ring holds (L, or 2 L where that fits too: then the noise of later steps is made aside)
inline size_t chain_lds_bytes(const asd_ctx* ctx, int ring) {
  return sizeof(float) * chain_layout(ctx->gmm->C, ctx->d, ctx->L, ctx->K, ring).total;
}
inline bool chain_fits(const asd_ctx* ctx, int ring) { return chain_lds_bytes(ctx, ring) + 2048 <= 160 * 1024; }

}  // namespace

// How many chains share a workgroup as a wavefront each (0: a chain takes a workgroup).  A lane walks its components by
// itself, and the instructions a model value costs it say up to where that is the faster way whatever else the call is: of 350
// random calls (d 1..16, C 1..600, L 2..64, 1..6000 chains), a wavefront / a workgroup a chain, 282 of at most 300 instructions
// 0.09..1.00.  Above them it depends on what the workgroup's form costs, its stages and, where chains share CUs, their number:
// 68 calls of 300..900 0.11..1.77, 14 of them above 1.02 (few chains); of (16, 64, 8) at 336, K 200, 8 chains, 240 / 216 us, of (8,
// 64, 16) at 416 176 / 198.  Those keep the workgroup.
constexpr int kWaveWork = 300;
static int wave_chains(const asd_ctx* ctx) {
  const int C = ctx->gmm->C, d = ctx->d;
  if (d > 4 * kWaveBlocks || ctx->L > 64) return 0;
  const WaveLayout l = wave_layout(C, d, ctx->L, ctx->K);
  if ((int64_t)l.per_lane * (2 * l.dq + 10) > kWaveWork) return 0;
  const size_t room = 158 * 1024 / sizeof(float);
  if (l.chain + l.chain_floats > room) return 0;
  // one a workgroup while there are CUs for all; else as many as a SIMD has places for, if LDS has
  int n = (int)std::min<int64_t>(8, ceil_div(ctx->B, 256));
  while (l.chain + n * l.chain_floats > room) --n;
  return n;
}

bool gmm_chain_supported(const asd_ctx* ctx) {
  if (ctx->kind != ASD_DEN_GMM || !ctx->gmm || ctx->L > 64 || ctx->d > 4096) return false;
  return chain_fits(ctx, ctx->L);
}

// Dynamic LDS above the default limit needs the attribute, once per kernel and size.
static hipError_t allow_lds(const void* kernel, size_t bytes, size_t* allowed) {
  if (bytes <= *allowed) return hipSuccess;
  const hipError_t e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
  if (e == hipSuccess) *allowed = bytes;
  return e;
}

template <int DB>
static asd_status launch_wave(asd_ctx* ctx, int cpw, const float* y0, float* traj, int32_t* rounds, RoundsOut out, hipStream_t st) {
  const GmmState* g = ctx->gmm;
  const WaveLayout l = wave_layout(g->C, ctx->d, ctx->L, ctx->K);
  const size_t bytes = sizeof(float) * (l.chain + cpw * l.chain_floats);
  static size_t allowed = 0;
  ASD_HIP(allow_lds((const void*)gmm_wave_sample_kernel<DB>, bytes, &allowed));
  hipLaunchKernelGGL(gmm_wave_sample_kernel<DB>, dim3((unsigned)ceil_div(ctx->B, cpw)), dim3(64 * std::max(4, cpw)), bytes, st,
                     ctx->B, ctx->K, ctx->L, ctx->d, g->C, cpw, ctx->key, ctx->c_x, ctx->c_0, ctx->sigma, ctx->tau, g->coef_tau,
                     g->means, g->musq, g->log_w, y0, traj, rounds, out, ctx->adaptive ? 1 : 0);
  ASD_HIP(hipGetLastError());
  return ASD_OK;
}

template <int NW, int PARTS>
static asd_status launch_chain(asd_ctx* ctx, int ring, size_t bytes, const float* y0, float* traj, int32_t* rounds, RoundsOut out,
                               hipStream_t st) {
  const GmmState* g = ctx->gmm;
  static size_t allowed = 0;
  ASD_HIP(allow_lds((const void*)gmm_chain_sample_kernel<NW, PARTS>, bytes, &allowed));
  hipLaunchKernelGGL((gmm_chain_sample_kernel<NW, PARTS>), dim3(ctx->B), dim3(64 * NW), bytes, st, ctx->K, ctx->L, ctx->d, g->C,
                     ctx->key, ctx->c_x, ctx->c_0, ctx->sigma, ctx->tau, g->coef_tau, g->means, g->musq, g->log_w, y0, traj, rounds,
                     out, ctx->adaptive ? 1 : 0, ring);
  ASD_HIP(hipGetLastError());
  return ASD_OK;
}

asd_status gmm_chain_sample(asd_ctx* ctx, const float* y0, float* traj, int32_t* rounds, hipStream_t st) {
  if (!gmm_chain_supported(ctx)) {
    set_error("chain-resident sampler: the mixture, the window and the schedule do not fit in LDS");
    return ASD_EUNSUPPORTED;
  }
  const RoundsOut out{ctx->chain_max, &ctx->report_dev->chain_rounds, ++ctx->chain_launches};
  const int cpw = wave_chains(ctx);
  if (cpw > 0) {
    switch ((ctx->d + 3) / 4) {
      case 1: ASD_TRY(launch_wave<1>(ctx, cpw, y0, traj, rounds, out, st)); break;
      case 2: ASD_TRY(launch_wave<2>(ctx, cpw, y0, traj, rounds, out, st)); break;
      case 3: ASD_TRY(launch_wave<3>(ctx, cpw, y0, traj, rounds, out, st)); break;
      default: ASD_TRY(launch_wave<4>(ctx, cpw, y0, traj, rounds, out, st)); break;
    }
  } else {
    const int ring = chain_fits(ctx, 2 * ctx->L) ? 2 * ctx->L : ctx->L;
    const size_t lds_bytes = chain_lds_bytes(ctx, ring);
    const int items = chain_items(ctx), nw = chain_waves(items, ctx->d, ctx->B), parts = chain_parts(items);
    if (nw == 4) ASD_TRY((launch_chain<4, 4>(ctx, ring, lds_bytes, y0, traj, rounds, out, st)));
    else if (nw == 8 && parts == 4) ASD_TRY((launch_chain<8, 4>(ctx, ring, lds_bytes, y0, traj, rounds, out, st)));
    else if (nw == 8) ASD_TRY((launch_chain<8, 8>(ctx, ring, lds_bytes, y0, traj, rounds, out, st)));
    else if (parts == 8) ASD_TRY((launch_chain<16, 8>(ctx, ring, lds_bytes, y0, traj, rounds, out, st)));
    else ASD_TRY((launch_chain<16, 16>(ctx, ring, lds_bytes, y0, traj, rounds, out, st)));
  }
  ASD_HIP(hipStreamSynchronize(st));
  ctx->last_rounds = (int32_t) * (const volatile uint32_t*)&ctx->report->chain_rounds;
  return ASD_OK;
}

}  // namespace asd
