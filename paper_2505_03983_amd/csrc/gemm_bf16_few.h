// bf16 x bf16 -> fp32 "NT" products of a few rows, on the slab layout of gemm_bf16_slab.h (same operands, same epilogues,
// same bits).
//
// What bounds such a call is latency: 64 rows of a 1024-wide layer are a microsecond of matrix work, and a tile that walks
// K through stages of 64 k pays a hand-over for each (7 us a launch, from 16 workgroups on 256 CUs).  Here an output tile
// is small enough (16 rows x 16 columns or a few of those) that most or all of its operands fit a CU's LDS at once: sixteen
// wavefronts have them on their way with the first instructions, and one wavefront per 16 x 16 block then runs through k in
// one go.  (K must be summed in order for the bits to match; with K shared among the wavefronts and partial sums added the
// same layers take 4.2 us instead of 5.1, but a sample's accept tests would then see other roundings than a larger
// batch's.  Accumulators passed from wavefront to wavefront instead: 0.15 us a pass, 7 us in all.)
//
// Of the 9000 cycles of 16 x 1024 x 1024, two planes, 3500 passed until half of the operands had landed and 4200 in the
// products, two thirds of that waiting for LDS: the loads were global ones, behind which the compiler waits for every read
// of LDS outstanding (load_to_lds), and it moved the reads up against their products.  As buffer loads, with the reads a batch ahead held
// in place, the products take 2900, the 64 dependent instructions' own latency: 4.8 -> 4.3 us a layer, 1536 x 1536 6.5 -> 5.8, 2048 x
// 2048 7.9 -> 7.1; one plane 3.8 -> 3.5, 5.2 -> 4.8, 6.0 -> 5.7.  (Stages of 8 slabs, whose first lands sooner: 4.9, a hand-over
// costs 400 cycles.  A wavefront that loads its operands into registers, with no hand-over at all: 6.5, sixty loads of it on
// their way are too few.)
//
// v_mfma_f32_16x16x32_bf16 adds its products in the order of two 32x32x16 (k 0..15, then 16..31), bit for bit.  One plane
// of A: an instruction takes a slab.  Two planes: an instruction takes 16 k, the hi terms in its lower k half, the lo terms
// in its upper one, the weights in both -- the order of the tiled kernel, at one instruction instead of two.  The weights
// are the first operand, so a lane ends up with four consecutive columns of one row, which is what the epilogues store.
//
// LDS: 16 rows of a slab are a block of one kilobyte (one direct load of a wavefront); a slab is PL MI blocks of A, then NJ of
// W; chunk c of row r sits in slot c ^ ((r >> 2) & 3) as in gemm_bf16_slab.h.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "gemm_bf16.h"
#include "gemm_bf16_slab.h"

namespace asd {

typedef float v4f_f __attribute__((ext_vector_type(4)));

// A workgroup tile is 16 MI rows x 16 NJ columns; SS slabs per stage, as many stages as LDS holds; PL planes of A.
template <int MI_, int NJ_, int SS_, int PL_>
struct FewRowsCfg {
  static constexpr int MI = MI_, NJ = NJ_, SS = SS_, PL = PL_;
  static constexpr int NW = 16, TILES = MI * NJ, BM = 16 * MI, BN = 16 * NJ;
  static constexpr int BPS = PL * MI + NJ;                     // blocks of a slab
  static constexpr int STAGE_BLOCKS = SS * BPS, WPS = NW / SS, LPW = BPS / WPS;   // WPS wavefronts load a slab, LPW blocks each
  static constexpr int FIT = 156 / STAGE_BLOCKS, STAGES = FIT < 4 ? FIT : 4;
  static constexpr size_t LDS_BYTES = (size_t)STAGES * STAGE_BLOCKS * 1024;
  static_assert(NW % SS == 0 && BPS % WPS == 0 && SS % 4 == 0 && STAGES >= 2, "stage shape");
  static_assert(TILES <= NW && kSlabRows % BM == 0 && kSlabRows % BN == 0, "tile shape");
};

template <class Cfg, class Epi>
__global__ __launch_bounds__(64 * Cfg::NW) void gemm_bf16_few_kernel(const int* __restrict__ M_dev, int M_max, int N,
                                                                     int nslabs, const uint16_t* __restrict__ A,
                                                                     int64_t a_slab, int64_t a_plane,
                                                                     const uint16_t* __restrict__ W, int64_t w_slab, Epi epi,
                                                                     int part_slabs) {
  constexpr int MI = Cfg::MI, NJ = Cfg::NJ, SS = Cfg::SS, PL = Cfg::PL, BPS = Cfg::BPS, LPW = Cfg::LPW, STAGES = Cfg::STAGES;
  extern __shared__ __attribute__((aligned(16))) uint8_t ldsb[];
  const int m0 = blockIdx.y * Cfg::BM, n0 = blockIdx.x * Cfg::BN;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int r = lane & 15, q = lane >> 4;

  // the 16 x 16 block this wavefront computes; what its epilogue reads of memory is requested first
  const bool fin = wave < Cfg::TILES;
  const int ti = wave / NJ, tj = wave % NJ;
  const int m = m0 + 16 * ti + r, n = n0 + 16 * tj + 4 * q;
  const bool nok = n < N;
  float4 prev = make_float4(0.f, 0.f, 0.f, 0.f), col = prev;
  if (fin) {
    if constexpr (Epi::kLoads) prev = epi.load4(min(m, M_max - 1), nok ? n : 0);
    col = epi.column4(nok ? n : 0);
  }
  const int nst = (nslabs + SS - 1) / SS;
  const uint32_t lane_off = (lane >> 2) * 64 + (((lane & 3) ^ ((lane >> 4) & 3)) * 16);
  const uint8_t* abase = reinterpret_cast<const uint8_t*>(A) + (int64_t)m0 * 64;
  const uint8_t* wbase = reinterpret_cast<const uint8_t*>(W) + (int64_t)n0 * 64;
  auto issue = [&](int st) {   // (blocks past the last slab repeat it; nobody reads them)
    uint8_t* dst = ldsb + ((st % STAGES) * SS + wave % SS) * (BPS * 1024);
    const int s = min(st * SS + wave % SS, nslabs - 1);
#pragma unroll
    for (int i = 0; i < LPW; ++i) {
      const int j = Cfg::WPS == 1 ? i : (wave / SS) * LPW + i;   // block of the slab
      const uint8_t* g = j < PL * MI ? abase + ((int64_t)s * a_slab + (int64_t)(j / MI) * a_plane + (j % MI) * 16 * 32) * 2
                                     : wbase + ((int64_t)s * w_slab + (j - PL * MI) * 16 * 32) * 2;
      load_to_lds(g, lane_off, dst + j * 1024);
    }
  };
#pragma unroll
  for (int s = 0; s < STAGES; ++s)
    if (s < nst) issue(s);
  float4 aux = make_float4(0.f, 0.f, 0.f, 0.f);   // what an epilogue can make ready while the loads are on their way
  if constexpr (Epi::kAux) {
    if (fin && nok) aux = epi.aux4(m, n);
  }
  // (the row count is itself a load from memory: asked for behind the others, it costs a live workgroup nothing)
  const int M = M_dev ? min(*M_dev, M_max) : M_max;
  if (m0 >= M) {
    wait_vmcnt<0>();   // nothing may land in LDS that is no longer ours
    return;
  }

  v4f_f acc = {0.f, 0.f, 0.f, 0.f};
  const int key = (r >> 2) & 3;
  // One plane: chunk q of a row.  Two: chunk 2 g + q % 2 for instruction g, hi rows for q < 2, lo rows for the others.
  const int a_off = (PL == 2 ? (q >> 1) * MI * 1024 : 0) + ti * 1024 + r * 64;
  const int w_off = (PL * MI + tj) * 1024 + r * 64;
  const int cp[2] = {(PL == 2 ? (q & 1) ^ key : q ^ key) * 16, ((2 + (q & 1)) ^ key) * 16};
  // sums of part_slabs slabs each, added in order (what a K split over workgroups gives; usually one part is all of K)
  v4f_f sum = acc;
  int next = part_slabs;   // slab at which the next part starts
  auto close_part = [&](int slab) {
    if (slab != next) return;
    if (next == part_slabs) sum = acc;
    else sum += acc;
    acc = (v4f_f){0.f, 0.f, 0.f, 0.f};
    next += part_slabs;
  };
  constexpr int H = PL, U = 4 / PL;   // instructions per slab; slabs per batch of fragment reads
  for (int st = 0; st < nst; ++st) {
    wait_stages<LPW, STAGES - 1>(min(nst - 1 - st, STAGES - 1));
    lds_handover();
    if (fin) {
      const uint8_t* sb = ldsb + (st % STAGES) * (Cfg::STAGE_BLOCKS * 1024);
      const int ns = min(SS, nslabs - st * SS);   // even
      v8bf af[2][U][H], wf[2][U][H];
      auto read_one = [&](int buf, int s0, int u, int g) {
        af[buf][u][g] = *reinterpret_cast<const v8bf*>(sb + (s0 + u) * (BPS * 1024) + a_off + cp[g]);
        wf[buf][u][g] = *reinterpret_cast<const v8bf*>(sb + (s0 + u) * (BPS * 1024) + w_off + cp[g]);
      };
      auto read = [&](int buf, int s0) {
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
          for (int g = 0; g < H; ++g) read_one(buf, s0, u, g);
      };
      auto mma = [&](int buf, int s0) {
#pragma unroll
        for (int u = 0; u < U; ++u)
          if (s0 + u < ns) {
            close_part(st * SS + s0 + u);
#pragma unroll
            for (int g = 0; g < H; ++g)
              acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[buf][u][g], af[buf][u][g], acc, 0, 0, 0);
          }
      };
      if (ns == SS && (next <= st * SS ? part_slabs >= SS : next >= st * SS + SS)) {
        // a full stage of one part: straight-line code, reads a batch ahead.  (Left to itself the compiler moves every read
        // up against the product that needs it, and the loop pays the latency of LDS for each.)
        close_part(st * SS);
        read(0, 0);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int s0 = 0; s0 < SS; s0 += U) {
#pragma unroll
          for (int u = 0; u < U; ++u)
#pragma unroll
            for (int g = 0; g < H; ++g) {
              if (s0 + U < SS) read_one((s0 / U + 1) & 1, s0 + U, u, g);
              acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[(s0 / U) & 1][u][g], af[(s0 / U) & 1][u][g], acc, 0, 0, 0);
              __builtin_amdgcn_sched_barrier(0);
            }
        }
      } else {
        for (int s0 = 0; s0 < ns; s0 += U) {   // (reads past ns stay inside the stage: SS is a multiple of U)
          read(0, s0);
          mma(0, s0);
        }
      }
    }
    if (st + STAGES < nst) {   // the stage's memory is refilled once nobody reads it
      lds_handover();
      issue(st + STAGES);
    }
  }
  if (nslabs > part_slabs) acc = sum + acc;
  if (fin && m < M && nok) {
    const float4 v = make_float4(acc[0], acc[1], acc[2], acc[3]);
    if constexpr (Epi::kAux) epi.store4(m, n, v, prev, col, aux);
    else epi.store4(m, n, v, prev, col);
  }
}

template <class Cfg, class Epi>
inline hipError_t launch_gemm_bf16_few(const int* M_dev, int M, int N, int K, SlabMat A, SlabMat W, Epi epi, hipStream_t st,
                                       int splits = 1) {
  if (splits < 1 || (slab_count(K) / 2) % splits != 0) return hipErrorInvalidValue;
  if (M > A.rows || N > W.rows || A.rows % kSlabRows || W.rows % kSlabRows) return hipErrorInvalidValue;
  auto kern = gemm_bf16_few_kernel<Cfg, Epi>;
  static bool attr_set = false;  // dynamic LDS above the default limit needs the attribute once per kernel
  if (!attr_set) {
    hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)Cfg::LDS_BYTES);
    if (e != hipSuccess) return e;
    attr_set = true;
  }
  hipLaunchKernelGGL(kern, dim3((unsigned)((N + Cfg::BN - 1) / Cfg::BN), (unsigned)((M + Cfg::BM - 1) / Cfg::BM)),
                     dim3(64 * Cfg::NW), Cfg::LDS_BYTES, st, M_dev, M, N, slab_count(K), A.p, A.rows * 32, A.plane, W.p,
                     W.rows * 32, epi, slab_count(K) / splits);
  return hipGetLastError();
}

}  // namespace asd
