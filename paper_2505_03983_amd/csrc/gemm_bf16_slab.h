// bf16 x bf16 -> fp32 "NT" GEMM for gfx950:  acc[m][n] = sum_k A[m][k] * W[n][k], operands in slab layout, a multi-stage
// direct-to-LDS pipeline in front of the matrix cores.
//
// Slab layout.  A matrix [rows, K] is stored as K/32 slabs of [rows][32] bf16: element (r, k) lies at
// (k / 32) * rows * 32 + r * 32 + k % 32 (rows and the number of slabs padded with zeros).  Both operands are ours to lay
// out -- activations are written by the epilogues below, weights are copied once -- and in this form the 16 rows x 32 k a
// wavefront fetches with one global_load_lds_dwordx4 are one kilobyte of consecutive memory, and so are the kilobytes of
// the rows next to them: nothing depends on the row pitch, and a stage can be as short as 32 k, which is what lets a
// 128 x 256 tile with two planes of A (32 KB a slab) keep four stages in a CU's LDS.
//
// Pipeline.  A bf16 MFMA consumes a slab in less time than a load takes to arrive, so the loads of STAGES - 1 stages are
// in flight: global_load_lds_dwordx4 moves 16 bytes per lane from L2 straight into LDS, completion is tracked with
// s_waitcnt vmcnt, and one bare barrier per stage hands a landed stage over while the one just consumed is refilled.
// Loads, fragment reads and the hand-over are slotted between MFMAs (see the loop).
//
// The loads are buffer loads (load_to_lds): behind global ones the compiler waited for every outstanding LDS read wherever an
// MFMA needs one, which undid the reads ahead.  us a layer before / now: 1984 x 4096 x 4096 130 / 128 with two planes, 75
// / 72 with one, 456 rows 39.4 / 37.7; 720 x 1536 x 1536, one plane, 14.6 / 12.9.
//
// LDS layout of a stage: per slab the A rows of every plane, then the W rows, 64 bytes a row = 4 chunks of 16 bytes.
// LDS serves 256 bytes per clock, 16 lanes of a 128-bit read; chunk c of row r sits in chunk slot c ^ ((r >> 2) & 3),
// so the 16 rows of a fragment read fall into 16 different 16-byte slots of a 256-byte line.  The permutation is applied
// on the global side of the load (inside a row's own 64 bytes).
//
// Two-plane A operand (PL = 2): A is given as the sum of two bf16 matrices of the same shape, a_plane elements apart
// (activations kept to 16 significant bits as hi + lo, see mlp.hip).  Every (A fragment, W fragment) pair is multiplied
// twice, once per plane, into the same accumulator: the weights are loaded once for both.  Every tile shape accumulates
// an element's products in the same order (k ascending in groups of 16, hi plane before lo), so a result does not depend
// on the shape that computed it.
//
// Split K (gridDim.z > 1): for a handful of rows the kernel is a stream of the weight matrix, and HBM only delivers its
// bandwidth with ~16 MB in flight -- more workgroups than the output has tiles.  The z-th workgroup of a tile contracts
// the z-th share of K and leaves its fp32 partial tile in scratch; splitk_finish_kernel then adds the partials in z order
// and runs the epilogue.  (Finishing inside the GEMM, by whichever workgroup of a tile arrives last, was measured: the
// device-scope fences it needs write back and invalidate an XCD's whole L2 and cost more than the second launch.)
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "gemm_bf16.h"

namespace asd {

constexpr int kSlabRows = 256;   // rows of a slab-layout matrix are padded to this (the tallest tile): no row clamps

inline int64_t slab_rows(int64_t rows) { return (rows + kSlabRows - 1) / kSlabRows * kSlabRows; }
inline int slab_count(int K) { return (K + 63) / 64 * 2; }                             // even: a stage may hold two
inline size_t slab_elems(int64_t rows, int K) { return (size_t)slab_rows(rows) * slab_count(K) * 32; }

// BM x BN workgroup tile, SPS slabs of 32 k per stage, STAGES stages, WGM x WGN wavefronts (each owns a
// (BM/WGM) x (BN/WGN) sub-tile), PL planes of A.
// AHEAD: fragments are read a whole stage ahead instead of a group of 16 k (small tiles, see the loop).
template <int BM_, int BN_, int SPS_, int STAGES_, int WGM_, int WGN_, int PL_, bool AHEAD_ = false>
struct SlabCfg {
  static constexpr bool AHEAD = AHEAD_;
  static constexpr int BM = BM_, BN = BN_, SPS = SPS_, STAGES = STAGES_, WGM = WGM_, WGN = WGN_, PL = PL_;
  static constexpr int NW = WGM * WGN, THREADS = 64 * NW;
  static constexpr int WM = BM / WGM, WN = BN / WGN;          // wavefront sub-tile
  static constexpr int MI = WM / 32, NJ = WN / 32;
  static constexpr int AR = PL * BM, ROWS = AR + BN;          // rows of a slab in LDS
  static constexpr int A_LOADS = AR / 16 / NW, W_LOADS = BN / 16 / NW;  // wave-loads (16 rows each) per wavefront and slab
  static constexpr int LPSL = A_LOADS + W_LOADS, LPS = SPS * LPSL;      // ... per slab and per stage
  static constexpr int SLAB_BYTES = ROWS * 64, STAGE_BYTES = SPS * SLAB_BYTES;
  static constexpr int PIPE_BYTES = STAGES * STAGE_BYTES, OUT_BYTES = BM * BN * 4;
  static constexpr size_t LDS_BYTES = PIPE_BYTES > OUT_BYTES ? PIPE_BYTES : OUT_BYTES;   // the epilogue parks the tile
  static constexpr int NG = 2 * SPS;                          // groups of 16 k per stage
  static_assert(PL == 1 || PL == 2, "A operand planes");
  static_assert(WM % 32 == 0 && WN % 32 == 0 && STAGES >= 3, "tile shape");
  static_assert(AR % (16 * NW) == 0 && BN % (16 * NW) == 0, "wave-loads must divide evenly among the wavefronts");
  static_assert(LDS_BYTES <= 160 * 1024, "LDS of a CU");
  static_assert(LPS * (STAGES - 1) <= 63, "vmcnt range");
  static_assert(kSlabRows % BM == 0 && kSlabRows % BN == 0, "padded rows");
  // loads of a later stage issued inside group g
  static constexpr int loads_in_group(int g) { return LPS / NG + (g < LPS % NG ? 1 : 0); }
  static constexpr int loads_before_group(int g) { return g == 0 ? 0 : loads_before_group(g - 1) + loads_in_group(g - 1); }
};

// Wait until at most `stages` * LPS of this wavefront's loads are outstanding.
template <int LPS, int MAX>
__device__ __forceinline__ void wait_stages(int stages) {
  if constexpr (MAX == 0) {
    wait_vmcnt<0>();
  } else {
    if (stages >= MAX) wait_vmcnt<LPS * MAX>();
    else wait_stages<LPS, MAX - 1>(stages);
  }
}

// A [planes][K/32][a_rows][32], W [K/32][w_rows][32].  M comes from device memory (compacted row plan).
template <class Cfg, class Epi, int CALL>
__global__ __launch_bounds__(Cfg::THREADS) void gemm_bf16_slab_kernel(const int* __restrict__ M_dev, int M_max, int N,
                                                                      int nslabs, const uint16_t* __restrict__ A,
                                                                      int64_t a_slab, int64_t a_plane,
                                                                      const uint16_t* __restrict__ W, int64_t w_slab,
                                                                      Epi epi, float* __restrict__ part) {
  constexpr int BM = Cfg::BM, BN = Cfg::BN, SPS = Cfg::SPS, STAGES = Cfg::STAGES, MI = Cfg::MI, NJ = Cfg::NJ, NW = Cfg::NW;
  constexpr int AR = Cfg::AR, PL = Cfg::PL, AI = PL * MI;   // AI: A fragments per k group (all planes)
  constexpr int WM = Cfg::WM, WN = Cfg::WN, NG = Cfg::NG;
  constexpr int A_LOADS = Cfg::A_LOADS, LPSL = Cfg::LPSL, LPS = Cfg::LPS;
  extern __shared__ __attribute__((aligned(16))) uint8_t ldsb[];

  const int M = M_dev ? min(*M_dev, M_max) : M_max;
  const int m0 = blockIdx.y * BM, n0 = blockIdx.x * BN;
  if (m0 >= M) return;

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // uniform: addresses of the direct loads stay scalar
  const int wm = wave / Cfg::WGN, wn = wave % Cfg::WGN;
  const int l32 = lane & 31, half = lane >> 5;

  const int splits = gridDim.z;
  const int nk = nslabs / SPS / splits;                       // stages of this workgroup's share of K
  const int s0 = blockIdx.z * nk * SPS;                       // its first slab

  // loader: a wave-load covers 16 rows of a slab; lane L fills chunk slot L of that kilobyte
  const uint32_t lane_off = (lane >> 2) * 64 + (((lane & 3) ^ ((lane >> 4) & 3)) * 16);
  const uint8_t* abase = reinterpret_cast<const uint8_t*>(A) + ((int64_t)s0 * a_slab + (int64_t)m0 * 32) * 2;
  const uint8_t* wbase = reinterpret_cast<const uint8_t*>(W) + ((int64_t)s0 * w_slab + (int64_t)n0 * 32) * 2;
  // wave-loads first .. first+count-1 of stage kt (per slab: A loads, then W loads) into the LDS stage at `sb`
  auto issue = [&](int kt, uint8_t* sb, int first, int count) {
#pragma unroll
    for (int q = 0; q < LPS; ++q) {
      if (q < first || q >= first + count) continue;
      const int sl = q / LPSL, p = q % LPSL;
      const int blk = wave + NW * (p < A_LOADS ? p : p - A_LOADS);   // block of 16 rows
      if (p < A_LOADS) {
        const int row = blk * 16, plane = row / BM;
        const uint8_t* g = abase + ((int64_t)(kt * SPS + sl) * a_slab + (int64_t)plane * a_plane + (int64_t)(row - plane * BM) * 32) * 2;
        load_to_lds(g, lane_off, sb + sl * Cfg::SLAB_BYTES + blk * 1024);
      } else {
        const uint8_t* g = wbase + ((int64_t)(kt * SPS + sl) * w_slab + (int64_t)blk * 16 * 32) * 2;
        load_to_lds(g, lane_off, sb + sl * Cfg::SLAB_BYTES + AR * 64 + blk * 1024);
      }
    }
  };

  v16f_b acc[MI][NJ];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

  constexpr int G = AI * NJ;                         // MFMAs per group of 16 k
#pragma unroll
  for (int s = 0; s < STAGES - 1; ++s)
    if (s < nk) issue(s, ldsb + s * Cfg::STAGE_BYTES, 0, LPS);

  const int key = (l32 >> 2) & 3;                    // swizzle key of this lane's rows (tile offsets are multiples of 16)
  const int a_row = (wm * WM + l32) * 64, w_row = AR * 64 + (wn * WN + l32) * 64;
  int cp[2];
#pragma unroll
  for (int ks = 0; ks < 2; ++ks) cp[ks] = ((ks * 2 + half) ^ key) * 16;

  constexpr int NBUF = Cfg::AHEAD ? 2 * NG : 2;      // fragment buffers, one per group of 16 k
  v8bf af[NBUF][AI], wf[NBUF][NJ];
  auto read_frags = [&](const uint8_t* sb, int g, int buf) {   // group g of the stage at sb
    const uint8_t* s = sb + (g >> 1) * Cfg::SLAB_BYTES;
#pragma unroll
    for (int i = 0; i < AI; ++i)   // fragment i: plane i / MI, 32-row block i % MI
      af[buf][i] = *reinterpret_cast<const v8bf*>(s + (i / MI) * (BM * 64) + a_row + (i % MI) * 32 * 64 + cp[g & 1]);
#pragma unroll
    for (int j = 0; j < NJ; ++j) wf[buf][j] = *reinterpret_cast<const v8bf*>(s + w_row + j * 32 * 64 + cp[g & 1]);
  };
  auto mma = [&](int buf, int first, int count) {  // MFMAs first .. first+count-1 of a group, row-major over (i, j)
#pragma unroll
    for (int q = 0; q < G; ++q)
      if (q >= first && q < first + count)
        acc[(q / NJ) % MI][q % NJ] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[buf][q / NJ], wf[buf][q % NJ],
                                                                             acc[(q / NJ) % MI][q % NJ], 0, 0, 0);
  };

  if constexpr (Cfg::AHEAD) {
    // Small tiles: a wavefront has a couple of MFMAs per group, which do not cover the latency of an LDS read, and no
    // neighbour on its SIMD to do so.  All fragments of stage kt + 1 are read before the MFMAs of stage kt; the barrier
    // in front of those reads also says that everybody's reads of stage kt are over (their wait below), so the loads of
    // stage kt + STAGES go straight into its memory.
    if (STAGES - 1 < nk) issue(STAGES - 1, ldsb + (STAGES - 1) * Cfg::STAGE_BYTES, 0, LPS);
    auto hand_over = [&](int behind) {   // stage after `behind` stages still in flight has landed, for every wavefront
      wait_stages<LPS, STAGES - 1>(behind);
      if constexpr (NW > 1) lds_handover();
      else asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    };
    auto hand_over_steady = [&]() {
      wait_vmcnt<LPS * (STAGES - 2)>();
      if constexpr (NW > 1) lds_handover();
      else asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    };
    auto read_stage = [&](const uint8_t* sb, int buf) {
#pragma unroll
      for (int g = 0; g < NG; ++g) read_frags(sb, g, buf * NG + g);
    };
    hand_over(nk - 1);
    read_stage(ldsb, 0);
    int cur = 0;
    // steady: stages kt + 1 .. kt + STAGES exist, no branches (a branch would end the compiler's view of which LDS reads
    // are outstanding, and it would wait for those just issued)
    auto step = [&](int kt, auto buf_c, auto steady_c) {
      constexpr int buf = decltype(buf_c)::value;
      constexpr bool steady = decltype(steady_c)::value;
      uint8_t* mine = ldsb + cur * Cfg::STAGE_BYTES;
      cur = cur + 1 == STAGES ? 0 : cur + 1;
      if (steady || kt + 1 < nk) {
        if constexpr (steady) hand_over_steady();
        else hand_over(min(nk - 2 - kt, STAGES - 2));
        read_stage(ldsb + cur * Cfg::STAGE_BYTES, buf ^ 1);
        if (steady || kt + STAGES < nk) issue(kt + STAGES, mine, 0, LPS);
      }
#pragma unroll
      for (int g = 0; g < NG; ++g) mma(buf * NG + g, 0, G);
      if constexpr (steady) {
        constexpr int T = NG * G, R = NG * (AI + NJ);   // MFMAs and fragment reads of a step
        sched_pairs<0x100, (R + 1) / 2 < T ? (R + 1) / 2 : T, 2>();
        sched_pairs<0x010, T - ((R + 1) / 2 < T ? (R + 1) / 2 : T), 1>();
      }
    };
    int kt = 0;
    for (; kt + STAGES + 1 < nk; kt += 2) {
      step(kt, std::integral_constant<int, 0>(), std::true_type());
      step(kt + 1, std::integral_constant<int, 1>(), std::true_type());
    }
    for (; kt < nk; kt += 2) {
      step(kt, std::integral_constant<int, 0>(), std::false_type());
      if (kt + 1 < nk) step(kt + 1, std::integral_constant<int, 1>(), std::false_type());
    }
  } else {
  // ---- software pipeline, rotated so that everything that is not an MFMA runs in the shadow of MFMAs:
  //   prologue : loads of stages 0..STAGES-2 in flight, stage 0 landed, its first fragments read
  //   stage kt : NG groups of 16 k.  Each group issues its MFMAs with the next group's fragment reads
  //              (two behind each of the first MFMAs) and its share of the direct loads of stage
  //              kt+STAGES-1 (one behind each following MFMA; that stage's memory was released by the
  //              barrier of the previous iteration) slotted in.
  //              Half-way through the last group the wavefront waits for its loads of stage kt+1 and for its
  //              own reads of stage kt, meets the others at the barrier (after which nobody reads stage kt's
  //              memory again) and reads the first fragments of stage kt+1 -- while the rest of the group
  //              executes.
  constexpr int H1 = (G + 1) / 2, H2 = G - H1;       // MFMAs of the last group before / after the hand-over
  constexpr int RD = AI + NJ, SLOTS = (RD + 1) / 2, RLAST = RD - 2 * (SLOTS - 1);
  constexpr int REM = G > SLOTS ? G - SLOTS : 0;     // MFMAs of a group left after the read slots
  wait_stages<LPS, STAGES - 2>(nk - 1);   // stage 0 landed; the other prologue stages may be in flight
  lds_handover();
  read_frags(ldsb, 0, 0);

  int cur = 0, nst = STAGES - 1;          // LDS stages of kt and of kt + STAGES - 1
  // steady: stages kt + 1 .. kt + STAGES - 1 exist, and the last of them is fetched now -- no branches, so that the stage is one scheduling region, the
  // interleaving asked for holds, and the compiler knows which LDS reads an MFMA has to wait for (behind a branch it
  // waits for all of them, those just issued for the next group included)
  auto step = [&](int kt, auto steady_c) {
    constexpr bool steady = decltype(steady_c)::value;
    const uint8_t* sb = ldsb + cur * Cfg::STAGE_BYTES;
    uint8_t* nb = ldsb + nst * Cfg::STAGE_BYTES;
    const int nxt = kt + STAGES - 1;
    nst = cur;                               // (the stage after the last one wraps to the one consumed now)
    cur = cur + 1 == STAGES ? 0 : cur + 1;
#pragma unroll
    for (int g = 0; g < NG - 1; ++g) {
      constexpr int L0 = Cfg::loads_in_group(0);  // groups may differ by one load; hints use the larger count
      read_frags(sb, g + 1, (g + 1) & 1);
      if constexpr (steady) issue(nxt, nb, Cfg::loads_before_group(g), Cfg::loads_in_group(g));
      mma(g & 1, 0, G);
      sched_pairs<0x100, SLOTS - 1, 2>();
      sched_pairs<0x100, 1, RLAST>();
      sched_pairs<0x010, (L0 < REM ? L0 : REM), 1>();
      sched_mfma<REM - (L0 < REM ? L0 : REM)>();
    }
    // last group, first part
    constexpr int LB = Cfg::loads_in_group(NG - 1);
    if constexpr (steady) issue(nxt, nb, Cfg::loads_before_group(NG - 1), LB);
    mma((NG - 1) & 1, 0, H1);
    sched_pairs<0x010, (LB < H1 ? LB : H1), 1>();
    sched_mfma<H1 - (LB < H1 ? LB : H1)>();
    if (steady || kt + 1 < nk) {
      // This wavefront's loads of stage kt+1 must have landed; those of the stages behind it may stay in flight.
      if constexpr (steady) wait_vmcnt<LPS * (STAGES - 2)>();
      else wait_stages<LPS, STAGES - 2>(nk - 2 - kt);
      lds_handover();
      read_frags(ldsb + cur * Cfg::STAGE_BYTES, 0, 0);
    }
    mma((NG - 1) & 1, H1, H2);
    sched_pairs<0x100, (SLOTS - 1 < H2 ? SLOTS - 1 : H2), 2>();
  };
  int kt = 0;
  for (; kt + STAGES - 1 < nk; ++kt) step(kt, std::true_type());
  for (; kt < nk; ++kt) step(kt, std::false_type());
  }

  // Epilogue through LDS (the pipeline stages are free now): each wavefront parks its WM x WN fp32
  // sub-tile in its own LDS region, then walks it row by row with 16-byte accesses, so global traffic
  // is row-contiguous and the code is a short loop rather than 16*MI*NJ unrolled scalar stores.
  lds_handover();  // every wavefront is done reading the last stage
  float* stage = reinterpret_cast<float*>(ldsb) + wave * (WM * WN);
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r)
        stage[(i * 32 + 8 * (r >> 2) + 4 * half + (r & 3)) * WN + j * 32 + l32] = acc[i][j][r];
  // the region is private to this wavefront: LDS operations of one wavefront complete in order
  constexpr int LPR = WN / 4;        // lanes per row (one float4 each)
  constexpr int RPI = 64 / LPR;      // rows per iteration
  const int lrow = lane / LPR, lcol = (lane % LPR) * 4;
  // The residual stream is read and rewritten in place: all reads of a batch of rows are issued
  // before its first write, so a batch costs one memory round trip.
  constexpr int ITERS = WM / RPI, BATCH = ITERS < 16 ? ITERS : 16;
  static_assert(ITERS % BATCH == 0, "epilogue batching");
  const int n = n0 + wn * WN + lcol;
  const bool nok = n < N;
  if (splits > 1) {
    float* dst = part + ((int64_t)blockIdx.z * M_max + m0 + wm * WM + lrow) * N + n;
#pragma unroll 4
    for (int it = 0; it < ITERS; ++it)
      if (nok && m0 + wm * WM + it * RPI + lrow < M)
        *reinterpret_cast<float4*>(dst + (int64_t)it * RPI * N) =
            *reinterpret_cast<const float4*>(&stage[(it * RPI + lrow) * WN + lcol]);
    return;
  }
  // (a lane's columns are the same in every row: what depends on them only is fetched once.  Loads past the last row or
  // column repeat it, so that a batch is one run of loads and one of stores with no wait in between.)
  const float4 col = epi.column4(nok ? n : 0);
#pragma unroll
  for (int it0 = 0; it0 < ITERS; it0 += BATCH) {
    float4 v[BATCH], prev[BATCH];
#pragma unroll
    for (int b = 0; b < BATCH; ++b) {
      const int row = (it0 + b) * RPI + lrow;
      prev[b] = Epi::kLoads ? epi.load4(min(m0 + wm * WM + row, M - 1), nok ? n : 0) : make_float4(0.f, 0.f, 0.f, 0.f);
      v[b] = *reinterpret_cast<const float4*>(&stage[row * WN + lcol]);
    }
#pragma unroll
    for (int b = 0; b < BATCH; ++b)   // (keeps the loads up here: sunk into the conditional stores they would wait for each other)
      asm volatile("" : "+v"(prev[b].x), "+v"(prev[b].y), "+v"(prev[b].z), "+v"(prev[b].w));
#pragma unroll
    for (int b = 0; b < BATCH; ++b) {
      const int m = m0 + wm * WM + (it0 + b) * RPI + lrow;
      if (m < M && nok) epi.store4(m, n, v[b], prev[b], col);
    }
  }
}

// One thread per four columns of a row: partials added in z order, then the epilogue.
template <class Epi>
__global__ __launch_bounds__(256) void splitk_finish_kernel(const int* __restrict__ M_dev, int M_max, int N, int splits,
                                                            const float* __restrict__ part, Epi epi) {
  const int M = M_dev ? min(*M_dev, M_max) : M_max;
  const int m = blockIdx.y;
  const int n = (blockIdx.x * 256 + threadIdx.x) * 4;
  if (m >= M || n >= N) return;
  const float4 prev = Epi::kLoads ? epi.load4(m, n) : make_float4(0.f, 0.f, 0.f, 0.f);
  float4 v = *reinterpret_cast<const float4*>(part + (int64_t)m * N + n);
  for (int z = 1; z < splits; ++z) {
    const float4 q = *reinterpret_cast<const float4*>(part + ((int64_t)z * M_max + m) * N + n);
    v.x += q.x; v.y += q.y; v.z += q.z; v.w += q.w;
  }
  epi.store4(m, n, v, prev, epi.column4(n));
}

// A slab-layout matrix: base, rows it was laid out with, elements between its planes.
struct SlabMat {
  const uint16_t* p;
  int64_t rows;
  int64_t plane;
};

// splits > 1 needs (number of 64-wide slab pairs) % splits == 0 and `part` of splits * M * N floats.
template <class Cfg, int CALL, class Epi>
inline hipError_t launch_gemm_bf16_slab(const int* M_dev, int M, int N, int K, SlabMat A, SlabMat W, Epi epi, hipStream_t st,
                                        int splits = 1, float* part = nullptr) {
  const int nslabs = slab_count(K);
  if (splits < 1 || (nslabs / 2) % splits != 0 || (splits > 1 && !part)) return hipErrorInvalidValue;
  if (M > A.rows || N > W.rows || A.rows % kSlabRows || W.rows % kSlabRows) return hipErrorInvalidValue;
  dim3 grid((unsigned)((N + Cfg::BN - 1) / Cfg::BN), (unsigned)((M + Cfg::BM - 1) / Cfg::BM), (unsigned)splits);
  auto kern = gemm_bf16_slab_kernel<Cfg, Epi, CALL>;
  static bool attr_set = false;  // dynamic LDS above the default limit needs the attribute once per kernel
  if (!attr_set) {
    hipError_t e = hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize,
                                       (int)Cfg::LDS_BYTES);
    if (e != hipSuccess) return e;
    attr_set = true;
  }
  hipLaunchKernelGGL(kern, grid, dim3(Cfg::THREADS), Cfg::LDS_BYTES, st, M_dev, M, N, nslabs, A.p, A.rows * 32, A.plane,
                     W.p, W.rows * 32, epi, part);
  if (splits > 1)
    hipLaunchKernelGGL(splitk_finish_kernel<Epi>, dim3((unsigned)((N / 4 + 255) / 256), (unsigned)M), dim3(256), 0, st,
                       M_dev, M, N, splits, part, epi);
  return hipGetLastError();
}

}  // namespace asd
