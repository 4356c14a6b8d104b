// What the GEMM kernels share: tile and ring geometry, launch arguments, the
// GELU and the LDS swizzle.
#pragma once

#include "engine_sync.h"

namespace bfsgemm {

using namespace bfsdev;

constexpr int kTile = 256, kBK = 32;
constexpr int kLoadW = 2, kMmaW = 8, kEpiW = 2, kWaves = 12;
constexpr uint32_t kSlotBytes = 2 * kTile * kBK * 2;     // A + B of one K step
constexpr uint32_t kESlotBytes = kMmaW * 32 * 32 * 2;     // 8 bf16 blocks
constexpr int kMaxSteps = 128;                            // K steps of the K-unrolled program

struct GemmParams {
  SyncCommon sc;
  InstrWaits bias, load, mma, spill, epi;
  InstrWaits spill_once;    // kernels on parts: SPILL's waits that are constant during loop C (spill: the others)
  const __bf16 *a;
  const __bf16 *bt;
  const float *bias_v;
  __bf16 *c;
  const int32_t *trips;
  const int64_t *trip_off;
  int32_t m, n, k;
  int32_t ring, e_ring;
  int32_t tiles_m, tiles_n;
  int32_t xcd_map;          // 1: group tiles per XCD
  int32_t n_whole;          // grids of whole tiles and parts: how many are whole
  int32_t n_loops;          // 3 (top, K, C) or 2 (top, C: the K-unrolled program)
  // K-unrolled program: counter slots of the top-level LOAD and MMA
  // instructions, and the dependency id of each step's wait (debug log)
  int32_t c_load, c_mma;
  uint16_t dep_mma[kMaxSteps], dep_load[kMaxSteps];
};

// x Phi(x) with the tail Phi(-|x|) = erfc(|x| / sqrt 2) / 2 as 2^P(|x|): P is a
// degree 7 fit of log2 Phi(-a) over a <= 6.5 (least squares, weighted by the
// error it causes in the result and reweighted towards equal peaks), its
// leading coefficient held negative so that the tail vanishes beyond (also at
// infinity).  Error below 4e-7 for |x| <= 12 and 5e-8 rms over N(0, 1), all of
// it fp32 rounding; the rational form of erf (Abramowitz & Stegun 7.1.26) has
// 4.7e-7 and 8.4e-8.  The epilogue is bound by vector instructions, and this
// takes one transcendental instead of two: 15 issue slots of a wave instead
// of 21.
__device__ __forceinline__ float gelu_erf(float x) {
  const float a = __builtin_fabsf(x);
  float p = -9.999999975e-07f;
  p = __builtin_fmaf(p, a, 4.391759649e-05f);
  p = __builtin_fmaf(p, a, -8.149240748e-04f);
  p = __builtin_fmaf(p, a, 8.176802658e-03f);
  p = __builtin_fmaf(p, a, -5.351847410e-02f);
  p = __builtin_fmaf(p, a, -4.587108195e-01f);
  p = __builtin_fmaf(p, a, -1.151217103e+00f);
  p = __builtin_fmaf(p, a, -9.999918342e-01f);
  const float tail = __builtin_amdgcn_exp2f(p);
  return x * (x < 0.0f ? tail : 1.0f - tail);
}

__device__ __forceinline__ uint32_t swz(uint32_t row, uint32_t chunk) {
  return row * 64u + ((chunk ^ ((row >> 2) & 3u)) << 4);
}

// Barrier-free, uninstrumented launches of the looped program: whole tiles or
// parts of them, K steps in pairs.  False (nothing launched, P as it was) if the
// ring's depth is odd, LOAD waits for the MMA before it, SPILL's waits are not of
// the program's usual kinds, or a ring of two slots does better step by step.
bool launch_parts(GemmParams &P, int n_wg, hipStream_t s, bfs_status &st);

}  // namespace bfsgemm
