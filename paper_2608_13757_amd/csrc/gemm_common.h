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

__device__ __forceinline__ float gelu_erf(float x) {
  const float z = x * 0.70710678118654752f;
  const float a = __builtin_fabsf(z);
  const float t = __builtin_amdgcn_rcpf(1.0f + 0.3275911f * a);
  const float poly =
      t * (0.254829592f + t * (-0.284496736f + t * (1.421413741f + t * (-1.453152027f + t * 1.061405429f))));
  const float erf_a = 1.0f - poly * __expf(-a * a);
  const float erf_z = __builtin_copysignf(erf_a, z);
  return 0.5f * x * (1.0f + erf_z);
}

__device__ __forceinline__ uint32_t swz(uint32_t row, uint32_t chunk) {
  return row * 64u + ((chunk ^ ((row >> 2) & 3u)) << 4);
}

// Barrier-free, uninstrumented launches of the looped program: whole tiles or
// parts of them, K steps in pairs.  False (nothing launched, P as it was) if the
// ring's depth is odd or SPILL's waits are not of the program's usual kinds.
bool launch_parts(GemmParams &P, int n_wg, hipStream_t s, bfs_status &st);

}  // namespace bfsgemm
