// What the MoE kernels share: ring geometry, launch arguments and SiLU.
#pragma once

#include "engine_sync.h"

namespace bfsmoe {

using namespace bfsdev;

constexpr int kBK = 32;
constexpr int kLoadW = 2, kMmaW = 8, kEpiW = 2, kWaves = 12;
// ring slot: the token rows of one K step (8 KiB for M-tiles of 128 rows,
// 16 KiB for 256), then 256 weight rows (16 KiB)
constexpr uint32_t a_slot_bytes(int bm) { return (uint32_t)bm * kBK * 2; }
constexpr uint32_t slot_bytes(int bm) { return a_slot_bytes(bm) + 256 * kBK * 2; }
constexpr uint32_t kESlotBytes = kMmaW * 32 * 32 * 2;

struct MoeParams {
  SyncCommon sc;
  InstrWaits acql, load, mma, acqe, spill, epi;
  const int32_t *work;
  const int32_t *perm;
  const int32_t *eoff;
  const __bf16 *a;          // x (phase 1) or h (phase 2)
  const __bf16 *w0;         // W_gate (phase 1) or W_down (phase 2)
  const __bf16 *w1;         // W_up (phase 1)
  __bf16 *out;              // h (phase 1) or y (phase 2)
  const int32_t *trips;
  const int64_t *trip_off;
  int32_t kdim, ndim, ring, e_ring;
};

__device__ __forceinline__ uint32_t swz(uint32_t row, uint32_t chunk) {
  return row * 64u + ((chunk ^ ((row >> 2) & 3u)) << 4);
}

__device__ __forceinline__ float silu(float g) { return g * __builtin_amdgcn_rcpf(1.0f + __expf(-g)); }

// Barrier-free, uninstrumented launches: K steps in pairs, work items split where
// the grid leaves compute units idle, row blocks past the expert's count left
// out.  bm: the program's M-tile height; linear: MMA->LOAD read linearized.
// False (nothing launched) if the rings do not allow it or whole items are faster.
bool launch_parts(const MoeParams &P, int phase, int bm, bool linear, int n_wg, hipStream_t s, bfs_status &st);

}  // namespace bfsmoe
