// bf16 GEMM + bias + GELU on parts of a tile (the family's contract, engines
// and layouts are those of kern_gemm.hip).
//
// Grids that leave compute units idle: each 256 x 256 tile of the program
// runs as four workgroups of 128 x 128 or two of 256 x 128, the program's
// engines, waves, counters and dependencies on a part of the tile; every
// element keeps its order of K and so its bits.  A part reads LDS and HBM more
// per MFMA (sub-tiles of 64 x 32 or 64 x 64 per wave), which is why full grids
// keep whole tiles.
//
// What bounds a part is the hand-off between the engines: a wave has 4 or 8
// MFMAs per K step, too few to hide a counter poll and an LDS round trip
// under, and the program's ring allows four steps in flight.  So both engines
// take two steps at a time, waiting once, for the second one's threshold (the
// larger), and signalling both together; the MFMA waves read the next step's
// fragments into a second register set before the MFMAs of the current one;
// and a slot pair holds rows of 128 bytes (64 of K), so that every load
// instruction covers whole cache lines (16 rows of 64 bytes each move 16 TB/s
// from L2 at most, 8 rows of 128 bytes 27 TB/s).
#include <algorithm>
#include <string>

#include "gemm_common.h"

using namespace bfsdev;
using namespace bfsgemm;

namespace {

constexpr uint32_t kSpinPolls = 64;

// Part of kTM rows and kTN columns: the MFMA waves as kWM x kWN sub-tiles of
// 32 kRB rows and 32 kCB columns.
template <int kTM, int kTN>
struct Part {
  static constexpr int kWN = kTM == kTN ? 4 : 2, kWM = kMmaW / kWN, kRB = kTM / (32 * kWM), kCB = kTN / (32 * kWN);
  static constexpr uint32_t kASlot = kTM * kBK * 2, kSlot = kASlot + kTN * kBK * 2;   // one K step: A rows, B rows
};

// Byte offset of 16-byte chunk c (0 .. 7) of a 128-byte row: 16 rows read at
// one chunk cover all banks.
__device__ __forceinline__ uint32_t swz128(uint32_t row, uint32_t c) { return row * 128u + ((c ^ ((row >> 1) & 7u)) << 4); }

// The part at row block tm and column block tn (in units of parts) of the
// program's workgroup pwg.
template <int kTM, int kTN>
__device__ __forceinline__ void run_part(const GemmParams &P, unsigned char *lds, int tm, int tn, int pwg) {
  using G = Part<kTM, kTN>;
  uint32_t *cnt = reinterpret_cast<uint32_t *>(lds);
  const uint32_t ring = lds_addr(lds) + kCntBytes, ering = ring;
  const uint32_t bias_l = ring + (uint32_t)P.ring * G::kSlot;
  const int wave = wave_id();
  const uint32_t lane = lane_id();
  const int m0 = tm * kTM, n0 = tn * kTN;

  Sync<BFS_MODE_BARRIER_FREE, false, kSpinPolls, true> S(P.sc, lds_addr(cnt), wave, pwg);
  const int64_t *toff = P.trip_off + (int64_t)pwg * P.n_loops;
  uint32_t trip_k = (uint32_t)ldc(P.trips + ldc(toff + 1));
  uint32_t trip_c = (uint32_t)ldc(P.trips + ldc(toff + 2));
  if (trip_k > (uint32_t)(P.k / kBK) || trip_c > 8u) {
    report_input(P.sc.err, 2u, (uint32_t)pwg, 0u, trip_k, trip_c, (uint32_t)wave);
    trip_k = min(trip_k, (uint32_t)(P.k / kBK));
    trip_c = min(trip_c, 8u);
  }
  // The program's chunk (of a tile's eight) of block (rb, cb) of MFMA wave
  // (wm, wn): chunks beyond trip_c are not stored.
  auto chunk_of = [](uint32_t wm, uint32_t wn, uint32_t rb, uint32_t cb) {
    return ((wm * G::kRB + rb) & 3u) * 2u + ((wn * G::kCB + cb) & 1u);
  };
  Regs g;

  if (wave < kLoadW) {
    // ------------------------------------------------------------ load engine
    const uint32_t ew = (uint32_t)wave;
    Site<1> s_bias, s_load;
    S.enter(s_bias, P.bias, g, 0);
    S.wait(s_bias, P.bias, g, 1, 0, [] {});
    // BIAS: 16 bytes from each of kTN / 4 lanes; it lands with the first pair of steps and retires before it
    if (wave == 0 && !S.aborted && lane < (uint32_t)kTN / 4u)
      __builtin_amdgcn_global_load_lds((const void *)(P.bias_v + n0 + 4 * lane), (BFS_LDS void *)(uintptr_t)bias_l, 16, 0, 0);
    // Whole tiles: each wave loads half of every pair (64 KiB for one wave take
    // longer to issue than the other pair's MFMAs last; 256 tiles, K = 4096:
    // 129 us with a pair per wave, 124 split).  Smaller parts: the two waves
    // take the pairs in turn, so that neither waits for a landed load while
    // the other's slots come free (64 tiles in quarters, K = 2048: 32.1 us,
    // split 32.9).  A wave has no part in the other's pairs: those retire on
    // it at once, in order (its counter word counts every LOAD).
    constexpr bool kBoth = kTM == kTile && kTN == kTile;
    constexpr uint32_t kRows = kBoth ? 16u : 8u, kStep = kBoth ? 2u : 4u;   // rows per load, K steps per pass
    S.enter(s_load, P.load, g, 1);
    const char *abase = reinterpret_cast<const char *>(P.a + (size_t)m0 * P.k);
    const char *bbase = reinterpret_cast<const char *>(P.bt + (size_t)n0 * P.k);
    // load j: rows kRows j + r_in and the chunk that belongs at position
    // lane % 8; a single last step (n = 1): the lanes of its second half, which
    // K does not have, read the first half's bytes again (never used)
    constexpr int kALoads = kTM / (int)kRows, kBLoads = kTN / (int)kRows;
    const uint32_t r_in = (kBoth ? 8u * ew : 0u) + (lane >> 3);
    uint32_t voff[kALoads];
    auto offsets = [&](uint32_t n) __attribute__((always_inline)) {
      const uint32_t keep = n == 1u ? 3u : 7u;
#pragma unroll
      for (int j = 0; j < kALoads; ++j) {
        const uint32_t row = kRows * j + r_in, chunk = (lane & 7u) ^ ((row >> 1) & 7u);
        voff[j] = (row * (uint32_t)P.k + 8u * (chunk & keep)) * 2u;
      }
    };
    offsets(2u);
    const uint32_t last_slot = (uint32_t)P.ring / 2u - 1u;         // slot pairs: one or two
    auto retire = [&](uint32_t n) {
      if (P.load.update >= 0 && n > 0) lds_add(S.word((uint32_t)P.load.update, ew), n);
    };
    const uint32_t first = kBoth ? 0u : 2u * ew;
    if (first != 0u || trip_k == 0u) {
      wait_vm<0>();
      S.signal(P.bias.update, ew);
    }
    if (first != 0u) retire(min(trip_k, 2u));          // pair 0 is wave 0's
    for (uint32_t it = first; it < trip_k; it += kStep) {
      const uint32_t n = min(trip_k - it, 2u);
      g.r1 = it + n;
      g.h1 = it + n;
      S.wait_affine(s_load, P.load, g, it + n, it + n - 1u, [] {});
      if (!S.aborted) {
        const uint32_t dst = ring + ((it >> 1) & last_slot) * 2u * G::kSlot + (kBoth ? 1024u * ew : 0u);
        const size_t kb = (size_t)it * (kBK * 2);
        if (n == 1u) offsets(1u);
#pragma unroll
        for (int j = 0; j < kALoads; ++j) {
          asm volatile("" : "+v"(voff[j]));   // keep the offset a 32-bit value at its use
          __builtin_amdgcn_global_load_lds((const void *)(abase + kb + voff[j]), (BFS_LDS void *)(uintptr_t)(dst + j * (kRows * 128u)), 16, 0, 0);
        }
#pragma unroll
        for (int j = 0; j < kBLoads; ++j) {
          asm volatile("" : "+v"(voff[j]));
          __builtin_amdgcn_global_load_lds((const void *)(bbase + kb + voff[j]),
                                           (BFS_LDS void *)(uintptr_t)(dst + 2u * G::kASlot + j * (kRows * 128u)), 16, 0, 0);
        }
        wait_vm<0>();
      }
      if (it == 0u) S.signal(P.bias.update, ew);
      retire(n + (kBoth ? 0u : min(trip_k - it - n, 2u)));         // and the other wave's next pair
    }
  } else if (wave < kLoadW + kMmaW) {
    // ------------------------------------------------------------ MFMA engine
    const uint32_t ew = (uint32_t)(wave - kLoadW);
    const uint32_t wm = ew / G::kWN, wn = ew % G::kWN;
    f32x16 acc[G::kRB][G::kCB];
#pragma unroll
    for (int rb = 0; rb < G::kRB; ++rb)
#pragma unroll
      for (int cb = 0; cb < G::kCB; ++cb) acc[rb][cb] = f32x16{};
    Site<1> s_mma, s_spill;
    Site<3> s_once;
    S.enter(s_mma, P.mma, g, 1);
    const uint32_t l32 = lane & 31u, lhi = lane >> 5;
    // this lane's chunk of slice 0 (16 of K) in its first A and B row; slice
    // s is the offset XOR 32 s, the next block of 32 rows 4096 bytes on
    const uint32_t a_off = ring + swz128(wm * 32u * G::kRB + l32, lhi);
    const uint32_t b_off = ring + 2u * G::kASlot + swz128(wn * 32u * G::kCB + l32, lhi);
    auto rd = [](uint32_t addr) { return __builtin_bit_cast(bf16x8, *(const BFS_LDS u32x4 *)(uintptr_t)addr); };
    uint32_t pslot = 0;                      // slot pair
    const uint32_t pairs = (uint32_t)P.ring / 2u;
    if constexpr (kTM == kTile && kTN == kTile) {
      // Whole tile: 128 accumulators per lane leave room for the fragments of
      // one slice.  Each A fragment is refilled with the next slice's as soon
      // as its two MFMAs are issued, the B pair after the last row block, so
      // that the next slice's LDS reads run under these MFMAs; the scheduling
      // barriers keep the compiler from hoisting the refills (a second
      // register set) or sinking them.
      bf16x8 fa[G::kRB], fb[G::kCB];
      for (uint32_t it = 0; it < trip_k; it += 2) {
        const uint32_t n = min(trip_k - it, 2u);
        g.r1 += n;
        g.h1 += n;
        S.wait_affine(s_mma, P.mma, g, g.h1, g.r1 - 1, [] {});
        const uint32_t base = pslot * 2u * G::kSlot;
        pslot = pslot + 1 == pairs ? 0u : pslot + 1;
#pragma unroll
        for (int cb = 0; cb < G::kCB; ++cb) fb[cb] = rd(b_off + base + 4096u * cb);
#pragma unroll
        for (int rb = 0; rb < G::kRB; ++rb) fa[rb] = rd(a_off + base + 4096u * rb);
        auto slice = [&](int s, bool refill) __attribute__((always_inline)) {
          const uint32_t x = 32u * (s + 1);
#pragma unroll
          for (int rb = 0; rb < G::kRB; ++rb) {
#pragma unroll
            for (int cb = 0; cb < G::kCB; ++cb)
              acc[rb][cb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[cb], fa[rb], acc[rb][cb], 0, 0, 0);
            if (refill) {
              fa[rb] = rd((a_off ^ x) + base + 4096u * rb);
              if (rb == G::kRB - 1) {
#pragma unroll
                for (int cb = 0; cb < G::kCB; ++cb) fb[cb] = rd((b_off ^ x) + base + 4096u * cb);
              }
            }
            __builtin_amdgcn_sched_barrier(0);
          }
        };
        // MMA retires from the slots once its last reads are issued (LDS
        // executes them before the signal)
        slice(0, true);
        if (n == 2u) {
          slice(1, true);
          slice(2, true);
        }
        if (P.mma.update >= 0) lds_add(S.word((uint32_t)P.mma.update, ew), n);
        slice(3, false);
      }
    } else {
      struct Frags {
        bf16x8 a[2][G::kRB], b[2][G::kCB];     // [slice of the step][block]
      };
      // Reads the fragments of step h of a pair (0: after the wait for the pair,
      // or for the last single step; 1).  MMA retires from the pair once its
      // last reads are issued (LDS executes the reads before the signal).
      auto fetch = [&](Frags &f, int h, uint32_t n) __attribute__((always_inline)) {
        if (h == 0) {
          g.r1 += n;
          g.h1 += n;
          S.wait_affine(s_mma, P.mma, g, g.h1, g.r1 - 1, [] {});
        }
        const uint32_t base = pslot * 2u * G::kSlot;
#pragma unroll
        for (int s = 0; s < 2; ++s) {
          const uint32_t x = 32u * (2 * h + s);
#pragma unroll
          for (int cb = 0; cb < G::kCB; ++cb) f.b[s][cb] = rd((b_off ^ x) + base + 4096u * cb);
#pragma unroll
          for (int rb = 0; rb < G::kRB; ++rb) f.a[s][rb] = rd((a_off ^ x) + base + 4096u * rb);
        }
        if (h == 1 || n == 1u) {
          if (P.mma.update >= 0) lds_add(S.word((uint32_t)P.mma.update, ew), n);
          pslot = pslot + 1 == pairs ? 0u : pslot + 1;
        }
      };
      auto mma = [&](const Frags &f) __attribute__((always_inline)) {
#pragma unroll
        for (int s = 0; s < 2; ++s)
#pragma unroll
          for (int rb = 0; rb < G::kRB; ++rb)
#pragma unroll
            for (int cb = 0; cb < G::kCB; ++cb)
              acc[rb][cb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.b[s][cb], f.a[s][rb], acc[rb][cb], 0, 0, 0);
      };
      Frags f0, f1;                            // even and odd steps
      const uint32_t full = trip_k / 2;
      if (full > 0) {
        fetch(f0, 0, 2);
        for (uint32_t p = 1; p < full; ++p) {
          fetch(f1, 1, 2);
          mma(f0);
          fetch(f0, 0, 2);
          mma(f1);
        }
        fetch(f1, 1, 2);
        mma(f0);
        if (trip_k & 1u) fetch(f0, 0, 1);
        mma(f1);
      } else if (trip_k & 1u) {
        fetch(f0, 0, 1);
      }
      if (trip_k & 1u) mma(f0);
    }
    // SPILL: the waits that stay the same for all chunks once, then per chunk
    // the epilogue slot's
    S.enter(s_once, P.spill_once, g, 2);
    S.enter(s_spill, P.spill, g, 2);
    S.wait_affine(s_once, P.spill_once, g, 1, g.r2, [] {});
#pragma unroll
    for (uint32_t c = 0; c < G::kRB * G::kCB; ++c) {
      const uint32_t rb = c / G::kCB, cb = c % G::kCB;
      g.r2 += 1;
      g.h2 = c + 1;
      S.wait_affine(s_spill, P.spill, g, c + 1, g.r2 - 1, [] {});
      if (!S.aborted && chunk_of(wm, wn, rb, cb) < trip_c) {
        const uint32_t blk = ering + (c & (uint32_t)(P.e_ring - 1)) * kESlotBytes + ew * 2048u;
        const f32x16 v = acc[rb][cb];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const uint32_t ncol = (wn * G::kCB + cb) * 32u + 8u * j + 4u * lhi;      // first of 4 columns
          const f32x4 bb = *(const BFS_LDS f32x4 *)(uintptr_t)(bias_l + 4u * ncol);
          const float x0 = gelu_erf(v[4 * j + 0] + bb.x), x1 = gelu_erf(v[4 * j + 1] + bb.y);
          const float x2 = gelu_erf(v[4 * j + 2] + bb.z), x3 = gelu_erf(v[4 * j + 3] + bb.w);
          const bf16x2 p01 = __builtin_convertvector(f32x2{x0, x1}, bf16x2);
          const bf16x2 p23 = __builtin_convertvector(f32x2{x2, x3}, bf16x2);
          const u32x2 q = {__builtin_bit_cast(uint32_t, p01), __builtin_bit_cast(uint32_t, p23)};
          *(BFS_LDS u32x2 *)(uintptr_t)(blk + l32 * 64u + (8u * j + 4u * lhi) * 2u) = q;
        }
      }
      S.signal(P.spill.update, ew);
    }
  } else {
    // -------------------------------------------------------- epilogue engine
    const uint32_t ew = (uint32_t)(wave - kLoadW - kMmaW);
    Site<1> s_epi;
    g.r1 = trip_k;
    g.h1 = trip_k;
    S.enter(s_epi, P.epi, g, 2);
    for (uint32_t c = 0; c < G::kRB * G::kCB; ++c) {
      const uint32_t rb = c / G::kCB, cb = c % G::kCB;
      g.r2 += 1;
      g.h2 = c + 1;
      S.wait_affine(s_epi, P.epi, g, c + 1, g.r2 - 1, [] {});
      if (!S.aborted) {
        const uint32_t eslot = c & (uint32_t)(P.e_ring - 1);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const uint32_t v = ew * 4u + q;              // MFMA wave whose block this is
          const uint32_t vm = v / G::kWN, vn = v % G::kWN;
          if (chunk_of(vm, vn, rb, cb) >= trip_c) continue;
          const uint32_t blk = ering + eslot * kESlotBytes + v * 2048u;
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            const uint32_t row = 16u * h + (lane >> 2), cc = lane & 3u;
            const u32x4 d = *(const BFS_LDS u32x4 *)(uintptr_t)(blk + row * 64u + cc * 16u);
            const size_t gm = (size_t)m0 + (vm * G::kRB + rb) * 32u + row;
            const size_t gn = (size_t)n0 + (vn * G::kCB + cb) * 32u + 8u * cc;
            *reinterpret_cast<u32x4 *>(P.c + gm * P.n + gn) = d;
          }
        }
      }
      S.signal(P.epi.update, ew);
    }
  }
  drain_all();
}

// Tile of the program's workgroup p.
__device__ __forceinline__ void tile_of(const GemmParams &P, int p, int &tm, int &tn) {
  if (P.xcd_map) {
    const int br = P.tiles_m / 4, bc = P.tiles_n / 2, xcd = p & 7, local = p >> 3;
    tm = (xcd >> 1) * br + local / bc;
    tn = (xcd & 1) * bc + local % bc;
  } else {
    tm = p / P.tiles_n;
    tn = p % P.tiles_n;
  }
}

__device__ __forceinline__ void clear_counters(unsigned char *lds) {
  uint32_t *cnt = reinterpret_cast<uint32_t *>(lds);
  for (int i = threadIdx.x; i < bfs::kMaxSlots * bfs::kMaxWavesPerEngine; i += blockDim.x) cnt[i] = 0;
  __syncthreads();
}

// Every tile in parts of kTM x kTN; the parts that share A or B rows run on
// one XCD, as whole tiles do.
template <int kTM, int kTN>
__global__ void __launch_bounds__(768) gemm_part_kernel(GemmParams P) {
  extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
  clear_counters(lds);
  constexpr int kUp = kTile / kTM, kBy = kTile / kTN;   // parts of a tile one above the other and beside each other
  const int wg = blockIdx.x, qm = kUp * P.tiles_m, qn = kBy * P.tiles_n;
  int tm, tn, pwg;
  if (P.xcd_map) {
    const int xcd = wg & 7, local = wg >> 3;
    const int br = qm / 4, bc = qn / 2;
    tm = (xcd >> 1) * br + local / bc;
    tn = (xcd & 1) * bc + local % bc;
    const int pbr = P.tiles_m / 4, pbc = P.tiles_n / 2, ptm = tm / kUp, ptn = tn / kBy;
    pwg = ((ptm % pbr) * pbc + ptn % pbc) * 8 + (ptm / pbr) * 2 + ptn / pbc;
  } else {
    tm = wg / qn;
    tn = wg % qn;
    pwg = (tm / kUp) * P.tiles_n + tn / kBy;
  }
  run_part<kTM, kTN>(P, lds, tm, tn, pwg);
}

// The first P.n_whole workgroups of the program as whole tiles, the rest in
// parts of kTM x kTN.
template <int kTM, int kTN>
__global__ void __launch_bounds__(768) gemm_mixed_kernel(GemmParams P) {
  extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
  clear_counters(lds);
  constexpr int kUp = kTile / kTM, kBy = kTile / kTN;
  int tm, tn;
  if ((int)blockIdx.x < P.n_whole) {
    tile_of(P, blockIdx.x, tm, tn);
    run_part<kTile, kTile>(P, lds, tm, tn, blockIdx.x);
  } else {
    const int q = blockIdx.x - P.n_whole, pwg = P.n_whole + q / (kUp * kBy), sub = q % (kUp * kBy);
    tile_of(P, pwg, tm, tn);
    run_part<kTM, kTN>(P, lds, tm * kUp + sub / kBy, tn * kBy + sub % kBy, pwg);
  }
}

}  // namespace

// Which grids run in parts (us at K = 4096 and in brackets at K = 512; whole
// tiles, halves, quarters on 256 compute units):
//   64 tiles    95 (27)   64 (19)   52 (14)     a quarter each: one round
//   128 tiles  100 (29)   76 (21)  103 (26)     a half each: one round
//   168 tiles   97 (28)  132 (36)  147 (36)     whole tiles: one round
// Beyond 256 tiles the last round of whole tiles, if it leaves half of the
// compute units or more idle, runs in parts by the same rule (272 tiles: 160
// against 207 us in two rounds of whole tiles).
bool bfsgemm::launch_parts(GemmParams &P, int n_wg, hipStream_t s, bfs_status &st) {
  constexpr int kCUs = 256;
  if (P.ring % 2 != 0) return false;       // the ring is used in pairs of slots
  // A pair of loads waits for what its second step does, so that must not be an
  // MMA of the pair itself: an offset of 1 leaves one step in flight (K step by
  // K step instead).
  for (int j = 0; j < P.load.n; ++j)
    if ((P.load.w[j].w.w2 & 0xffffu) < 2u) return false;
  // SPILL's waits on loops outside C are constant during its trip
  InstrWaits once = P.spill, chunk = P.spill;
  once.n = chunk.n = 0;
  for (int j = 0; j < P.spill.n; ++j) {
    InstrWaits &to = P.spill.w[j].kind == kWaitConst ? once : chunk;
    to.w[to.n++] = P.spill.w[j];
  }
  if (!bfs::no_dynamic(chunk) || !bfs::waits_fit({{&once, 3}, {&chunk, 1}})) return false;
  const int rest = n_wg % kCUs;
  int parts = rest == 0 ? 1 : 4 * rest <= kCUs ? 4 : 2 * rest <= kCUs ? 2 : 1;
  // halves: the epilogue slots in use must fit the smaller ring
  if (parts == 2 && (size_t)std::min(P.e_ring, 4) * kESlotBytes > (size_t)P.ring * Part<256, 128>::kSlot) parts = 1;
  // A ring of two slots holds one pair, so that a whole tile's loads and MMAs
  // take turns: single steps overlap.  (us step by step and in pairs, 256 tiles:
  // K = 4096 139 and 151, 512 34 and 32, 96 23 and 19; 168 tiles, K = 4096, 120
  // and 145; 128 tiles, not in halves as four epilogue slots do not fit there,
  // K = 1024 43 and 46.)
  if (P.ring == 2 && parts == 1 && P.k > 512) return false;
  P.spill_once = once;
  P.spill = chunk;
  P.n_whole = n_wg - rest;
  auto go = [&](auto kern, uint32_t slot, int columns, int grid) {
    const size_t lds = kCntBytes + (size_t)P.ring * slot + 4 * columns;
    hipError_t e = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) {
      st = bfs::fail(BFS_E_DEVICE, std::string("gemm attribute: ") + hipGetErrorString(e));
      return;
    }
    hipLaunchKernelGGL(kern, dim3(grid), dim3(64 * kWaves), lds, s, P);
    e = hipGetLastError();
    st = e == hipSuccess ? BFS_OK : bfs::fail(BFS_E_DEVICE, std::string("gemm launch: ") + hipGetErrorString(e));
  };
  const int grid = P.n_whole + parts * rest;
  if (parts == 1) go(gemm_part_kernel<256, 256>, Part<256, 256>::kSlot, 256, grid);
  else if (P.n_whole > 0 && parts == 4) go(gemm_mixed_kernel<128, 128>, Part<256, 256>::kSlot, 256, grid);
  else if (P.n_whole > 0) go(gemm_mixed_kernel<256, 128>, Part<256, 256>::kSlot, 256, grid);
  else if (parts == 4) go(gemm_part_kernel<128, 128>, Part<128, 128>::kSlot, 128, grid);
  else go(gemm_part_kernel<256, 128>, Part<256, 128>::kSlot, 128, grid);
  return true;
}
