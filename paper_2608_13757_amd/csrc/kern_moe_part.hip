// MoE grouped GEMM on parts of the program's work items (the family's
// contract, engines and dependencies are those of kern_moe.hip), for
// barrier-free uninstrumented launches.
//
// A work item (expert, 256 weight rows, run of M-tiles) is cut into units of
// kPM token rows by kPN weight rows; a workgroup runs every sm-th unit of the
// item's rows (and one of sn column parts), with the program's loops, waves,
// counters and dependencies on a unit in place of an M-tile.  Every output
// element keeps its order of K and so its bits.
//
// What bounds a unit is the way of its rows from L2 into LDS: 64 KiB per pair
// of K steps for 0.86 us of MFMAs, with two pairs in the ring, so a pair's
// loads have to land within one pair's MFMAs.
//
//   * K steps go in pairs: one wait, for the second step's threshold, and rows
//     of 128 bytes (64 of K) in the ring, so that every load instruction covers
//     whole cache lines.  Both load waves load half of each pair: with a pair
//     per wave in turn its 64 load instructions issue one after another (one
//     expert of 256 rows, K = 4096: 115 us; split 84 us; single steps of
//     64-byte rows 94 us).
//   * A unit's token rows past the expert's count are not loaded, multiplied or
//     stored, by blocks of 32 rows.  Blocks alternate between the MFMA waves
//     that share a column block, so a unit with v valid blocks takes
//     ceil(v / 2) blocks' MFMAs; units without valid rows are not run.
//   * An item's units go to several workgroups: on small grids to fill the
//     compute units, on large ones to run together (they read the same weights).
//
// 32768 tokens, 64 experts, K = 4096 and 1408 (us of phase 1 and 2 with whole
// items in single steps, then here): 1100 and 570, 951 and 497.
#include <string>
#include <type_traits>

#include "moe_common.h"

using namespace bfsdev;
using namespace bfsmoe;

namespace {

constexpr uint32_t kSpinPolls = 64;

// Units of kPM token rows and kPN weight rows: the MFMA waves as kWM x kWN,
// each with kRB blocks of 32 token rows (block kWM rb + wm of the unit) and two
// blocks of 32 weight rows (phase 1: gate and up of the same 32 columns).
template <int kPM_, int kPN_>
struct Unit {
  static constexpr int kPM = kPM_, kPN = kPN_;
  static constexpr int kWN = kPN / 64, kWM = kMmaW / kWN, kRB = kPM / (32 * kWM);
  static constexpr uint32_t kASlot = kPM * kBK * 2, kSlot = kASlot + kPN * kBK * 2;   // one K step: token rows, weight rows
};

struct Split {
  int32_t bm;        // the program's M-tile height
  int32_t sm, sn;    // workgroups of an item: units of its rows in turn, column parts
  int32_t n_wg;      // items
  int32_t items;     // ... rounded up to a multiple of 8
  int32_t table;     // moe_many_kernel: byte offset of its items in LDS
  int32_t slots;     // ring slots in LDS (even)
};

// Byte offset of 16-byte chunk c (0 .. 7) of a 128-byte row: 16 rows read at
// one chunk cover all banks.
__device__ __forceinline__ uint32_t swz128(uint32_t row, uint32_t c) { return row * 128u + ((c ^ ((row >> 1) & 7u)) << 4); }

// A work item: its expert, first output column and M-tile, the expert's first
// grouped row and row count, and the M loop's trip.
struct Item {
  int32_t expert, n0, mt0, e_lo, e_cnt;
  uint32_t trip_m;
};

__device__ __forceinline__ Item read_item(const MoeParams &P, int wg) {
  Item x;
  x.expert = ldc(P.work + 4 * wg + 0);
  x.n0 = ldc(P.work + 4 * wg + 1);
  x.mt0 = ldc(P.work + 4 * wg + 2);
  x.e_lo = ldc(P.eoff + x.expert);
  x.e_cnt = ldc(P.eoff + x.expert + 1) - x.e_lo;
  x.trip_m = (uint32_t)ldc(P.trips + ldc(P.trip_off + (int64_t)wg * 4 + 1));
  return x;
}

// The units of item wg that fall to its workgroup sub (of sm * sn).
template <int kPhase, int kPM, int kPN>
__device__ __forceinline__ void run_units(const MoeParams &P, const Split &D, unsigned char *lds, int wg, int sub,
                                          const Item &I) {
  using G = Unit<kPM, kPN>;
  uint32_t *cnt = reinterpret_cast<uint32_t *>(lds);
  const uint32_t ring = lds_addr(lds) + kCntBytes;
  const uint32_t ering = P.e_ring == 0 ? ring : ring + (uint32_t)D.slots * G::kSlot;

  const int sm = sub / D.sn, sn = sub % D.sn;
  const int wave = wave_id();
  const uint32_t lane = lane_id(), l32 = lane & 31u, lhi = lane >> 5;
  const int32_t expert = I.expert, mt0 = I.mt0, e_lo = I.e_lo, e_cnt = I.e_cnt;
  const int32_t n0 = I.n0 + sn * (kPhase == 1 ? kPN / 2 : kPN);
  const int64_t *toff = P.trip_off + (int64_t)wg * 4;
  uint32_t trip_m = I.trip_m;
  const int64_t k_off = ldc(toff + 2), c_off = ldc(toff + 3);
  const uint32_t ksteps = (uint32_t)(P.kdim / kBK);
  const uint32_t max_m = (uint32_t)max(0, (e_cnt + D.bm - 1) / D.bm - mt0);
  if (trip_m > max_m) {
    report_input(P.sc.err, 1u, (uint32_t)wg, 1u, trip_m, max_m, (uint32_t)wave);
    trip_m = max_m;
  }
  // units of the item with valid rows, and this workgroup's share of them
  const int32_t row_lo = mt0 * D.bm, row_hi = min(row_lo + (int32_t)trip_m * D.bm, e_cnt);
  const int32_t units = row_hi > row_lo ? (row_hi - row_lo + kPM - 1) / kPM : 0;
  const uint32_t trip_u = units > sm ? (uint32_t)((units - sm + D.sm - 1) / D.sm) : 0u;
  if (trip_u == 0u) return;
  auto unit_row = [&](uint32_t i) { return row_lo + (sm + (int32_t)i * D.sm) * kPM; };
  // 32-row blocks of a unit that hold rows of the expert
  auto blocks_of = [&](int32_t row0) { return (uint32_t)(min(row_hi - row0, kPM) + 31) / 32u; };

  for (int i = threadIdx.x; i < bfs::kMaxSlots * bfs::kMaxWavesPerEngine; i += blockDim.x) cnt[i] = 0;
  __syncthreads();
  Sync<BFS_MODE_BARRIER_FREE, false, kSpinPolls, true> S(P.sc, lds_addr(cnt), wave, wg);
  constexpr uint32_t kChunks = kPhase == 1 ? (uint32_t)G::kRB : 2u * G::kRB;   // per unit
  const uint32_t pairs = (uint32_t)D.slots / 2u;
  Regs g;
  Site<1> sa, sb, sc;               // one per wait site of the engine (each has one wait)
  uint32_t pslot = 0;               // slot pair

  if (wave < kLoadW) {
    // ------------------------------------------------------------ load engine
    const uint32_t ew = (uint32_t)wave;
    // per pair and wave, 8 rows each: load j of wave ew covers rows 16 j + 8 ew ..
    constexpr int kALoads = kPM / 16, kBLoads = kPN / 16;
    // this lane's row there is r_in on; chunk: the 16 bytes of its row that
    // belong at position lane % 8
    const uint32_t r_in = 8u * ew + (lane >> 3);
    const uint32_t chunk = (lane & 7u) ^ ((r_in >> 1) & 7u);
    // the token ids of a unit's rows (gathered through perm in phase 1) are
    // loaded during the previous unit
    int32_t prow[kALoads];
    auto load_rows = [&](uint32_t i) __attribute__((always_inline)) {
      const int32_t m0 = unit_row(i);
#pragma unroll
      for (int j = 0; j < kALoads; ++j) {
        const int32_t r = min(m0 + 16 * j + (int32_t)r_in, e_cnt - 1);
        prow[j] = kPhase == 1 ? P.perm[e_lo + r] : e_lo + r;
      }
    };
    load_rows(0);
    S.enter(sa, P.acql, g, 1);
    for (uint32_t i = 0; i < trip_u; ++i) {
      g.r1 += 1;
      g.h1 = i + 1;
      S.wait(sa, P.acql, g, i + 1, g.r1 - 1, [] {});            // ACQL
      S.signal(P.acql.update, ew);
      // the K and C loops have static trips; a trip table that disagrees is
      // reported (the static trips run)
      const int32_t m0 = unit_row(i);
      if (wave == 0) {
        const int32_t mi = (m0 - row_lo) / D.bm, chunks = kPhase == 1 ? D.bm / 64 : D.bm / 32;
        const int32_t tk = ldc(P.trips + k_off + mi), tc = ldc(P.trips + c_off + mi);
        if (tk != (int32_t)ksteps || tc != chunks)
          report_input(P.sc.err, 2u, (uint32_t)wg, (uint32_t)mi, (uint32_t)tk, (uint32_t)tc, (uint32_t)wave);
      }
      // source rows as 32-bit per-lane byte offsets from a wave-uniform base
      // that advances with K (no vector address arithmetic in the loop)
      uint32_t voff[kALoads];
      uint32_t over = 0;              // offsets beyond 32 bits
#pragma unroll
      for (int j = 0; j < kALoads; ++j) {
        const uint64_t off = ((uint64_t)(uint32_t)prow[j] * (uint32_t)P.kdim + 8u * chunk) * 2u;
        over = max(over, (uint32_t)(off >> 32) != 0u ? (uint32_t)prow[j] : 0u);
        voff[j] = (uint32_t)off;
      }
      if (__ballot(over != 0u) != 0ull) {
        report_input(P.sc.err, 3u, (uint32_t)wg, i, over, 0u, (uint32_t)wave);
        S.aborted = 1u;
      }
      // phase 1: the first half of the weight rows is W_gate's, the second W_up's
      constexpr int kHalf = kPhase == 1 ? kBLoads / 2 : kBLoads;
      uint32_t woff[kBLoads];
#pragma unroll
      for (int j = 0; j < kBLoads; ++j)
        woff[j] = ((16u * (uint32_t)(j % kHalf) + r_in) * (uint32_t)P.kdim + 8u * chunk) * 2u;
      if (i + 1 < trip_u) load_rows(i + 1);
      uint32_t blocks = blocks_of(m0);
      const size_t eb = ((size_t)expert * P.ndim + (size_t)n0) * P.kdim * 2;
      const char *w0 = reinterpret_cast<const char *>(P.w0) + eb;
      const char *w1 = kPhase == 1 ? reinterpret_cast<const char *>(P.w1) + eb : w0;
      S.enter(sb, P.load, g, 2);
      const uint32_t k0 = g.r2;
      for (uint32_t it = 0; it < ksteps; it += 2) {
        const uint32_t n = min(ksteps - it, 2u);
        g.r2 = k0 + it + n;
        g.h2 = it + n;
        S.wait_affine(sb, P.load, g, it + 2u, g.r2 - 1, [] {});   // (a single last step's pair of slots too)
        if (!S.aborted) {
          uint32_t sl = pslot + (it >> 1);
          sl -= sl >= pairs ? (sl / pairs) * pairs : 0u;
          const uint32_t dst = ring + sl * 2u * G::kSlot;
          const size_t kb = (size_t)it * (kBK * 2);
          const char *ab = reinterpret_cast<const char *>(P.a) + kb, *wb0 = w0 + kb, *wb1 = w1 + kb;
          // a single last step: the lanes of its second half, which K does
          // not have, read the first half's bytes again (never used; it is
          // the unit's last step, so the offsets need not be put back)
          if (n == 1u) {
            const uint32_t back = (chunk & 4u) * 16u;
#pragma unroll
            for (int j = 0; j < kALoads; ++j) voff[j] -= back;
#pragma unroll
            for (int j = 0; j < kBLoads; ++j) woff[j] -= back;
          }
          asm volatile("" : "+s"(blocks));   // (compared here, not kept as masks)
#pragma unroll
          for (int j = 0; j < kALoads; ++j) {
            if ((uint32_t)(j / 2) < blocks) {
              asm volatile("" : "+v"(voff[j]));   // keep the offset a 32-bit value at its use
              __builtin_amdgcn_global_load_lds((const void *)(ab + voff[j]), (BFS_LDS void *)(uintptr_t)(dst + 2048u * j + 1024u * ew), 16, 0, 0);
            }
          }
#pragma unroll
          for (int j = 0; j < kBLoads; ++j) {
            asm volatile("" : "+v"(woff[j]));
            __builtin_amdgcn_global_load_lds((const void *)((j < kHalf ? wb0 : wb1) + woff[j]),
                                             (BFS_LDS void *)(uintptr_t)(dst + 2u * G::kASlot + 2048u * j + 1024u * ew), 16, 0, 0);
          }
          wait_vm<0>();
        }
        if (P.load.update >= 0) lds_add(S.word((uint32_t)P.load.update, ew), n);
      }
      g.r2 = k0 + ksteps;
      g.h2 = ksteps;
      pslot = (pslot + (ksteps + 1u) / 2u) % pairs;
      g.r3 += kChunks;
      g.h3 = kChunks;
    }
  } else if (wave < kLoadW + kMmaW) {
    // ------------------------------------------------------------ MFMA engine
    const uint32_t ew = (uint32_t)(wave - kLoadW);
    const uint32_t wm = ew / G::kWN, wn = ew % G::kWN;
    // this lane's chunk of slice 0 (16 of K) in its first token row and in its
    // row of the two weight blocks; slice s is the offset XOR 32 s, token
    // block rb another 4096 kWM rb bytes on
    const uint32_t brow0 = kPhase == 1 ? 32u * wn + l32 : 64u * wn + l32;
    constexpr uint32_t b_step = (kPhase == 1 ? kPN / 2 : 32) * 128u;
    uint32_t a_off = ring + swz128(32u * wm + l32, lhi), b_off = ring + 2u * G::kASlot + swz128(brow0, lhi);
    auto rd = [](uint32_t addr) { return __builtin_bit_cast(bf16x8, *(const BFS_LDS u32x4 *)(uintptr_t)addr); };
    S.enter(sb, P.acqe, g, 1);
    f32x16 acc[2][G::kRB];            // [weight block][token block]
    // waits for the next pair (or last single step) of n steps; its offset in the ring
    auto wait_pair = [&](uint32_t n) __attribute__((always_inline)) {
      g.r2 += n;
      g.h2 += n;
      S.wait_affine(sa, P.mma, g, g.h2, g.r2 - 1, [] {});
      return pslot * 2u * G::kSlot;
    };
    // MMA retires from the pair once its last reads are issued (LDS executes
    // a wave's reads before the signal that follows them)
    auto release = [&](uint32_t n) __attribute__((always_inline)) {
      if (P.mma.update >= 0) lds_add(S.word((uint32_t)P.mma.update, ew), n);
      pslot = pslot + 1 == pairs ? 0u : pslot + 1;
    };
    // The K loop on this wave's first `mine` token blocks (its first one always:
    // one loop with a branch per further block keeps the accumulators in place,
    // a loop for each count does not).
    auto k_loop = [&](uint32_t mine) __attribute__((always_inline)) {
      if constexpr (G::kRB == 4) {
        // 128 accumulators per lane leave room for the fragments of one
        // slice: each is refilled with the next slice's as soon as its MFMAs
        // are issued; the scheduling barriers keep the compiler from hoisting
        // the refills (a second register set) or sinking them
        bf16x8 fa[G::kRB], fb[2];
        for (uint32_t it = 0; it < ksteps; it += 2) {
          const uint32_t n = min(ksteps - it, 2u);
          const uint32_t base = wait_pair(n);
          fb[0] = rd(b_off + base);
          fb[1] = rd(b_off + base + b_step);
#pragma unroll
          for (int rb = 0; rb < G::kRB; ++rb) fa[rb] = rd(a_off + base + 4096u * G::kWM * rb);
          auto slice = [&](int s, auto refill) __attribute__((always_inline)) {
            asm volatile("" : "+v"(a_off), "+v"(b_off));   // (no register for every slice's offset)
            const uint32_t a_s = (a_off ^ (32u * (s + 1))) + base, b_s = (b_off ^ (32u * (s + 1))) + base;
#pragma unroll
            for (int rb = 0; rb < G::kRB; ++rb) {
              asm volatile("" : "+s"(mine));   // (compared here, not kept as masks)
              if (rb == 0 || (uint32_t)rb < mine) {
                acc[0][rb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[0], fa[rb], acc[0][rb], 0, 0, 0);
                acc[1][rb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[1], fa[rb], acc[1][rb], 0, 0, 0);
                if constexpr (decltype(refill)::value) fa[rb] = rd(a_s + 4096u * G::kWM * rb);
              }
              __builtin_amdgcn_sched_barrier(0);
            }
            if constexpr (decltype(refill)::value) {
              fb[0] = rd(b_s);
              fb[1] = rd(b_s + b_step);
            }
          };
          using Refill = std::true_type;
          using NoRefill = std::false_type;
          slice(0, Refill{});
          if (n == 2u) {
            slice(1, Refill{});
            slice(2, Refill{});
          }
          release(n);
          slice(3, NoRefill{});
        }
      } else {
        // the next step's fragments are read into a second register set before
        // the MFMAs of the current one
        struct Frags {
          bf16x8 a[2][G::kRB], b[2][2];      // [slice of the step][block]
        };
        uint32_t base = 0;
        auto fetch = [&](Frags &f, int h, uint32_t n) __attribute__((always_inline)) {
          if (h == 0) base = wait_pair(n);
#pragma unroll
          for (int s = 0; s < 2; ++s) {
            const uint32_t x = 32u * (2 * h + s);
            f.b[s][0] = rd((b_off ^ x) + base);
            f.b[s][1] = rd((b_off ^ x) + base + b_step);
#pragma unroll
            for (int rb = 0; rb < G::kRB; ++rb) f.a[s][rb] = rd((a_off ^ x) + base + 4096u * G::kWM * rb);
          }
          if (h == 1 || n == 1u) release(n);
        };
        auto mma = [&](const Frags &f) __attribute__((always_inline)) {
#pragma unroll
          for (int rb = 0; rb < G::kRB; ++rb)
            if (rb == 0 || (uint32_t)rb < mine) {
#pragma unroll
              for (int s = 0; s < 2; ++s) {
                acc[0][rb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.b[s][0], f.a[s][rb], acc[0][rb], 0, 0, 0);
                acc[1][rb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.b[s][1], f.a[s][rb], acc[1][rb], 0, 0, 0);
              }
            }
        };
        Frags f0, f1;
        const uint32_t full = ksteps / 2;
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
          if (ksteps & 1u) fetch(f0, 0, 1);
          mma(f1);
        } else {
          fetch(f0, 0, 1);
        }
        if (ksteps & 1u) mma(f0);
      }
    };
    for (uint32_t i = 0; i < trip_u; ++i) {
      g.r1 += 1;
      g.h1 = i + 1;
#pragma unroll
      for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int rb = 0; rb < G::kRB; ++rb) acc[b][rb] = f32x16{};
      const uint32_t v = blocks_of(unit_row(i));
      const uint32_t mine = v > wm ? (v - wm + G::kWM - 1) / G::kWM : 0u;   // this wave's blocks
      S.enter(sa, P.mma, g, 2);
      g.h2 = 0;
      k_loop(mine);
      S.wait(sb, P.acqe, g, i + 1, g.r1 - 1, [] {});                    // ACQE
      S.signal(P.acqe.update, ew);
      S.enter(sc, P.spill, g, 3);
#pragma unroll
      for (uint32_t c = 0; c < kChunks; ++c) {
        constexpr uint32_t kCB = kPhase == 1 ? 1u : 2u;          // chunk = token block (phase 1), times weight block (2)
        const uint32_t rb = c / kCB, cb = c % kCB;
        g.r3 += 1;
        g.h3 = c + 1;
        S.wait_affine(sc, P.spill, g, c + 1, g.r3 - 1, [] {});
        if (!S.aborted && rb < mine) {
          const uint32_t eslot = P.e_ring == 0 ? c : (P.e_ring == 2 ? ((g.r3 - 1) & 1u) : 0u);
          const uint32_t blk = ering + eslot * kESlotBytes + ew * 2048u;
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            float x[4];
#pragma unroll
            for (int e = 0; e < 4; ++e)
              x[e] = kPhase == 1 ? silu(acc[0][rb][4 * j + e]) * acc[1][rb][4 * j + e] : acc[cb][rb][4 * j + e];
            const u32x2 q = {__builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{x[0], x[1]}, bf16x2)),
                             __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{x[2], x[3]}, bf16x2))};
            *(BFS_LDS u32x2 *)(uintptr_t)(blk + l32 * 64u + (8u * j + 4u * lhi) * 2u) = q;
          }
        }
        S.signal(P.spill.update, ew);
      }
    }
  } else {
    // -------------------------------------------------------- epilogue engine
    const uint32_t ew = (uint32_t)(wave - kLoadW - kMmaW);
    // this wave stores the blocks of MFMA waves 4 ew .. 4 ew + 3, which have
    // kWs different places wm among the token blocks; lane rows 16 h + lane / 4
    constexpr int kWs = 4 / G::kWN;
    for (uint32_t i = 0; i < trip_u; ++i) {
      g.r1 += 1;
      g.h1 = i + 1;
      const int32_t m0 = unit_row(i);
      int32_t tok[G::kRB][kWs][2];
#pragma unroll
      for (int rb = 0; rb < G::kRB; ++rb)
#pragma unroll
        for (int w = 0; w < kWs; ++w)
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            const int32_t r = m0 + 32 * (G::kWM * rb + kWs * (int32_t)ew + w) + 16 * h + (int32_t)(lane >> 2);
            tok[rb][w][h] = r < row_hi ? (kPhase == 1 ? e_lo + r : P.perm[e_lo + r]) : -1;
          }
      g.r2 += ksteps;
      g.h2 = ksteps;
      S.enter(sa, P.epi, g, 3);
#pragma unroll
      for (uint32_t c = 0; c < kChunks; ++c) {
        constexpr uint32_t kCB = kPhase == 1 ? 1u : 2u;
        const uint32_t rb = c / kCB, cb = c % kCB;
        g.r3 += 1;
        g.h3 = c + 1;
        S.wait_affine(sa, P.epi, g, c + 1, g.r3 - 1, [] {});
        if (!S.aborted) {
          const uint32_t eslot = P.e_ring == 0 ? c : (P.e_ring == 2 ? ((g.r3 - 1) & 1u) : 0u);
          const uint32_t cc = lane & 3u;
          // the chunk's segments into registers, then EPI retires from its
          // slot (LDS executes the reads before the signal), then the stores
          u32x4 d[4][2];
#pragma unroll
          for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int h = 0; h < 2; ++h)
              d[q][h] = *(const BFS_LDS u32x4 *)(uintptr_t)(ering + eslot * kESlotBytes + (ew * 4u + q) * 2048u +
                                                            (16u * h + (lane >> 2)) * 64u + cc * 16u);
          S.signal(P.epi.update, ew);
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const int w = q / G::kWN, wn = q % G::kWN;
            const uint32_t col = (uint32_t)n0 + (kPhase == 1 ? 32u * wn : 64u * wn + 32u * cb) + 8u * cc;
#pragma unroll
            for (int h = 0; h < 2; ++h)
              if (tok[rb][w][h] >= 0)
                *reinterpret_cast<u32x4 *>(P.out + (size_t)tok[rb][w][h] * P.ndim + col) = d[q][h];
          }
        } else {
          S.signal(P.epi.update, ew);
        }
      }
    }
  }
  drain_all();
}

// Workgroup b of the launch: item b % items and its workgroup b / items.  The
// first workgroups of all items come first, so that workgroups without units
// (runs shorter than sm units) do not alternate with the others (workgroups go
// to the shader engines of an XCD in turn).  An item's workgroups keep its XCD
// (workgroup w runs on XCD w % 8).
template <int kPhase, int kPM>
__global__ void __launch_bounds__(768) moe_part_kernel(MoeParams P, Split D) {
  extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
  const int wg = blockIdx.x % D.items;
  if (wg < D.n_wg) run_units<kPhase, kPM, 256>(P, D, lds, wg, blockIdx.x / D.items, read_item(P, wg));
}

// Many items: workgroups that stay, kPerXcd on each XCD.  The units of an XCD's
// items (item w belongs to XCD w % 8), counted along the items in order, go to
// its workgroups in turn, so that the units of an item, which read the same
// weights, run at about the same time and share them in L2 (with a workgroup
// per item each M-tile reads them from memory again), and the last round is
// made of the smallest experts' units.  The items and the sums of units up to
// each are kept in LDS behind the ring (read from memory for each unit they
// cost it some microseconds).
constexpr int kPerXcd = 32, kAlone = 1 << 20;   // kAlone: units of an item that far apart (one unit)

template <int kPhase, int kPM>
__global__ void __launch_bounds__(768) moe_many_kernel(MoeParams P, Split D) {
  extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
  const int x = blockIdx.x % 8, n_x = D.items / 8;
  const uint32_t table = lds_addr(lds) + (uint32_t)D.table;
  uint32_t total = 0;
  for (int c = 0; c < n_x; c += 64) {       // every wave counts, the first one writes
    const int i = c + (int)lane_id(), item = 8 * i + x;
    uint32_t upto = 0;
    u32x4 w{}, v{};
    if (i < n_x && item < D.n_wg) {
      const int32_t e = P.work[4 * item], n0 = P.work[4 * item + 1], mt0 = P.work[4 * item + 2];
      const uint32_t trip_m = (uint32_t)P.trips[P.trip_off[(int64_t)item * 4 + 1]];
      const int32_t e_lo = P.eoff[e], e_cnt = P.eoff[e + 1] - e_lo, left = e_cnt - mt0 * D.bm;
      const uint32_t rows = left <= 0 ? 0u : trip_m > (uint32_t)left / (uint32_t)D.bm ? (uint32_t)left : trip_m * (uint32_t)D.bm;
      upto = (rows + kPM - 1u) / kPM;
      w = u32x4{(uint32_t)e, (uint32_t)n0, (uint32_t)mt0, (uint32_t)e_lo};
      v = u32x4{(uint32_t)e_cnt, trip_m, 0u, 0u};
    }
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {      // inclusive sums
      const uint32_t u = __shfl_up(upto, d);
      if ((int)lane_id() >= d) upto += u;
    }
    upto += total;
    v.z = upto;
    if (threadIdx.x < 64 && i < n_x) {
      *(BFS_LDS u32x4 *)(uintptr_t)(table + 32u * (uint32_t)i) = w;
      *(BFS_LDS u32x4 *)(uintptr_t)(table + 32u * (uint32_t)i + 16u) = v;
    }
    total = __builtin_amdgcn_readlane(upto, 63);
  }
  int c = 0;
  for (uint32_t unit = blockIdx.x / 8; unit < total; unit += kPerXcd) {
    __syncthreads();                        // the table is written; the unit before is done in every wave
    uint64_t hit = 0;
    while (true) {                          // the first item whose sum exceeds unit (unit < total: there is one)
      const int i = min(c + (int)lane_id(), n_x - 1);
      hit = __ballot(*(const BFS_LDS uint32_t *)(uintptr_t)(table + 32u * (uint32_t)i + 24u) > unit);
      if (hit != 0ull) break;
      c += 64;
    }
    const int at = c + __builtin_ctzll(hit);
    const u32x4 w = *(const BFS_LDS u32x4 *)(uintptr_t)(table + 32u * (uint32_t)at);
    const u32x4 v = *(const BFS_LDS u32x4 *)(uintptr_t)(table + 32u * (uint32_t)at + 16u);
    const uint32_t before = at > 0 ? uniform(*(const BFS_LDS uint32_t *)(uintptr_t)(table + 32u * (uint32_t)at - 8u)) : 0u;
    const Item I{(int32_t)uniform(w.x), (int32_t)uniform(w.y), (int32_t)uniform(w.z), (int32_t)uniform(w.w),
                 (int32_t)uniform(v.x), uniform(v.y)};
    run_units<kPhase, kPM, 256>(P, D, lds, 8 * at + x, (int)(unit - before), I);
  }
  // Trips beyond the expert's M-tiles, once on each XCD: an item without rows has
  // no unit that would report them.
  if (blockIdx.x < 8u && threadIdx.x < 64u) {
    for (int c0 = 0; c0 < n_x; c0 += 64) {
      const int i = min(c0 + (int)lane_id(), n_x - 1);
      const u32x4 w = *(const BFS_LDS u32x4 *)(uintptr_t)(table + 32u * (uint32_t)i);
      const u32x4 v = *(const BFS_LDS u32x4 *)(uintptr_t)(table + 32u * (uint32_t)i + 16u);
      const uint32_t max_m = (uint32_t)(max((int32_t)v.x - (int32_t)w.z * D.bm, 0) + D.bm - 1) / (uint32_t)D.bm;
      const uint64_t bad = __ballot(v.y > max_m);
      if (bad == 0ull) continue;
      const int at = __builtin_ctzll(bad);
      report_input(P.sc.err, 1u, (uint32_t)(8 * (c0 + at) + x), 1u, (uint32_t)__builtin_amdgcn_readlane((int)v.y, at),
                   (uint32_t)__builtin_amdgcn_readlane((int)max_m, at), 0u);
    }
  }
}

// At most kScan items: in quarters of 128 x 128 if these fit the compute units
// at once, else as moe_part_kernel.  How many there are the routing decides, so
// every wave counts them from the items' trips, and finds the workgroup's own
// in the sums: a workgroup per possible quarter of every item (16) would cost
// 1 us per 256 of them that have none (32 experts, 280 rows, K = 768 and 512:
// both phases 50 us, so 31).  (us of phase 1 and 2 in whole units, in quarters:
// 8 experts of 128 rows, K = 2048 and 1408, 176 and 128 quarters, 43 and 33, 33
// and 25; 2048 ragged rows, K = 1024 and 1408, 440 and 160 quarters, 31 and 39,
// 38 and 25.)  The workgroup's item comes out of LDS, where every wave keeps what
// it counts: read from memory again it cost 1.5 us (128 items of a few rows, K =
// 256: 12.7 us, so 11.2; whole items without a count 9.8), and kept in the lanes'
// registers these went to scratch memory (2048 rows, K = 1024 and 1408, both phases:
// 56.5 us from memory, 55.9 from the lanes, so 55.5).
constexpr int kScan = 128, kCUs = 256;

template <int kPhase, int kPM>
__global__ void __launch_bounds__(768) moe_small_kernel(MoeParams P, Split D) {
  extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
  // (both halves' loads first: two levels deep, from cold lines)
  int32_t e[kScan / 64], n0[kScan / 64], mt0[kScan / 64], lo[kScan / 64], hi[kScan / 64];
  uint32_t trip[kScan / 64];
  {
    int64_t at[kScan / 64];
#pragma unroll
    for (int h = 0; h < kScan / 64; ++h) {
      const int i = min(64 * h + (int)lane_id(), D.n_wg - 1);
      e[h] = P.work[4 * i];
      n0[h] = P.work[4 * i + 1];
      mt0[h] = P.work[4 * i + 2];
      at[h] = P.trip_off[(int64_t)i * 4 + 1];
    }
#pragma unroll
    for (int h = 0; h < kScan / 64; ++h) {
      lo[h] = P.eoff[e[h]];
      hi[h] = P.eoff[e[h] + 1];
      trip[h] = (uint32_t)P.trips[at[h]];
    }
  }
  // The items in the ring's memory, which no load fills before every wave has
  // reached the barrier in run_units, its item read.  (Every wave writes all of
  // them, the same values, so that none waits for another.)
  const uint32_t table = lds_addr(lds) + kCntBytes;
  static_assert(32 * kScan <= 2 * Unit<128, 128>::kSlot, "the items fit the smallest ring");
#pragma unroll
  for (int h = 0; h < kScan / 64; ++h) {
    const uint32_t row = table + 32u * (64u * h + lane_id());
    *(BFS_LDS u32x4 *)(uintptr_t)row = u32x4{(uint32_t)e[h], (uint32_t)n0[h], (uint32_t)mt0[h], (uint32_t)lo[h]};
    *(BFS_LDS u32x4 *)(uintptr_t)(row + 16u) = u32x4{(uint32_t)(hi[h] - lo[h]), trip[h], 0u, 0u};
  }
  auto item_of = [&](int w) __attribute__((always_inline)) {
    const uint32_t row = table + 32u * (uint32_t)w;
    const u32x4 a = *(const BFS_LDS u32x4 *)(uintptr_t)row, b = *(const BFS_LDS u32x4 *)(uintptr_t)(row + 16u);
    return Item{(int32_t)uniform(a.x), (int32_t)uniform(a.y), (int32_t)uniform(a.z), (int32_t)uniform(a.w),
                (int32_t)uniform(b.x), uniform(b.y)};
  };
  // quarters up to and with items lane and 64 + lane (an item without rows but
  // with a trip has two, so that the trip is checked as any other's)
  uint32_t own[kScan / 64], upto[kScan / 64], quarters = 0;
#pragma unroll
  for (int h = 0; h < kScan / 64; ++h) {
    // (32 bits: rows first cut to the expert's, trips to as many tiles)
    const int32_t left = max(hi[h] - lo[h] - mt0[h] * D.bm, 0);
    const uint32_t rows = trip[h] > (uint32_t)left ? (uint32_t)left : min((uint32_t)left, trip[h] * (uint32_t)D.bm);
    own[h] = 64 * h + (int)lane_id() < D.n_wg && trip[h] != 0u ? 2u * max((rows + 127u) / 128u, 1u) : 0u;
    upto[h] = own[h];
#pragma unroll
    for (int x = 1; x < 64; x <<= 1) {
      const uint32_t below = __shfl_up(upto[h], x);
      upto[h] += (int)lane_id() >= x ? below : 0u;
    }
    upto[h] += quarters;
    quarters = uniform(__shfl(upto[h], 63));
  }
  if (quarters <= (uint32_t)kCUs) {
    // quarter q here: neighbours in q (an item's) on one XCD
    const uint32_t per = (quarters + 7u) / 8u, q = (blockIdx.x % 8u) * per + blockIdx.x / 8u;
    if (blockIdx.x / 8u >= per || q >= quarters) return;
    int wg = 0;
    uint32_t sub = 0, parts = 2;
#pragma unroll
    for (int h = kScan / 64 - 1; h >= 0; --h) {
      const uint64_t above = __ballot(upto[h] > q);
      if (above != 0ull) {
        const int at = __builtin_ctzll(above);
        wg = 64 * h + at;
        parts = uniform(__shfl(own[h], at));
        sub = q - (uniform(__shfl(upto[h], at)) - parts);
      }
    }
    Split Q = D;
    Q.sm = (int32_t)(parts / 2u);
    Q.sn = 2;
    run_units<kPhase, 128, 128>(P, Q, lds, wg, (int)sub, item_of(wg));
    return;
  }
  const int wg = blockIdx.x % D.items, sub = blockIdx.x / D.items;
  if (wg < D.n_wg && sub < D.sm) run_units<kPhase, kPM, 256>(P, D, lds, wg, sub, item_of(wg));
}

}  // namespace

bool bfsmoe::launch_parts(const MoeParams &P, int phase, int bm, bool linear, int n_wg, hipStream_t s, bfs_status &st) {
  // Pairs of steps take an even number of ring slots, one less than an odd
  // ring (one more does not fit beside the epilogue slots of M-tiles of 128:
  // whole items instead, 16384 tokens, 32 experts, K = 4096 and 1408: 1167 us
  // of both phases, in four slots 885).  A pair at steps s and s + 1 waits for
  // the MMAs of step s + 1 - ring, and MMA retires steps in twos from the start
  // of a unit: with an odd ring that step is the first of its two, so the pair
  // ring - 1 before is free.  Read linearized, MMA->LOAD counts steps across
  // M-tiles, where a single last step would break the twos.
  const int slots = P.ring & ~1, ksteps = P.kdim / kBK;
  if (linear && ksteps % 2 != 0) return false;
  // Whole items stay where units do not win back what they cost.  (Time of whole
  // items over units, the geometric mean of calls of mixed expert sizes and, in
  // brackets, the range: within it the rows per expert decide, which the host
  // does not know.)
  //   One pair of slots, from a ring of three: 129 .. 192 items 1.15 (0.76 ..
  //   2.6), 193 .. 768 items 0.95 (0.66 .. 1.8).
  //   M-tiles of 128 rows, more than 384 items: phase 1, K <= 512, 0.94 (0.80 ..
  //   1.14), above 1.07; phase 2, K <= 256, 0.98 (0.78 .. 1.08), above 1.03.  Up
  //   to 384 items 1.0 .. 1.4 over every range of K (0.74 .. 3.4).
  //   M-tiles of 256 rows: 1.05 .. 2 over every range (0.89 .. 3.5).
  if (P.ring == 3 && n_wg > 192) return false;
  if (bm == 128 && n_wg > 384 && P.kdim <= (phase == 1 ? 512 : 256)) return false;
  auto go = [&](auto part, auto many, auto small, auto unit) -> bool {
    using G = decltype(unit);
    const int chunks = phase == 1 ? G::kRB : 2 * G::kRB;
    const size_t ring = (size_t)slots * G::kSlot;
    const size_t base = kCntBytes + ring + (size_t)P.e_ring * kESlotBytes;
    // Up to four workgroups for an item's units (runs of four M-tiles) while
    // the items are few; beyond `few` of them, workgroups that stay and take the
    // units in turn.  The rows per expert decide which is faster, and the host
    // does not know them; the line is where it pays on average.  Phase 1, us split
    // and in turn, items in brackets: [224] 145 and 109, [248] 413 and 363, [304]
    // 483 and 448, [448] 88 and 67, [1040] 1048 and 951 (a workgroup per item),
    // but [352] 770 and 824, [376] 117 and 129; 32 experts [352] of 16, 256, 512
    // and 1024 rows each, K = 2048, 98 and 110, 139 and 144, 231 and 209, 448 and
    // 383.  (Units in turn stay on their item's XCD, so one expert with most of
    // the rows and one column tile fills one XCD only: 4 experts, 28140 Zipf(1)
    // rows, K = 256, 128 columns, [216], 42 against 29 in whole items.)  Phase 2's
    // units are shorter and store twice the chunks: [176] 44 and 48, [312] 214 and
    // 220, [448] 254 and 233, [512] 390 and 417, [720] 349 and 254, [1520] 515 and
    // 497.
    const int few = phase == 1 ? kScan : 512;
    const int items = (n_wg + 7) / 8 * 8;
    const size_t table = (size_t)items / 8 * 32;
    const bool is_small = n_wg <= kScan, is_many = n_wg > few && base + table <= 160 * 1024;
    const int sm = is_many ? kAlone : n_wg > 512 ? 1 : 4;
    const size_t lds = base + (is_many ? table : 0);
    // (quarters take half of the ring and of the chunks or less)
    if (lds > 160 * 1024 || (P.e_ring == 0 && (size_t)chunks * kESlotBytes > ring)) return false;
    const int grid = is_many ? 8 * kPerXcd : is_small && items * sm < kCUs ? kCUs : items * sm;
    const auto kern = is_many ? many : is_small ? small : part;
    hipError_t e = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) {
      st = bfs::fail(BFS_E_DEVICE, std::string("moe attribute: ") + hipGetErrorString(e));
      return true;
    }
    hipLaunchKernelGGL(kern, dim3(grid), dim3(64 * kWaves), lds, s, P, Split{bm, sm, 1, n_wg, items, (int)base, slots});
    e = hipGetLastError();
    st = e == hipSuccess ? BFS_OK : bfs::fail(BFS_E_DEVICE, std::string("moe launch: ") + hipGetErrorString(e));
    return true;
  };
  // Units as high as the program's M-tiles.  (us of phase 1 and 2 in whole
  // items, in units of 256, of 128 rows: 16 experts, 8192 rows, K = 2048 and
  // 1408: 206 and 155, 151 and 82, 183 and 85.  M-tiles of 128 rows, 32
  // experts, K = 2048 and 1024: 187 and 98, units of 128: 171 and 93.)
  if (bm == 128)
    return phase == 1 ? go(moe_part_kernel<1, 128>, moe_many_kernel<1, 128>, moe_small_kernel<1, 128>, Unit<128, 256>{})
                      : go(moe_part_kernel<2, 128>, moe_many_kernel<2, 128>, moe_small_kernel<2, 128>, Unit<128, 256>{});
  return phase == 1 ? go(moe_part_kernel<1, 256>, moe_many_kernel<1, 256>, moe_small_kernel<1, 256>, Unit<256, 256>{})
                    : go(moe_part_kernel<2, 256>, moe_many_kernel<2, 256>, moe_small_kernel<2, 256>, Unit<256, 256>{});
}
