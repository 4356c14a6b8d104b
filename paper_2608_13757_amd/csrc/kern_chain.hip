// Two-engine chain: a load engine streams 256-element fp32 tiles through an
// LDS ring, a vector engine accumulates a scaled copy of every tile.  One
// wave per engine; the program is a two-level nest A{ B{ ... } }:
//
//   A{ E0: ACQ                                  (no datapath)
//      B{ E0: LOAD  X[n] -> ring[(rhat_B - 1) % R]   (n = r_B - 1 + base[wg])
//         E1: CONS  acc += c * ring[(rhat_B - 1) % R] } }
//   E1: STORE acc -> out[wg]
//
// Dependencies (from the plan, Eq. 5 on the loop registers): LOAD->CONS at
// offset 0, CONS->LOAD at offset R (a slot is refilled only after its tile
// was read, inside one trip of B), CONS->ACQ at offset 1 (case C3 at A: the
// next trip of B starts filling slot 0 again only after the previous trip's
// reads).  Barrier mode synchronizes both waves before each loop statement
// and at every iteration end, with static ordinals in a region.
//
// What bounds it: one workgroup runs a serial chain of hand-offs, so memory
// latency must stay out of the chain.  The tiles of a workgroup are adjacent
// in memory and their number is the sum of B's trips, so the load engine
// fetches them ahead of the waits, kStage tiles in flight, by direct-to-LDS
// loads (16 bytes per lane) into a staging ring that only it uses.  LOAD then
// is a copy from staging to the ring slot, held in a register before the wait
// of its slot, and retires at once (LDS executes the counter add after the
// write).  The last loads of a workgroup repeat its last tile, so that the
// counted vmcnt wait is the same for every tile.  The vector engine takes up
// to four tiles that the last observed counter covers in one LDS round trip,
// with one counter add.  One workgroup, 16 iterations of A, trips of B up to
// 8: 16.9 us against 26.5 us with the loads issued after each wait into the
// ring itself, which exposed the memory latency in every iteration of A.
//
// Family contract (BFS_KERNEL_CHAIN): loops top -> A -> B; engines of one
// wave each; ACQ (opcode 0, E0) in A before B; LOAD (1, E0) and CONS (2, E1)
// in B, both slotted by rhat_B modulo R = ring_slots[0] (1..8), LOAD tiles
// indexed by r_B; STORE (3, E1) at the top level after A; tile_elems 256.
// Buffers: [0] int64 tile base per workgroup, [1] fp32 input tiles
// [n][256], [2] fp32 output [n_wg][256].
#include <string>

#include "engine_sync.h"

using namespace bfsdev;

namespace {

constexpr int kTileFloats = 256;
constexpr uint32_t kTileBytes = kTileFloats * 4;
constexpr uint32_t kStage = 8;           // tiles in flight ahead of the ring

struct ChainParams {
  SyncCommon sc;
  InstrWaits acq, load, cons, store;
  const int32_t *trips;
  const int64_t *trip_off;
  const int64_t *base;
  const float *x;
  float *out;
  int32_t ring;
  float scale;
};

// Sum over the 64 lanes, wave-uniform.
__device__ __forceinline__ uint32_t wave_sum(uint32_t v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += (uint32_t)__shfl_xor((int)v, o);
  return uniform(v);
}

template <int kMode, bool kInstr>
__global__ void __launch_bounds__(128) chain_kernel(ChainParams P) {
  extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
  uint32_t *cnt = reinterpret_cast<uint32_t *>(lds);
  unsigned char *ring = lds + kCntBytes;
  for (int i = threadIdx.x; i < bfs::kMaxSlots * bfs::kMaxWavesPerEngine; i += blockDim.x) cnt[i] = 0;
  __syncthreads();

  const int wave = wave_id();
  const uint32_t lane = lane_id();
  const int wg = blockIdx.x;
  Sync<kMode, kInstr> S(P.sc, lds_addr(cnt), wave, wg);
  const int64_t *toff = P.trip_off + (int64_t)wg * 3;
  const uint32_t trip_a = (uint32_t)ldc(P.trips + ldc(toff + 1));
  const int64_t off_b = ldc(toff + 2);
  const int64_t tbase = ldc(P.base + wg);
  const uint32_t R = (uint32_t)P.ring;
  const uint32_t ring_l = lds_addr(ring) + 16u * lane;     // this lane's 16 bytes of slot 0
  Regs g;
  // trips of B, 64 iterations of A at a time, one per lane
  uint32_t trips_b = lane < trip_a ? (uint32_t)P.trips[off_b + lane] : 0u;
  asm volatile("" : "+v"(trips_b));
  auto trip_of = [&](uint32_t ia) {
    if (ia > 0u && (ia & 63u) == 0u) {
      trips_b = ia + lane < trip_a ? (uint32_t)P.trips[off_b + ia + lane] : 0u;
      asm volatile("" : "+v"(trips_b));   // arrived here, so that no other iteration waits for loads in flight
    }
    return (uint32_t)__builtin_amdgcn_readlane((int)trips_b, (int)(ia & 63u));
  };

  // Barrier-free, uninstrumented launches: one compare with the last observed
  // counter value per wait, then polls without sleeping (the two waves share
  // no issue slots with others worth yielding to).
  constexpr bool kLean = kMode == BFS_MODE_BARRIER_FREE && !kInstr;
  const uint32_t limit = P.sc.watchdog > 0xffffffffull ? 0xffffffffu : (uint32_t)P.sc.watchdog;
  auto affine = [](const Site<1> &st, uint32_t t) {    // threshold of iteration t (0: no wait)
    const int32_t v = st.base[0] + (int32_t)((st.mk[0] >> 16) * t);
    return st.n > 0u && t > (st.mk[0] & 0xffffu) && v > 0 ? (uint32_t)v : 0u;
  };
  // The waits of LOAD and CONS are on loop B's own iterations (producer and
  // shared loop B): their base moves by N per iteration of B.
  auto next_trip = [](Site<1> &st, uint32_t trip) { st.base[0] += (int32_t)((st.mk[0] >> 16) * trip); };
  auto spin = [&](Site<1> &st, uint32_t thr, const InstrWaits &iw, uint32_t instance) __attribute__((always_inline)) {
    if (thr <= st.seen[0] || S.aborted) return;
    const uint32_t addr = st.meta[0] & 0xffffu;
    for (uint32_t polls = 0;; ++polls) {
      const uint32_t v = uniform(lds_poll(addr));
      st.seen[0] = v;
      if (v >= thr) return;
      if (polls >= limit) {
        report_deadlock(P.sc.err, iw.w[0].w.w3 & 0xffffu, (uint32_t)wg, instance, thr, v, (uint32_t)wave);
        S.aborted = 1u;
        return;
      }
      if (polls >= 256u) __builtin_amdgcn_s_sleep(2);
    }
  };

  if (wave == 0) {
    // ------------------------------------------------------------ load engine
    // tiles of this workgroup: the sum of B's trips
    uint32_t n_tiles = trips_b;
    for (uint32_t i = lane + 64u; i < trip_a; i += 64u) n_tiles += (uint32_t)P.trips[off_b + i];
    n_tiles = wave_sum(n_tiles);
    const char *src = reinterpret_cast<const char *>(P.x + tbase * kTileFloats) + 16u * lane;
    const uint32_t stage = lds_addr(ring) + R * kTileBytes, stage_l = stage + 16u * lane;
    uint32_t fetch = 0, fslot = 0, tslot = 0;    // next tile to fetch and its staging slot; staging slot to read next
    auto fetch_one = [&]() {
      __builtin_amdgcn_global_load_lds((const void *)(src + (int64_t)min(fetch, n_tiles - 1u) * kTileBytes),
                                       (BFS_LDS void *)(uintptr_t)(stage + fslot * kTileBytes), 16, 0, 0);
      fetch += 1;
      fslot = (fslot + 1u) % kStage;
    };
    f32x4 tile = {};
    // the oldest staged tile into registers (kStage loads are in flight, so
    // at most kStage - 1 may remain), then its staging slot is refilled
    auto take = [&]() {
      asm volatile("s_waitcnt vmcnt(%2)\n\tds_read_b128 %0, %1\n\ts_waitcnt lgkmcnt(0)"
                   : "=v"(tile)
                   : "v"(stage_l + tslot * kTileBytes), "n"(kStage - 1)
                   : "memory");
      tslot = (tslot + 1u) % kStage;
      fetch_one();
    };
    if (n_tiles > 0) {
      for (uint32_t i = 0; i < kStage; ++i) fetch_one();
      take();
    }
    Site<1> s_acq, s_load;
    S.sync_point(S.word(0, 0));                        // before loop A
    S.enter(s_acq, P.acq, g, 1);                       // (a C3 wait: evaluated at each iteration of A)
    if (kLean) S.enter(s_load, P.load, g, 2);
    for (uint32_t ia = 0; ia < trip_a; ++ia) {
      g.r1 += 1;
      g.h1 = ia + 1;
      const uint32_t trip_b = trip_of(ia);
      if constexpr (kLean) {
        // ACQ and LOAD by running thresholds; both mostly wait for CONS, so
        // what ACQ observed serves LOAD too
        if (P.acq.n > 0) spin(s_acq, S.threshold_plain(P.acq.w[0].w, g), P.acq, ia);
        S.signal(P.acq.update, 0);
        if ((s_acq.meta[0] & 0xffffu) == (s_load.meta[0] & 0xffffu)) s_load.seen[0] = max(s_load.seen[0], s_acq.seen[0]);
        uint32_t slot_l = ring_l;
        for (uint32_t ib = 0; ib < trip_b; ++ib) {
          spin(s_load, affine(s_load, ib + 1), P.load, g.r2 + ib);
          asm volatile("ds_write_b128 %0, %1" ::"v"(slot_l), "v"(tile) : "memory");
          S.signal(P.load.update, 0);
          take();                                      // the next tile, before the waits it may have to pass
          slot_l = slot_l + kTileBytes == ring_l + R * kTileBytes ? ring_l : slot_l + kTileBytes;
        }
        g.r2 += trip_b;
        g.h2 = trip_b;
        next_trip(s_load, trip_b);
        continue;
      }
      // ACQ: its waits; everything before it has retired
      S.wait(s_acq, P.acq, g, ia + 1, g.r1 - 1, [] {});
      S.signal(P.acq.update, 0);
      S.sync_point(S.word(0, 0));                      // before loop B
      S.enter(s_load, P.load, g, 2);
      uint32_t slot = 0;
      for (uint32_t ib = 0; ib < trip_b; ++ib) {
        g.r2 += 1;
        g.h2 = ib + 1;
        S.wait_affine(s_load, P.load, g, ib + 1, g.r2 - 1, [] {});
        if (!S.aborted) {
          asm volatile("ds_write_b128 %0, %1" ::"v"(ring_l + slot * kTileBytes), "v"(tile) : "memory");
          S.signal(P.load.update, 0);
          take();                                      // the next tile, before the waits it may have to pass
        } else {
          S.signal(P.load.update, 0);
        }
        S.sync_point(S.word(0, 0));                    // end of a B iteration (barrier mode)
        slot = (slot + 1 == R) ? 0u : slot + 1;
      }
      S.sync_point(S.word(0, 0));                      // end of an A iteration
    }
  } else {
    // ---------------------------------------------------------- vector engine
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    const float c = P.scale;
    Site<1> s_cons, s_store;
    if (kLean) S.enter(s_cons, P.cons, g, 2);
    S.sync_point(S.word(1, 0));                        // before loop A
    for (uint32_t ia = 0; ia < trip_a; ++ia) {
      g.r1 += 1;
      g.h1 = ia + 1;
      const uint32_t trip_b = trip_of(ia);
      S.sync_point(S.word(1, 0));                      // before loop B
      if (!kLean) S.enter(s_cons, P.cons, g, 2);
      uint32_t slot = 0;
      if constexpr (kLean) {
        // Tiles that the observed counter covers, four or two at a time: with
        // one LOAD per count (N = 1) the threshold of iteration t is base + t.
        const bool unit = (s_cons.mk[0] >> 16) == 1u && (s_cons.mk[0] & 0xffffu) == 0u && s_cons.n == 1u;
        auto at = [&](uint32_t i) {                    // slot i places on
          const uint32_t sl = slot + i;
          return ring_l + (sl >= R ? sl - R : sl) * kTileBytes;   // (at most R tiles wait in the ring)
        };
        auto read = [&](uint32_t i) { return *(const BFS_LDS f32x4 *)(uintptr_t)at(i); };
        auto add = [&](const f32x4 &v) {
#pragma unroll
          for (int j = 0; j < 4; ++j) acc[j] = acc[j] + c * v[j];
        };
        // LDS executes the counter add after the reads before it
        auto signal = [&](uint32_t k) {
          if (P.cons.update >= 0) lds_add(S.word((uint32_t)P.cons.update, 0), k);
        };
        for (uint32_t ib = 0; ib < trip_b;) {
          spin(s_cons, affine(s_cons, ib + 1), P.cons, g.r2 + ib);
          const uint32_t have = S.aborted || !unit ? 1u : min(s_cons.seen[0] - (uint32_t)s_cons.base[0], trip_b) - ib;
          uint32_t k = 1;
          if (have >= 4u) {
            k = 4;
            const f32x4 v0 = read(0), v1 = read(1), v2 = read(2), v3 = read(3);
            signal(4);
            add(v0);
            add(v1);
            add(v2);
            add(v3);
          } else if (have >= 2u) {
            k = 2;
            const f32x4 v0 = read(0), v1 = read(1);
            signal(2);
            add(v0);
            add(v1);
          } else {
            const f32x4 v0 = read(0);
            signal(1);
            add(v0);
          }
          ib += k;
          slot += k;
          if (slot >= R) slot -= R;
        }
        g.r2 += trip_b;
        g.h2 = trip_b;
        next_trip(s_cons, trip_b);
        continue;
      }
      for (uint32_t ib = 0; ib < trip_b; ++ib) {
        g.r2 += 1;
        g.h2 = ib + 1;
        S.wait_affine(s_cons, P.cons, g, ib + 1, g.r2 - 1, [] {});
        if (!S.aborted) {
          const f32x4 v = *(const BFS_LDS f32x4 *)(uintptr_t)(ring_l + slot * kTileBytes);
#pragma unroll
          for (int j = 0; j < 4; ++j) acc[j] = acc[j] + c * v[j];
        }
        // the slot has been read: LDS executes the add after the read
        S.signal(P.cons.update, 0);
        S.sync_point(S.word(1, 0));                    // end of a B iteration (barrier mode)
        slot = (slot + 1 == R) ? 0u : slot + 1;
      }
      S.sync_point(S.word(1, 0));                      // end of an A iteration
    }
    // STORE (top level, after loop A)
    S.enter(s_store, P.store, g, 0);
    S.wait(s_store, P.store, g, 1, 0, [] {});
    if (!S.aborted) __builtin_nontemporal_store(acc, reinterpret_cast<f32x4 *>(P.out + (int64_t)wg * kTileFloats + 4 * lane));
    if (P.store.update >= 0) {
      drain_all();
      S.signal(P.store.update, 0);
    }
  }
  drain_all();
  S.finish(lane);
}

}  // namespace

namespace bfs {

bfs_status launch_chain(const bfs_plan *p, DevImage *img, const void *const *bufs, int32_t nbufs,
                        const int32_t *trips, const int64_t *trip_off, int32_t n_wg, void *stream, uint32_t *dbg,
                        int64_t dbg_cap, const bfs_run_opts &o) {
  // structure: top{ A{ ACQ(E0); B{ LOAD(E0) CONS(E1) } }; STORE(E1) }
  if (p->n_loops != 3 || p->loop_parent[1] != 0 || p->loop_parent[2] != 1)
    return fail(BFS_E_UNSUPPORTED, "chain: loops must be top -> A -> B");
  if (p->n_engines != 2 || p->waves_per_engine[0] != 1 || p->waves_per_engine[1] != 1)
    return fail(BFS_E_UNSUPPORTED, "chain: two engines of one wave");
  if (p->tile_elems != kTileFloats) return fail(BFS_E_UNSUPPORTED, "chain: tile_elems must be 256");
  int ins_acq = -1, ins_load = -1, ins_cons = -1, ins_store = -1;
  for (size_t i = 0; i < p->instr_engine.size(); ++i) {
    const int op = p->instr_opcode[i], e = p->instr_engine[i], par = p->instr_parent[i];
    if (op == 0 && e == 0 && par == 1 && ins_acq < 0) ins_acq = (int)i;
    else if (op == 1 && e == 0 && par == 2 && ins_load < 0) ins_load = (int)i;
    else if (op == 2 && e == 1 && par == 2 && ins_cons < 0) ins_cons = (int)i;
    else if (op == 3 && e == 1 && par == 0 && ins_store < 0) ins_store = (int)i;
    else return fail(BFS_E_UNSUPPORTED, "chain: unexpected instruction " + std::to_string(i));
  }
  if (ins_acq < 0 || ins_load < 0 || ins_cons < 0 || ins_store < 0)
    return fail(BFS_E_UNSUPPORTED, "chain: needs ACQ, LOAD, CONS and STORE");
  // ACQ precedes loop B in A's body
  auto acq_first = [&]() {
    for (int it = p->body_off[1]; it < p->body_off[2]; ++it) {
      if (p->body_kind[it] == 1) return false;
      for (int j = p->block_off[p->body_id[it]]; j < p->block_off[p->body_id[it] + 1]; ++j)
        if (p->block_instrs[j] == ins_acq) return true;
    }
    return false;
  };
  if (!acq_first()) return fail(BFS_E_UNSUPPORTED, "chain: ACQ must precede loop B");
  const int R = p->ring_slots[0];
  const int32_t *la = &p->instr_args[8 * ins_load];
  const int32_t *ca = &p->instr_args[8 * ins_cons];
  const int32_t *sa = &p->instr_args[8 * ins_store];
  // slot = (rhat_B - 1) % R for both; LOAD reads input buffer 1 at tile r_B
  if (R < 1 || R > 8 || la[0] != 1 || la[1] != 0 || la[2] != -1 || la[4] != 2 || la[5] != R || la[6] != 2 ||
      ca[0] != 0 || ca[1] != 0 || ca[2] != -1 || ca[4] != 2 || ca[5] != R || sa[0] != 0 || sa[1] != 2)
    return fail(BFS_E_UNSUPPORTED, "chain: ring of 1..8 slots indexed by rhat_B, tiles by r_B, one accumulator");
  if (!has_dep(p, ins_load, ins_cons, 0) || !has_dep(p, ins_cons, ins_load, R) || !has_dep(p, ins_cons, ins_acq, 1))
    return fail(BFS_E_UNSUPPORTED, "chain: needs LOAD->CONS(0), CONS->LOAD(ring), CONS->ACQ(1)");
  if (nbufs < 3 || !bufs[0] || !bufs[1] || !bufs[2]) return fail(BFS_E_INVALID, "chain: needs [base, x, out]");
  if (!trips || !trip_off) return fail(BFS_E_INVALID, "chain: needs trip tables");
  const std::vector<DevWait> dw = device_waits(p);
  ChainParams P{};
  if (!fill_waits(p, dw, ins_acq, P.acq) || !fill_waits(p, dw, ins_load, P.load) ||
      !fill_waits(p, dw, ins_cons, P.cons) || !fill_waits(p, dw, ins_store, P.store))
    return fail(BFS_E_RESOURCE, "chain: at most 4 waits per instruction");
  if (!waits_fit({{&P.acq, 1}, {&P.load, 1}, {&P.cons, 1}, {&P.store, 1}}))
    return fail(BFS_E_RESOURCE, "chain: more waits on an instruction than its engine loop takes");
  if (p->mode == BFS_MODE_BARRIER_FREE && (!no_dynamic(P.load) || !no_dynamic(P.cons)))
    return fail(BFS_E_UNSUPPORTED, "chain: a B-loop wait depends on a loop register other than the B loop's");
  P.trips = trips;
  P.trip_off = trip_off;
  P.base = static_cast<const int64_t *>(bufs[0]);
  P.x = static_cast<const float *>(bufs[1]);
  P.out = static_cast<float *>(const_cast<void *>(bufs[2]));
  P.sc = sync_common(img, dbg, dbg_cap, o, 2);
  P.ring = R;
  P.scale = __builtin_bit_cast(float, ca[7]);
  const size_t lds = kCntBytes + (size_t)(R + kStage) * kTileBytes;
  const bool instr = dbg || o.dev_stats || o.fault_dep >= 0;
  hipStream_t s = (hipStream_t)stream;
  auto go = [&](auto kern) -> bfs_status {
    hipLaunchKernelGGL(kern, dim3(n_wg), dim3(128), lds, s, P);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(BFS_E_DEVICE, std::string("chain launch: ") + hipGetErrorString(e));
    return BFS_OK;
  };
  if (p->mode == BFS_MODE_BARRIER)
    return instr ? go(chain_kernel<BFS_MODE_BARRIER, true>) : go(chain_kernel<BFS_MODE_BARRIER, false>);
  return instr ? go(chain_kernel<BFS_MODE_BARRIER_FREE, true>) : go(chain_kernel<BFS_MODE_BARRIER_FREE, false>);
}

}  // namespace bfs
