// Generic tile-machine interpreter: one wavefront per engine walks its
// projection of the statement tree, maintains the loop registers of
// Section 5.1 (r: entries since the start, rhat: entries in the current
// trip), evaluates every wait before issuing an instruction, executes the
// instruction's datapath and retires it by incrementing its counter.
//
// Family contract (BFS_KERNEL_INTERP): every engine has one wave; buffers are
//   [0] const int64 tile base per workgroup, [1] const fp32 input tiles,
//   [2] fp32 output tiles.
// Opcodes (see the program description): 0 no-op, 1 load tile into a ring
// slot, 2 acc += c * slot, 3 store acc to output tile wg, 4 slot + c into a
// second ring, 5 store a slot to output tile gidx.
//
// What bounds it: the chain of dependent accesses behind each instruction
// (code word, descriptors, loop registers, counter poll) and the memory
// latency of its load.  So:
//   * the engine's program and the loop registers live in vector registers,
//     one code word, descriptor or loop per lane, read with v_readlane (a few
//     clocks) instead of from memory or LDS.  That takes at most 64 code words
//     and 64 waits per engine; longer programs read the same tables with
//     scalar loads (kLanes false).
//   * loads go directly to LDS and stay in flight, up to 8 tiles, with
//     stores counted in the same queue; they retire in issue order with
//     counted vmcnt waits: the oldest when the queue is full, one at a time
//     while the engine is blocked on a wait (its consumers may be waiting for
//     exactly those), all of them before any other instruction retires and at
//     every barrier.  Instrumented launches retire each instruction at once.
//   * a wait already met by the last observed counter value (counters only
//     grow, barrier mode aside) is not polled again.
//   * an innermost loop of one instruction with at most two waits (the usual
//     one: an engine's projection holds its own instructions only) is decoded
//     once and run without the dispatch, which is some 300 scalar instructions
//     per iteration and trip on the general path and 40 here: thresholds, slots
//     and tiles are carried incrementally, trips are read 64 at a time, and
//     where the loop around it holds nothing else (or a no-op before it, an
//     acquire) the trips follow one another.
// The ring program (64 outer iterations, 4 slots, 1024 workgroups, 303 MB of
// tiles) takes 164 us, 492 us with every instruction dispatched, and 1705 us
// with tables, loop registers and execution counts read from memory and LDS and
// every instruction drained before the next.
#include <type_traits>

#include "bfs_internal.h"
#include "device_sync.h"

using namespace bfsdev;

namespace {

constexpr int kMaxInstrsInterp = 256;
constexpr uint32_t kMaxPending = 8;     // vector-memory instructions in flight per engine

typedef __attribute__((ext_vector_type(4))) float f32x4;

// One of an inner loop's waits, decoded, and its state in a run of trips: the
// threshold is run, growing by N with r of loop P, while rhat of loop S > kk.
// (Members by name: arrays, even with unrolled indexes, went to scratch memory.)
struct InnerWait {
  uint32_t addr = 0, dep = 0, k = 0, lP = 0, lS = 0, mask = 0;
  int32_t N = 0, c = 0;
};
struct InnerWaitState {
  int32_t run, step, step_a;
  uint32_t kk, met;
};

struct InterpParams {
  const int32_t *code;          // code words, 4 x int32
  const int32_t *engine_off;    // [3][n_engines + 1]: first code word, instruction row, wait row
  const int32_t *waits;         // wait rows, 8 x int32
  const int32_t *args;          // instruction rows: args[8]
  const int32_t *trips;
  const int64_t *trip_off;
  const int64_t *base;
  const float *x;
  float *out;
  uint32_t *dbg;
  int64_t dbg_cap;
  uint32_t *err;
  uint64_t *stats;              // per-wave statistics (null: off)
  uint64_t watchdog;
  int32_t fault_dep, fault_delta;
  int32_t n_loops, n_engines, tile;
  int32_t wide_x, wide_out;     // tiles of 256 in a 16-byte aligned buffer: one 16-byte access per lane
  uint32_t fallback_loops;      // bit l: drain barrier at the end of every iteration of loop l
  int32_t ring_off[4];          // float offsets in the ring area
  int32_t acc_off;
  int32_t data_floats;
  int32_t lds_data_off;         // byte offset in dynamic LDS
  int32_t lds_snap_off, snap_words;   // per-engine allocation: running counts and snapshots per wave
};

__device__ __forceinline__ uint32_t rl(uint32_t v, uint32_t lane) {
  return (uint32_t)__builtin_amdgcn_readlane((int)v, (int)lane);
}

// v with lane l replaced by x (l and x wave-uniform)
__device__ __forceinline__ uint32_t wl(uint32_t v, uint32_t l, uint32_t x) { return lane_id() == l ? x : v; }

// a % b; ring depths are small and often powers of two
__device__ __forceinline__ uint32_t umod(uint32_t a, uint32_t b) {
  if ((b & (b - 1u)) == 0u) return a & (b - 1u);
  return a < b ? a : a % b;
}

// At most n <= 15 vector-memory instructions outstanding (fewer for the counts
// that no queue of kMaxPending equal entries leaves).
__device__ __forceinline__ void wait_at_most(uint32_t n) {
  n = uniform(n);
  if (n < 4u) {
    if (n < 2u) {
      if (n == 0u) wait_vm<0>(); else wait_vm<1>();
    } else {
      if (n == 2u) wait_vm<2>(); else wait_vm<3>();
    }
  } else if (n < 8u) {
    if (n < 6u) {
      if (n == 4u) wait_vm<4>(); else wait_vm<5>();
    } else {
      if (n == 6u) wait_vm<6>(); else wait_vm<7>();
    }
  } else {
    if (n < 12u) wait_vm<8>(); else wait_vm<12>();
  }
}

// kLanes: the engine's code words, instruction rows and wait rows each fit
// the 64 lanes of a register (the launcher checks); otherwise they are read
// with scalar loads.
template <int kMode, bool kInstr, bool kLanes, bool kInner = false>
__global__ void __launch_bounds__(512) interp_kernel(InterpParams P) {
  extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
  uint32_t *cnt = reinterpret_cast<uint32_t *>(lds);            // [64 slots][8 waves]
  const int wave = wave_id();
  const uint32_t lane = lane_id();
  const int wg = blockIdx.x;
  const uint32_t e = (uint32_t)wave, E1 = (uint32_t)P.n_engines + 1u;
  float *data = reinterpret_cast<float *>(lds + P.lds_data_off);

  // The engine's program: lane i holds code word i, instruction row i and
  // wait row i.  (Loaded before the zeroing below so that the latencies
  // overlap.)
  const uint32_t code0 = (uint32_t)ldc(P.engine_off + e), code1 = (uint32_t)ldc(P.engine_off + e + 1);
  const uint32_t row0 = (uint32_t)ldc(P.engine_off + E1 + e), row1 = (uint32_t)ldc(P.engine_off + E1 + e + 1);
  const uint32_t wait0 = (uint32_t)ldc(P.engine_off + 2 * E1 + e), wait1 = (uint32_t)ldc(P.engine_off + 2 * E1 + e + 1);
  uint32_t cw[4] = {}, ar[8] = {}, wr[8] = {};
  if (kLanes) {
    if (lane < code1 - code0)
#pragma unroll
      for (int j = 0; j < 4; ++j) cw[j] = (uint32_t)P.code[4 * (code0 + lane) + j];
    if (lane < row1 - row0)
#pragma unroll
      for (int j = 0; j < 8; ++j) ar[j] = (uint32_t)P.args[8 * (row0 + lane) + j];
    if (lane < wait1 - wait0)
#pragma unroll
      for (int j = 0; j < 8; ++j) wr[j] = (uint32_t)P.waits[8 * (wait0 + lane) + j];
  }
  auto code = [&](uint32_t pc, int j) __attribute__((always_inline)) { return kLanes ? rl(cw[j], pc) : (uint32_t)ldc(P.code + 4 * (code0 + pc) + j); };
  auto arg = [&](uint32_t row, int j) __attribute__((always_inline)) { return kLanes ? rl(ar[j], row) : (uint32_t)ldc(P.args + 8 * (row0 + row) + j); };
  auto wrow = [&](uint32_t w, int j) __attribute__((always_inline)) { return kLanes ? rl(wr[j], w) : (uint32_t)ldc(P.waits + 8 * (wait0 + w) + j); };
  // Loop registers and trip-table offsets, loop l in lane l (at most 32).
  uint32_t rv = lane == 0 ? 1u : 0u, hv = rv, tv = rv;
  uint32_t off_lo = 0, off_hi = 0;
  if (lane < (uint32_t)P.n_loops) {
    const int64_t o = P.trip_off[(int64_t)wg * P.n_loops + lane];
    off_lo = (uint32_t)o;
    off_hi = (uint32_t)((uint64_t)o >> 32);
  }
  const int64_t tbase = P.base ? ldc(P.base + wg) : 0;   // programs without loads and stores need none

  // Zero counters, snapshots and data (rings and accumulators).
  for (int i = threadIdx.x; i < bfs::kMaxSlots * bfs::kMaxWavesPerEngine; i += blockDim.x) cnt[i] = 0;
  // per-engine allocation: words 0 .. kMaxEngines - 1 hold the running count
  // of each producer engine's instructions up to this wave's position, then
  // the dependencies' snapshots
  uint32_t *snap_p = reinterpret_cast<uint32_t *>(lds + P.lds_snap_off) + wave * P.snap_words;
  for (int i = lane; i < P.snap_words; i += 64) snap_p[i] = 0;
  for (int i = threadIdx.x; i < P.data_floats; i += blockDim.x) data[i] = 0.f;
  __syncthreads();
  // The program has arrived: taken here, so that the compiler does not place
  // a wait for these loads (which would wait for every load in flight) at
  // their uses in the loop.
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    if (j < 4) asm volatile("" : "+v"(cw[j]));
    asm volatile("" : "+v"(ar[j]), "+v"(wr[j]));
  }
  asm volatile("" : "+v"(off_lo), "+v"(off_hi));

  const uint32_t snap = lds_addr(snap_p);
  const uint32_t cnt_base = lds_addr(cnt), data_l = lds_addr(data);
  auto counter = [&](uint32_t slot) __attribute__((always_inline)) { return cnt_base + 4u * slot * (uint32_t)bfs::kMaxWavesPerEngine; };
  const uint32_t own_words = counter(e);
  uint32_t *log_entries = nullptr;
  uint32_t nlog = 0;
  if (kInstr && P.dbg) {
    const int64_t nw = (int64_t)gridDim.x * P.n_engines;
    log_entries = P.dbg + nw + ((int64_t)wg * P.n_engines + wave) * 4 * P.dbg_cap;
  }
  WaveStats stt;
  if (kInstr && P.stats) {
    stt.on = true;
    stt.t_start = now_ticks();
  }
  const uint32_t limit = P.watchdog > 0xffffffffull ? 0xffffffffu : (uint32_t)P.watchdog;
  const uint32_t T = (uint32_t)P.tile;
  const uint32_t ld_ops = P.wide_x ? 1u : T / 64u, st_ops = P.wide_out ? 1u : T / 64u;   // accesses per tile
  uint32_t aborted = 0;
  uint32_t seen = 0;                       // lane w: last observed counter value of wait w (w < 64)

  // Issued, unretired loads and stores, oldest first: counter slot + 1 (0
  // none) in 8 bits each.  All entries of the queue have the same number of
  // vector-memory instructions (ops), which the counted waits rely on: a
  // change of it empties the queue first.
  uint64_t queue = 0;
  uint32_t pending = 0, ops = 1;
  uint32_t in_flight_pc = ~0u;             // instruction whose accesses the whole queue holds (~0: of several)
  auto add_slot = [&](uint32_t slot1) __attribute__((always_inline)) {
    if (slot1 != 0u) lds_add(counter(slot1 - 1u), 1u);
  };
  auto retire_one = [&]() __attribute__((always_inline)) {
    pending -= 1;
    wait_at_most(pending * ops);
    add_slot((uint32_t)queue & 0xffu);
    queue >>= 8;
  };
  auto retire_all = [&]() __attribute__((always_inline)) {
    if (pending > 0) {
      wait_vm<0>();
      for (; pending > 0; --pending, queue >>= 8) add_slot((uint32_t)queue & 0xffu);
    }
  };
  auto issued = [&](uint32_t slot1) __attribute__((always_inline)) {      // one more instruction of `ops` accesses is in flight
    queue |= (uint64_t)slot1 << (8u * pending);
    pending += 1;
    in_flight_pc = ~0u;
    if (kInstr) retire_all();
    else if (pending == kMaxPending || (pending + 1u) * ops > 16u) retire_one();
  };
  auto want_ops = [&](uint32_t n) __attribute__((always_inline)) {
    if (ops != n) {
      retire_all();
      ops = n;
    }
  };
  auto barrier_point = [&]() __attribute__((always_inline)) {             // Section 3.4: drain, meet, reset, meet
    retire_all();
    const uint64_t t0 = (kInstr && stt.on) ? now_ticks() : 0;
    region_sync(own_words, 1);
    if (kInstr && stt.on) stt.barrier += now_ticks() - t0;
    seen = 0;                              // the counters were reset
  };
  // Poll until the counter reaches thr, retiring what this engine holds.
  auto poll_until = [&](uint32_t addr, uint32_t thr, uint32_t dep, uint32_t inst) __attribute__((always_inline)) -> uint32_t {
    uint32_t polls = 0;
    while (true) {
      const uint32_t v = uniform(lds_poll(addr));
      if (v >= thr) return v;
      if (pending > 0) {
        retire_one();
        continue;
      }
      if (++polls > limit) {
        report_deadlock(P.err, dep, (uint32_t)wg, inst, thr, v, (uint32_t)wave);
        aborted = 1u;
        return v;
      }
      if (polls > 16u) __builtin_amdgcn_s_sleep(1);
    }
  };

  // Datapath pieces shared by the general path and the inner loop.
  auto ring_at = [&](uint32_t id) __attribute__((always_inline)) {        // 0 .. 3, selected without indexing (stays in scalar registers)
    return (uint32_t)(id == 0 ? P.ring_off[0] : id == 1 ? P.ring_off[1] : id == 2 ? P.ring_off[2] : P.ring_off[3]);
  };
  auto load_tile = [&](uint32_t dst, const float *src) __attribute__((always_inline)) {
    want_ops(ld_ops);
    if (P.wide_x) {
      __builtin_amdgcn_global_load_lds((const void *)(src + 4 * lane), (BFS_LDS void *)(uintptr_t)dst, 16, 0, 0);
    } else {
      for (uint32_t i = 0; i < T; i += 64u)
        __builtin_amdgcn_global_load_lds((const void *)(src + i + lane), (BFS_LDS void *)(uintptr_t)(dst + 4u * i), 4, 0, 0);
    }
  };
  // writes one tile to HBM as st_ops stores, in flight
  auto store_tile = [&](uint32_t src, float *dst) __attribute__((always_inline)) {
    want_ops(st_ops);
    if (P.wide_out) {
      *reinterpret_cast<f32x4 *>(dst + 4 * lane) = *(const BFS_LDS f32x4 *)(uintptr_t)(src + 16u * lane);
    } else {
      for (uint32_t i = 0; i < T; i += 64u) dst[i + lane] = *(const BFS_LDS float *)(uintptr_t)(src + 4u * (i + lane));
    }
  };
  auto scale_acc = [&](uint32_t acc, uint32_t src, float c) __attribute__((always_inline)) {         // acc += c * slot
    if (T == 256u) {
      BFS_LDS f32x4 *a = (BFS_LDS f32x4 *)(uintptr_t)(acc + 16u * lane);
      f32x4 v = *a;
      const f32x4 x = *(const BFS_LDS f32x4 *)(uintptr_t)(src + 16u * lane);
#pragma unroll
      for (int j = 0; j < 4; ++j) v[j] = v[j] + c * x[j];
      *a = v;
    } else {
      for (uint32_t i = lane; i < T; i += 64u) {
        BFS_LDS float *a = (BFS_LDS float *)(uintptr_t)(acc + 4u * i);
        *a = *a + c * *(const BFS_LDS float *)(uintptr_t)(src + 4u * i);
      }
    }
  };
  auto add_const = [&](uint32_t dst, uint32_t src, float c) __attribute__((always_inline)) {         // slot + c
    for (uint32_t i = lane; i < T; i += 64u)
      *(BFS_LDS float *)(uintptr_t)(dst + 4u * i) = *(const BFS_LDS float *)(uintptr_t)(src + 4u * i) + c;
  };

  // Trips of one loop, read 64 at a time: lane i holds entry tw_first + i of
  // the trip list of loop tw_loop.  next_trip: entry i of loop l, of which
  // `left` more follow for sure (those of its parent's remaining iterations);
  // called with nothing in flight where it has to read.
  uint32_t tw = 0, tw_loop = ~0u, tw_first = 0, tw_n = 0;
  auto has_trip = [&](uint32_t l, uint32_t i) __attribute__((always_inline)) { return l == tw_loop && i - tw_first < tw_n; };
  auto read_trips = [&](uint32_t l, uint32_t i, uint32_t left) __attribute__((always_inline)) {
    const int64_t o = (int64_t)((uint64_t)rl(off_lo, l) | (uint64_t)rl(off_hi, l) << 32);
    tw_loop = l;
    tw_first = i;
    tw_n = min(left, 63u) + 1u;
    if (lane < tw_n) tw = (uint32_t)P.trips[o + (int64_t)i + lane];
    asm volatile("" : "+v"(tw));           // waited for here
  };

  // The last inner loop found at an instruction, decoded (see below).
  struct Inner {
    uint32_t pc = ~0u;                     // the instruction it was decoded from
    bool ok = false, nest = false;
    uint32_t l = 0, a = 0, op = 0, slot1 = 0, wait = 0, n_waits = 0;
    InnerWait w0, w1;
    bool pre = false;                      // a no-op before the loop in the loop around it (an acquire)
    int32_t a2 = 0, a4 = 0;
    uint32_t a3 = 0, a5 = 0, a6 = 0, src = 0, dst = 0;
    float k_const = 0.f;
  } F;
  auto decode = [&](bool on, uint32_t row) __attribute__((always_inline)) {
    InnerWait x;
    if (on) {
      const uint32_t q0 = wrow(row, 0);
      x.addr = counter(q0 & 0xffu);
      x.dep = wrow(row, 1);
      x.k = wrow(row, 2);
      x.lP = (q0 >> 8) & 0xffu;
      x.lS = (q0 >> 16) & 0xffu;
      x.mask = (q0 >> 24) & 1u;
      x.N = (int32_t)wrow(row, 4);
      x.c = x.N * (int32_t)wrow(row, 3) + (x.N - (int32_t)wrow(row, 5));
    }
    return x;
  };
  // Runs the decoded loop from its first iteration of a trip on; returns the
  // code words it passes.
  // (The no-op before the loop in the general form only: with a form of its own
  // for wide loads the chain program took 214 us instead of 266, but the ring
  // program, which has no such no-op, 181 instead of 168.)
  enum { LOAD_WIDE, SCALE_256, OTHER };
  auto run_inner = [&](auto which) __attribute__((always_inline)) -> uint32_t {
    constexpr int kWhich = decltype(which)::value;
    constexpr bool kWide = kWhich == LOAD_WIDE, kPre = kWhich == OTHER;
    const bool tiles = kWide || (kWhich == OTHER && (F.op == 1u || F.op == 5u));
    const uint32_t l = F.l, a = F.a, own = counter(F.slot1 - 1u);
    uint32_t r = rl(rv, l), n = rl(tv, l);               // r of the trip's first iteration
    uint32_t ra = rl(rv, a), ha = rl(hv, a);
    const uint32_t ta = F.nest ? rl(tv, a) : ha;
    // What is in flight from here on is this instruction's, so that the queue
    // is a count.  (Told by the instruction, not by the queue's counter slots:
    // those of instructions that nothing waits for are alike, and a store must
    // not read its slot before a load ahead of it has landed there.  n_ops is a
    // sum: a choice between captured variables would keep all of them in
    // scratch memory.)
    const uint32_t is_ld = F.op == 1u, is_st = F.op == 5u;
    const uint32_t n_ops = is_ld * ld_ops + is_st * st_ops + (1u - is_ld - is_st) * ops;
    const uint64_t same = (uint64_t)F.slot1 * 0x0101010101010101ull;
    if (in_flight_pc != F.pc) retire_all();
    in_flight_pc = F.pc;
    ops = n_ops;
    const uint32_t most = max(min(kMaxPending, 16u / ops), 1u) - 1u;   // in flight after an instruction
    auto signal = [&](uint32_t m) __attribute__((always_inline)) {
      if (F.slot1 != 0u) lds_add(own, m);
    };
    auto start = [&](const InnerWait &w, uint32_t row) __attribute__((always_inline)) {
      InnerWaitState x;
      x.run = w.N * (int32_t)rl(rv, w.lP) - w.c;
      x.step = w.lP == l ? w.N : 0;
      x.step_a = w.lP == a ? w.N : 0;
      x.kk = !w.mask ? 0u : w.lS == l ? w.k : (rl(hv, w.lS) > w.k ? 0u : ~0u);
      x.met = row < 64u ? rl(seen, row & 63u) : 0u;
      return x;
    };
    InnerWaitState x0 = start(F.w0, F.wait), x1 = start(F.w1, F.wait + 1u);
    auto block = [&](const InnerWait &w, InnerWaitState &x, uint32_t inst) __attribute__((always_inline)) {
      uint32_t polls = 0;
      while (true) {
        x.met = uniform(lds_poll(w.addr));
        if ((int32_t)x.met >= x.run) break;
        if (pending > 0) {
          pending -= 1;
          wait_at_most(pending * ops);
          signal(1u);
        } else if (++polls > limit) {
          report_deadlock(P.err, w.dep, (uint32_t)wg, inst, (uint32_t)x.run, x.met, (uint32_t)wave);
          aborted = 1u;
          break;
        } else if (polls > 16u) {
          __builtin_amdgcn_s_sleep(1);
        }
      }
    };
    auto wait = [&](const InnerWait &w, InnerWaitState &x, uint32_t h) __attribute__((always_inline)) {
      if (x.run > (int32_t)x.met && h > x.kk && !aborted) block(w, x, r - 1u);
      x.run += x.step;
    };
    const bool pre = kPre && F.pre;
    const uint32_t pre_slot1 = pre ? code(F.pc - 2u, 0) >> 24 : 0u, pre_wait = pre ? code(F.pc - 2u, 2) : 0u;
    const uint32_t pre_n = pre ? code(F.pc - 2u, 3) : 0u;
    const InnerWait p0 = decode(pre_n > 0u, pre_wait), p1 = decode(pre_n > 1u, pre_wait + 1u);
    InnerWaitState y0 = start(p0, pre_wait), y1 = start(p1, pre_wait + 1u);
    // a wait of the no-op, whose threshold is evaluated at each iteration
    auto wait_pre = [&](const InnerWait &w, InnerWaitState &y) __attribute__((always_inline)) {
      const uint32_t rP = w.lP == l ? r - 1u : w.lP == a ? ra + 0u : rl(rv, w.lP);
      const uint32_t hS = w.lS == l ? n + 0u : w.lS == a ? ha + 0u : rl(hv, w.lS);
      y.run = w.mask && hS <= w.k ? 0 : w.N * (int32_t)rP - w.c;
      if (y.run > (int32_t)y.met && !aborted) block(w, y, ra - 1u);
    };
    auto flush = [&]() __attribute__((always_inline)) {
      if (pending > 0) {
        wait_vm<0>();
        signal(pending);
        pending = 0;
      }
    };
    // slot and tile
    const bool p4 = F.a4 >= 0, p2 = F.a2 >= 0;
    uint32_t s4 = p4 ? umod(rl(hv, (uint32_t)F.a4) - 1u, F.a5) : 0u;
    uint32_t s2 = p2 ? umod(rl(rv, (uint32_t)F.a2) - 1u, F.a3) : 0u;
    const uint32_t mul2 = p2 ? F.a5 : 0u;
    const uint32_t d4 = F.a4 == (int32_t)l ? 1u : 0u, d2 = F.a2 == (int32_t)l ? 1u : 0u;
    int64_t tile = tiles ? (tbase + (int64_t)rl(rv, F.a6) - 1) * (int64_t)T : 0;
    const int64_t d6 = tiles && F.a6 == l ? (int64_t)T : 0;
    while (true) {
      for (uint32_t h = 1; h <= n; ++h, ++r) {
        wait(F.w0, x0, h);
        wait(F.w1, x1, h);
        const uint32_t slot = 4u * T * (s4 + s2 * mul2);
        if (tiles && !aborted) {
          if (kWide)
            __builtin_amdgcn_global_load_lds((const void *)(P.x + tile + 4 * lane), (BFS_LDS void *)(uintptr_t)(F.dst + slot), 16, 0, 0);
          else if (F.op == 1u)
            load_tile(F.dst + slot, P.x + tile);
          else
            store_tile(F.src + slot, P.out + tile);
          if (pending >= most) {
            if (kWide) wait_vm<kMaxPending - 1>(); else wait_at_most(pending * ops);
            signal(1u);
          } else {
            pending += 1;
          }
        } else {
          if (!aborted) {
            if (kWhich == SCALE_256 || F.op == 2u) scale_acc(F.dst, F.src + slot, F.k_const);
            else add_const(F.dst + slot, F.src + slot, F.k_const);
          }
          signal(1u);
        }
        s4 = s4 + d4 == F.a5 ? 0u : s4 + d4;
        s2 = s2 + d2 == F.a3 ? 0u : s2 + d2;
        tile += d6;
      }
      if (ha == ta) break;
      // the next iteration of the loop around it, which holds nothing else (but
      // the no-op)
      ra += 1u;
      ha += 1u;
      if (pre) {
        wait_pre(p0, y0);
        wait_pre(p1, y1);
        flush();
        add_slot(pre_slot1);
      }
      if (!has_trip(l, ra - 1u)) {
        flush();
        read_trips(l, ra - 1u, ta - ha);
      }
      n = rl(tw, ra - 1u - tw_first);
      x0.run += x0.step_a;
      x1.run += x1.step_a;
      if (F.w0.mask && F.w0.lS == a) x0.kk = ha > F.w0.k ? 0u : ~0u;
      if (F.w1.mask && F.w1.lS == a) x1.kk = ha > F.w1.k ? 0u : ~0u;
      if (d4) s4 = 0u;
      if (F.a4 == (int32_t)a) s4 = s4 + 1u == F.a5 ? 0u : s4 + 1u;
      if (F.a2 == (int32_t)a) s2 = s2 + 1u == F.a3 ? 0u : s2 + 1u;
      if (tiles && F.a6 == a) tile += (int64_t)T;
    }
    if (kWhich == OTHER && F.op == 4u) drain_lds();      // a load into the slot (direct to LDS) may follow
    if (F.n_waits > 0u && F.wait < 64u) seen = wl(seen, F.wait, x0.met);
    if (F.n_waits > 1u && F.wait + 1u < 64u) seen = wl(seen, F.wait + 1u, x1.met);
    if (pre_n > 0u && pre_wait < 64u) seen = wl(seen, pre_wait, y0.met);
    if (pre_n > 1u && pre_wait + 1u < 64u) seen = wl(seen, pre_wait + 1u, y1.met);
    queue = pending > 0 ? same & ((1ull << (8u * pending)) - 1ull) : 0ull;
    rv = wl(rv, l, r - 1u);
    hv = wl(hv, l, n);
    tv = wl(tv, l, n);
    if (!F.nest) return 2u;
    rv = wl(rv, a, ra);
    hv = wl(hv, a, ha);
    return 3u;
  };

  uint32_t pc = 0;
  while (true) {
    const uint32_t w0 = code(pc, 0), kind = w0 & 0xffu;
    const uint32_t w1 = code(pc, 1), w2 = code(pc, 2), w3 = code(pc, 3);
    // A loop of one instruction with at most two waits (the usual innermost
    // loop of an engine): all that the general path below decodes for each
    // instruction and loop end is decoded once for the loop and evaluated once
    // per trip, and the iterations of a trip follow one another.
    if (kInner && kind == bfs::CODE_INSTR && !aborted &&
        (code(pc + 1, 0) & 0xffu) == (uint32_t)bfs::CODE_END && code(pc + 1, 2) + 1u == pc) {
      if (pc != F.pc) {
        F.pc = pc;
        F.op = (w0 >> 8) & 0xffu;
        F.slot1 = w0 >> 24;
        F.wait = w2;
        F.n_waits = w3;
        F.l = code(pc + 1, 1);
        // the loop around it, if it holds nothing but this loop and at most a
        // no-op before it
        F.a = pc > 0u ? code(pc - 1u, 3) : 0u;
        F.nest = (code(pc + 2, 0) & 0xffu) == (uint32_t)bfs::CODE_END && code(pc + 2, 1) == F.a &&
                 ((P.fallback_loops >> F.a) & 1u) == 0u;
        const uint32_t first = code(pc + 2, 2) + 1u, n0 = pc > 1u ? code(pc - 2u, 0) : 0u;   // first word of its body
        F.pre = F.nest && first + 2u == pc && (n0 & 0xffffu) == (uint32_t)bfs::CODE_INSTR && code(pc - 2u, 3) <= 2u;
        F.nest = F.pre || (F.nest && first + 1u == pc);
        F.ok = ((P.fallback_loops >> F.l) & 1u) == 0u && w3 <= 2u &&
               (F.op == 1u || F.op == 2u || F.op == 4u || F.op == 5u);
        // (waits on snapshots stay on the general path)
        for (uint32_t w = w2; F.ok && w < w2 + w3; ++w) F.ok = wrow(w, 6) == 0u;
        if (F.pre)
          for (uint32_t w = code(pc - 2u, 2); F.ok && w < code(pc - 2u, 2) + code(pc - 2u, 3); ++w) F.ok = wrow(w, 6) == 0u;
        F.w0 = decode(F.ok && w3 > 0u, w2);
        F.w1 = decode(F.ok && w3 > 1u, w2 + 1u);
        if (F.ok) {
          F.a2 = (int32_t)arg(w1, 2);
          F.a3 = arg(w1, 3);
          F.a4 = (int32_t)arg(w1, 4);
          F.a5 = arg(w1, 5);
          F.a6 = arg(w1, 6);
          F.k_const = __uint_as_float(arg(w1, 7));
          const uint32_t a0 = arg(w1, 0), a1 = arg(w1, 1);
          F.src = data_l + 4u * ring_at(a0);
          F.dst = data_l + 4u * (F.op == 2u ? (uint32_t)P.acc_off + a1 * T : ring_at(a1));
        }
      }
      if (F.ok && rl(hv, F.l) == 1u) {
        if (F.op == 1u && P.wide_x && !F.pre) pc += run_inner(std::integral_constant<int, LOAD_WIDE>{});
        else if (F.op == 2u && T == 256u && !F.pre) pc += run_inner(std::integral_constant<int, SCALE_256>{});
        else pc += run_inner(std::integral_constant<int, OTHER>{});
        continue;
      }
    }
    if (__builtin_expect(kind == bfs::CODE_INSTR, 1)) {
      // CODE_INSTR: w0 = kind | opcode << 8 | innermost loop << 16 | (counter
      // slot + 1) << 24, w1 its row, w2 its first wait row, w3 its waits.  The
      // innermost loop runs it once per iteration: r counts its executions.
      const uint32_t op = (w0 >> 8) & 0xffu, n_waits = w3, slot1 = w0 >> 24;
      const uint32_t inst = rl(rv, (w0 >> 16) & 0xffu) - 1u;
      for (uint32_t w = w2; w < w2 + n_waits; ++w) {
        const uint32_t q0 = wrow(w, 0), dep = wrow(w, 1);
        const uint32_t mask = (q0 >> 24) & 1u, linear = (q0 >> 25) & 1u;
        uint32_t thr;
        if (kMode == BFS_MODE_BARRIER) {
          thr = wrow(w, 3);
        } else {
          const uint32_t k = wrow(w, 2), q3 = wrow(w, 3), slots = wrow(w, 6);
          const uint32_t lS = (q0 >> 16) & 0xffu, hS = rl(hv, lS);
          if (slots > 0u) {
            // per-engine: the snapshot of iteration r_S - k (or the latest
            // one), under the mask of Eq. 5
            const uint32_t rS = rl(rv, lS);
            const bool owed = linear ? rS > k : (!mask || hS > k);
            const uint32_t idx = slots > 1u ? umod(rS - k, slots) : 0u;
            thr = owed ? uniform(lds_poll(snap + 4u * (q3 + idx))) : 0u;
          } else {
            thr = eq5(rl(rv, (q0 >> 8) & 0xffu), hS, (int)k, (int)q3, (int)wrow(w, 4), (int)wrow(w, 5), (int)mask);
          }
        }
        if (kInstr && (int)dep == P.fault_dep) thr += (uint32_t)P.fault_delta;
        uint32_t obs = 0;
        if (!aborted && thr > 0u && (kInstr || w >= 64u || thr > rl(seen, w & 63u))) {
          const uint64_t t0 = (kInstr && stt.on) ? now_ticks() : 0;
          obs = poll_until(counter(q0 & 0xffu), thr, dep, inst);
          if (w < 64u) seen = wl(seen, w, obs);
          if (kInstr && stt.on) {
            stt.blocked += now_ticks() - t0;
            stt.n_blocked += 1;
          }
        }
        if (kInstr) log_wait(log_entries, P.dbg_cap, nlog, dep, inst, thr, obs);
      }
      // Datapath.
      bool in_flight = false;                // retires later, in order
      if (!aborted && op != 0u) {
        // ring slot and tile index
        auto slot_of = [&]() __attribute__((always_inline)) {
          const int32_t a2 = (int32_t)arg(w1, 2), a4 = (int32_t)arg(w1, 4);
          uint32_t s = a4 >= 0 ? umod(rl(hv, (uint32_t)a4) - 1u, arg(w1, 5)) : 0u;
          if (a2 >= 0) s += umod(rl(rv, (uint32_t)a2) - 1u, arg(w1, 3)) * arg(w1, 5);
          return s;
        };
        auto tile_of = [&]() __attribute__((always_inline)) { return (tbase + (int64_t)rl(rv, arg(w1, 6)) - 1) * (int64_t)T; };
        if (op == 1u) {          // load
          load_tile(data_l + 4u * (ring_at(arg(w1, 1)) + slot_of() * T), P.x + tile_of());
          in_flight = true;
        } else {
          // the engine's earlier loads have landed before it reads a slot, and
          // retire before this instruction does
          retire_all();
          const float c = __uint_as_float(arg(w1, 7));
          if (op == 2u) {        // acc += c * slot
            scale_acc(data_l + 4u * ((uint32_t)P.acc_off + arg(w1, 1) * T),
                      data_l + 4u * (ring_at(arg(w1, 0)) + slot_of() * T), c);
          } else if (op == 3u) { // store acc
            store_tile(data_l + 4u * ((uint32_t)P.acc_off + arg(w1, 0) * T), P.out + (int64_t)wg * T);
            in_flight = true;
          } else if (op == 4u) { // slot + c
            const uint32_t s = slot_of() * T;
            add_const(data_l + 4u * (ring_at(arg(w1, 1)) + s), data_l + 4u * (ring_at(arg(w1, 0)) + s), c);
          } else if (op == 5u) { // store slot
            store_tile(data_l + 4u * (ring_at(arg(w1, 0)) + slot_of() * T), P.out + tile_of());
            in_flight = true;
          }
        }
      }
      // Retire in program order.  LDS executes a wave's operations in issue
      // order, so the add lands after the instruction's LDS reads and writes.
      if (in_flight) {
        issued(slot1);
      } else {
        retire_all();
        add_slot(slot1);
        if (op == 4u) drain_lds();           // a load into the slot (direct to LDS) may follow
      }
      pc += 1;
      continue;
    }
    if (kind == bfs::CODE_END) {           // w1 loop, w2 its loop word
      const uint32_t l = w1;
      if (kMode == BFS_MODE_BARRIER) {
        barrier_point();
      } else if ((P.fallback_loops >> l) & 1u) {
        // Section 5.2 fallback: everything issued in this iteration of l has
        // retired on every engine before any engine starts the next one.
        // Every engine walks the same loop tree with the same trip table, so
        // all waves meet the same sequence of barriers.
        retire_all();
        drain_all();
        __builtin_amdgcn_s_barrier();
      }
      const uint32_t h = rl(hv, l);
      if (h < rl(tv, l)) {
        rv = wl(rv, l, rl(rv, l) + 1u);
        hv = wl(hv, l, h + 1u);
        pc = w2 + 1;
      } else {
        pc += 1;
      }
      continue;
    }
    if (kind == bfs::CODE_LOOP) {          // w1 loop, w2 its end word, w3 parent
      if (kMode == BFS_MODE_BARRIER) barrier_point();
      const uint32_t l = w1, rp = rl(rv, w3);
      // the trip: entry rp - 1 of the loop's list; those of the parent's
      // remaining iterations follow it, so up to 64 are read at once
      if (!has_trip(l, rp - 1u)) {
        retire_all();
        read_trips(l, rp - 1u, rl(tv, w3) - rl(hv, w3));
      }
      const uint32_t t = rl(tw, rp - 1u - tw_first);
      tv = wl(tv, l, t);
      if (t == 0) {
        hv = wl(hv, l, 0u);
        pc = w2 + 1;
      } else {
        rv = wl(rv, l, rl(rv, l) + 1u);
        hv = wl(hv, l, 1u);
        pc += 1;
      }
      continue;
    }
    if (kind == bfs::CODE_HALT) break;
    if (kind == bfs::CODE_TRACK) {         // w1 producer engine, w2 instructions passed
      const uint32_t a = snap + 4u * w1;
      lds_store(a, uniform(lds_poll(a)) + w2);
      pc += 1;
      continue;
    }
    {                                      // CODE_SNAP
      // the producer engine's running count right after the producer's
      // position, kept for the iteration of S it belongs to (w0: engine and
      // S; w1 snapshots kept, w2 the first one's word)
      const uint32_t idx = w1 > 1u ? umod(rl(rv, (w0 >> 16) & 0xffu), w1) : 0u;
      lds_store(snap + 4u * (w2 + idx), uniform(lds_poll(snap + 4u * ((w0 >> 8) & 0xffu))));
      pc += 1;
      continue;
    }
  }
  retire_all();
  if (kInstr && P.dbg && lane == 0) P.dbg[(int64_t)wg * P.n_engines + wave] = nlog;
  if (kInstr && stt.on && lane == 0) {
    uint64_t *o = P.stats + ((int64_t)wg * P.n_engines + wave) * 8;
    o[0] = now_ticks() - stt.t_start;
    o[1] = stt.blocked;
    o[2] = stt.n_blocked;
    o[3] = stt.barrier;
    o[4] = 0;
    o[5] = 0;
    o[6] = 0;
    o[7] = 0;
  }
}

}  // namespace

namespace bfs {

bfs_status launch_interp(const bfs_plan *p, DevImage *img, const void *const *bufs, int32_t nbufs,
                         const int32_t *trips, const int64_t *trip_off, int32_t n_wg, void *stream,
                         uint32_t *dbg, int64_t dbg_cap, const bfs_run_opts &o) {
  for (int e = 0; e < p->n_engines; ++e)
    if (p->waves_per_engine[e] != 1) return fail(BFS_E_UNSUPPORTED, "interpreter runs one wave per engine");
  if ((int)p->instr_engine.size() > kMaxInstrsInterp) return fail(BFS_E_RESOURCE, "interpreter: > 256 instructions");
  if (!trips || !trip_off) return fail(BFS_E_INVALID, "interpreter needs trip tables");
  if (nbufs < 3) return fail(BFS_E_INVALID, "interpreter needs buffers [base, x, out]");
  InterpParams P{};
  P.code = img->code;
  P.engine_off = img->engine_off;
  P.waits = img->waits;
  P.args = img->instr_args;
  P.trips = trips;
  P.trip_off = trip_off;
  P.base = static_cast<const int64_t *>(bufs[0]);
  P.x = static_cast<const float *>(bufs[1]);
  P.out = static_cast<float *>(const_cast<void *>(bufs[2]));
  P.dbg = dbg;
  P.dbg_cap = dbg_cap;
  P.err = img->err;
  P.stats = o.dev_stats;
  P.watchdog = o.watchdog_polls;
  P.fault_dep = o.fault_dep;
  P.fault_delta = o.fault_delta;
  P.n_loops = p->n_loops;
  P.n_engines = p->n_engines;
  P.fallback_loops = p->fallback_loops;
  P.tile = p->tile_elems > 0 ? p->tile_elems : 64;
  P.wide_x = P.tile == 256 && reinterpret_cast<uintptr_t>(bufs[1]) % 16 == 0;
  P.wide_out = P.tile == 256 && reinterpret_cast<uintptr_t>(bufs[2]) % 16 == 0;
  int64_t off = 0;
  for (int i = 0; i < 4; ++i) {
    P.ring_off[i] = (int32_t)off;
    off += (int64_t)p->ring_slots[i] * P.tile;
  }
  P.acc_off = (int32_t)off;
  off += (int64_t)(p->n_accs > 0 ? p->n_accs : 0) * P.tile;
  const int64_t data_floats = off + 4 * P.tile;
  P.data_floats = (int32_t)data_floats;
  const int counters_bytes = kMaxSlots * kMaxWavesPerEngine * 4;
  P.lds_data_off = counters_bytes;
  P.snap_words = p->mode == BFS_MODE_BARRIER_FREE && p->alloc == BFS_ALLOC_PER_ENGINE ? p->snap_words : 0;
  P.lds_snap_off = (int32_t)(P.lds_data_off + data_floats * 4);
  const size_t lds_bytes = (size_t)P.lds_snap_off + (size_t)p->n_engines * P.snap_words * 4;
  // The limit a program is held to includes 1408 bytes per engine for loop
  // registers and per-instruction words, the family's documented footprint
  // (they are held in registers).
  if (lds_bytes + (size_t)p->n_engines * (3 * kMaxLoops + kMaxInstrsInterp) * 4 > 160 * 1024)
    return fail(BFS_E_RESOURCE, "interpreter: LDS footprint over 160 KiB");
  // the program in registers: at most 64 code words and 64 waits per engine
  bool lanes = true;
  for (int e = 0; e < p->n_engines; ++e)
    lanes = lanes && p->code_off[e + 1] - p->code_off[e] <= 64 && img->n_waits[e] <= 64;
  const bool instr = dbg || o.dev_stats || o.fault_dep >= 0;
  auto go = [&](auto kern) -> bfs_status {
    hipError_t err = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_bytes);
    if (err != hipSuccess) return fail(BFS_E_DEVICE, std::string("hipFuncSetAttribute: ") + hipGetErrorString(err));
    hipLaunchKernelGGL(kern, dim3(n_wg), dim3(64 * p->n_engines), lds_bytes, (hipStream_t)stream, P);
    err = hipGetLastError();
    if (err != hipSuccess) return fail(BFS_E_DEVICE, std::string("interp launch: ") + hipGetErrorString(err));
    return BFS_OK;
  };
  if (p->mode == BFS_MODE_BARRIER) {
    if (instr) return lanes ? go(interp_kernel<BFS_MODE_BARRIER, true, true>) : go(interp_kernel<BFS_MODE_BARRIER, true, false>);
    return lanes ? go(interp_kernel<BFS_MODE_BARRIER, false, true>) : go(interp_kernel<BFS_MODE_BARRIER, false, false>);
  }
  if (instr)
    return lanes ? go(interp_kernel<BFS_MODE_BARRIER_FREE, true, true>) : go(interp_kernel<BFS_MODE_BARRIER_FREE, true, false>);
  // The kernel with inner loops run without dispatch, if a loop of the program
  // is one and no engine tracks another's instances: those engines' loops hold
  // further words and stay on the general path, and the slowest engine sets the
  // pace (us with these loops and without: ring program, a counter per engine,
  // 256 workgroups 856 and 696, chain program, 191 workgroups 52.4 and 43.6;
  // a counter per loop, ring, 1024 workgroups 167 and 513, chain 269 and 655).
  bool inner = false, tracks = false;
  for (int e = 0; e < p->n_engines; ++e)
    for (int32_t pc = 0, n = p->code_off[e + 1] - p->code_off[e]; pc < n; ++pc) {
      const int32_t *w = &p->code[4 * (size_t)(p->code_off[e] + pc)];
      tracks = tracks || w[0] == CODE_TRACK || w[0] == CODE_SNAP;
      if (w[0] != CODE_INSTR || pc + 1 == n || w[4] != CODE_END || w[6] + 1 != pc) continue;
      const int32_t op = p->instr_opcode[w[1]];
      inner = inner || (((p->fallback_loops >> w[5]) & 1u) == 0u && (op == 1 || op == 2 || op == 4 || op == 5) &&
                        p->instr_wait_off[w[1] + 1] - p->instr_wait_off[w[1]] <= 2);
    }
  inner = inner && !tracks;
  if (inner)
    return lanes ? go(interp_kernel<BFS_MODE_BARRIER_FREE, false, true, true>)
                 : go(interp_kernel<BFS_MODE_BARRIER_FREE, false, false, true>);
  return lanes ? go(interp_kernel<BFS_MODE_BARRIER_FREE, false, true>) : go(interp_kernel<BFS_MODE_BARRIER_FREE, false, false>);
}

}  // namespace bfs
