// ems_kernels.hip -- gfx950 kernels of the transport loop.
//
// The paper steps the whole track population once per iteration with one
// kernel per species in three streams, appending secondaries to per-species
// "next" index arrays with an atomic counter and swapping current/next after
// each step (section 3).  On MI355X:
//  - one launch per iteration: its waves are dealt to the photons and to the
//    e-/e+ (a concatenated index space [e- | e+]), and go on with the other
//    species when their own is used up, so neither species' last waves leave
//    the device idle;
//  - the queues hold the tracks themselves (64-byte records); survivors are
//    rewritten compactly each iteration, so slots are reused by construction;
//  - a thread keeps stepping its track (a "visit") until a step creates
//    secondaries or ends the track, so the many boundary crossings of photons
//    in the thin slabs do not each cost a queue round trip; every step still
//    draws from its own (id, step) stream, so histories are unchanged;
//  - appends are aggregated per wave (ballot + popcount prefix, one atomic
//    per wave and species);
//  - secondaries are reserved against a per-species limit that always leaves
//    room for every survivor; a track whose secondaries do not fit is carried
//    from before that step, so a full queue defers work instead of losing it;
//  - the last block of the launch leaves the extents of the next queues to
//    the next launch, so a chain of launches needs no host round trip.
#include <hip/hip_runtime.h>

#include "ems_iteration.hpp"

namespace ems {

namespace {

constexpr int kBlock = 64 * kBlockWaves;
// lanes waiting in the world volume that make a wave compute their boundary
// distances together (box geometries)
#ifndef EMS_WORLD_BATCH
#define EMS_WORLD_BATCH 16
#endif
constexpr uint32_t kWorldBatch = EMS_WORLD_BATCH;
// s_waitcnt immediate for "all vector memory operations done" (vmcnt 0,
// expcnt and lgkmcnt at their maxima: not waited on)
constexpr int kWaitVmem = 0x0F70;

// Reserve `count` (0..3) consecutive slots per lane in an append counter with
// one atomic per wave; returns this lane's first slot.  Every lane of the wave
// must pass the same counter.
__device__ inline uint32_t wave_reserve(uint32_t* counter, uint32_t count) {
  const uint64_t b0 = __ballot(count & 1u);
  const uint64_t b1 = __ballot((count >> 1) & 1u);
  const uint32_t total = (uint32_t)(__popcll(b0) + 2 * __popcll(b1));
  if (total == 0) return 0;
  const uint64_t lt = __lanemask_lt();
  const uint32_t prefix = (uint32_t)(__popcll(b0 & lt) + 2 * __popcll(b1 & lt));
  const int leader = __ffsll((unsigned long long)(b0 | b1)) - 1;
  uint32_t base = 0;
  if ((int)__lane_id() == leader) base = atomicAdd(counter, total);
  base = __shfl(base, leader);
  return base + prefix;
}

// Next queue index for every lane with `want`: taken from the wave's own
// range [lo, hi), which is refilled a chunk at a time from the launch's
// global cursor, so a wave pays one global atomic per chunk instead of one
// per refill.  Every index below the cursor's final value is handed out
// exactly once (ranges are disjoint and none is dropped).
// A chunk is an eighth of an even share of what the wave knows to be left of
// the queue's n indices, between a whole wave's request and kCursorMax, so
// the launch still ends with small ones (40 000 x 10 GeV, mixed form: 64
// indices always 104.5 ms, 256 always 105.9, by what is left 102.6; 10^4 x
// 10 GeV 40.9, 43.7 and 40.9; 500 x 2 GeV 4.27, 5.75 and 4.25).
constexpr uint32_t kCursorMin = 64, kCursorMax = 256;
static_assert(kCursorMin >= 64, "a chunk must cover a whole wave's request");
__device__ inline uint32_t take_next(uint32_t* cursor, uint32_t pool, bool want, uint32_t& lo, uint32_t& hi,
                                     uint32_t n, uint32_t waves) {
  const uint64_t m = __ballot(want);
  const uint32_t wants = (uint32_t)__popcll(m);
  const uint32_t rank = (uint32_t)__popcll(m & __lanemask_lt());
  const uint32_t avail = hi - lo;
  uint32_t i = lo + rank;
  if (wants > avail) {
    // the rest of the old range, then a fresh chunk (wants <= 64 <= chunk)
    const uint32_t share = (n > hi ? n - hi : 0u) / 8u / waves;
    const uint32_t chunk = share < kCursorMin ? kCursorMin : (share > kCursorMax ? kCursorMax : share);
    uint32_t base = 0;
    const int leader = __ffsll((unsigned long long)m) - 1;
    if ((int)__lane_id() == leader) base = atomicAdd(cursor, chunk);
    base = __shfl(base, leader) + pool;
    if (rank >= avail) i = base + (rank - avail);
    lo = base + (wants - avail);
    hi = base + chunk;
  } else {
    lo += wants;
  }
  return i;
}

// Append slots in wave-private chunks.  A wave holds a range [lo, hi) of each
// append counter (Ctl::next) and refills it `chunk` slots at a time (one
// global atomic per chunk instead of one per batch: thousands of waves
// appending to the same few counters otherwise serialise on them).  Unused
// ends of the ranges are marked dead when the wave exits.  chunk = 1 is
// exact reservation (no unused slots).
struct Ranges {
  uint32_t lo[kNextCounters], hi[kNextCounters];  // uniform
};
// A wave's request to one counter: cnt (0..MAX) slots per lane; the lane's
// k-th slot is slot(k).
struct Take {
  uint32_t prefix, total, lo, avail, base;
  __device__ uint32_t slot(uint32_t k) const {
    const uint32_t x = prefix + k;
    return x < avail ? lo + x : base + (x - avail);
  }
};
template <int MAX = 1>
__device__ inline Take ask(const Ranges& rg, int c, uint32_t cnt) {
  const uint64_t b0 = __ballot(cnt & 1u);
  const uint64_t lt = __lanemask_lt();
  Take t;
  t.total = (uint32_t)__popcll(b0);
  t.prefix = (uint32_t)__popcll(b0 & lt);
  if constexpr (MAX > 1) {
    const uint64_t b1 = __ballot((cnt >> 1) & 1u);
    t.total += 2 * (uint32_t)__popcll(b1);
    t.prefix += 2 * (uint32_t)__popcll(b1 & lt);
  }
  t.lo = rg.lo[c];
  t.avail = rg.hi[c] - rg.lo[c];
  t.base = 0;
  return t;
}
// Serve up to five requests at once: the counters that have to be refilled
// are incremented by one instruction, lane c for counter c.  The increments
// complete at the memory side, some microseconds away: one after another
// they were most of a batch in a wave with few tracks.
struct Ask {
  int c;
  uint32_t chunk;
  Take* t;
};
template <int N>
__device__ inline void serve(Ctl* ctl, Ranges& rg, const Ask (&a)[N]) {
  uint32_t need[N], grab[N], any = 0, v = 0;
  const uint32_t lane = __lane_id();
#pragma unroll
  for (int i = 0; i < N; ++i) {
    const Take& t = *a[i].t;
    need[i] = t.total > t.avail ? t.total - t.avail : 0u;
    grab[i] = need[i] == 0u ? 0u : (need[i] > a[i].chunk ? need[i] : a[i].chunk);
    any |= need[i];
    if (lane == (uint32_t)a[i].c) v = grab[i];
  }
  uint32_t got = 0;
  if (any) {
    if (v) got = atomicAdd(&ctl->next[lane * kLine], v);
  }
#pragma unroll
  for (int i = 0; i < N; ++i) {
    const int c = a[i].c;
    if (need[i]) {
      const uint32_t base = (uint32_t)__builtin_amdgcn_readlane((int)got, c);
      a[i].t->base = base;
      rg.lo[c] = base + need[i];
      rg.hi[c] = base + grab[i];
    } else {
      rg.lo[c] += a[i].t->total;
    }
  }
}

// Per-iteration append plan by species (every wave of an iteration's launches
// computes the same, from the current queue sizes).  The chunk is the
// largest power of two up to EMS_APPEND_CHUNK for which all waves together
// leave unused at most a quarter of the current population and of the free
// room (so small populations append exactly); the secondary limit leaves
// room for every survivor plus the unused chunk ends of the home region, and
// less than that where room is scarce (secondary_limit).
// 128: 40 000 x 10 GeV, mixed form, 104.5 ms, 10^4 x 10 GeV 40.6 (64: 108.0 and
// 40.65, 256: 104.5 and 40.9, 1024: 109.5 and 41.2).
#ifndef EMS_APPEND_CHUNK
#define EMS_APPEND_CHUNK 128
#endif
struct Plan {
  uint32_t lim[3], chunk[3];
  uint32_t lim_s, chunk_s;  // appends to the next short buffer
};
// The current short electrons (ns) may all survive their first step into
// the next e- queue, so they count with the current e- tracks; the short
// launch's waves also append to that queue's home region.  New short
// electrons are e- of the next iteration as well: the e- secondary limit is
// shared, half of it (at most the short buffer's capacity) for the short
// buffer, so that the next iteration's e- and short electrons together
// again leave room for all their survivors.  The short buffer takes the e-
// chunk, bounded so that all waves together leave unused at most a quarter
// of its capacity.
// SHORT: the kernel variant routes short electrons (the plan is the same
// as without when the context has no short buffers).
template <bool SHORT>
__device__ inline Plan append_plan(const KArgs& a, uint32_t n0, uint32_t n1, uint32_t n2, uint32_t ns,
                                   uint32_t level) {
  Plan p;
  if constexpr (!SHORT) {
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      const uint64_t n = q == 0 ? n0 : (q == 1 ? n1 : n2);
      const uint64_t room = a.cap - n;
      const uint64_t waves = 2ull * a.waves;
      const uint64_t budget = (n < room ? n : room) / 4;
      uint32_t chunk = EMS_APPEND_CHUNK;
      while (chunk > 1 && waves * chunk > budget) chunk >>= 1;
      p.chunk[q] = chunk;
      const uint64_t slack = chunk > 1 ? (uint64_t)a.waves * chunk : 0;  // <= room / 4
      p.lim[q] = secondary_limit((uint32_t)(room - slack), a.cap, level);
    }
    p.lim_s = 0;
    p.chunk_s = 1;
    return p;
  }
  const uint64_t waves = 2ull * a.waves + (a.cap_s ? a.waves_s : 0u);
#pragma unroll
  for (int q = 0; q < 3; ++q) {
    const uint64_t n = q == 0 ? n0 : (q == 1 ? (uint64_t)n1 + ns : n2);
    const uint64_t room = n < a.cap ? a.cap - n : 0;
    const uint64_t budget = (n < room ? n : room) / 4;
    uint32_t chunk = EMS_APPEND_CHUNK;
    while (chunk > 1 && waves * chunk > budget) chunk >>= 1;
    const uint64_t home_waves = (uint64_t)a.waves + (q == 1 && a.cap_s ? a.waves_s : 0u);
    const uint64_t slack = chunk > 1 ? home_waves * chunk : 0;
    p.chunk[q] = chunk;
    p.lim[q] = secondary_limit((uint32_t)(room > slack ? room - slack : 0), a.cap, level);
  }
  uint32_t cs = p.chunk[1];
  while (cs > 1 && waves * cs > a.cap_s / 4) cs >>= 1;
  p.chunk_s = cs;
  p.lim_s = 0;
  if (a.cap_s) {
    const uint32_t half = p.lim[1] / 2;
    p.lim_s = (uint64_t)half < a.cap_s ? half : (uint32_t)a.cap_s;
    p.lim[1] -= p.lim_s;
  }
  return p;
}

// the interactions after which the parent track goes on
__device__ inline bool parent_survives(uint32_t process) {
  return process == kXCompton || process == kXMoller || process == kXBhabha || process == kXBrem;
}

// One slot per lane with `want` among the lanes executing this call (also in
// divergent code): one atomic per call for all of them.
__device__ inline unsigned long long active_append(unsigned long long* counter, bool want) {
  const uint64_t m = __ballot(want);
  if (m == 0) return 0;
  const int leader = __ffsll((unsigned long long)m) - 1;
  unsigned long long base = 0;
  if ((int)__lane_id() == leader) base = atomicAdd(counter, (unsigned long long)__popcll(m));
  base = __shfl(base, leader);
  return base + (unsigned long long)__popcll(m & __lanemask_lt());
}

__device__ inline uint32_t wave_sum(uint32_t v) {
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
  return v;
}
__device__ inline void wave_count(uint32_t* counter, uint32_t v) {
  const uint32_t s = wave_sum(v);
  if (__lane_id() == 0 && s) atomicAdd(counter, s);
}

// Launch tallies (Ctl::add): a wave sums each over its lanes, lane k keeps
// tally k, and they are added to the block's copy in LDS with one instruction;
// the block adds its copy to the launch's with another when it ends.  (The
// copy is of 32-bit words, as tables may fill LDS but for 80 bytes: a wave
// adds a sum that eight of could pass them, four waves with two loops each, to
// the launch's tally itself.)  (Where
// every lane adds to the same words the compiler sums them itself, one lane
// after another: some 5000 instructions at the end of each of a wave's loops.
// 300 requests 13.6 -> 12.6 ms, 32 x 1 GeV 1.80 -> 1.69, 500 x 2 GeV 4.07 ->
// 3.98, 10^4 x 10 GeV 40.55 -> 40.37.)
__device__ inline void clear_counts(uint32_t* cnt) {
  if (threadIdx.x < kAdds) cnt[threadIdx.x] = 0u;
}
// (the old value is waited for, so the addition is done)
__device__ inline void add_tally(Ctl* ctl, uint32_t k, unsigned long long v) {
  const unsigned long long old = atomicAdd(&ctl->add[k], v);
  asm volatile("" ::"v"((uint32_t)old));
}
// sum over a wave with all lanes active: within rows of 16 lanes, then the
// rows' totals (row_shr 1, 2, 4, 8; row_bcast 15 and 31)
__device__ inline uint32_t wave_total(uint32_t v) {
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xf, 0xf, true);
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xf, 0xf, true);
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xf, 0xf, true);
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xf, 0xf, true);
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xa, 0xf, false);
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xc, 0xf, false);
  return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}
struct Tallies {
  unsigned long long mine = 0;  // lane k: tally k
  __device__ void count(int k, uint32_t v) {
    // (halves: the sum of 64 counters may pass 32 bits)
    const unsigned long long s = wave_total(v & 0xFFFFu) + ((unsigned long long)wave_total(v >> 16) << 16);
    if (__lane_id() == (uint32_t)k) mine = s;
  }
  __device__ void add_to(Ctl* ctl, uint32_t* cnt) const {
    static_assert(2 * kBlockWaves <= 8, "eight sums below 2^29 fit a word");
    if (__lane_id() >= kAdds || !mine) return;
    if (mine >> 29) add_tally(ctl, __lane_id(), mine);
    else atomicAdd(&cnt[__lane_id()], (uint32_t)mine);
  }
};
// all waves of the block have counted (a barrier inside)
__device__ inline void publish_counts(Ctl* ctl, const uint32_t* cnt) {
  __syncthreads();
  if (threadIdx.x < kAdds) {
    const uint32_t v = cnt[threadIdx.x];
    if (v) add_tally(ctl, threadIdx.x, v);
  }
}

template <class R>
__device__ inline void store_track(const Queue<R>& q, uint32_t i, const Trk<R>& t, uint32_t vb) {
  q.store(i, t, (t.n << vb) | (uint32_t)t.slab);
}

// position of the idx-th track of a queue with `home` tracks in the bottom
// region (the rest are in the top region, counted downwards)
__device__ inline uint32_t queue_pos(uint32_t idx, uint32_t home, uint64_t cap) {
  return idx < home ? idx : (uint32_t)(cap - 1 - (idx - home));
}

// Tallies of one applied step: FP64 atomic scoring per (event, slab), energy
// ledger, optional per-event counts and step log.
struct DevSink {
  // deposits of consecutive steps into the same (event, slab) add up in the
  // lane and reach the tally with one atomic when the cell changes or the
  // lane finishes (summation order of FP64 atomics is unordered anyway)
  size_t acc_cell = 0;
  double acc_dep = 0.0;

  __device__ void flush(const KArgs& a) {
    if (acc_dep != 0.0) atomicAdd(&a.edep[acc_cell], acc_dep);
    acc_dep = 0.0;
  }

  // F: the kernel's optional parts; the per-step records (exits, full
  // ledger, step log) exist only with kFRecord
  template <int F, class R>
  __device__ void apply(const KArgs& a, int sp, const Trk<R>& t, const StepOut<R>& o, double e_before) {
    Ctl* const ctl = a.ctl;
    if (o.dep != 0.0) {
      const size_t cell = (size_t)t.ev * a.env.n_slabs + o.slab;
      if (cell != acc_cell) {
        flush(a);
        acc_cell = cell;
      }
      acc_dep += o.dep;
    }
    LedgerDev& L = a.ledger[t.ev];
    if (o.escaped != 0.0) atomicAdd(&L.escaped[0] + sp, o.escaped);
    if (o.killed != 0.0) atomicAdd(&L.killed, o.killed);
    if (o.pair) atomicAdd(&L.n_pair, (uint32_t)o.pair);
    if (o.annih) atomicAdd(&L.n_annih, (uint32_t)o.annih);
    if constexpr ((F & kFRecord) == 0) return;
    if (a.exit_cap) {
      // the track left the stack: its state at the exit point
      const bool out = o.escaped != 0.0;
      const unsigned long long i = active_append(&ctl->exit_n, out);
      if (out && i < a.exit_cap) {
        ExitRec& x = a.exits[i];
        x.event = t.ev;
        x.species = (uint32_t)sp;
        x.ekin = o.escaped;
        x.pos[0] = t.x;
        x.pos[1] = t.y;
        x.pos[2] = t.z;
        x.dir[0] = t.ux;
        x.dir[1] = t.uy;
        x.dir[2] = t.uz;
      }
    }
    if (a.flags & kFlagFullLedger) {
      atomicAdd(&L.n_steps, 1ull);
      if (o.clen != 0.0) atomicAdd(&L.charged_len, o.clen);
      if (o.null) atomicAdd(&L.n_null, 1ull);
      if (o.nsec > 0) atomicAdd(&L.n_created[0] + o.sec[0].sp, 1ull);
      if (o.nsec > 1) atomicAdd(&L.n_created[0] + o.sec[1].sp, 1ull);
    }
    if (a.flags & kFlagSteplog) {
      const unsigned long long ls = atomicAdd(&ctl->log_n, 1ull);
      if (ls < a.log_cap) {
        StepRec& r = a.log[ls];
        r.event = t.ev;
        r.species = (uint32_t)sp;
        r.id = t.id;
        r.step = t.n - 1;
        r.slab_after = t.slab;
        r.limiter = o.limiter;
        r.process = o.process;
        r.e_before = e_before;
        r.e_after = t.E;
        r.pos[0] = t.x;
        r.pos[1] = t.y;
        r.pos[2] = t.z;
        r.step_len = o.step_len;
        r.edep = o.dep;
      }
    }
  }
};

// Stage the table blocks of the launch's species (bit 0 of `which`: photons,
// bit 1: e-/e+), the slab planes, slab materials and material constants in
// LDS; returns the environment pointing there.
template <class R>
__device__ inline R* stage_tables(const void* src, uint32_t n, char*& lds) {
  R* dst = reinterpret_cast<R*>(lds);
  const R* t = static_cast<const R*>(src);
  for (uint32_t i = threadIdx.x; i < n; i += kBlock) dst[i] = t[i];
  lds += (n * sizeof(R) + 7) / 8 * 8;
  return dst;
}
// what a block holds in LDS
template <class R>
struct Staged {
  const R *tg, *tl;
  const double* zplane;
  const MatRT* mat;
  const uint32_t* slab_mat;
};
template <class R, int GEO>
__device__ Staged<R> stage(const KArgs& a, char* lds, uint32_t which) {
  Staged<R> st{nullptr, nullptr, nullptr, nullptr, nullptr};
  if (which & kPhotons) st.tg = stage_tables<R>(a.tab_g, a.n_mat * kGammaTables * a.env.nodes, lds);
  if (which & kLeptons) st.tl = stage_tables<R>(a.tab_l, a.n_mat * kLeptonTables * a.env.nodes, lds);
  double* zp = reinterpret_cast<double*>(lds);
  // a box geometry reads its volume materials from global memory
  const uint32_t nz = GEO == 1 ? 0u : a.env.n_slabs + 1, nsm = GEO == 1 ? 0u : a.env.n_slabs;
  for (uint32_t i = threadIdx.x; i < nz; i += kBlock) zp[i] = a.zplane[i];
  MatRT* mr = reinterpret_cast<MatRT*>(zp + nz);
  if (threadIdx.x < a.n_mat) mr[threadIdx.x] = a.mat[threadIdx.x];
  uint32_t* sm = reinterpret_cast<uint32_t*>(mr + a.n_mat);
  for (uint32_t i = threadIdx.x; i < nsm; i += kBlock) sm[i] = a.slab_mat[i];
  __syncthreads();
  st.zplane = zp;
  st.mat = mr;
  st.slab_mat = sm;
  return st;
}

// The kernel's arguments as its first parameter holds them, read anew: a
// wave needs some eighty scalars over one iteration of its loop, more than
// fit the scalar registers beside its own state, and a value that is kept
// is spilled to lanes of vector registers and fetched back one word an
// instruction.  Reading them again from the argument segment (scalar cache)
// where a part of the loop begins keeps them out of the other parts: spilled
// scalars of the FP64 kernel 228 -> 150 (fetches and stores of them 1554 ->
// 484 of 12 000 instructions), 10^4 x 10 GeV 48.9 -> 46.1 ms, 40 000 x 10 GeV
// in the mixed form 127.6 -> 118.6 ms.
__device__ __forceinline__ const KArgs& fresh_args() {
  using Arg = const __attribute__((address_space(4))) KArgs;
  Arg* p = (Arg*)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(p));
  return *(const KArgs*)p;
}
// The walk of the hierarchy from the world volume as a function of its own,
// for the FP64 kernels: it needs a hundred registers for a while, and inlined
// it had the loop's own values spilled around every step (1500 x 10 GeV in the
// tower block: 27.2 ms inlined, 25.6 so; with FP32 tracks, which leave it the
// registers, 9.15 ms inlined and 9.3 as a call).  `args`: the kernel's
// argument segment, the same for all lanes.
__device__ __noinline__ GeoPre walk_world(const KArgs* args, double x, double y, double z, double ux, double uy,
                                          double uz) {
  using Arg = const __attribute__((address_space(4))) KArgs;
  const uint64_t at = (uint64_t)args;
  Arg* a = (Arg*)((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)at) |
                  (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(at >> 32)) << 32);
  const double p[3] = {x, y, z}, u[3] = {ux, uy, uz};
  GeoPre g{0.0, Face{0, 0.0, 0, -1}};
  g.s = world_distance(((const KArgs*)a)->env.nav, p, u, g.fc);
  return g;
}

template <class R>
__device__ __forceinline__ StepReals<R> reals_of(const KArgs& a) {
  if constexpr (sizeof(R) == 4) return a.env32;
  else return a.env;
}
template <class R, int GEO>
__device__ __forceinline__ StepEnv<R> env_of(const KArgs& a, const Staged<R>& st) {
  StepEnv<R> e;
  e.tg = st.tg;
  e.tl = st.tl;
  e.zplane = GEO == 1 ? nullptr : st.zplane;
  e.slab_mat = GEO == 1 ? a.slab_mat : st.slab_mat;
  e.mat = st.mat;
  if constexpr (GEO == 1) e.nav = a.env.nav;
  e.elc = a.el_c;
  e.elt = static_cast<const R*>(a.el_tab);
  e.nodes = a.env.nodes;
  e.n_slabs = a.env.n_slabs;
  static_cast<StepReals<R>&>(e) = reals_of<R>(a);
  e.half_xy = a.env.half_xy;
  e.bz = a.env.bz;
  e.ecut = a.env.ecut;
  e.tcut = a.env.tcut;
  e.kcut = a.env.kcut;
  e.mask = a.env.mask;
  e.seed = a.env.seed;
  e.max_steps = a.env.max_steps;
  return e;
}

}  // namespace

// The visits of one species in one iteration: photons (PHOTONS) or e-/e+.
//
// Batched lane refill: the lanes of a wave keep stepping their tracks while
// more than refill_below (photons: photon_refill_below) of them are still
// inside a visit.  Then the lanes whose visit ended commit together
// (secondaries, survivors, carried tracks: a few atomics for the whole
// batch) and empty lanes take the next tracks of the queue from a
// per-launch cursor.  Lanes thus stay busy instead of waiting for the
// wave's longest visit, without paying one atomic per track.  The order in
// which tracks are visited does not change any result.

// Minimum resident waves per SIMD the register allocation must allow, per
// arithmetic type, geometry kind and optional parts.  FP64: 2 (at 3 the
// kernels spill 1 KB per lane: e-/e+ 31% slower).  FP32, slab stack: 3
// without optional parts (40 000 x 10 GeV 101.6 ms, at 4 107.5 ms; at 2 157
// ms when at 3 it was 135); with them
// and in box geometries 2 (1501 mixed-species events in a field 17.2 ms, at 3,
// with spills, 17.8 ms; towers 999 x 1 GeV 8.8 ms, at 3 9.6 ms).
#ifndef EMS_WAVES_F64
#define EMS_WAVES_F64 2
#endif
#ifndef EMS_WAVES_F32
#define EMS_WAVES_F32 3
#endif
#ifndef EMS_WAVES_F32_FIELD
#define EMS_WAVES_F32_FIELD 2
#endif
#ifndef EMS_WAVES_BOX_F32
#define EMS_WAVES_BOX_F32 2
#endif
template <class R, int GEO, int F>
constexpr int visit_waves() {
  if (sizeof(R) == 8) return EMS_WAVES_F64;
  if (GEO == 1) return EMS_WAVES_BOX_F32;
  return (F & ~kFShort) != 0 ? EMS_WAVES_F32_FIELD : EMS_WAVES_F32;
}
// What the waves of a launch share: the current queues' sizes, the append
// plan, and where the launch's tallies go.
struct Launch {
  uint32_t cur;
  Sizes z;
  Plan plan;
  float limit;  // MeV: tracks above it make no secondaries in this iteration
  uint32_t* cnt;  // block's tallies (LDS)
};

template <bool PHOTONS, class R, int GEO, int F>
__device__ __forceinline__ void visit_loop(Ctl* ctl, const Staged<R>& st, const Launch& ln, const WaveShare& share,
                                           Ranges& rg) {
  constexpr int KIND = PHOTONS ? 0 : 1;
  constexpr bool kShort = (F & kFShort) != 0;
  // a step changes the direction itself (before any interaction)
  constexpr bool kTurns = !PHOTONS && (F & (kFField | kFMsc)) != 0;
  // secondaries: photons make e- and e+, e-/e+ make photons and e-
  constexpr int kSecA = PHOTONS ? kElectron : kGamma, kSecB = PHOTONS ? kPositron : kElectron;
  // secondaries of one step: of a photon an e- and an e+ at most, of an e-/e+
  // two photons (annihilation) or one e-, so only photons are ever asked for
  // two at a time (with two of each allowed, and a copy of the track for the
  // state before its step: 10^4 x 10 GeV 40.3 ms, now 39.7; 40 000 x 10 GeV
  // in the mixed form 101.6 and 98.9; towers 24.9 and 23.5)
  constexpr int kMaxA = PHOTONS ? 1 : 2;
  const uint32_t nmine = PHOTONS ? ln.z.n0 : ln.z.n1 + ln.z.n2 + ln.z.np;
  const uint32_t nxt = ln.cur ^ 1u;
  const KArgs& a0 = fresh_args();
  const int max_visit = (int)(PHOTONS ? a0.photon_steps_per_visit : a0.steps_per_visit);
  const uint32_t refill_below = PHOTONS ? a0.photon_refill_below : a0.refill_below;
  const Plan& plan = ln.plan;
  // short-electron routing: compiled into the kFShort variants only
  const bool shorts = kShort && a0.cap_s != 0;
  DevSink sink;
  uint32_t* cursor = &ctl->cursor[PHOTONS ? 0u : kLine];
  const bool track_live = (F & kFRecord) && (a0.flags & kFlagEventLive) != 0;

  bool has = false;   // lane holds a track (inside a visit or waiting to commit)
  bool fin = false;   // its visit ended; outputs wait for the batch commit
  bool held = false;  // the visit's last step is not yet applied to the tallies
  bool drained = false;
  // queue indices held by this wave (uniform)
  uint32_t chunk_lo = share.first, chunk_hi = share.first + share.lanes;
  if (share.first >= share.pool) chunk_hi = chunk_lo;  // a helper has no share of its own
  const bool my_lane = __lane_id() < share.lanes;
  // Once the queue is used up nothing refills the lanes, and a wave that
  // let all of its lanes finish before it sampled their interactions
  // would hold the launch back by one chain of steps after another: it
  // takes a batch as soon as at most 3/16 of its lanes still step (of 64:
  // 12; 0, 4, 8, 16, 20, 24 measured on 1500 x 10 GeV with scattering and
  // fluctuations: 27.7, 24.1, 23.5, 23.4, 23.4, 23.5 ms; 12: 23.3 ms).
  const uint32_t drain_below = share.lanes * 3 / 16;
  const uint32_t world_min = share.lanes / 4 < kWorldBatch ? share.lanes / 4 : kWorldBatch;
  int sp = PHOTONS ? 0 : 1;
  Trk<R> t;
  // the track before its last step, for a step whose secondaries do not
  // fit (id, event and key do not change; the volume is o.slab, the step
  // number t.n - 1)
  double x0 = 0.0, y0 = 0.0, z0 = 0.0, e0 = 0.0;
  R ux0 = R(0), uy0 = R(0), uz0 = R(0);
  VisitState<R> vs;
  StepOut<R> o;
  o.nsec = 0;
  o.pending = false;
  uint32_t visits_e = 0, visits_p = 0, steps_e = 0, steps_p = 0, carried_n = 0;
  uint32_t made_a = 0, made_b = 0, made_s = 0;
  uint32_t kept_a = 0, kept_b = 0;  // home records written (own species; e+)
  // Box geometries: a step that starts in the world volume needs the
  // nearest box along the track, a walk of the hierarchy that costs the
  // whole wave as much as many ordinary steps however few lanes take it.
  // Such lanes wait (world_wait), also across batches, until kWorldBatch
  // of them do (a quarter of a wave with fewer lanes) or no other lane
  // steps; then the wave computes their distances together (world_ready,
  // world_pre) and they take their steps with them.
  bool world_ready = false;
  GeoPre world_pre{0.0, Face{0, 0.0, 0, -1}};
  // (charged tracks in a field search their boundary along the helix
  // within their own step limit: they take no straight-line distance)
  const bool world_batch = PHOTONS || !((F & kFField) && a0.env.bz != 0.0);
  const uint32_t world = GEO == 1 ? a0.env.nav.n_boxes : 0u;
  for (;;) {
    bool world_wait = false;
    if constexpr (GEO == 1)
      world_wait = world_batch && has && !fin && !world_ready && (uint32_t)t.slab == world;
    uint32_t stepping = (uint32_t)__popcll(__ballot(has && !fin && !world_wait));
    if constexpr (GEO == 1) {
      const uint32_t nw = (uint32_t)__popcll(__ballot(world_wait));
      if (nw && (nw >= world_min || stepping == 0)) {
        if (world_wait) {
          if constexpr (sizeof(R) == 8) {
            world_pre = walk_world(&fresh_args(), t.x, t.y, t.z, t.ux, t.uy, t.uz);
          } else {
            const double p[3] = {t.x, t.y, t.z}, u[3] = {(double)t.ux, (double)t.uy, (double)t.uz};
            world_pre.s = world_distance(fresh_args().env.nav, p, u, world_pre.fc);
          }
          world_ready = true;
          world_wait = false;
        }
        stepping += nw;
      }
    }
    // batch point: few lanes still stepping
    if (stepping == 0 || (drained ? stepping <= drain_below && __ballot(fin) != 0 : stepping <= refill_below)) {
      const KArgs& a = fresh_args();
      // (0) e-/e+: while the queue still has tracks, interactions are
      // sampled only once at least interact_min lanes wait for one (each
      // sampler costs the wave one pass however few lanes use it); until
      // then those lanes are parked: they keep their tracks and take no
      // part in this batch.  A wave whose lanes are all parked samples
      // them, so every wave ends (interact_min <= 64).
      const uint32_t npend = PHOTONS ? 0u : (uint32_t)__popcll(__ballot(fin && o.pending));
      const bool parked = !PHOTONS && !drained && npend < a.interact_min && fin && o.pending;
      const bool done = fin && !parked;  // visits this batch finishes
      // (1) prefetch the records of the tracks that the lanes free after
      // this batch will take; the loads are in flight during (2)
      // a parent that survives its interaction keeps its lane and goes on
      // stepping in this launch while it has steps left
      const bool will_continue = done && o.pending && parent_survives(o.process) && vs.steps < max_visit;
      const bool want = (!has || (done && !will_continue)) && !drained && my_lane;
      bool got = false;
      int nsp = PHOTONS ? 0 : 1;
      uint32_t nw = kDeadRecord;
      Trk<R> nt;
      if (__ballot(want) != 0) {
        const uint32_t i = take_next(cursor, share.pool, want, chunk_lo, chunk_hi, nmine, a.waves);
        got = want && i < nmine;
        // (with fewer than 64 lanes a wave the first shares hold every track)
        drained = share.lanes < 64u || __ballot(want && i >= nmine) != 0;
        if (got) {
          uint32_t idx = i, home = PHOTONS ? ln.z.h0 : ln.z.h1;
          if (!PHOTONS && i >= ln.z.n1) {
            nsp = 2;
            idx = i - ln.z.n1;
            home = ln.z.h2;
          }
          const bool spilled = !PHOTONS && (F & kFShort) && i >= ln.z.n1 + ln.z.n2;  // an e- from the spill buffer
          if (spilled) nsp = 1;
          const uint32_t pos = spilled ? i - ln.z.n1 - ln.z.n2 : queue_pos(idx, home, a.cap);
          const Queue<R> src = spilled ? short_view<R>(a, 2u) : queue_view<R>(a, ln.cur, (uint32_t)nsp);
          nw = src.load(pos, nt);
        }
      }
      // (2) the interactions selected by the lanes' last steps, sampled
      // together (one pass through each sampler the wave needs)
      if constexpr (!kTurns) {
        ux0 = t.ux;
        uy0 = t.uy;
        uz0 = t.uz;
      }
      if (done && o.pending) interact<KIND, F>(env_of<R, GEO>(a, st), t, o);
      // (3) the prefetched records have arrived; waiting here, before any
      // store of this batch is issued, keeps later uses of their fields
      // from waiting on those stores (vector memory completes in order)
      __builtin_amdgcn_s_waitcnt(kWaitVmem);
      bool take = got && nw != kDeadRecord;  // dead: refused secondary or unused chunk end
      nt.slab = (int32_t)(nw & ((1u << a.vol_bits) - 1u));
      nt.n = nw >> a.vol_bits;
      // a record that would index outside the tallies or the slab stack
      // is reported, never used
      if (take && (nt.slab >= (int32_t)a.env.n_slabs || nt.ev >= a.max_events)) {
        atomicOr(&ctl->error, kErrCorrupt);
        take = false;
      }
      // (4) commit the finished visits: reserve first, then write
      if (__ballot(done) != 0) {
        // secondaries into the top regions (a step commits only if all of
        // its secondaries fit), then survivors or carried tracks
        // e- secondaries below short_E go to the next short buffer
        const bool made = done && o.nsec > 0;
        const bool hold = made && (float)e0 + (sp == 2 ? (float)(2.0 * kMe) : 0.0f) > ln.limit;  // scarce room
        const bool s0 = shorts && made && !hold && o.sec[0].sp == kElectron && o.sec[0].E < a.short_E;
        const bool s1 = shorts && made && !hold && o.nsec > 1 && o.sec[1].sp == kElectron && o.sec[1].E < a.short_E;
        const bool in0 = made && !hold && !s0, in1 = made && !hold && o.nsec > 1 && !s1;  // to the queues
        const uint32_t da = (in0 && o.sec[0].sp == kSecA ? 1u : 0u) + (in1 && o.sec[1].sp == kSecA ? 1u : 0u);
        const uint32_t db = (in0 && o.sec[0].sp == kSecB ? 1u : 0u) + (in1 && o.sec[1].sp == kSecB ? 1u : 0u);
        const uint32_t ds = (s0 ? 1u : 0u) + (s1 ? 1u : 0u);
        // a home slot for every survivor that leaves the lane
        const bool leave = done && t.slab >= 0 && !will_continue;
        Take ta = ask<kMaxA>(rg, kNextSec + kSecA, da), tb = ask(rg, kNextSec + kSecB, db);
        Take th = ask(rg, kNextHome + (PHOTONS ? 0 : 1), leave && sp != 2 ? 1u : 0u);
        Take tp{0, 0, 0, 0, 0}, ts{0, 0, 0, 0, 0};
        if constexpr (!PHOTONS) tp = ask(rg, kNextHome + 2, leave && sp == 2 ? 1u : 0u);
        if (shorts) ts = ask(rg, kNextShort, ds);
        if constexpr (PHOTONS) {
          if constexpr (kShort) {
            const Ask asks[4] = {{kNextSec + kSecA, plan.chunk[kSecA], &ta}, {kNextSec + kSecB, plan.chunk[kSecB], &tb},
                                 {kNextHome, plan.chunk[0], &th}, {kNextShort, plan.chunk_s, &ts}};
            serve(ctl, rg, asks);
          } else {
            const Ask asks[3] = {{kNextSec + kSecA, plan.chunk[kSecA], &ta}, {kNextSec + kSecB, plan.chunk[kSecB], &tb},
                                 {kNextHome, plan.chunk[0], &th}};
            serve(ctl, rg, asks);
          }
        } else if constexpr (kShort) {
          const Ask asks[5] = {{kNextSec + kSecA, plan.chunk[kSecA], &ta}, {kNextSec + kSecB, plan.chunk[kSecB], &tb},
                               {kNextHome + 1, plan.chunk[1], &th}, {kNextHome + 2, plan.chunk[2], &tp},
                               {kNextShort, plan.chunk_s, &ts}};
          serve(ctl, rg, asks);
        } else {
          const Ask asks[4] = {{kNextSec + kSecA, plan.chunk[kSecA], &ta}, {kNextSec + kSecB, plan.chunk[kSecB], &tb},
                               {kNextHome + 1, plan.chunk[1], &th}, {kNextHome + 2, plan.chunk[2], &tp}};
          serve(ctl, rg, asks);
        }
        const uint32_t lim_a = plan.lim[kSecA], lim_b = plan.lim[kSecB];
        bool fits = !(da && ta.slot(0) >= lim_a) && !(db && tb.slot(0) >= lim_b);
        if (kMaxA > 1 && da > 1 && ta.slot(1) >= lim_a) fits = false;
        if (shorts && ds && ts.slot(0) >= plan.lim_s) fits = false;
        const bool commit = made && fits && !hold;
        const bool carry = made && !commit;  // back to the state before the last step
        const bool cont = done && t.slab >= 0 && !carry && will_continue;  // stays in the lane
        const bool keep = leave || carry;                                  // written to the next queue
        uint32_t hs = sp == 2 ? tp.slot(0) : th.slot(0);
        // carried tracks that were not to leave still need a home slot
        const bool late = carry && !leave;
        if (__ballot(late) != 0) {
          Take lh = ask(rg, kNextHome + (PHOTONS ? 0 : 1), late && sp != 2 ? 1u : 0u);
          Take lp{0, 0, 0, 0, 0};
          if constexpr (PHOTONS) {
            const Ask asks[1] = {{kNextHome, plan.chunk[0], &lh}};
            serve(ctl, rg, asks);
          } else {
            lp = ask(rg, kNextHome + 2, late && sp == 2 ? 1u : 0u);
            const Ask asks[2] = {{kNextHome + 1, plan.chunk[1], &lh}, {kNextHome + 2, plan.chunk[2], &lp}};
            serve(ctl, rg, asks);
          }
          if (late) hs = sp == 2 ? lp.slot(0) : lh.slot(0);
        }
        if (commit || (done && held && o.nsec == 0)) {
          sink.apply<F>(a, sp, t, o, e0);
          if (sp == 2) ++steps_p;
          else ++steps_e;
          made_a += da;
          made_b += db;
          made_s += ds;
        }
        if (carry) ++carried_n;
        if (done && track_live) {
          // net change of the event's live tracks: the visited track ends
          // or stays, committed secondaries join
          const int delta = (keep || cont ? 1 : 0) + (commit ? (int)(da + db + ds) : 0) - 1;
          if (delta != 0) atomicAdd(&a.live_ev[t.ev], delta);
        }
        // secondary number k to slot sl of its queue's top region (or, to
        // the short buffer, from the bottom); a refused one marks its slot
        // dead for the next iteration
        auto put = [&](const Queue<R>& dq, const Sec<R>& sec, uint32_t ps) {
          if (commit) {
            Trk<R> c;
            c.x = t.x;
            c.y = t.y;
            c.z = t.z;
            c.ux = sec.ux;
            c.uy = sec.uy;
            c.uz = sec.uz;
            c.E = sec.E;
            c.id = sec.id;
            c.ev = t.ev;
            c.key = t.key;
            c.n = 0;
            c.slab = o.slab;
            store_track(dq, ps, c, a.vol_bits);
          } else {
            dq.kill(ps);
          }
        };
        auto put_queue = [&](int q, int most, uint32_t d, const Take& tk, uint32_t lim) {
          if (!d) return;
          const Queue<R> dq = queue_view<R>(a, nxt, (uint32_t)q);
          const bool first = in0 && o.sec[0].sp == q;
          const uint32_t sl = tk.slot(0);
          if (sl < lim) put(dq, first ? o.sec[0] : o.sec[1], (uint32_t)(a.cap - 1 - sl));
          if (most > 1 && d > 1) {
            const uint32_t s2 = tk.slot(1);
            if (s2 < lim) put(dq, o.sec[1], (uint32_t)(a.cap - 1 - s2));
          }
        };
        put_queue(kSecA, kMaxA, da, ta, lim_a);
        put_queue(kSecB, 1, db, tb, lim_b);
        if (kShort && ds) {
          const Queue<R> sq = short_view<R>(a, nxt);
          const uint32_t sl = ts.slot(0);
          if (sl < plan.lim_s) put(sq, s0 ? o.sec[0] : o.sec[1], sl);
        }
        if (keep) {
          const Queue<R> dq = queue_view<R>(a, nxt, (uint32_t)sp);
          if (hs >= a.cap) {
            atomicOr(&ctl->error, kErrOverflow);
          } else {
            // (a track written here leaves the lane)
            if (carry) {
              t.x = x0;
              t.y = y0;
              t.z = z0;
              t.E = e0;
              t.ux = ux0;
              t.uy = uy0;
              t.uz = uz0;
              t.n -= 1;
              t.slab = o.slab;
            }
            store_track(dq, hs, t, a.vol_bits);
            if (sp == 2) ++kept_b;
            else ++kept_a;
          }
        }
        if (done) {
          has = cont;
          fin = false;
          held = false;
          o.nsec = 0;
          o.pending = false;
        }
        // a continuing photon has a new energy and direction
        if (PHOTONS && cont) photon_begin(env_of<R, GEO>(a, st), t, vs.pc);
      }
      // (5) the freed lanes take their prefetched tracks
      if (take) {
        t.x = nt.x;
        t.y = nt.y;
        t.z = nt.z;
        t.ux = nt.ux;
        t.uy = nt.uy;
        t.uz = nt.uz;
        t.E = nt.E;
        t.id = nt.id;
        t.ev = nt.ev;
        t.key = nt.key;
        t.n = nt.n;
        t.slab = nt.slab;
        sp = nsp;
        has = true;
        visit_begin<KIND>(env_of<R, GEO>(a, st), sp, t, vs);
        world_ready = false;
        if (sp == 2) ++visits_p;
        else ++visits_e;
      }
      if (__ballot(has) == 0) {
        if (drained) break;
        continue;
      }
      // tracks just taken that start in the world wait for a world pass
      if constexpr (GEO == 1)
        world_wait = world_batch && has && !fin && !world_ready && (uint32_t)t.slab == world;
    }

    // one step of every lane inside a visit
    if (has && !fin && !world_wait) {
      const KArgs& a = fresh_args();
      x0 = t.x;
      y0 = t.y;
      z0 = t.z;
      e0 = t.E;
      if constexpr (kTurns) {
        ux0 = t.ux;
        uy0 = t.uy;
        uz0 = t.uz;
      }
      fin = visit_step<KIND, R, GEO, F | kFWorldPre>(env_of<R, GEO>(a, st), sp, vs, t, o, max_visit,
                                                     world_ready ? &world_pre : nullptr);
      world_ready = false;
      held = o.pending;
      if (!held) {
        sink.apply<F>(a, sp, t, o, e0);
        if (sp == 2) ++steps_p;
        else ++steps_e;
      }
    }
  }

  sink.flush(fresh_args());
  constexpr int kOwn = PHOTONS ? 0 : 1;
  Tallies sums;
  sums.count(kAddSteps + kOwn, steps_e);
  sums.count(kAddVisits + kOwn, visits_e);
  sums.count(kAddKept + kOwn, kept_a);
  if constexpr (!PHOTONS) {
    sums.count(kAddSteps + 2, steps_p);
    sums.count(kAddVisits + 2, visits_p);
    sums.count(kAddKept + 2, kept_b);
  }
  sums.count(kAddMade + kSecA, made_a + (kSecA == kElectron ? made_s : 0u));
  sums.count(kAddMade + kSecB, made_b + (kSecB == kElectron ? made_s : 0u));
  sums.count(kAddMadeBy + kOwn, made_a + made_b + made_s);
  sums.count(kAddCarried, carried_n);
  if constexpr (kShort) sums.count(kAddMadeShort, made_s);
  sums.add_to(ctl, ln.cnt);
}

// The last block of an iteration to end folds the tallies into the totals
// and leaves the extents of the next queues to the next iteration.  Wave 0 of
// that block does it, a counter to a lane: every counter is fetched and
// cleared in one exchange each (they live at the memory side, some
// microseconds a round trip; one after another they took 9 us of every
// iteration).
template <bool SHORT>
__device__ inline void close_iteration(const KArgs& a, Ctl* ctl, const Launch& ln) {
  const uint32_t lane = __lane_id();
  uint32_t app = 0, error = 0;
  unsigned long long add = 0;
  // (the spill counter is read only)
  if (lane < kNextCounters) app = atomicAnd(&ctl->next[lane * kLine], lane == kNextSpill ? ~0u : 0u);
  if (lane < kAdds) add = atomicExch(&ctl->add[lane], 0ull);
  if (lane == 0) error = atomicOr(&ctl->error, 0u);
  auto next_of = [&](int c) { return (uint32_t)__builtin_amdgcn_readlane((int)app, c); };
  auto add_of = [&](int k) {
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)add, k);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(add >> 32), k);
    return (unsigned long long)lo | ((unsigned long long)hi << 32);
  };
  Appended n;
  n.shorts_real = SHORT ? (uint32_t)add_of(kAddMadeShort) : 0u;
  uint32_t live = n.shorts_real;
#pragma unroll
  for (int q = 0; q < 3; ++q) {
    n.real[q] = (uint32_t)(add_of(kAddMade + q) + add_of(kAddKept + q)) - (q == 1 ? n.shorts_real : 0u);
    live += n.real[q];
  }
  unsigned long long tot[kAdds];
#pragma unroll
  for (int q = 0; q < 3; ++q) {
    n.home[q] = next_of(kNextHome + q);
    n.sec[q] = next_of(kNextSec + q);
    n.lim[q] = ln.plan.lim[q];
  }
#pragma unroll
  for (int k = 0; k < kAdds; ++k) tot[k] = add_of(k);
  n.shorts = SHORT ? next_of(kNextShort) : 0u;
  n.lim_s = ln.plan.lim_s;
  n.spilled = SHORT ? next_of(kNextSpill) : 0u;
  const unsigned long long commits = tot[kAddSteps] + tot[kAddSteps + 1] + tot[kAddSteps + 2];
  const unsigned long long carried = tot[kAddCarried];
  if (lane != 0) return;
  const Extents& e = ctl->ext[ln.cur];
  const uint32_t r0 = e.n_real[0], r1 = e.n_real[1] + (SHORT ? e.n_short_real : 0u), r2 = e.n_real[2];
  if (a.flags & kFlagProfile) {
    if (ctl->iteration < a.profile_cap) {
      a.profile[(size_t)ctl->iteration * 3 + 0] = r0;
      a.profile[(size_t)ctl->iteration * 3 + 1] = r1;
      a.profile[(size_t)ctl->iteration * 3 + 2] = r2;
    }
  }
  if (r0 + r1 + r2 > 0) ctl->iteration += 1;
  if (carried > 0 && commits == 0 && ln.z.level >= kNoLevel) {  // nothing can move: queues too small
    atomicOr(&ctl->error, kErrStall);
    error |= kErrStall;
  }
  // how scarce room is (next_level)
  uint64_t least = a.cap;
  bool little = true;
#pragma unroll
  for (int q = 0; q < 3; ++q) {
    const uint32_t lim = n.lim[q] + (SHORT && q == 1 ? n.lim_s : 0u);
    const uint64_t used = (uint64_t)n.real[q] + (SHORT && q == 1 ? n.shorts_real : 0u);
    const uint64_t room = used < a.cap ? a.cap - used : 0;
    least = room < least ? room : least;
    if (tight(lim, a.cap)) little = little && tot[kAddMade + q] * 4 <= lim;
  }
  const uint32_t level = next_level(ln.z.level, carried, commits, least, a.cap, little);
  // the other record (the next short buffer becomes the current one with it)
  ctl->ext[ln.cur ^ 1u] = next_extents(n, live, level, error != 0 || e.stop);
#pragma unroll
  for (int q = 0; q < 3; ++q) {
    const uint32_t all = n.real[q] + (q == 1 ? n.shorts_real : 0u);
    ctl->peak[q] = all > ctl->peak[q] ? all : ctl->peak[q];
    ctl->steps[q] += tot[kAddSteps + q];
    ctl->visits[q] += tot[kAddVisits + q];
    ctl->created[q] += tot[kAddMade + q];
  }
  ctl->made_by[0] += tot[kAddMadeBy];
  ctl->made_by[1] += tot[kAddMadeBy + 1];
  ctl->deferred += carried;
  if constexpr (SHORT) ctl->steps_s += tot[kAddStepsShort];
  ctl->live = live;
  ctl->cursor[0] = 0;
  ctl->cursor[kLine] = 0;
  ctl->blocks_done = 0;
}

// One iteration: every track of the current queues is visited once.  The
// two species' loops do not depend on each other within an iteration (both
// read the current queues and append to the next), so one launch runs both:
// the waves are dealt to the species in proportion to their tracks, and a
// wave whose species is used up goes on with the other one, so the tail of
// one overlaps the other.  `which` names the species of the launch: both, or
// one after the other in a launch each (per-kernel timing, or tables that
// would cost resident blocks if both were staged); the launch of the e-/e+
// closes the iteration.
// Measured against two launches an iteration (with the counters' round trips
// one after another): 32 x 1 GeV 3.4 -> 2.2 ms, 500 x 2 GeV 8.1 -> 5.5 ms,
// 10^4 x 10 GeV 59.2 -> 55.1 ms, 1501 mixed-species events in a field, mixed
// form 28.6 -> 21.7 ms.  All waves on photons first, then on e-/e+, instead
// of dealt to both from the start: 10^4 x 10 GeV 56.9 ms, 2500 mixed-species
// events in a field 39.9 instead of 37.8 ms.
template <class R, int GEO, int F>
__global__ __launch_bounds__(kBlock, (visit_waves<R, GEO, F>())) void k_visit(KArgs a, uint32_t which) {
  extern __shared__ double lds_words[];
  __shared__ uint32_t cnt[kAdds];
  Ctl* ctl = a.ctl;
  constexpr bool kShort = (F & kFShort) != 0;
  Launch ln;
  ln.cnt = cnt;
  ln.cur = a.cur;
  ln.z = sizes_of<kShort>(ctl, ln.cur, a.cap_p);
  // secondary slots per species that leave room for all survivors
  ln.plan = append_plan<kShort>(a, ln.z.n0, ln.z.n1, ln.z.n2, ln.z.ns, ln.z.level);
  bool any_tight = false;
#pragma unroll
  for (int q = 0; q < 3; ++q) any_tight |= tight(ln.plan.lim[q] + (kShort && q == 1 ? ln.plan.lim_s : 0u), a.cap);
  ln.limit = any_tight ? energy_limit(ln.z.level) : __builtin_huge_valf();
  const bool stop = ctl->ext[ln.cur].stop != 0;
  const uint32_t ng = which & kPhotons && !stop ? ln.z.n0 : 0u;
  const uint32_t nl = which & kLeptons && !stop ? ln.z.n1 + ln.z.n2 + ln.z.np : 0u;
  // consecutive waves go to different blocks (and so CUs)
  const uint32_t w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) * gridDim.x + blockIdx.x;
  const Deal d = deal_launch(ng, nl, gridDim.x, w);
  const WaveShare &sg = d.sg, &sl = d.sl;
  const uint32_t workers = d.workers;
  if (blockIdx.x >= workers && (workers || blockIdx.x)) return;
  if (workers) {
    clear_counts(cnt);
    const Staged<R> st = stage<R, GEO>(a, reinterpret_cast<char*>(lds_words), which);
    Ranges rg{};
    const bool own_g = w < d.wg;
#pragma unroll 1
    for (int turn = 0; turn < 2; ++turn) {
      const bool photons = own_g == (turn == 0);
      // (a species without tracks or not in this launch; a wave helps only
      // where the shares left tracks over)
      if (photons ? ng == 0u || (turn == 1 && sg.lanes < 64u) : nl == 0u || (turn == 1 && sl.lanes < 64u)) continue;
      if (photons) {
        const WaveShare s = turn == 0 ? sg : WaveShare{64u, sg.pool, sg.pool};
        visit_loop<true, R, GEO, F>(ctl, st, ln, s, rg);
      } else {
        const WaveShare s = turn == 0 ? sl : WaveShare{64u, sl.pool, sl.pool};
        visit_loop<false, R, GEO, F>(ctl, st, ln, s, rg);
      }
    }
    // unused ends of the wave's append ranges hold no track
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      const Queue<R> dq = queue_view<R>(a, ln.cur ^ 1u, (uint32_t)q);
      const uint32_t lim = ln.plan.lim[q];
      const uint32_t send = rg.hi[kNextSec + q] < lim ? rg.hi[kNextSec + q] : lim;
      for (uint32_t x = rg.lo[kNextSec + q] + __lane_id(); x < send; x += 64) dq.kill(a.cap - 1 - x);
      for (uint32_t x = rg.lo[kNextHome + q] + __lane_id(); x < rg.hi[kNextHome + q]; x += 64) {
        if (x < a.cap) dq.kill(x);
      }
    }
    if (kShort && a.cap_s) {
      const Queue<R> sq = short_view<R>(a, ln.cur ^ 1u);
      const uint32_t send = rg.hi[kNextShort] < ln.plan.lim_s ? rg.hi[kNextShort] : ln.plan.lim_s;
      for (uint32_t x = rg.lo[kNextShort] + __lane_id(); x < send; x += 64) sq.kill(x);
    }
    publish_counts(ctl, cnt);
  }

  if (!(which & kLeptons)) return;
  // The block's increments are performed (every atomic at the memory side)
  // before its ticket is counted, so the block that draws the last ticket
  // sees them all; the records themselves are read by the next launch.
  if (threadIdx.x >= 64) return;
  __builtin_amdgcn_s_waitcnt(kWaitVmem);
  uint32_t ticket = 0;
  if (workers && threadIdx.x == 0) ticket = atomicAdd(&ctl->blocks_done, 1u);
  ticket = (uint32_t)__builtin_amdgcn_readfirstlane((int)ticket);
  if (!workers || ticket == workers - 1) close_iteration<kShort>(a, ctl, ln);
}

// Short electrons.  Most e- secondaries of a shower are slow (Compton and
// photo-electrons, delta rays) and end in their first step, ranged out.
// In the visit launch each of them costs a lane a record load, one step and
// a commit in a wave whose other lanes follow long tracks; here a launch of
// its own, at the start of the iteration, gives every lane one such track:
// one step, its tallies, and the survivor (if any) appended to the next e-
// queue as any e-/e+ survivor.  A track whose first step selects a discrete
// interaction is handed unchanged to this iteration's visit launch (spill
// buffer), which takes the same step again and samples the interaction
// there: every step still draws from its own (id, step) stream, so results
// and the iteration of every step are those of the visit launch.
// (without optional parts the step and a prefetched record fit 3 resident
// waves per SIMD in FP64, 5 in FP32; with them 3 and 4; in box geometries
// 2 and 3)
#ifndef EMS_WAVES_F64_SHORT
#define EMS_WAVES_F64_SHORT 3
#endif
#ifndef EMS_WAVES_F32_SHORT
#define EMS_WAVES_F32_SHORT 5
#endif
template <class R, int GEO, int F>
constexpr int short_waves() {
  if (GEO == 1) return sizeof(R) == 8 ? 2 : 3;  // box navigation needs more registers
  return sizeof(R) == 8 ? (F == 0 ? EMS_WAVES_F64_SHORT : 3) : (F == 0 ? EMS_WAVES_F32_SHORT : 4);
}
template <class R, int GEO, int F>
__global__ __launch_bounds__(kBlock, (short_waves<R, GEO, F>())) void k_short(KArgs a) {
  extern __shared__ double lds_words[];
  char* lds = reinterpret_cast<char*>(lds_words);
  __shared__ uint32_t cnt[kAdds];
  Ctl* ctl = a.ctl;
  const uint32_t cur = a.cur;
  const Sizes z = sizes_of<true>(ctl, cur, a.cap_p);
  const uint32_t ns = z.ns, spilled = ctl->ext[cur].spilled;
  if (blockIdx.x >= (ns + kBlock - 1) / kBlock || ctl->ext[cur].stop) return;
  clear_counts(cnt);
  const Staged<R> st = stage<R, GEO>(a, lds, kLeptons);
  const StepEnv<R> env = env_of<R, GEO>(a, st);
  const Plan plan = append_plan<true>(a, z.n0, z.n1, z.n2, ns, z.level);
  DevSink sink;
  const bool track_live = (F & kFRecord) && (a.flags & kFlagEventLive) != 0;
  const Queue<R> src = short_view<R>(a, cur);
  const Queue<R> spill = short_view<R>(a, 2u);
  const Queue<R> dst = queue_view<R>(a, cur ^ 1u, (uint32_t)kElectron);
  // wave-private append ranges: next e- home, spill buffer
  Ranges rg{};
  // spill appends: all waves' unused chunk ends fit in the spill buffer's
  // room beyond cap_s (at most ns <= cap_s tracks spill)
  uint32_t chunk_p = plan.chunk[1] < 64u ? plan.chunk[1] : 64u;
  while (chunk_p > 1 && (uint64_t)a.waves_s * chunk_p > a.cap_p - a.cap_s) chunk_p >>= 1;
  uint32_t steps = 0, loads = 0, kept = 0;
  // the record of the lane's next track is loaded while the current one
  // steps (the step reads only LDS, so nothing waits for those loads early)
  auto load = [&](uint32_t i, Trk<R>& t, uint32_t& w) {
    w = kDeadRecord;
    if (i < ns) {
      w = src.load(i, t);
    }
  };
  const uint32_t stride = gridDim.x * kBlock;
  Trk<R> t;
  uint32_t w;
  load(blockIdx.x * kBlock + threadIdx.x, t, w);
  for (uint32_t base = blockIdx.x * kBlock; base < ns; base += stride) {
    Trk<R> tn;
    uint32_t wn;
    load(base + stride + threadIdx.x, tn, wn);
    bool has = w != kDeadRecord;
    t.slab = (int32_t)(w & ((1u << a.vol_bits) - 1u));
    t.n = w >> a.vol_bits;
    if (has && (t.slab >= (int32_t)a.env.n_slabs || t.ev >= a.max_events)) {
      atomicOr(&ctl->error, kErrCorrupt);
      has = false;
    }
    const Trk<R> first = t;
    StepOut<R> o;
    o.nsec = 0;
    bool to_spill = false, alive = false;
    if (has) {
      ++loads;
      clear_out(t, o);
      lepton_step<R, GEO, F>(env, false, t, o);
      if (o.pending) {
        to_spill = true;
      } else {
        watchdog(env, t, o);
        sink.apply<F>(a, kElectron, t, o, first.E);
        ++steps;
        alive = t.slab >= 0;
        if (track_live && !alive) atomicAdd(&a.live_ev[t.ev], -1);
      }
    }
    Take th = ask(rg, kNextHome + 1, alive ? 1u : 0u), tp = ask(rg, kNextSpill, to_spill ? 1u : 0u);
    const Ask asks[2] = {{kNextHome + 1, plan.chunk[1], &th}, {kNextSpill, chunk_p, &tp}};
    serve(ctl, rg, asks);
    if (alive) {
      const uint32_t hs = th.slot(0);
      if (hs >= a.cap) {
        atomicOr(&ctl->error, kErrOverflow);
      } else {
        store_track(dst, hs, t, a.vol_bits);
        ++kept;
      }
    }
    if (to_spill) {
      const uint32_t ps = tp.slot(0) - spilled;
      if (ps >= a.cap_p) atomicOr(&ctl->error, kErrOverflow);
      else store_track(spill, ps, first, a.vol_bits);
    }
    t = tn;
    w = wn;
  }
  sink.flush(a);
  for (uint32_t x = rg.lo[kNextHome + 1] + __lane_id(); x < rg.hi[kNextHome + 1]; x += 64) {
    if (x < a.cap) dst.kill(x);
  }
  // (counted from the range's start: the counter is not cleared, and may wrap)
  for (uint32_t k = __lane_id(); k < rg.hi[kNextSpill] - rg.lo[kNextSpill]; k += 64) {
    const uint32_t x = rg.lo[kNextSpill] + k - spilled;
    if (x < a.cap_p) spill.kill(x);
  }
  Tallies sums;
  sums.count(kAddSteps + 1, steps);
  sums.count(kAddStepsShort, steps);
  sums.count(kAddVisits + 1, loads);
  sums.count(kAddKept + 1, kept);
  sums.add_to(ctl, cnt);
  publish_counts(ctl, cnt);
}

#ifndef EMS_SLAB_F32_TU
// Zero `words` 8-byte words at p and then `ntail` single bytes at tail, with
// plain vector stores (grid-stride).  The library clears its device memory
// with this kernel instead of memset nodes, which a caller capturing the
// stream into a graph could not rely on.
__global__ __launch_bounds__(kBlock) void k_fill_zero(unsigned long long* p, uint64_t words, unsigned char* tail,
                                                      uint32_t ntail) {
  const uint64_t stride = (uint64_t)gridDim.x * kBlock;
  for (uint64_t i = (uint64_t)blockIdx.x * kBlock + threadIdx.x; i < words; i += stride) p[i] = 0ull;
  if (blockIdx.x == 0 && threadIdx.x < ntail) tail[threadIdx.x] = 0;
}

// Atomic-throughput probe: FP64 adds of 1.0, the instruction of the deposit
// tallies, to cells drawn by a fixed hash of the op index (grid-stride).
__global__ __launch_bounds__(kBlock) void k_atomic_probe(double* cells, uint64_t n_cells, uint64_t n_ops) {
  const uint64_t stride = (uint64_t)gridDim.x * kBlock;
  for (uint64_t i = (uint64_t)blockIdx.x * kBlock + threadIdx.x; i < n_ops; i += stride) {
    uint64_t h = i * 0x9E3779B97F4A7C15ull;
    h ^= h >> 29;
    h *= 0xBF58476D1CE4E5B9ull;
    h ^= h >> 32;
    atomicAdd(&cells[h % n_cells], 1.0);
  }
}

// Injection: prepared tracks appended to the home regions of the current
// queues.
template <class R>
__global__ __launch_bounds__(kBlock) void k_inject(KArgs a, const InjRec* rec, uint32_t n) {
  Ctl* ctl = a.ctl;
  const uint32_t cur = a.cur;
  Extents& e = ctl->ext[cur];
  for (uint32_t base = blockIdx.x * kBlock; base < n; base += gridDim.x * kBlock) {
    const uint32_t i = base + threadIdx.x;
    const bool active = i < n;
    InjRec r{};
    if (active) r = rec[i];
    for (int qs = 0; qs < 3; ++qs) {
      const uint32_t cnt = (active && (int)r.sp == qs) ? 1u : 0u;
      const uint32_t slot = wave_reserve(&e.n_home[qs], cnt);
      const bool fits = cnt && slot + e.n_sec[qs] < a.cap;
      wave_count(&e.n_real[qs], fits ? 1u : 0u);
      if (!cnt) continue;
      if (!fits) {
        atomicOr(&ctl->error, kErrOverflow);
        continue;
      }
      Trk<R> t;
      t.x = r.x;
      t.y = r.y;
      t.z = r.z;
      t.ux = (R)r.ux;
      t.uy = (R)r.uy;
      t.uz = (R)r.uz;
      t.E = r.E;
      t.id = r.id;
      t.ev = r.ev;
      t.key = r.key;
      t.n = 0;
      t.slab = r.slab;
      store_track(queue_view<R>(a, cur, (uint32_t)qs), slot, t, a.vol_bits);
      if (a.flags & kFlagEventLive) atomicAdd(&a.live_ev[r.ev], 1);
    }
  }
}

// Zero the deposits, ledger and live counter of the listed rows (one block
// per row, grid-stride over the list).
__global__ __launch_bounds__(kBlock) void k_reset_rows(KArgs a, const uint32_t* rows, uint32_t n) {
  for (uint32_t i = blockIdx.x; i < n; i += gridDim.x) {
    const uint32_t r = rows[i];
    if (r >= a.max_events) continue;
    double* e = a.edep + (size_t)r * a.env.n_slabs;
    for (uint32_t k = threadIdx.x; k < a.env.n_slabs; k += kBlock) e[k] = 0.0;
    unsigned long long* l = reinterpret_cast<unsigned long long*>(a.ledger + r);
    for (uint32_t k = threadIdx.x; k < sizeof(LedgerDev) / 8; k += kBlock) l[k] = 0ull;
    if (threadIdx.x == 0) a.live_ev[r] = 0;
  }
}

// Copy the deposits and ledger of the listed rows to a compact staging area:
// entry i holds n_slabs doubles, then the row's ledger.
__global__ __launch_bounds__(kBlock) void k_gather_rows(KArgs a, const uint32_t* rows, uint32_t n, char* out) {
  const size_t stride = (size_t)a.env.n_slabs * 8 + sizeof(LedgerDev);
  for (uint32_t i = blockIdx.x; i < n; i += gridDim.x) {
    const uint32_t r = rows[i];
    if (r >= a.max_events) continue;
    double* o = reinterpret_cast<double*>(out + i * stride);
    const double* e = a.edep + (size_t)r * a.env.n_slabs;
    for (uint32_t k = threadIdx.x; k < a.env.n_slabs; k += kBlock) o[k] = e[k];
    unsigned long long* lo = reinterpret_cast<unsigned long long*>(o + a.env.n_slabs);
    const unsigned long long* li = reinterpret_cast<const unsigned long long*>(a.ledger + r);
    for (uint32_t k = threadIdx.x; k < sizeof(LedgerDev) / 8; k += kBlock) lo[k] = li[k];
  }
}

// live count after injection (one thread); after an injection that did not
// fit nothing is stepped
__global__ void k_census(KArgs a) {
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    Ctl* c = a.ctl;
    Extents& e = c->ext[a.cur];
    uint32_t live = e.n_short_real;
    for (int q = 0; q < 3; ++q) {
      const uint32_t n = e.n_real[q] + (q == 1 ? e.n_short_real : 0u);
      c->peak[q] = n > c->peak[q] ? n : c->peak[q];
      live += e.n_real[q];
    }
    c->live = live;
    if (c->error) e.stop = 1;
  }
}

#endif  // EMS_SLAB_F32_TU

// Kernel variants.  A part that is compiled in costs registers and spills also
// where it is off, so a context launches the smallest variant that covers its
// configuration (KArgs::feat).  Both kinds of geometry: no parts, or all.  A
// slab stack also: the field; the field and the records (the offload server);
// scattering and fluctuations; the field and compounds.  Variants with the
// short-electron routing exist for no parts, the field and the records, and
// all (each would be built twice otherwise).
// Against the variant with all parts: 1500 x 10 GeV with scattering and
// fluctuations 14.78 -> 13.44 ms, PbWO4 1501 mixed-species events in a field,
// mixed form 17.09 -> 16.64, 37 x 1 GeV 2.38 -> 2.28; the field alone against
// the field with the records: 2500 mixed-species events 27.83 -> 26.42 ms, 48
// tracks 0.364 -> 0.343.
template <class R, int GEO>
const void* visit_fn(uint32_t feat) {
  if (feat == 0) return reinterpret_cast<const void*>(&k_visit<R, GEO, 0>);
  if (feat == kFShort) return reinterpret_cast<const void*>(&k_visit<R, GEO, kFShort>);
  if constexpr (GEO == 0) {
    if (feat == (kFField | kFRecord)) return reinterpret_cast<const void*>(&k_visit<R, GEO, kFField | kFRecord>);
    if (feat == (kFField | kFRecord | kFShort))
      return reinterpret_cast<const void*>(&k_visit<R, GEO, kFField | kFRecord | kFShort>);
    if (feat == kFField) return reinterpret_cast<const void*>(&k_visit<R, GEO, kFField>);
    if (feat == kFAlong) return reinterpret_cast<const void*>(&k_visit<R, GEO, kFAlong>);
    if (feat == kFFieldCompound) return reinterpret_cast<const void*>(&k_visit<R, GEO, kFFieldCompound>);
  }
  if (feat == (kFAll & ~kFShort)) return reinterpret_cast<const void*>(&k_visit<R, GEO, kFAll & ~kFShort>);
  return reinterpret_cast<const void*>(&k_visit<R, GEO, kFAll>);
}
// the short launch takes the visit launch's optional parts (its own work is
// the short path, so the routing bit does not apply to it)
template <class R, int GEO>
const void* short_fn(uint32_t feat) {
  feat &= ~(uint32_t)kFShort;
  if (feat == 0) return reinterpret_cast<const void*>(&k_short<R, GEO, 0>);
  if constexpr (GEO == 0) {
    if (feat == (kFField | kFRecord)) return reinterpret_cast<const void*>(&k_short<R, GEO, kFField | kFRecord>);
  }
  return reinterpret_cast<const void*>(&k_short<R, GEO, kFAll>);
}
// the visit kernel, or the short launch's
template <class R, int GEO>
const void* kernel_of(const KArgs& a, bool shorts) {
  return shorts ? short_fn<R, GEO>(a.feat) : visit_fn<R, GEO>(a.feat);
}
#ifdef EMS_SLAB_F32_TU
const void* kernel_of_slab_f32(const KArgs& a, bool shorts) { return kernel_of<float, 0>(a, shorts); }
#else
// The mixed-form kernels of the slab stack come from a translation unit of
// their own (ems_kernels_slab_f32.hip), built with another instruction
// scheduler (see build.py).
const void* kernel_of_slab_f32(const KArgs& a, bool shorts);
const void* kernel_for(const KArgs& a, bool shorts) {
  if (a.geo == 1) return a.precision ? kernel_of<float, 1>(a, shorts) : kernel_of<double, 1>(a, shorts);
  return a.precision ? kernel_of_slab_f32(a, shorts) : kernel_of<double, 0>(a, shorts);
}
// LDS of a visit launch of the species `which`
uint32_t visit_lds(const KArgs& a, uint32_t which) {
  return which == kPhotons ? a.lds_g : (which == kLeptons ? a.lds_l : a.lds_gl);
}
// one iteration is the short-electron launch (with short buffers), then one
// visit launch of both species or one of each
hipError_t launch_short(const KArgs& a, uint32_t blocks, hipStream_t s) {
  KArgs arg = a;
  void* args[] = {&arg};
  return hipLaunchKernel(kernel_for(a, true), dim3(blocks), dim3(kBlock), args, a.lds_l, s);
}
hipError_t launch_visit(const KArgs& a, uint32_t which, uint32_t blocks, hipStream_t s) {
  KArgs arg = a;
  void* args[] = {&arg, &which};
  return hipLaunchKernel(kernel_for(a, false), dim3(blocks), dim3(kBlock), args, visit_lds(a, which), s);
}
hipError_t launch_inject(const KArgs& a, const InjRec* rec, uint32_t n, hipStream_t s) {
  const uint32_t want = (n + kBlock - 1) / kBlock;
  const uint32_t blocks = n == 0 ? 1 : (want < 4096 ? want : 4096);
  if (a.precision) hipLaunchKernelGGL(k_inject<float>, dim3(blocks), dim3(kBlock), 0, s, a, rec, n);
  else hipLaunchKernelGGL(k_inject<double>, dim3(blocks), dim3(kBlock), 0, s, a, rec, n);
  return hipGetLastError();
}
hipError_t launch_reset_rows(const KArgs& a, const uint32_t* rows, uint32_t n, hipStream_t s) {
  const uint32_t blocks = n == 0 ? 1 : (n < 1024 ? n : 1024);
  hipLaunchKernelGGL(k_reset_rows, dim3(blocks), dim3(kBlock), 0, s, a, rows, n);
  return hipGetLastError();
}
hipError_t launch_gather_rows(const KArgs& a, const uint32_t* rows, uint32_t n, char* out, hipStream_t s) {
  const uint32_t blocks = n == 0 ? 1 : (n < 1024 ? n : 1024);
  hipLaunchKernelGGL(k_gather_rows, dim3(blocks), dim3(kBlock), 0, s, a, rows, n, out);
  return hipGetLastError();
}
hipError_t launch_atomic_probe(double* cells, uint64_t n_cells, uint64_t n_ops, hipStream_t s) {
  const uint64_t want = (n_ops + kBlock - 1) / kBlock;
  const uint32_t blocks = (uint32_t)(want < 16384 ? (want ? want : 1) : 16384);
  hipLaunchKernelGGL(k_atomic_probe, dim3(blocks), dim3(kBlock), 0, s, cells, n_cells, n_ops);
  return hipGetLastError();
}
hipError_t launch_fill_zero(void* p, uint64_t bytes, hipStream_t s) {
  if (bytes == 0) return hipSuccess;
  if (reinterpret_cast<uintptr_t>(p) % 8) return hipErrorInvalidValue;
  const uint64_t words = bytes / 8;
  const uint64_t want = (words + kBlock - 1) / kBlock;
  const uint32_t blocks = (uint32_t)(want == 0 ? 1 : (want < 8192 ? want : 8192));
  hipLaunchKernelGGL(k_fill_zero, dim3(blocks), dim3(kBlock), 0, s, static_cast<unsigned long long*>(p), words,
                     static_cast<unsigned char*>(p) + words * 8, (uint32_t)(bytes % 8));
  return hipGetLastError();
}
hipError_t launch_census(const KArgs& a, hipStream_t s) {
  hipLaunchKernelGGL(k_census, dim3(1), dim3(64), 0, s, a);
  return hipGetLastError();
}
// blocks of the visit launch of `which` and of the short launch (which = 0)
// that fit on one CU (registers and LDS), for the variants the context
// launches
hipError_t visit_occupancy(const KArgs& a, uint32_t which, int* per_cu) {
  const void* f = kernel_for(a, which == 0);
  const uint32_t lds = which == 0 ? a.lds_l : visit_lds(a, which);
  // (the largest of the kernel's launches: the attribute is the kernel's)
  const uint32_t most = which == 0 || a.split ? (a.lds_l > a.lds_g ? a.lds_l : a.lds_g) : a.lds_gl;
  hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)most);
  if (e != hipSuccess) return e;
  return hipOccupancyMaxActiveBlocksPerMultiprocessor(per_cu, f, kBlock, lds);
}
#endif  // EMS_SLAB_F32_TU

}  // namespace ems
