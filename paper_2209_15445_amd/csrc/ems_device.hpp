// ems_device.hpp -- device-side data layout shared by the kernels and the
// host runtime: track queues, the loop-control block, kernel arguments.
#pragma once
#include "ems_step.hpp"

namespace ems {

// One species queue buffer: records of position and energy in FP64, 64-bit
// id, direction in the arithmetic type R, then event row, RNG event key, and
// step count and volume packed in one word (n << b | volume, b = 12 for the
// slab stack, more for a large box geometry; all ones marks a dead slot).  76
// bytes per track in the FP64 form, 64 in the mixed form.  The six buffers
// (2 x 3 species) are consecutive blocks of cap * track_bytes.
// A record is 64 bytes, read and written with four 16-byte operations (the
// FP64 form keeps the last three words, 12 bytes, in an array of their own
// behind the records): consecutive lanes use consecutive records, so whole
// cache lines are moved either way, and a batch of a wave needs four or five
// memory instructions and two base addresses where an array per field took
// eleven of each (and spilled the addresses from the scalar registers).
// 40 000 x 10 GeV, mixed form: 135.5 ms with an array per field, 129.6 ms with
// records; HBM bytes of a photon launch (10^5 x 10 GeV) 3.72 and 2.54 GB.
constexpr uint32_t kSlabBits = 12, kSlabMask = (1u << kSlabBits) - 1;
constexpr uint32_t kMaxSlabs = kSlabMask;                 // slab indices 0..4094
constexpr uint32_t kMaxBoxes = 1u << 24;
constexpr uint32_t kMaxStepsPerTrack = (1u << 20) - 1;    // step counts fit 20 bits
constexpr uint32_t kDeadRecord = 0xFFFFFFFFu;
struct alignas(16) TrackRec64 {
  double x, y, z, E, ux, uy, uz;
  uint64_t id;
};
struct TrackTail64 {
  uint32_t ev, key, ns;
};
struct alignas(16) TrackRec32 {
  double x, y, z, E;
  float ux, uy, uz;
  uint32_t ns;
  uint64_t id;
  uint32_t ev, key;
};
template <class R>
constexpr size_t track_bytes() {
  return sizeof(R) == 8 ? sizeof(TrackRec64) + sizeof(TrackTail64) : sizeof(TrackRec32);
}
static_assert(sizeof(TrackRec64) == 64 && sizeof(TrackTail64) == 12 && sizeof(TrackRec32) == 64, "track records");

template <class R>
struct Queue;
template <>
struct Queue<double> {
  TrackRec64* rec;
  TrackTail64* tail;
  EMS_HD void kill(uint32_t i) const { tail[i].ns = kDeadRecord; }
  EMS_HD void store(uint32_t i, const Trk<double>& t, uint32_t ns) const {
    rec[i] = TrackRec64{t.x, t.y, t.z, t.E, t.ux, t.uy, t.uz, t.id};
    tail[i] = TrackTail64{t.ev, t.key, ns};
  }
  // the record without t.n and t.slab; returns their packed word
  EMS_HD uint32_t load(uint32_t i, Trk<double>& t) const {
    const TrackRec64 r = rec[i];
    const TrackTail64 e = tail[i];
    t.x = r.x;
    t.y = r.y;
    t.z = r.z;
    t.E = r.E;
    t.ux = r.ux;
    t.uy = r.uy;
    t.uz = r.uz;
    t.id = r.id;
    t.ev = e.ev;
    t.key = e.key;
    return e.ns;
  }
};
template <>
struct Queue<float> {
  TrackRec32* rec;
  EMS_HD void kill(uint32_t i) const { rec[i].ns = kDeadRecord; }
  EMS_HD void store(uint32_t i, const Trk<float>& t, uint32_t ns) const {
    rec[i] = TrackRec32{t.x, t.y, t.z, t.E, t.ux, t.uy, t.uz, ns, t.id, t.ev, t.key};
  }
  EMS_HD uint32_t load(uint32_t i, Trk<float>& t) const {
    const TrackRec32 r = rec[i];
    t.x = r.x;
    t.y = r.y;
    t.z = r.z;
    t.E = r.E;
    t.ux = r.ux;
    t.uy = r.uy;
    t.uz = r.uz;
    t.id = r.id;
    t.ev = r.ev;
    t.key = r.key;
    return r.ns;
  }
};

EMS_HD void view_at(char* b, uint64_t cap, Queue<double>& q) {
  q.rec = reinterpret_cast<TrackRec64*>(b);
  q.tail = reinterpret_cast<TrackTail64*>(q.rec + cap);
}
EMS_HD void view_at(char* b, uint64_t, Queue<float>& q) { q.rec = reinterpret_cast<TrackRec32*>(b); }

// Loop control, written by the block that closes an iteration.
//
// Each next-queue buffer of capacity cap has two regions: survivors and
// carried tracks of that species fill it from the bottom (home region), new
// secondaries from the top (position cap-1-s for secondary slot s).  The
// secondaries of species q may use at most cap - n_cur[q] slots, which leaves
// room for every survivor, so a step whose secondaries do not fit is simply
// not taken: the track is carried unchanged and stepped again later (its
// random numbers depend only on its id and step count).
constexpr uint32_t kLine = 32;  // words of a cache line
constexpr int kNextCounters = 8, kNextHome = 0, kNextSec = 3, kNextShort = 6, kNextSpill = 7;
// launch tallies (Ctl::add), by species where [3]
enum : int {
  kAddSteps = 0,        // [3] steps taken
  kAddVisits = 3,       // [3] track records loaded
  kAddMade = 6,         // [3] secondaries written
  kAddKept = 9,         // [3] records written to the home regions
  kAddMadeBy = 12,      // [2] secondaries by launch (photon, e-/e+)
  kAddCarried = 14,     // tracks carried unstepped
  kAddMadeShort = 15,   // e- secondaries written to the short buffer (in kAddMade too)
  kAddStepsShort = 16,  // steps of the short launch (in kAddSteps too)
  kAdds = 17
};
// The queues of one iteration, by buffer.  The launches of an iteration read
// the record of the current buffer (KArgs::cur, alternating from iteration to
// iteration) and its close writes the other one: a block may start after the
// iteration was closed (another context's work may hold the device, or the
// grid may exceed it) and still has to read what the blocks before it read.
struct Extents {
  uint32_t n_home[3];  // tracks in the home region
  uint32_t n_sec[3];   // tracks in the secondary region
  // Live records: the extents n_home + n_sec may include dead slots (unused
  // ends of wave-private append chunks); n_real counts the live tracks.
  uint32_t n_real[3];
  // Short electrons (KArgs::short_E): extent and live records of the short
  // buffer, and the spill counter before the iteration.
  uint32_t n_short, n_short_real, spilled;
  uint32_t held;  // octaves held back: kNoLevel less the energy level (ems_iteration.hpp)
  uint32_t stop;  // an error was seen: nothing is stepped any more
};
struct Ctl {
  Extents ext[2];
  uint32_t blocks_done;   // completion ticket of the running launch
  uint32_t iteration;
  uint32_t live;          // tracks in the next iteration's queues
  uint32_t error;         // kErr* bits
  uint32_t peak[3];
  unsigned long long steps[3], created[3], deferred, log_n;
  unsigned long long visits[3];  // track records loaded (one per visit)
  unsigned long long made_by[2];  // secondary records written (photons, e-/e+)
  unsigned long long exit_n;  // outgoing tracks recorded (may exceed the capacity)
  unsigned long long steps_s;  // e- steps taken by the short launches
  // tallies of the running iteration, folded into the totals above when it
  // ends
  unsigned long long add[kAdds];
  // The counters every wave draws from, each alone in its cache line: they
  // are incremented at the memory side, where the requests for one line
  // wait for each other (in one line with each other and the fields above:
  // 10^4 x 10 GeV 43.1 ms, 40 000 x 10 GeV in the mixed form 111.4, 500 x
  // 2 GeV 4.49; each in its own: 40.9, 104.5 and 4.27).
  // Append counters: home (0..2) and secondary regions (3..5) of the next
  // queues by species, next short buffer (6), and the spill buffer (7: tracks
  // the short launch hands to the e-/e+ loop; never cleared during a batch,
  // its slots count from Extents::spilled).
  alignas(128) uint32_t next[kNextCounters * kLine];
  alignas(128) uint32_t cursor[2 * kLine];  // queue indices handed out (photons, e-/e+)
};
enum : uint32_t { kErrOverflow = 1u, kErrStall = 2u, kErrCorrupt = 4u };

// Track prepared on the host for injection (slab located, direction unit,
// RNG event key of its row).
struct InjRec {
  double x, y, z, ux, uy, uz, E;
  uint64_t id;
  uint32_t ev, sp;
  int32_t slab;
  uint32_t key;
};

// Outgoing track, laid out as a primary record of the public header.
struct ExitRec {
  uint32_t event, species;
  double ekin, pos[3], dir[3];
};

// Per-event ledger as laid out in the public header.
struct LedgerDev {
  double edep, escaped[3], killed, charged_len;
  unsigned long long n_steps, n_created[3], n_null;
  uint32_t n_pair, n_annih;
};

struct StepRec {
  uint32_t event, species;
  uint64_t id;
  uint32_t step;
  int32_t slab_after;
  uint32_t limiter, process;
  double e_before, e_after, pos[3], step_len, edep;
};

enum : uint32_t { kFlagSteplog = 1u, kFlagFullLedger = 2u, kFlagProfile = 4u, kFlagEventLive = 8u, kFlagTiming = 16u };

struct KArgs {
  char* qbase;         // six queue buffers, see queue_view
  Ctl* ctl;
  double* edep;        // [rows][n_slabs]
  LedgerDev* ledger;   // [rows]
  const void* tab_g;   // photon table block [mat][3][nodes] (double or float)
  const void* tab_l;   // lepton table block [mat][12][nodes]
  const double* zplane;
  const uint32_t* slab_mat;
  const MatRT* mat;
  const double* el_c;   // element screening constants [mat][4][2]
  const void* el_tab;   // partial pair / brems totals [mat][4][2][nodes] (double or float)
  StepRec* log;
  uint32_t* profile;   // [profile_cap][3]
  int32_t* live_ev;    // [rows] live tracks per event (kFlagEventLive)
  uint64_t cap;        // tracks per species per buffer
  uint32_t cur;        // this iteration's buffer and extents (0/1)
  uint64_t qstride;    // bytes of a queue buffer (cap records)
  uint32_t max_events;  // tally rows
  uint64_t log_cap;
  uint32_t profile_cap;
  uint32_t flags;
  uint32_t n_mat;
  uint32_t lds_g, lds_l, lds_gl;  // dynamic LDS of a launch: photon, lepton tables, both
  uint32_t split;             // photons and e-/e+ in a launch each
  uint32_t steps_per_visit;   // steps a thread may take per launch
  uint32_t refill_below;      // batch commit/refill when at most this many lanes still step
  uint32_t interact_min;      // e-/e+: sample a batch's interactions once this many wait
  uint32_t photon_steps_per_visit, photon_refill_below;  // the photon kernel's own two
  uint32_t precision;  // 0: FP64 kernels, 1: mixed kernels
  uint32_t waves;             // waves of a visit launch
  ExitRec* exits;             // outgoing tracks (exit_cap records)
  uint64_t exit_cap;
  uint32_t geo;               // geometry kind: 0 slab stack, 1 boxes
  uint32_t feat;              // optional parts (kF* bits) of the kernels launched
  uint32_t vol_bits;          // low bits of the packed word that hold the volume
  StepEnv<double> env;  // scalars; its pointers are set per block
  StepReals<float> env32;  // env's StepReals in the mixed form's arithmetic type
  // Short electrons: e- secondaries below short_E (0: none) are appended to
  // a buffer of their own (two of cap_s records, current and next) and take
  // their first step in a launch of their own at the start of the next
  // iteration; a track whose first step selects an interaction goes to the
  // spill buffer (cap_p records) for the e-/e+ of that iteration's visit launch.
  char* sbase;                // the two short buffers, then the spill buffer
  uint64_t cap_s, cap_p;
  double short_E;
  uint32_t waves_s;           // waves of the short launch
};

// queue of species sp in buffer buf (0/1)
template <class R>
EMS_HD Queue<R> queue_view(const KArgs& a, uint32_t buf, uint32_t sp) {
  Queue<R> q;
  // (by selection: sp may differ between lanes, the rest does not)
  const uint64_t at = sp == 0 ? 0ull : (sp == 1 ? a.qstride : 2 * a.qstride);
  view_at(a.qbase + (buf ? 3 * a.qstride : 0ull) + at, a.cap, q);
  return q;
}
// short buffer b (0/1) and the spill buffer (b = 2), laid out as queues
template <class R>
EMS_HD Queue<R> short_view(const KArgs& a, uint32_t b) {
  Queue<R> q;
  view_at(a.sbase + (size_t)b * a.cap_s * track_bytes<R>(), b == 2 ? a.cap_p : a.cap_s, q);
  return q;
}

}  // namespace ems
