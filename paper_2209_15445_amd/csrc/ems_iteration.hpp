// ems_iteration.hpp -- the queues an iteration's launches read, how a visit
// launch is dealt to its waves, and what its close leaves to the next
// iteration (device code, also run by a host check).
#pragma once
#include "ems_device.hpp"

namespace ems {

constexpr uint32_t kBlockWaves = 4;  // waves of a visit block
// species of a visit launch
enum : uint32_t { kPhotons = 1u, kLeptons = 2u };

// Scarce room goes to the lower energies.  A queue that is filled with tracks
// whose next steps all need a slot never moves again, so queues too small for
// a shower have to be kept from filling with tracks that take long to end.
// Once an iteration had to carry tracks (steps refused for want of room), and
// while less than a quarter of some queue is free, tracks above an energy of
// 2^(level - 10) MeV make no secondaries (they are carried), and an iteration
// takes at most half of such a queue's room.  The level follows the room: down an octave an
// iteration while less than an eighth of a queue is free (two below a
// thirty-second), up one while little of what there was is taken, up two when
// nothing had to be carried, and up four when nothing moved at all; the batch
// fails only if nothing moves without a level.  The energies of a step's
// secondaries add up to less than the track's (a positron's with its rest
// energy), so what is let through ends in tracks that are let through.
// Queues that hold the whole shower never come to this.
// Times in queues of a fourth, an eighth and a sixteenth of the largest
// population, with this rule and (in brackets) with photons waiting while less
// than an eighth of the e- queue was free: 500 x 2 GeV FP64 10.6, 33.9, 70.6 ms
// (10.0, no end, no end), mixed form 9.9, 23.6, 51.5 (9.8, 38.6, no end), in
// the tower block FP64 21.2, 70.8, 161 (20.0, 49.0, no end); 2000 x 5 GeV FP64
// 19.3, 32.2, 62.6 (19.2, 32.0, 116.5).  (Limited only where a secondary goes to
// a scarce queue: 82.6 and 232 ms in a sixteenth, and more registers.)
constexpr uint32_t kNoLevel = 24;  // (16 GeV: no limit)
EMS_HD bool tight(uint64_t room, uint64_t cap) { return room < cap / 4; }
EMS_HD uint32_t secondary_limit(uint32_t room, uint64_t cap, uint32_t level) {
  return level < kNoLevel && tight(room, cap) && room > 2 ? room - room / 2 : room;
}
EMS_HD float energy_limit(uint32_t level) {
  return level < kNoLevel ? __builtin_ldexpf(1.0f, (int)level - 10) : __builtin_huge_valf();
}
// least: free slots of the fullest next queue; little: at most a quarter of
// every tight queue's limit was taken
EMS_HD uint32_t next_level(uint32_t level, uint64_t carried, uint64_t commits, uint64_t least, uint64_t cap,
                           bool little) {
  const uint32_t up = carried == 0 ? 2 : (commits == 0 ? 4 : (little || !tight(least, cap) ? 1 : 0));
  const uint32_t down = least < cap / 32 ? 2 : (least < cap / 8 ? 1 : 0);
  if (carried && commits && down) return level > down ? level - down : 0u;
  return level + up < kNoLevel ? level + up : kNoLevel;
}

// the current queues: home regions, all tracks by species, short buffer,
// and the tracks the short launch spilled to the e-/e+ loop
struct Sizes {
  uint32_t h0, h1, h2, n0, n1, n2, ns, np, level;
};
template <bool SHORT>
EMS_HD Sizes sizes_of(const Ctl* ctl, uint32_t cur, uint64_t cap_p) {
  const Extents& e = ctl->ext[cur];
  Sizes z;
  z.h0 = e.n_home[0];
  z.h1 = e.n_home[1];
  z.h2 = e.n_home[2];
  z.n0 = z.h0 + e.n_sec[0];
  z.n1 = z.h1 + e.n_sec[1];
  z.n2 = z.h2 + e.n_sec[2];
  z.ns = SHORT ? e.n_short : 0u;
  z.level = kNoLevel - e.held;
  const uint32_t np = SHORT ? ctl->next[kNextSpill * (int)kLine] - e.spilled : 0u;
  z.np = (uint64_t)np < cap_p ? np : (uint32_t)cap_p;
  return z;
}

// How one species' tracks are dealt to `waves` of a launch's waves: `lanes`
// lanes of a wave hold tracks, wave w of them starts with the queue indices
// [first, first + lanes), and indices from `pool` on are handed out by the
// launch's cursor.
// A population that does not fill the device is dealt evenly over the waves:
// what bounds such a launch is the chain of dependent steps of its slowest
// wave, and a wave pays for every path that any of its lanes takes, so a wave
// with one track runs its steps several times faster than one with 64.
// 32 x 1 GeV (at most 6000 tracks at once, 2048 waves): 6.7 ms a batch with
// 64 tracks to a wave, 3.2 ms dealt evenly.
struct WaveShare {
  uint32_t lanes, first, pool;
};
EMS_HD WaveShare wave_share(uint32_t n, uint32_t w, uint32_t waves) {
  WaveShare s;
  const uint32_t even = n / waves + (n % waves != 0);
  s.lanes = even >= 64u ? 64u : (even > 1u ? even : 1u);
  s.first = w * s.lanes;
  s.pool = waves * s.lanes;
  return s;
}

// A visit launch's waves: the first wg of them start with photons (shares
// sg), the rest with e-/e+ (sl).  The waves with a share come first, and only
// their blocks (below `workers`) take part: the others end at once, without
// drawing a ticket (an iteration without tracks, of which a chunk may hold a
// dozen: 10 us with 512 tickets).  They may do so because every block of a
// launch computes the same numbers, whenever it starts (see Extents).
struct Deal {
  WaveShare sg, sl;
  uint32_t wg, workers;
};
EMS_HD Deal deal_launch(uint32_t ng, uint32_t nl, uint32_t blocks, uint32_t w) {
  Deal d;
  const uint32_t waves = blocks * kBlockWaves;
  uint32_t wg = (uint32_t)((uint64_t)waves * ng / ((uint64_t)ng + nl + (ng + nl == 0u)));
  if (ng) wg = wg < 1u ? 1u : wg;
  if (nl) wg = wg < waves ? wg : waves - 1u;
  d.sg = wave_share(ng, w, wg ? wg : 1u);
  const uint32_t wl = waves - wg;
  if (d.sg.lanes < 64u) wg = (ng + d.sg.lanes - 1) / d.sg.lanes;
  d.sl = wave_share(nl, w - wg, wl ? wl : 1u);
  const uint32_t used = wg + (d.sl.lanes < 64u ? (nl + d.sl.lanes - 1) / d.sl.lanes : wl);
  d.wg = wg;
  d.workers = used < blocks ? used : blocks;
  return d;
}

// What an iteration leaves to the next: extents from the append counters
// (refused slots lie above the limits), live records as counted.
struct Appended {
  uint32_t home[3], sec[3], lim[3], real[3];
  uint32_t shorts, lim_s, shorts_real, spilled;
};
EMS_HD Extents next_extents(const Appended& n, uint32_t live, uint32_t level, uint32_t stop) {
  Extents e;
  for (int q = 0; q < 3; ++q) {
    // with no live track left the dead slots need no visit
    e.n_home[q] = live ? n.home[q] : 0u;
    e.n_sec[q] = live ? (n.sec[q] < n.lim[q] ? n.sec[q] : n.lim[q]) : 0u;
    e.n_real[q] = n.real[q];
  }
  e.n_short = live ? (n.shorts < n.lim_s ? n.shorts : n.lim_s) : 0u;
  e.n_short_real = n.shorts_real;
  e.spilled = n.spilled;
  e.held = kNoLevel - level;
  e.stop = stop;
  return e;
}

}  // namespace ems
