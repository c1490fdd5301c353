// Host check of how a visit launch is dealt and closed (ems_iteration.hpp):
// the blocks of a launch start in any order and at any time, also after the
// block that draws the last ticket has closed the iteration.  Every queue
// index has to be taken exactly once, the iteration closed exactly once, and
// no block may take anything after the close.
// Each launch is run a second time on a model that reads what its own close
// wrote (one record for both): the check has to see that one fail.
#include <cstdio>
#include <memory>
#include <random>
#include <vector>

#include "../paper_2209_15445_amd/csrc/ems_iteration.hpp"

using namespace ems;

namespace {

std::mt19937_64 rng(4);
uint32_t below(uint32_t n) { return (uint32_t)(rng() % n); }
// populations: none, a few, about one to a wave, more than the waves hold
uint32_t population(uint32_t waves) {
  switch (below(5)) {
    case 0: return 0;
    case 1: return below(8);
    case 2: return below(2 * waves + 1);
    case 3: return below(64 * waves + 1);
    default: return below(130 * waves + 1);
  }
}

constexpr uint64_t kCapP = 1u << 20;

struct Run {
  Ctl* ctl;
  Appended next;  // what this iteration will have appended
  bool one_record;
  long faults = 0, late = 0;

  template <bool SHORT>
  void close(uint32_t cur) {
    next.spilled = SHORT ? ctl->next[kNextSpill * (int)kLine] : 0u;
    uint32_t live = next.shorts_real;
    for (uint32_t r : next.real) live += r;
    ctl->ext[cur ^ 1u] = next_extents(next, live, kNoLevel, 0);
    if (one_record) ctl->ext[cur] = ctl->ext[cur ^ 1u];
    ctl->cursor[0] = ctl->cursor[kLine] = 0;
    ctl->blocks_done = 0;
  }

  // one launch of `blocks` blocks
  template <bool SHORT>
  void launch(uint32_t cur, uint32_t which, uint32_t blocks) {
    const Sizes all = sizes_of<SHORT>(ctl, cur, kCapP);
    const uint32_t n[2] = {which & kPhotons ? all.n0 : 0u, which & kLeptons ? all.n1 + all.n2 + all.np : 0u};
    std::vector<uint8_t> taken[2] = {std::vector<uint8_t>(n[0]), std::vector<uint8_t>(n[1])};
    auto take = [&](int k, uint32_t i) {
      if (i >= n[k] || taken[k][i]++) ++faults;
    };
    struct Started {
      uint32_t b, ng, nl, workers;
    };
    std::vector<uint32_t> waiting(blocks);
    for (uint32_t b = 0; b < blocks; ++b) waiting[b] = b;
    std::vector<Started> running;
    int closes = 0;
    while (!waiting.empty() || !running.empty()) {
      if (!waiting.empty() && (running.empty() || below(3) == 0)) {
        // a block starts: it reads its launch's sizes
        const uint32_t k = below((uint32_t)waiting.size()), b = waiting[k];
        waiting[k] = waiting.back();
        waiting.pop_back();
        const Sizes z = sizes_of<SHORT>(ctl, cur, kCapP);
        const uint32_t ng = which & kPhotons ? z.n0 : 0u, nl = which & kLeptons ? z.n1 + z.n2 + z.np : 0u;
        const uint32_t workers = deal_launch(ng, nl, blocks, b).workers;
        late += closes != 0;
        if (b >= workers && (workers || b)) continue;
        if (closes) ++faults;  // works on what the next launch will take
        running.push_back({b, ng, nl, workers});
        continue;
      }
      // a block ends: its waves' shares, what the cursors still hand out, its
      // ticket
      const uint32_t k = below((uint32_t)running.size());
      const Started s = running[k];
      running[k] = running.back();
      running.pop_back();
      for (uint32_t v = 0; s.workers && v < kBlockWaves; ++v) {
        const uint32_t w = v * blocks + s.b;
        const Deal d = deal_launch(s.ng, s.nl, blocks, w);
        const bool own_g = w < d.wg;
        for (int turn = 0; turn < 2; ++turn) {
          const bool photons = own_g == (turn == 0);
          const WaveShare& q = photons ? d.sg : d.sl;
          const uint32_t m = photons ? s.ng : s.nl;
          if (m == 0u || (turn == 1 && q.lanes < 64u)) continue;
          const int sp = photons ? 0 : 1;
          if (turn == 0 && q.first < q.pool)
            for (uint32_t i = q.first; i < q.first + q.lanes && i < m; ++i) take(sp, i);
          if (q.lanes < 64u) continue;
          uint32_t* cursor = &ctl->cursor[sp * kLine];
          const uint32_t chunk = 64u << below(3);
          for (uint32_t at = 0; at < m; ) {
            at = *cursor + q.pool;
            *cursor += chunk;
            for (uint32_t i = at; i < at + chunk && i < m; ++i) take(sp, i);
          }
        }
      }
      if (!(which & kLeptons)) continue;
      if (s.workers == 0 || ctl->blocks_done++ == s.workers - 1) {
        close<SHORT>(cur);
        ++closes;
      }
    }
    for (int k = 0; k < 2; ++k)
      for (uint8_t t : taken[k]) faults += t != 1;
    faults += closes != (which & kLeptons ? 1 : 0);
    faults += ctl->blocks_done != 0;
  }
};

template <bool SHORT>
long iterations(bool one_record, long* late) {
  auto ctl = std::make_unique<Ctl>();
  Run r{ctl.get(), {}, one_record};
  for (int it = 0; it < 4000; ++it) {
    const uint32_t sizes[] = {1, 2, 3, 7, 64, 200}, blocks = sizes[below(it % 50 ? 5 : 6)], cur = it & 1;
    for (int q = 0; q < 3; ++q) {
      const uint32_t p = population(blocks * kBlockWaves);
      r.next.home[q] = below(p + 1);
      r.next.sec[q] = p - r.next.home[q];
      r.next.lim[q] = ~0u;
      r.next.real[q] = p;
    }
    r.next.shorts = r.next.shorts_real = SHORT ? population(blocks * kBlockWaves) : 0u;
    r.next.lim_s = ~0u;
    // the short launch hands some of its tracks over
    if (SHORT) ctl->next[kNextSpill * (int)kLine] += below(ctl->ext[cur].n_short + 1);
    if (it == 2000) ctl->next[kNextSpill * (int)kLine] = ctl->ext[cur].spilled = ~0u - 3u;  // (the counter wraps)
    if (it % 3 == 0) {
      r.launch<SHORT>(cur, kPhotons, blocks);
      r.launch<SHORT>(cur, kLeptons, blocks);
    } else {
      r.launch<SHORT>(cur, kPhotons | kLeptons, blocks);
    }
    if (r.faults && one_record) break;
  }
  *late += r.late;
  return r.faults;
}

// the limits of scarce room: a free slot may be taken, an iteration leaves
// some room while more than two are free, nothing is limited without a level,
// and where nothing moves the level is soon gone
long limits() {
  long faults = 0;
  for (uint64_t cap : {64ull, 256ull, 4096ull, 1ull << 20, 1ull << 28}) {
    for (uint32_t level = 0; level <= kNoLevel; ++level) {
      for (uint64_t room : {(uint64_t)0, (uint64_t)1, (uint64_t)2, (uint64_t)3, cap / 32, cap / 8, cap / 4 - 1, cap / 4, cap}) {
        const uint32_t lim = secondary_limit((uint32_t)room, cap, level);
        faults += lim > room || (room && !lim);
        if (level == kNoLevel || !tight(room, cap)) faults += lim != room;
        else if (room > 2) faults += lim == room;
        const uint32_t stuck = next_level(level, 5, 0, room, cap, true), none = next_level(level, 0, 5, room, cap, true);
        faults += stuck != (level + 4 < kNoLevel ? level + 4 : kNoLevel) || none < level;
        for (bool little : {false, true}) faults += next_level(level, 5, 5, room, cap, little) > kNoLevel;
      }
    }
    faults += energy_limit(kNoLevel) < 1e30f || energy_limit(10) != 1.0f;
    // full queues lower the level to the bottom
    uint32_t level = kNoLevel;
    for (int i = 0; i < 12; ++i) level = next_level(level, 1, 1, 0, cap, false);
    faults += level != 0;
  }
  return faults;
}

}  // namespace

int main() {
  long late = 0, unused = 0;
  const long a = iterations<false>(false, &late), b = iterations<true>(false, &late);
  const long x = iterations<false>(true, &unused), y = iterations<true>(true, &unused);
  std::printf("%ld blocks started after a close; faults %ld, %ld; with one record %ld, %ld\n", late, a, b, x, y);
  const long l = limits();
  std::printf("limits of scarce room: %ld faults\n", l);
  return a == 0 && b == 0 && l == 0 && late > 1000 && x > 0 && y > 0 ? 0 : 1;
}
