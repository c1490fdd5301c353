// ems_primaries.hip -- a batch's way in and out: its restart, the check,
// staging and id passes that ems_enqueue_device runs on primaries handed over
// in device memory before the tracks are injected (the host path computes the
// same on the host), and the rows read back by the host.
#include <hip/hip_runtime.h>

#include "ems_runtime.hpp"

namespace ems {

namespace {

constexpr int kBlock = 256;

// Primaries handed over in device memory (section 4: the particles of a
// region given to the library; here already resident in HBM).  A primary
// is accepted under the conditions of the host path: row below max_events,
// a species, finite positive energy, a finite non-zero direction, and a
// position inside the geometry (a volume found for it in a box geometry;
// inside the stack's z range and its half width for a slab stack).
__device__ inline bool primary_valid(const KArgs& a, const PrimRec& q) {
#pragma clang fp contract(off)
  const double d2 = q.dir[0] * q.dir[0] + q.dir[1] * q.dir[1] + q.dir[2] * q.dir[2];
  if (!(q.event < a.max_events && q.species <= 2u && q.E > 0.0 && isfinite(q.E) && d2 > 0.0 && isfinite(d2)))
    return false;
  if (a.geo) {
    if (!(isfinite(q.pos[0]) && isfinite(q.pos[1]) && isfinite(q.pos[2]))) return false;
    return bvh_locate(a.env.nav, q.pos, q.dir) >= 0;
  }
  const uint32_t n = a.env.n_slabs;
  return q.pos[2] >= a.zplane[0] && q.pos[2] <= a.zplane[n] && fabs(q.pos[0]) <= a.env.half_xy &&
         fabs(q.pos[1]) <= a.env.half_xy;
}

// slab holding z (planes zp[0..n]); a point on a plane belongs to the slab
// its direction enters
__device__ inline int32_t slab_of(const double* zp, uint32_t n, double z, double uz) {
  if (z >= zp[n]) return (int32_t)n - 1;
  uint32_t lo = 0, hi = n;  // zp[lo] <= z < zp[hi]
  while (hi - lo > 1) {
    const uint32_t mid = (lo + hi) / 2;
    if (zp[mid] <= z) lo = mid;
    else hi = mid;
  }
  if (lo > 0 && z == zp[lo] && uz < 0.0) lo -= 1;
  return (int32_t)lo;
}

// Check pass over n device primaries: chk[0] = n - i for the first invalid
// primary i (0: all valid), chk[1 + s] = primaries of species s.  chk is
// zero on entry.
__global__ __launch_bounds__(kBlock) void k_check_primaries(KArgs a, const PrimRec* p, uint64_t n,
                                                            unsigned long long* chk) {
  const uint64_t stride = (uint64_t)gridDim.x * kBlock;
  for (uint64_t base = (uint64_t)blockIdx.x * kBlock; base < n; base += stride) {
    const uint64_t i = base + threadIdx.x;
    bool ok = true;
    uint32_t sp = 3;
    if (i < n) {
      const PrimRec q = p[i];
      ok = primary_valid(a, q);
      sp = ok ? q.species : 3u;
      if (!ok) atomicMax(&chk[0], (unsigned long long)(n - i));
    }
    for (uint32_t s = 0; s < 3; ++s) {
      const uint32_t c = (uint32_t)__popcll(__ballot(sp == s));
      if (__lane_id() == 0 && c) atomicAdd(&chk[1 + s], (unsigned long long)c);
    }
  }
}

// Injection record of a valid primary (direction normalised, volume
// located, the row's event key); its id is set later.
__device__ inline InjRec staged(const KArgs& a, const PrimRec& q, const uint32_t* keys) {
  // the length as the host computes it: products and sums rounded one by
  // one (no fused multiply-add), then a correctly rounded root and quotients
#pragma clang fp contract(off)
  const double nrm = sqrt(q.dir[0] * q.dir[0] + q.dir[1] * q.dir[1] + q.dir[2] * q.dir[2]);
  InjRec r;
  r.x = q.pos[0];
  r.y = q.pos[1];
  r.z = q.pos[2];
  r.ux = q.dir[0] / nrm;
  r.uy = q.dir[1] / nrm;
  r.uz = q.dir[2] / nrm;
  r.E = q.E;
  r.id = 0;
  r.ev = q.event;
  r.sp = q.species;
  if (a.geo) {
    const double pp[3] = {r.x, r.y, r.z}, uu[3] = {r.ux, r.uy, r.uz};
    r.slab = bvh_locate(a.env.nav, pp, uu);
  } else {
    r.slab = slab_of(a.zplane, a.env.n_slabs, r.z, r.uz);
  }
  r.key = keys[q.event];
  return r;
}

// Stage pass: the injection records of k valid device primaries; ids are set
// by k_primary_ids.
__global__ __launch_bounds__(kBlock) void k_stage_primaries(KArgs a, const PrimRec* p, uint32_t k,
                                                            const uint32_t* keys, InjRec* out) {
  for (uint32_t i = blockIdx.x * kBlock + threadIdx.x; i < k; i += gridDim.x * kBlock) out[i] = staged(a, p[i], keys);
}

// Ids of a group of up to 1024 primaries: the running index of a primary
// within its row, in input order, continuing from the row's count so far
// (row_next).  A block of 1024 threads has the group's (row, position) keys
// in LDS and sorts them (bitonic) unless they come in row order, as a batch
// made event by event does; a primary's rank is its distance from its row's
// first key, and the row's last key adds the group's count to row_next, which
// returns the row's base.  put(position, id) is called once for each.
constexpr uint32_t kIdGroup = 1024;
struct IdGroup {
  unsigned long long key[kIdGroup], base[kIdGroup];
  int head[kIdGroup / 64];  // last row start in each wave's keys (-1: none)
};
template <class Put>
__device__ inline void group_ids(IdGroup& s, bool in, uint32_t ev, unsigned long long* row_next, Put put) {
  const uint32_t t = threadIdx.x;
  s.key[t] = in ? ((unsigned long long)ev << 10 | t) : ~0ull;
  __syncthreads();
  if (!__syncthreads_and(t == 0 || s.key[t - 1] <= s.key[t])) {
    for (uint32_t size = 2; size <= kIdGroup; size <<= 1) {
      for (uint32_t j = size >> 1; j > 0; j >>= 1) {
        const uint32_t o = t ^ j;
        if (o > t) {
          const unsigned long long x = s.key[t], y = s.key[o];
          const bool up = (t & size) == 0;
          if ((x > y) == up) {
            s.key[t] = y;
            s.key[o] = x;
          }
        }
        __syncthreads();
      }
    }
  }
  const unsigned long long kk = s.key[t];
  const bool valid = kk != ~0ull;
  const unsigned long long row = kk >> 10;
  const bool first = valid && (t == 0 || (s.key[t - 1] >> 10) != row);
  const bool last = valid && (t == kIdGroup - 1 || (s.key[t + 1] >> 10) != row);
  // start of the key's row: the last row start at or before it
  const unsigned long long starts = __ballot(first);
  const int wave = (int)(t / 64), begin = wave * 64;
  if (__lane_id() == 0) s.head[wave] = starts ? begin + 63 - __clzll((long long)starts) : -1;
  __syncthreads();
  const unsigned long long upto = starts & (__lanemask_lt() | 1ull << __lane_id());
  int start = upto ? begin + 63 - __clzll((long long)upto) : -1;
  for (int w = wave - 1; w >= 0 && start < 0; --w) start = s.head[w];
  if (last) s.base[start] = atomicAdd(&row_next[row], (unsigned long long)((int)t - start + 1));
  __syncthreads();
  if (valid) put((uint32_t)(kk & (kIdGroup - 1)), s.base[start] + (unsigned long long)((int)t - start));
  __syncthreads();
}
__global__ __launch_bounds__(kIdGroup) void k_primary_ids(InjRec* rec, uint32_t n, unsigned long long* row_next) {
  __shared__ IdGroup s;
  for (uint32_t g = 0; g < n; g += kIdGroup) {
    const bool in = g + threadIdx.x < n;
    group_ids(s, in, in ? rec[g + threadIdx.x].ev : 0u, row_next,
              [&](uint32_t pos, unsigned long long id) { rec[g + pos].id = id; });
  }
}

// A batch of at most 1024 device primaries in one launch of one block
// instead of five launches and a copy: check, ids, injection records and the
// tracks, which are appended only if all primaries are valid and the queues
// have room for them (pend: tracks enqueued before).  res as k_check_primaries
// leaves it; it may be host memory.  32 primaries: the call went from 69 to
// 47 us.
template <class R>
__global__ __launch_bounds__(kIdGroup) void k_few_primaries(KArgs a, const PrimRec* p, uint32_t n,
                                                            const uint32_t* keys, unsigned long long* row_next,
                                                            Pending pend, unsigned long long* res) {
  __shared__ IdGroup s;
  __shared__ unsigned long long ids[kIdGroup];
  __shared__ uint32_t per_wave[3][kIdGroup / 64];
  __shared__ uint32_t bad;
  const uint32_t t = threadIdx.x, wave = t / 64;
  const bool in = t < n;
  if (t == 0) bad = n;
  PrimRec q{};
  if (in) q = p[t];
  const bool ok = in && primary_valid(a, q);
  const uint32_t sp = ok ? q.species : 3u;
  uint32_t rank = 0;
  for (uint32_t k = 0; k < 3; ++k) {
    const unsigned long long m = __ballot(sp == k);
    if (sp == k) rank = (uint32_t)__popcll(m & __lanemask_lt());
    if (__lane_id() == 0) per_wave[k][wave] = (uint32_t)__popcll(m);
  }
  __syncthreads();
  if (in && !ok) atomicMin(&bad, t);
  uint32_t total[3] = {0, 0, 0};
  for (uint32_t k = 0; k < 3; ++k)
    for (uint32_t w = 0; w < kIdGroup / 64; ++w) {
      if (sp == k && w < wave) rank += per_wave[k][w];
      total[k] += per_wave[k][w];
    }
  __syncthreads();
  bool room = bad == n;
  for (uint32_t k = 0; k < 3; ++k) room = room && pend.n[k] + total[k] <= a.cap;
  if (t == 0) {
    res[0] = n - bad;
    for (uint32_t k = 0; k < 3; ++k) res[1 + k] = total[k];
  }
  if (!room) return;
  group_ids(s, in, q.event, row_next, [&](uint32_t pos, unsigned long long id) { ids[pos] = id; });
  Ctl* ctl = a.ctl;
  const uint32_t cur = a.cur;
  Extents& e = ctl->ext[cur];
  const uint32_t home = in ? e.n_home[sp] : 0u, sec = in ? e.n_sec[sp] : 0u;
  if (in) {
    const InjRec r = staged(a, q, keys);
    const uint32_t slot = home + rank;
    if (slot + sec < a.cap) {
      Trk<R> tr;
      tr.x = r.x;
      tr.y = r.y;
      tr.z = r.z;
      tr.ux = (R)r.ux;
      tr.uy = (R)r.uy;
      tr.uz = (R)r.uz;
      tr.E = r.E;
      tr.id = ids[t];
      tr.ev = r.ev;
      tr.key = r.key;
      tr.n = 0;
      tr.slab = r.slab;
      queue_view<R>(a, cur, sp).store(slot, tr, (uint32_t)r.slab);
      if (a.flags & kFlagEventLive) atomicAdd(&a.live_ev[r.ev], 1);
      atomicAdd(&e.n_real[sp], 1u);
    } else {
      atomicOr(&ctl->error, kErrOverflow);
    }
  }
  __syncthreads();  // (all have read the extents)
  if (t < 3) e.n_home[t] += t == 0 ? total[0] : (t == 1 ? total[1] : total[2]);
}

// Restart of a batch: the tallies to zero, and the control block but for the
// extents of the queues (empty after a run).  One launch instead of three
// or four, and nothing the host waits for (it read the control block and
// wrote it back): the call went from 34 to 3.6 us with 48 events.
struct Spans {
  uint4* p[3];
  uint64_t n[3];  // 16-byte words
};
__global__ __launch_bounds__(kBlock) void k_restart(Ctl* ctl, uint32_t cur, Spans z) {
  const uint64_t stride = (uint64_t)gridDim.x * kBlock;
#pragma unroll
  for (int k = 0; k < 3; ++k)
    for (uint64_t i = (uint64_t)blockIdx.x * kBlock + threadIdx.x; i < z.n[k]; i += stride)
      z.p[k][i] = make_uint4(0u, 0u, 0u, 0u);
  if (blockIdx.x) return;
  static_assert(sizeof(Ctl) % 4 == 0, "cleared by words");
  Extents e{};
  if (threadIdx.x == 0) {
    e = ctl->ext[cur];
    e.spilled = 0;
    e.stop = 0;
    e.held = 0;
  }
  __syncthreads();
  for (uint32_t i = threadIdx.x; i < sizeof(Ctl) / 4; i += kBlock) reinterpret_cast<uint32_t*>(ctl)[i] = 0u;
  __syncthreads();
  if (threadIdx.x == 0) ctl->ext[cur] = e;
}

// Rows to memory of the host, a block to a row at a time: deposits as they
// are, and the ledger with the sum of the row's deposits, added one after
// another as the host does (so no second copy of the deposits is read for
// it).  500 ledgers of 100 columns 51 -> 19 us, 48 rows of deposits 35 -> 21.
__global__ __launch_bounds__(kBlock) void k_read_rows(KArgs a, uint32_t first, uint32_t n, double* edep,
                                                      LedgerDev* led) {
  static_assert(kSumCols <= kBlock, "a column to a thread");
  __shared__ double dep[kSumCols];
  const uint32_t nc = a.env.n_slabs;
  for (uint32_t i = blockIdx.x; i < n; i += gridDim.x) {
    const double* e = a.edep + (size_t)(first + i) * nc;
    if (edep)
      for (uint32_t k = threadIdx.x; k < nc; k += kBlock) edep[(size_t)i * nc + k] = e[k];
    if (led) {
      if (threadIdx.x < nc) dep[threadIdx.x] = e[threadIdx.x];
      const unsigned long long* from = reinterpret_cast<const unsigned long long*>(a.ledger + first + i);
      unsigned long long* to = reinterpret_cast<unsigned long long*>(led + i);
      if (threadIdx.x < sizeof(LedgerDev) / 8 && threadIdx.x != offsetof(LedgerDev, edep) / 8)
        to[threadIdx.x] = from[threadIdx.x];
      __syncthreads();
      if (threadIdx.x == 0) {
        double sum = 0.0;
        for (uint32_t k = 0; k < nc; ++k) sum += dep[k];
        led[i].edep = sum;
      }
      __syncthreads();
    }
  }
}

}  // namespace

hipError_t launch_check_primaries(const KArgs& a, const void* p, uint64_t n, unsigned long long* chk, hipStream_t s) {
  const uint64_t want = (n + kBlock - 1) / kBlock;
  const uint32_t blocks = (uint32_t)(want < 4096 ? (want ? want : 1) : 4096);
  hipLaunchKernelGGL(k_check_primaries, dim3(blocks), dim3(kBlock), 0, s, a, static_cast<const PrimRec*>(p), n, chk);
  return hipGetLastError();
}
hipError_t launch_stage_primaries(const KArgs& a, const void* p, uint32_t k, const uint32_t* keys,
                                  unsigned long long* row_next, InjRec* out, hipStream_t s) {
  const uint32_t want = (k + kBlock - 1) / kBlock;
  const uint32_t blocks = want < 4096 ? (want ? want : 1) : 4096;
  hipLaunchKernelGGL(k_stage_primaries, dim3(blocks), dim3(kBlock), 0, s, a, static_cast<const PrimRec*>(p), k, keys,
                     out);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_primary_ids, dim3(1), dim3(kIdGroup), 0, s, out, k, row_next);
  return hipGetLastError();
}

hipError_t launch_few_primaries(const KArgs& a, const void* p, uint32_t n, const uint32_t* keys,
                                unsigned long long* row_next, const Pending& pend, unsigned long long* res,
                                hipStream_t s) {
  static_assert(kFewPrimaries <= kIdGroup, "one block takes them all");
  const PrimRec* q = static_cast<const PrimRec*>(p);
  if (a.precision)
    hipLaunchKernelGGL(k_few_primaries<float>, dim3(1), dim3(kIdGroup), 0, s, a, q, n, keys, row_next, pend, res);
  else
    hipLaunchKernelGGL(k_few_primaries<double>, dim3(1), dim3(kIdGroup), 0, s, a, q, n, keys, row_next, pend, res);
  return hipGetLastError();
}

hipError_t launch_restart(const KArgs& a, const Span (&z)[3], hipStream_t s) {
  Spans v{};
  uint64_t words = 1;
  for (int k = 0; k < 3; ++k) {
    v.p[k] = static_cast<uint4*>(z[k].p);
    v.n[k] = z[k].bytes / 16;
    words = v.n[k] > words ? v.n[k] : words;
  }
  const uint64_t want = (words + kBlock - 1) / kBlock;
  const uint32_t blocks = (uint32_t)(want < 4096 ? want : 4096);
  hipLaunchKernelGGL(k_restart, dim3(blocks), dim3(kBlock), 0, s, a.ctl, a.cur, v);
  return hipGetLastError();
}
hipError_t launch_read_rows(const KArgs& a, uint32_t first, uint32_t n, double* edep, LedgerDev* led, hipStream_t s) {
  hipLaunchKernelGGL(k_read_rows, dim3(n < 2048 ? n : 2048), dim3(kBlock), 0, s, a, first, n, edep, led);
  return hipGetLastError();
}

}  // namespace ems
