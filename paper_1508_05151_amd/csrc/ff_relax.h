// Tile relaxation: the scheduler of the propagation sweeps (device side).
//
// A sweep of Eq. 2 assigns every grid point the best of its own value, its
// vertical and its horizontal predecessor's new value.  The dependencies run
// right and down only (sweep-transformed coordinates), so the assignment has
// exactly one solution, and any order of evaluation that ends with every
// point consistent with its two predecessors ends in that solution: the value
// raster order gives.  A sweep therefore starts every tile of the grid at
// once, on whatever its neighbours hold, and solves a tile again when a
// border value that it read has changed since.  A change rarely crosses more
// than a few tiles (a better flow spreads until it meets a better one), so
// most tiles settle in their second or third visit instead of waiting for the
// whole field above and to the left of them.
//
// Tiles are kTileH grid rows of kTileW columns, row i shifted left by i
// columns (a parallelogram along the anti-diagonals: a wavefront that works
// on one anti-diagonal per step has all its rows busy in every step).  Tile
// (v, u) reads the borders of (v, u - 1), of (v - 1, u + 1) and, one word, of
// (v - 1, u).
//
// Per tile one counter of unanswered requests: base + 1 before the first
// visit, base when settled.  Whoever raises a counter from base owns the
// tile's next visit and either makes it itself or queues it; a visit reads
// the counter before the borders, and takes what it read off afterwards, so
// a request that came in between keeps the tile owned.  Border words carry
// value, cost and the launch's tag in 64 bits (single-copy atomic, so never
// torn); a word without this launch's tag means the neighbour still holds
// its input value.  Stores that another workgroup may read, and all stores
// to the sweep's output, are agent-scope (workgroups sit on several XCDs
// whose L2 caches are not coherent) and complete before the counter is
// touched.
//
// A workgroup without a tile waits for one to be queued, so that a burst of
// requests finds workgroups ready; surplus ones leave.  It waits only once
// every workgroup of the launch has started, and leaves otherwise: it holds a
// place on the chip, and one that has not started still owes its first visits.
// So a launch needs one place to end, however many the chip has left for it:
// the workgroup that starts last finds all started and drains the queue.
// What every workgroup shares is kept off the visits: with a ticket and a count
// of owed visits touched on each of them, one memory channel set the pace of
// the whole chip (8.8 instead of 6.2 ms per 1024x436 pair).  The words that
// count starts are sixteen for the same reason (eight pairs: 1 % slower with 32;
// SIFT 161x119: 1 % slower with one per 32 workgroups).
#pragma once

#include "ff_internal.h"

namespace ff {

constexpr int kTileH = 16, kTileW = 16;   // rows, columns
__host__ __device__ __forceinline__ int tiles_x(int Gw) { return (Gw + kTileH - 1 + kTileW - 1) / kTileW; }
__host__ __device__ __forceinline__ int tiles_y(int Gh) { return (Gh + kTileH - 1) / kTileH; }

constexpr int kRelaxIdle = 96;   // workgroups that wait for work, about: more only crowd the words they poll
constexpr int kRelaxStart = 16;  // words that count the workgroups started, block b on word b % 16

__device__ __forceinline__ uint64_t rt_clock() { return __builtin_amdgcn_s_memrealtime(); }

// global-address-space accesses throughout: a flat access also counts as an
// LDS operation and, while pending, turns a wait for some loads into a wait
// for all of them
template <class T>
__device__ __forceinline__ __attribute__((address_space(1))) T* gp(T* p) {
  return (__attribute__((address_space(1))) T*)p;
}
template <class T>
__device__ __forceinline__ T ld_coh(const T* p) {
  return __hip_atomic_load(gp(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <class T>
__device__ __forceinline__ void st_coh(T* p, T v) {
  __hip_atomic_store(gp(p), v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <class T>
__device__ __forceinline__ T add_coh(T* p, T v) {
  return __hip_atomic_fetch_add(gp(p), v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <class T>
__device__ __forceinline__ T swap_coh(T* p, T v) {
  return __hip_atomic_exchange(gp(p), v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// every memory operation of this wavefront before this point has completed
__device__ __forceinline__ void mem_wait() {
  __atomic_signal_fence(__ATOMIC_SEQ_CST);
  __builtin_amdgcn_s_waitcnt(0);
  __atomic_signal_fence(__ATOMIC_SEQ_CST);
}

// One launch's scheduler words, all zero before it, each in a line of its own
// (an operation on a word that every workgroup uses takes its turn at one
// memory channel); one wavefront per workgroup calls the functions below,
// every lane with the same arguments (the other wavefronts' memory operations
// have completed).
struct RelaxCtl {
  int32_t head, pad0[31];   // tickets drawn for queued tiles
  int32_t tail, pad1[31];   // tiles queued
  int32_t pend;             // (visits owed) - T; -T when the sweep has settled
  int32_t beat, pad2[30];   // raised by every kBeatVisits-th visit of a workgroup
  struct {
    int32_t n, pad[31];
  } started[kRelaxStart];
};
static_assert(sizeof(RelaxCtl) == (3 + kRelaxStart) * 128, "one line per word");
struct RelaxQ {
  RelaxCtl* ctl;
  int32_t* ring;       // queued tiles + 1, 0 where empty; empty again when the launch ends
  int cap;             // ring entries, >= tiles of any launch
  int T, G;            // tiles and workgroups of this launch (G <= T)
  int32_t* status;     // FF_ERR_DEVICE if the watchdog fired
  uint64_t timeout;    // its limit, in 10 ns ticks
};

// The watchdog: a waiting workgroup gives up when neither pend nor beat has
// changed for the limit.  pend changes when a workgroup waits or queues tiles;
// one that goes from tile to tile without either (its first visits, a chain of
// single revisits) raises beat every kBeatVisits of them.  So it fires on a
// sweep at work only if that many visits take longer than the limit.
constexpr int kBeatVisits = 32;

// A workgroup's own words.  done: visits it has answered for and not yet taken
// off the owed ones (one operation on the shared word per wait instead of one
// per visit).
struct RelaxWg {
  int mine;     // its first visits: tiles block, block + G, ..
  int done;
  int visits;
};
__device__ __forceinline__ RelaxWg relax_begin(const RelaxQ& q, int block) {
  if ((threadIdx.x & 63) == 0) add_coh(&q.ctl->started[block % kRelaxStart].n, 1);
  return {block, 0, 0};
}

// A queued tile to visit, or -1 to leave.
__device__ __forceinline__ int relax_wait(const RelaxQ& q, RelaxWg& w) {
  const int lane = threadIdx.x & 63;
  int old = 0;
  if (lane == 0) old = add_coh(&q.ctl->pend, -w.done);
  const int all = (q.G + kRelaxStart - 1 - lane) / kRelaxStart;   // workgroups counted on word `lane`
  const bool some = lane < kRelaxStart && ld_coh(&q.ctl->started[lane].n) < all;
  old = __builtin_amdgcn_readfirstlane(old);
  if (old - w.done == -q.T) return -1;
  w.done = 0;
  if (__ballot(some)) return -1;
  // enough workgroups wait already?
  const int h = __builtin_amdgcn_readfirstlane(ld_coh(&q.ctl->head));
  const int tl = __builtin_amdgcn_readfirstlane(ld_coh(&q.ctl->tail));
  if (h - tl >= kRelaxIdle) return -1;
  int pos = 0;
  if (lane == 0) pos = add_coh(&q.ctl->head, 1);
  pos = __builtin_amdgcn_readfirstlane(pos);
  int32_t* const slot = q.ring + pos % q.cap;
  uint64_t t0 = rt_clock();
  uint64_t last = ~0ull;
  for (int it = 0;; ++it) {
    if (__builtin_amdgcn_readfirstlane(ld_coh(slot)) != 0) {
      // tickets a ring apart share a slot: an entry is taken by whoever clears
      // it, and the other one waits on for the next
      int v = 0;
      if (lane == 0) v = swap_coh(slot, 0);
      const int st = ld_coh(q.status);
      v = __builtin_amdgcn_readfirstlane(v);
      // (an abandoned launch may leave entries behind)
      if (__builtin_amdgcn_readfirstlane(st) != 0) return -1;
      if (v != 0) return v - 1;
    }
    if ((it & 3) == 3) {
      const uint64_t pb = ld_coh(reinterpret_cast<const uint64_t*>(&q.ctl->pend));
      const int p = __builtin_amdgcn_readfirstlane((int)(uint32_t)pb);
      const int b = __builtin_amdgcn_readfirstlane((int)(uint32_t)(pb >> 32));
      if (p == -q.T || __builtin_amdgcn_readfirstlane(ld_coh(q.status)) != 0) return -1;
      const uint64_t seen = ((uint64_t)(uint32_t)b << 32) | (uint32_t)p;
      if (seen != last) {
        last = seen;
        t0 = rt_clock();
      } else if (rt_clock() - t0 > q.timeout) {
        if (lane == 0) st_coh(q.status, (int32_t)FF_ERR_DEVICE);
        return -1;
      }
    }
    __builtin_amdgcn_s_sleep(4);
  }
}

// End of a visit of tile `self` (counter words cnt[], tile numbers local to
// the field, the field's tiles starting at g0): its stores have completed.
// handled: requests the visit answered.  to_r / to_bl / to_b: whether border
// values that tile self + 1 / self + nu - 1 / self + nu reads have changed.
// Returns the next tile (global number) this workgroup owns, or -1; w.done is
// raised when the visit leaves nothing owed in its place.
__device__ __forceinline__ int relax_done(const RelaxQ& q, int32_t* cnt, int base, int self, int nu, int g0,
                                          int handled, bool to_r, bool to_bl, bool to_b, RelaxWg& w) {
  const int lane = threadIdx.x & 63;
  const bool on = lane == 0 || (lane == 1 && to_r) || (lane == 2 && to_b) || (lane == 3 && to_bl);
  const int tile = self + (lane == 1 ? 1 : lane == 2 ? nu : lane == 3 ? nu - 1 : 0);
  bool owned = false;
  if (on) {
    const int old = add_coh(cnt + tile, lane == 0 ? -handled : 1);
    owned = lane == 0 ? old - handled != base : old == base;
  }
  if (++w.visits % kBeatVisits == 0 && lane == 0) add_coh(&q.ctl->beat, 1);
  const uint64_t m = __ballot(owned);
  if (m == 0) {
    ++w.done;
    return -1;
  }
  const int first = __ffsll((unsigned long long)m) - 1;
  const uint64_t rest = m & (m - 1);
  if (rest) {
    // the visits are owed before anyone can make them
    const int k = __popcll(rest);
    int pos = 0;
    const int pay = k - w.done;   // what is owed less what was answered for
    w.done = 0;
    if (lane < 2) pos = add_coh(lane == 0 ? &q.ctl->tail : &q.ctl->pend, lane == 0 ? k : pay);
    mem_wait();
    pos = __builtin_amdgcn_readfirstlane(pos) + __popcll(rest & ((1ull << lane) - 1));
    if ((rest >> lane) & 1) {
      // an entry still there is one that a running workgroup holds a ticket
      // for and is about to take: no more than T tiles are queued at a time, so
      // later entries have been taken
      int32_t* const slot = q.ring + pos % q.cap;
      const uint64_t t0 = rt_clock();
      for (;;) {
        int32_t want = 0;
        if (__hip_atomic_compare_exchange_strong(gp(slot), &want, g0 + tile + 1, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                 __HIP_MEMORY_SCOPE_AGENT))
          break;
        if (ld_coh(q.status) != 0) break;
        if (rt_clock() - t0 > q.timeout) {
          st_coh(q.status, (int32_t)FF_ERR_DEVICE);
          break;
        }
        __builtin_amdgcn_s_sleep(1);
      }
    }
  }
  return g0 + __builtin_amdgcn_readlane(tile, first);
}

// The tile after a visit that left the workgroup with tile `next`, or none
// (-1): that one, its next first visit, or a queued tile; -1 to leave.  first:
// no earlier visit of the tile in this launch.
__device__ __forceinline__ int relax_next(const RelaxQ& q, RelaxWg& w, int next, bool& first) {
  first = false;
  if (next >= 0) return next;
  if (w.mine < q.T) {
    w.mine += q.G;
    first = w.mine < q.T;
  }
  return first ? w.mine : relax_wait(q, w);
}

// Border words: flow | cost | launch tag
__device__ __forceinline__ uint64_t xch_pack(int32_t f, int32_t cst, uint32_t tag) {
  const uint32_t c16 = cst == kInf ? 0xFFFFu : (uint32_t)cst;
  return (uint64_t)(uint32_t)f | ((uint64_t)(c16 | (tag << 16)) << 32);
}

}  // namespace ff
