// The tile relaxation's scheduler (csrc/ff_relax.h, this very header) run on
// the host: workgroups of one wavefront as fibers under a discrete-event
// simulation with a chosen number of places on the chip, random latencies,
// random stalls, on a small relaxation problem with a known solution.
//
//   relax_host NU NV G SLOTS SEED STALL VISIT TIMEOUT SLOW SHUFFLE
//
// NU x NV tiles; G workgroups, SLOTS of them on the chip at once, started in
// order of their number or (SHUFFLE) in any; of a million operations STALL are
// 500 times as long; a visit lasts VISIT ticks, tile 0's first one SLOW of
// them; TIMEOUT: the watchdog's limit in ticks.  Prints one line:
//   status S wrong W twice D left L visits V
// W: tiles whose value differs from the raster-order solution; D: visits that
// began while another one of the same tile ran; L: counters, queue entries or
// owed visits not back to rest.
#include <stdio.h>
#include <stdlib.h>
#include <algorithm>
#include <ucontext.h>

#include <memory>
#include <queue>
#include <random>
#include <vector>

#include "ff_relax.h"

namespace {
constexpr int kLanes = 16;      // of a wavefront, enough for everything the scheduler does
constexpr size_t kStack = 1 << 15;
enum State { kReady, kCollective, kMemory, kDone };

struct Lane {
  ucontext_t ctx;
  std::unique_ptr<char[]> stack;
  State st = kReady;
  uint64_t value = 0;
};
struct Wg {
  Lane l[kLanes];
  uint64_t got[kLanes];
  int block = 0;
  uint64_t latency = 0;
};

std::mt19937_64 rng;
uint64_t now;
int stall;
ucontext_t home;
Wg* wg;
int lane_now;

void leave(State st) {
  Lane& l = wg->l[lane_now];
  l.st = st;
  swapcontext(&l.ctx, &home);
}
void wait(uint64_t ticks) {
  if ((int)(rng() % 1000000) < stall) ticks *= 500;
  if (ticks > wg->latency) wg->latency = ticks;
  leave(kMemory);
}
}  // namespace

namespace sim {
Idx thread_idx() { return {(unsigned)lane_now}; }
uint64_t collective(uint64_t v, int lane) {
  wg->l[lane_now].value = v;
  leave(kCollective);
  if (lane >= 0) return wg->got[lane];
  uint64_t m = 0;
  for (int i = 0; i < kLanes; ++i) m |= wg->got[i] ? 1ull << i : 0;
  return m;
}
void memory() { wait(60 + rng() % 60); }
void sleep(int n) { wait(1 + 3 * n); }
uint64_t clock() { return now; }
}  // namespace sim

namespace {
// the problem: every tile takes the least of its own value and of its left,
// lower-left-above and upper neighbour's plus a weight
struct Problem {
  int nu, nv, T, visit, slow;
  std::vector<int> own, val, cnt, ring, busy, wl, wd, wu;
  std::vector<uint64_t> word;
  std::vector<uint8_t> seen;
  ff::RelaxCtl ctl{};
  int32_t status = 0;
  ff::RelaxQ q{};
  long visits = 0, twice = 0;
} P;

int solve(int t, int l, int d, int u) {
  int v = P.own[t];
  if (t % P.nu > 0 && l + P.wl[t] < v) v = l + P.wl[t];
  if (t >= P.nu && t % P.nu + 1 < P.nu && d + P.wd[t] < v) v = d + P.wd[t];
  if (t >= P.nu && u + P.wu[t] < v) v = u + P.wu[t];
  return v;
}

// as the sweeps' visits: counter, borders, work, results, words, requests
int visit(int t, bool first, ff::RelaxWg& w) {
  using namespace ff;
  const int lane = threadIdx.x, base = -1;
  const int handled = __builtin_amdgcn_readfirstlane(ld_coh(&P.cnt[t]) - base);
  int changed = 0;
  if (lane == 0) {
    ++P.visits;
    if (P.busy[t]++) ++P.twice;
    auto border = [&](int nb) {
      const uint64_t w = ld_coh(&P.word[nb]);
      return w ? (int)(uint32_t)w : P.own[nb];
    };
    int l = 0, d = 0, u = 0;
    if (t % P.nu > 0) l = border(t - 1);
    if (t >= P.nu && t % P.nu + 1 < P.nu) d = border(t - P.nu + 1);
    if (t >= P.nu) u = border(t - P.nu);
    const int was = first ? P.own[t] : P.val[t];
    wait((uint64_t)P.visit * (t == 0 && first ? P.slow : 1));
    P.val[t] = solve(t, l, d, u);
    changed = P.val[t] != was;
    if (changed) st_coh(&P.word[t], (uint64_t)1 << 32 | (uint32_t)P.val[t]);
    --P.busy[t];
  }
  changed = __builtin_amdgcn_readfirstlane(changed);
  const bool right = t % P.nu + 1 < P.nu, down = t + P.nu < P.T;
  return relax_done(P.q, P.cnt.data(), base, t, P.nu, 0, handled, changed && right, changed && down && t % P.nu > 0,
                    changed && down, w);
}

void lane_main() {
  using namespace ff;
  RelaxWg w = relax_begin(P.q, wg->block);
  int gt = w.mine;
  bool first = true;
  do gt = relax_next(P.q, w, visit(gt, first, w), first);
  while (gt >= 0);
  leave(kDone);
}

void start(Wg& w) {
  for (Lane& l : w.l) {
    l.st = kReady;
    if (!l.stack) l.stack.reset(new char[kStack]);
    getcontext(&l.ctx);
    l.ctx.uc_stack.ss_sp = l.stack.get();
    l.ctx.uc_stack.ss_size = kStack;
    l.ctx.uc_link = &home;
    makecontext(&l.ctx, lane_main, 0);
  }
}

// runs w until it waits for memory; false: it has ended
bool step(Wg& w) {
  wg = &w;
  w.latency = 0;
  for (;;) {
    int waiting = 0, ended = 0;
    for (lane_now = 0; lane_now < kLanes; ++lane_now) {
      Lane& l = w.l[lane_now];
      if (l.st == kReady) swapcontext(&home, &l.ctx);
      waiting += l.st == kMemory;
      ended += l.st == kDone;
    }
    if (ended == kLanes) return false;
    if (waiting) {
      for (Lane& l : w.l)
        if (l.st == kMemory) l.st = kReady;
      return true;
    }
    for (int i = 0; i < kLanes; ++i) {
      w.got[i] = w.l[i].value;
      if (w.l[i].st != kCollective) {
        printf("lanes apart\n");
        exit(2);
      }
      w.l[i].st = kReady;
    }
  }
}
}  // namespace

int main(int argc, char** argv) {
  if (argc != 11) return 2;
  int a[11];
  for (int i = 1; i < 11; ++i) a[i] = atoi(argv[i]);
  P.nu = a[1];
  P.nv = a[2];
  P.T = P.nu * P.nv;
  const int G = std::min(a[3], P.T), slots = a[4];
  rng.seed(a[5]);
  stall = a[6];
  P.visit = a[7];
  P.slow = a[9];
  for (int t = 0; t < P.T; ++t) {
    P.own.push_back(t == 0 ? 0 : (int)(rng() % 400));
    P.wl.push_back((int)(rng() % (P.nv == 1 ? 1 : 60)));
    P.wd.push_back((int)(rng() % 60));
    P.wu.push_back((int)(rng() % 60));
  }
  P.val = P.own;
  P.cnt.assign(P.T, 0);
  P.busy.assign(P.T, 0);
  P.ring.assign(P.T, 0);
  P.word.assign(P.T, 0);
  P.q.ctl = &P.ctl;
  P.q.ring = P.ring.data();
  P.q.cap = P.q.T = P.T;
  P.q.G = G;
  P.q.status = &P.status;
  P.q.timeout = (uint64_t)a[8];

  std::vector<int> order(G);
  for (int i = 0; i < G; ++i) order[i] = i;
  if (a[10])
    for (int i = G - 1; i > 0; --i) std::swap(order[i], order[rng() % (i + 1)]);
  std::vector<std::unique_ptr<Wg>> chip;
  typedef std::pair<uint64_t, int> Event;   // time, place
  std::priority_queue<Event, std::vector<Event>, std::greater<Event>> events;
  int next = 0;
  for (; next < std::min(G, slots); ++next) {
    chip.emplace_back(new Wg);
    chip.back()->block = order[next];
    start(*chip.back());
    events.push({(uint64_t)next, next});
  }
  while (!events.empty()) {
    const Event e = events.top();
    events.pop();
    now = e.first;
    Wg& w = *chip[e.second];
    if (step(w)) {
      events.push({now + w.latency, e.second});
    } else if (next < G) {
      w.block = order[next++];
      start(w);
      events.push({now + 10, e.second});
    }
  }
  long wrong = 0, left = P.ctl.pend != -P.T;
  std::vector<int> ref(P.T);
  for (int t = 0; t < P.T; ++t) {
    ref[t] = solve(t, t > 0 ? ref[t - 1] : 0, t >= P.nu ? ref[t - P.nu + 1] : 0, t >= P.nu ? ref[t - P.nu] : 0);
    wrong += ref[t] != P.val[t];
    left += (P.cnt[t] != -1) + (P.ring[t] != 0);
  }
  printf("status %d wrong %ld twice %ld left %ld visits %ld\n", P.status, wrong, P.twice, left, P.visits);
  return 0;
}
