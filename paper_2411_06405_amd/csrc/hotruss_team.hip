// hotruss_team.hip -- rounds run by one team of workgroups inside one launch.
//
// Most peel rounds are small: on Chung-Lu and R-MAT graphs the median round
// peels under ten edges, and run as four kernels over the whole chip it takes
// about 35 us of which nearly all is launch gaps, cold caches (every kernel
// boundary drops the L2 contents other XCDs may have changed) and dependent
// loads from HBM.  A team is the workgroups of one slot that sit on one XCD:
// they share that XCD's L2, so they can meet at a barrier of 0.7 us (32
// workgroups of 1,024 threads: one flag word each, all polled together; 29 us
// with a device-scope fence per wave, 20 us over the whole chip) and hand each
// other data through the L2 (85 ns a dependent load) without any fence.  A
// team runs rounds back to back until one of its steps is large enough for
// the whole chip; it then leaves that step, and the rest of the round, to the
// round kernels that follow in the same graph.
//
// A team's round takes 15 to 25 us on such graphs (Chung-Lu 100k h = 2: level
// scan 3.4 over all rounds, of which 38% begin with one, marking 2.6, ball change
// 7, support update 5.3, barriers 5), bound by the chain of dependent accesses,
// now to the L2.  Before and after, ms a call: uniform random 200 h = 2 1.8 and
// 1.2 to 1.5; Chung-Lu 5,001 h = 3 194 and 114; 32 clique-planted graphs in one
// batch 216 and 116; a session of 24 mixed requests 306 and 166 to 175; without
// allocations, where the host had to look at every round, Chung-Lu 1,500 h = 2
// 44.6 and 8.7.  One graph whose rounds are mostly large gains nothing from it
// (R-MAT 16 h = 2: 1,237 by teams alone, 987 by the chip); which of the two runs
// is decided by their progress (see Pace).
//
// What makes it safe:
//  * A team is whoever arrived: its workgroups join by a counter, the first
//    one closes it after a bounded wait, and late ones return, as do those
//    that come to a full team (TEAM_MAX).  Every member
//    is running when the team starts, so a barrier never waits for a
//    workgroup that has yet to be scheduled, whatever else shares the GPU.
//  * Members check that they are on the same XCD (XCC_ID register).
//  * Words that other members write are read with ld<true>() (device-scope
//    relaxed loads, served by the L2), stores and atomics are complete in the
//    L2 before the writer's barrier flag is (s_waitcnt).
//  * Every counter that a step accumulates exists per round parity, so that
//    it can be reset while no member reads or adds to it.
//  * Every wait is bounded; one that runs out ends the decomposition with an
//    internal error.
#include "hotruss_dev.h"

namespace hotruss {

constexpr uint32_t TEAM_THREADS = 1024, TEAM_CAP = 2048, TEAM_WAVES = TEAM_THREADS / WAVE;
constexpr uint32_t TEAM_JOIN_POLLS = 256;       // about 20 us
constexpr uint32_t TEAM_SPIN = 1u << 24;        // over a second: only a fault gets there

// Up to where a team takes a step; beyond, the whole chip is faster.  One graph:
// 1,024 ball-change items and 16,384 support items (Chung-Lu 100k h = 2, with
// half, once, twice and 16 times that: 229, 213, 218, 247 ms; BA 12,345: 19.9,
// 19.4, 19.9, 20.5).  Several graphs share the chip and wait for each other's
// large steps, so their teams go on longer: 4,096 and 32,768 (32 graphs in a
// batch, with an eighth, a quarter, once and four times that: 130, 120, 108,
// 106 ms; a session of 24: 184, 178, 172, 181).
struct TeamLimits {
  uint32_t rounds;   // rounds per launch (the host looks in between)
  uint32_t peeled;   // edges peeled by one round; 0: none, the chip runs all rounds
  uint32_t items;    // work items of one ball-change level
  uint32_t support;  // work items of one support update
};

__global__ void k_team_reset(const Dev* __restrict__ dp) { reset_team(*dp); }

// The slots that have rounds to run (more than one slot).
__global__ void __launch_bounds__(1024) k_team_plan(const Dev* __restrict__ devs, uint32_t S,
                                                    uint32_t* __restrict__ plan) {
  __shared__ uint32_t s_w[TEAM_WAVES], s_run;
  if (threadIdx.x == 0) s_run = 0;
  __syncthreads();
  for (uint32_t base = 0; base < S; base += 1024) {
    const uint32_t i = base + threadIdx.x;
    bool act = false;
    if (i < S) {
      const Ctl* c = devs[i].ctl;
      act = !c->done && !c->halt && !c->err;
    }
    const uint64_t b = __ballot(act);
    if (lane_id() == 0) s_w[threadIdx.x / WAVE] = (uint32_t)__popcll(b);
    __syncthreads();
    uint32_t at = s_run;
    for (uint32_t w = 0; w < threadIdx.x / WAVE; ++w) at += s_w[w];
    at += (uint32_t)__popcll(b & ((1ull << lane_id()) - 1));
    if (act) plan[1 + at] = i;
    __syncthreads();
    if (threadIdx.x == 0)
      for (uint32_t w = 0; w < TEAM_WAVES; ++w) s_run += s_w[w];
    __syncthreads();
  }
  if (threadIdx.x == 0) plan[0] = s_run;
}

struct TeamLds {
  uint32_t me, n, ok;
  uint32_t mn[TEAM_WAVES], cn[TEAM_WAVES], at;
};

__device__ __forceinline__ uint32_t xcc_id() {
  return __builtin_amdgcn_s_getreg(20 | (31 << 11)) & 15u;  // HW_REG_XCC_ID
}

// Join the team of a slot; false: too late, on another XCD, or failed.
__device__ bool team_join(Team* t, uint32_t expected, TeamLds& s) {
  if (threadIdx.x == 0) {
    uint32_t n = 0, me = 0;
    const uint32_t x = xcc_id() + 1, first = atomicCAS(&t->xcc, 0u, x);
    if (first == 0 || first == x) {
      me = atomicAdd(&t->joined, 1u);
      if (me == 0) {
        for (uint32_t i = 0; i < TEAM_JOIN_POLLS && ld<true>(&t->joined) < expected; ++i) {}
        n = team_size(atomicExch(&t->joined, TEAM_CLOSED));
        __hip_atomic_store(&t->size, n, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      } else if (team_admits(me)) {  // not after TEAM_CLOSED, nor once the team is full
        for (uint32_t i = 0; i < TEAM_SPIN && !n; ++i) n = ld<true>(&t->size);
      }
    }
    s.me = me;
    s.n = n;
  }
  __syncthreads();
  return s.n != 0;
}

// All members reach barrier `ep`; everything they wrote before it is in the
// L2 when it returns.  false: a member did not come (all give up).
__device__ bool team_barrier(Team* t, uint32_t me, uint32_t n, uint32_t ep, TeamLds& s) {
  asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
  __syncthreads();
  if (n == 1) return true;
  if (threadIdx.x < WAVE) {
    if (threadIdx.x == 0)
      __hip_atomic_store(&t->flag[me], ep, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    bool all = false;
    for (uint32_t i = 0; i < TEAM_SPIN && !all; ++i)
      all = __ballot(threadIdx.x < n && ld<true>(&t->flag[threadIdx.x]) < ep) == 0;
    if (threadIdx.x == 0) s.ok = all;
  }
  __syncthreads();
  return s.ok != 0;
}

// Smallest live support of the member's edges and how many have it; mine:
// this thread's own minimum.
__device__ void team_scan(const Dev& d, uint32_t me, uint32_t n, TeamLds& s, uint32_t* mine) {
  const uint32_t stride = n * TEAM_THREADS;
  uint32_t e = me * TEAM_THREADS + threadIdx.x, mn = SUP_GONE, cn = 0;
  auto take = [&](uint32_t v) {
    if (v < mn) {
      mn = v;
      cn = 0;
    }
    cn += v == mn;
  };
  for (; e + 7 * stride < d.m; e += 8 * stride) {
    uint32_t v[8];
#pragma unroll
    for (uint32_t u = 0; u < 8; ++u) v[u] = ld<true>(d.sup + e + u * stride);
#pragma unroll
    for (uint32_t u = 0; u < 8; ++u) take(v[u]);
  }
  for (; e < d.m; e += stride) take(ld<true>(d.sup + e));
  *mine = mn;
  const uint32_t wm = wave_min(mn), wc = wave_sum(mn == wm ? cn : 0u);
  if (lane_id() == 0) {
    s.mn[threadIdx.x / WAVE] = wm;
    s.cn[threadIdx.x / WAVE] = wc;
  }
  __syncthreads();
  if (threadIdx.x < WAVE) {
    const uint32_t m = lane_id() < TEAM_WAVES ? s.mn[lane_id()] : SUP_GONE;
    const uint32_t gm = wave_min(m);
    const uint32_t gc = wave_sum(lane_id() < TEAM_WAVES && m == gm ? s.cn[lane_id()] : 0u);
    if (lane_id() == 0) {
      d.team->smin[me] = gm;
      d.team->scnt[me] = gc;
    }
  }
}

// List the member's edges whose support is mn in R, from s.at on.
__device__ void team_collect(const Dev& d, uint32_t p, uint32_t mn, uint32_t mine, uint32_t me,
                             uint32_t n, TeamLds& s) {
  if (!__ballot(mine == mn)) return;  // none in this wave's edges
  const uint32_t stride = n * TEAM_THREADS;
  for (uint32_t b = me * TEAM_THREADS + (threadIdx.x & ~(WAVE - 1)); b < d.m; b += stride) {
    const uint32_t e = b + lane_id();
    const bool take = mine == mn && e < d.m && ld<true>(d.sup + e) == mn;
    if (!__ballot(take)) continue;
    const uint32_t i = wave_reserve<true>(&s.at, take ? 1u : 0u);
    if (take) d.R[p][i] = e;
  }
}

__device__ __forceinline__ uint64_t* cnt_items(Ctl* c, uint32_t j, uint32_t p) {
  return reinterpret_cast<uint64_t*>(&c->cnt[j][p].nit);  // nit, iovf
}
__device__ __forceinline__ uint64_t* cnt_events(Ctl* c, uint32_t j, uint32_t p) {
  return reinterpret_cast<uint64_t*>(&c->cnt[j][p].nev);  // nev, ovf
}

// Counters of one parity back to zero (one wave).
__device__ __forceinline__ void team_reset_lists(Ctl* c, uint32_t h, uint32_t q, uint32_t lane) {
  if (lane >= 1 && lane <= h + 1) {
    __hip_atomic_store(cnt_items(c, lane, q), 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    __hip_atomic_store(cnt_events(c, lane, q), 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  }
  if (lane == 0) c->nPushc[q].v = 0;
}

__device__ void team_run(const Dev& d, uint32_t me, uint32_t n, const TeamLimits& lim,
                         LevelLds<TEAM_THREADS, TEAM_CAP>& lv, TeamLds& s) {
  Ctl* c = d.ctl;
  Team* t = d.team;
  uint32_t r = c->r, k = c->k, nR = c->nRc.v, live = c->live, compact_at = c->compact_at;
  bool jump = c->jump != 0;
  const bool leader = me == 0;
  const uint32_t tid = threadIdx.x, wave = tid / WAVE, lane = lane_id();
  const uint32_t nthreads = n * TEAM_THREADS, nwaves = n * TEAM_WAVES;
  const uint32_t wid = wave * n + me;  // wave in the team, workgroups first
  uint32_t ep = 0, rounds = 0, levels = 0, compactions = 0, overflows = 0, phase = c->phase;
  // book-keeping: the first member's last wave, which has the least else to do
  const bool book = leader && wave == TEAM_WAVES - 1;
  uint64_t events = 0;  // lane j has level j's
  bool done = false;
#define TEAM_BARRIER()                        \
  do {                                        \
    if (!team_barrier(t, me, n, ++ep, s)) {   \
      if (tid == 0) {                         \
        c->failed = 1;                        \
        c->done = 1;                          \
        d.status[0] = 3;                      \
      }                                       \
      return;                                 \
    }                                         \
  } while (0)
  TEAM_BARRIER();  // every member has read the state above
  bool resume = phase != ROUND_CLOSED;  // the round kernels have run the rest of a round
  if (resume && phase == 0) {
    if (book) {
      team_reset_lists(c, d.h, (r & 1) ^ 1, lane);
      if (lane == 0) c->cnt[1][r & 1].nev = 2 * nR;
    }
    TEAM_BARRIER();
  }
  while (true) {
    const uint32_t p = r & 1, q = p ^ 1;
    bool last = nR == live;  // the round that peels every remaining edge updates nothing
    if (!resume) {
      // the previous round's event lists, lane j level j's; marks of a level
      // whose list overflowed are cleared by the whole chip
      uint64_t prev = 0;
      if (lane >= 1 && lane <= d.h) prev = ld<true>(cnt_events(c, lane, q));
      phase = ROUND_CLOSED;
      if (rounds >= lim.rounds) break;
      // (testing: steps that are forced through the round kernels)
      const bool whole = __ballot((prev >> 32) != 0) || (d.serial & 12u);
      if (!whole && lim.peeled && (live <= compact_at || (d.serial & 16u))) {
        compact_rows<true>(d, wid, nwaves);
        compact_at = compact_next(live);
        ++compactions;
        TEAM_BARRIER();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");  // rows are read through the L1
      }
      if (jump) {
        // level jump: the minimum of the live supports, and the edges at it
        uint32_t mine;
        team_scan(d, me, n, s, &mine);
        TEAM_BARRIER();
        const uint32_t v = lane < n ? ld<true>(&t->smin[lane]) : SUP_GONE;
        const uint32_t mn = wave_min(v);
        uint32_t total;
        const uint32_t before = wave_excl_scan(lane < n && v == mn ? ld<true>(&t->scnt[lane]) : 0u,
                                               &total);
        if (whole || total > lim.peeled) {
          if (leader)
            for (uint32_t i = tid; i < d.nminpart; i += TEAM_THREADS) d.minpart[i] = mn;
          nR = 0;
          phase = 0;
          break;
        }
        k = mn + 2;
        nR = total;
        ++levels;
        const uint32_t at = __shfl(before, me, WAVE);
        if (tid == 0) s.at = at;
        __syncthreads();
        team_collect(d, p, mn, mine, me, n, s);
        TEAM_BARRIER();
      } else if (whole || nR > lim.peeled) {
        phase = 0;
        break;
      }
      const RoundCtx rc{r, k, p, nR};
      const uint32_t* R = d.R[p];
      // one edge per wavefront, dealt to workgroups first; in large rounds one
      // per lane
      if (nR <= 4 * nwaves) {
        for (uint32_t i = wid; i < nR; i += nwaves) mark_edge_wave<true>(d, rc, ld<true>(R + i), i);
      } else {
        for (uint32_t b = wid * WAVE; b < nR; b += nthreads) {
          const uint32_t i = b + lane;
          mark_edge<true>(d, rc, i < nR, i < nR ? ld<true>(R + i) : 0u, i);
        }
      }
      // clear the previous round's marks, from the waves that marked no edge on
      for (uint32_t j = d.h == 1 ? 1 : 2; j <= d.h; ++j)
        clear_marks<true>(d, j, q, (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)prev, (int)j),
                          (nwaves - 1 - wid) * WAVE + lane, nthreads);
      TEAM_BARRIER();
      if (book) {
        team_reset_lists(c, d.h, q, lane);  // the previous round's lists are read
        if (lane == 0) c->cnt[1][p].nev = 2 * nR;  // both directions of every peeled edge
      }
      last = nR == live;
      uint32_t step = 2;
      for (; !last && step <= d.h; ++step) {
        const uint64_t w = ld<true>(cnt_items(c, step, p));
        const uint32_t ni = (uint32_t)w;
        if (w >> 32 || ni > lim.items) break;
        level_step<TEAM_THREADS, TEAM_CAP, true>(d, rc, step, ni, me, n, lv);
        TEAM_BARRIER();
      }
      if (!last && step <= d.h) {
        phase = step;
        break;
      }
      if (!last) {
        const uint64_t w = ld<true>(cnt_items(c, d.h + 1, p));
        const uint32_t ni = (uint32_t)w;
        if (w >> 32 || ni > lim.support) {
          phase = d.h + 1;
          break;
        }
        support_step<true, 2>(d, rc, ni, me, n, TEAM_WAVES, nullptr);
        TEAM_BARRIER();
      }
    }
    resume = false;
    // close the round
    const uint32_t pushed = last ? 0u : ld<true>(&c->nPushc[p].v);
    if (book) {
      const bool level = lane >= 1 && lane <= d.h + 1;
      const uint64_t w = level ? ld<true>(cnt_events(c, lane, p)) : 0;
      const uint64_t i = level ? ld<true>(cnt_items(c, lane, p)) : 0;
      events += lane == 1 ? 2 * nR : (uint32_t)w;
      overflows += __ballot(((w | i) >> 32) != 0) != 0;
    }
    live -= nR;
    ++r;
    ++rounds;
    jump = pushed == 0;
    nR = pushed;
    phase = ROUND_CLOSED;
    if (live == 0) {
      done = true;
      break;
    }
  }
#undef TEAM_BARRIER
  if (!book) return;
  if (lane >= 1 && lane <= d.h) c->levents[lane] += events;
  const uint64_t top = __shfl(events, d.h, WAVE);
  if (lane == 0) {
    c->r = r;
    c->k = k;
    c->nRc.v = nR;
    c->live = live;
    c->jump = jump;
    c->phase = phase;
    c->compact_at = compact_at;
    c->levels += levels;
    c->compactions += compactions;
    c->overflows += overflows;
    c->events += top;
    d.status[2] = live;
    d.status[3] = r;
    if (done) {
      c->done = 1;
      d.status[0] = 1;
    }
  }
}

// One workgroup per CU (its registers leave room for no second one; nothing but
// speed depends on it).  Workgroups are dealt to the XCDs in turn, so block b is
// taken to be on XCD b mod 8; the slots of an XCD share its workgroups evenly
// (fewer than eight slots: the first XCD with a free CU takes a slot, and the
// others' workgroups return).
__global__ void __launch_bounds__(TEAM_THREADS) k_team(const Dev* __restrict__ devs,
                                                       const uint32_t* __restrict__ plan,
                                                       TeamLimits lim) {
  __shared__ LevelLds<TEAM_THREADS, TEAM_CAP> lv;
  __shared__ TeamLds s;
  const uint32_t A = plan ? plan[0] : 1;
  if (!A) return;
  for (uint32_t i = threadIdx.x; i < TEAM_CAP; i += TEAM_THREADS) lv.flag[i] = 0;
  const uint32_t xcd = blockIdx.x & 7, i = blockIdx.x >> 3, per = gridDim.x >> 3;
  const uint32_t nx = A >= 8 ? (A - xcd + 7) / 8 : 1;  // slots of this XCD
  const uint32_t share = min(nx, per);
  for (uint32_t a = i % share; a < nx; a += share < nx ? per : nx) {
    const Dev& d = devs[plan ? plan[1 + (A >= 8 ? xcd + 8 * a : xcd % A)] : 0];
    if (!plan && (d.ctl->done || d.ctl->halt || d.ctl->err)) return;
    __syncthreads();
    if (team_join(d.team, share < nx ? 1u : (per - a + nx - 1) / nx, s))
      team_run(d, s.me, s.n, lim, lv, s);
  }
}

}  // namespace hotruss
