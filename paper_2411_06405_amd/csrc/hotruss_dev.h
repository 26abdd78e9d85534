// hotruss_dev.h -- device-side state and helpers shared by the libhotruss
// kernels (gfx950, wave64).  Internal header of the GPU library.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

// The team kernel (hotruss_team.hip) hands data from workgroup to workgroup of
// one XCD by what this chip does and HIP's memory model does not promise: loads
// of device scope are served by the XCD's L2, stores and atomics of workgroup
// scope are complete there after s_waitcnt vmcnt(0), and XCC_ID names the XCD.
// On another chip each of these has to be looked at first.
#if defined(__HIP_DEVICE_COMPILE__) && !defined(__gfx950__)
#error "hotruss is written for gfx950: see the team kernel's use of the L2"
#endif

namespace hotruss {

constexpr uint32_t HMAX = 16;            // largest hop threshold with its own ball level
constexpr uint32_t ALIVE = 0xffffffffu;  // srem value of a slot whose edge is still in S
constexpr uint32_t SUP_GONE = 0xffffffffu;   // sup value of a peeled edge
constexpr uint32_t SLOT_GONE = 0x80000000u;  // in the low word of ce: the slot's edge is peeled
constexpr int WAVE = 64;
constexpr uint32_t CHUNK = 64;           // slots (or bitset words) per work item
constexpr uint32_t MIN_PART = 1024;      // partial-minimum slots of the level-jump reduction
constexpr uint32_t DEG_BUCKETS = 256;    // degree classes of the renumbering
constexpr uint32_t NSTAT = 8;            // work counters kept in stats mode
constexpr uint32_t STAT_GRID = 6144;     // most workgroups a counted kernel may use

// error bits in Ctl::err (set by the validation kernels)
constexpr uint32_t ERR_ROWPTR = 1u, ERR_COL = 2u, ERR_ORDER = 4u, ERR_LOOP = 8u,
                   ERR_ASYM = 16u, ERR_COUNT = 32u;

// Work item kinds.  A work item covers at most CHUNK consecutive CSR slots
// (or bitset words) of one vertex, so that a wavefront handles it in one step.
//   KIND_A_SLOTS  level j = 2, x lost its neighbour z:   candidates (x, y), y in the
//                 old neighbourhood of z (slots with srem >= r); extra: (x, z)
//   KIND_A_WORDS  level j >= 3, x lost its neighbour z:  candidates (x, w), w in z's
//                 old (j-1)-ball (bitset words [base, base+len))
//   KIND_B_SLOTS  w left z's (j-1)-ball: candidates (y, w), y a live neighbour of z
//                 (slots with srem > r); extra: (z, w)
// Item = {x, y, base, meta}: meta = kind << 30 | extra << 29 | len << 22 | vstart.
constexpr uint32_t KIND_A_SLOTS = 0, KIND_A_WORDS = 1, KIND_B_SLOTS = 2;

struct Item {
  uint32_t x, y, base, meta;
};

__host__ __device__ inline uint32_t item_meta(uint32_t kind, uint32_t extra, uint32_t len,
                                              uint32_t vstart) {
  return (kind << 30) | (extra << 29) | (len << 22) | vstart;
}
__device__ inline uint32_t meta_kind(uint32_t m) { return m >> 30; }
__device__ inline uint32_t meta_extra(uint32_t m) { return (m >> 29) & 1u; }
__device__ inline uint32_t meta_len(uint32_t m) { return (m >> 22) & 127u; }
__device__ inline uint32_t meta_vstart(uint32_t m) { return m & ((1u << 22) - 1); }

// List lengths of one level in a round of one parity.  Items and events have a
// cache line each, and so have the other counters that many wavefronts add to:
// device-scope atomics on one line serialise at about 11 ns each (with the
// peel-set and item counters on one line, the first marking of Chung-Lu 100k
// h = 1 took 690 us instead of 275).
struct alignas(128) Cnt {
  uint32_t nit;   // work items (level h+1: support items)
  uint32_t iovf;  // work item list overflowed
  alignas(128) uint32_t nev;  // ball-change events
  uint32_t ovf;   // event list overflowed
};

struct alignas(128) LineCounter {
  uint32_t v;
};

// Device control block: the whole round state lives on the device so that
// the round driver never needs the host between rounds.
struct Ctl {
  uint32_t err;
  uint32_t nact;     // rows in use: vertices from nact on are isolated (renumbered graphs)
  uint32_t words;    // words of a bitset row that can hold a vertex below nact (even)
  uint32_t nlong;    // renumbered graphs: rows of 64 slots or more (they come first)
  uint32_t k;        // current level: edges with sup <= k-2 are peeled
  uint32_t r;        // index of the current peel round
  uint32_t phase;    // first step of this round that the round kernels run: 0 mark, j level
                     // j, h+1 support; ROUND_CLOSED: none, the round has not begun
  uint32_t compact_at;  // compact the adjacency rows once live falls to this
  uint32_t live;     // edges still in S
  uint32_t levels;   // levels visited
  uint32_t done;     // decomposition finished (read by the host with halt)
  uint32_t halt;     // a work list overflowed: the host re-runs the step in windows
  uint32_t halt_step;  // step that halted: level j (2..h), or h+1 for the support update
  uint32_t jump;     // this round starts with a level jump
  // A support query keeps the words up to here, and on a renumbered graph the
  // buckets; the rest is the rounds' (see ctl_bytes).
  uint32_t bucket[DEG_BUCKETS];  // vertices per degree bucket, then where each starts
  uint64_t events;   // top-level ball-change events (statistics)
  uint64_t overflows;
  Cnt cnt[HMAX + 2][2];  // per level (h+1: support items) and round parity
  LineCounter nRc;       // |R_r|, edges peeled in the current round
  LineCounter nPushc[2];          // edges whose support crossed k-2 in a round of this parity
  uint32_t compactions;  // adjacency compactions done (statistics)
  uint32_t failed;       // a wait of the team kernel ran out: the decomposition is abandoned
  uint32_t recovering;   // the host is re-running an overflowed step in windows
  // stats mode: method-level work count (support evaluations and bytes of the
  // re-evaluating peeling method on the same round schedule)
  uint32_t acct_nch;     // vertices whose h-ball changed this round (listed)
  uint32_t acct_nv;      // ball builds of this round (listed)
  uint32_t acct_incomplete;  // an event list overflowed: the count is a lower bound
  uint64_t acct_evals;
  uint64_t acct_bytes;
  uint64_t levents[HMAX + 1];  // ball-change events per level, all rounds
  // stats mode: work counters, level kernel [0..5), support kernel [5..8)
  uint64_t stat[NSTAT];
};

// Bytes of a control block: of a decomposition (full), or of the initial pass.
constexpr __host__ __device__ size_t ctl_bytes(bool full, bool renumber) {
  return full ? sizeof(Ctl) : renumber ? offsetof(Ctl, events) : offsetof(Ctl, bucket);
}

constexpr uint32_t ROUND_CLOSED = 0xffu;

// Where the workgroups of one slot's team (see k_team) meet.  Zeroed between
// launches of the team kernel.
constexpr uint32_t TEAM_MAX = 64;
struct alignas(128) Team {
  uint32_t xcc;     // 1 + the XCD of the team (0: unclaimed)
  uint32_t joined;  // members so far; from TEAM_CLOSED on, too late
  uint32_t size;    // members, once closed
  uint32_t pad[29];
  uint32_t flag[TEAM_MAX];  // per member: the last barrier it reached
  uint32_t smin[TEAM_MAX];  // per member: level-jump minimum of its edges ...
  uint32_t scnt[TEAM_MAX];  // ... and how many of them have it
};
constexpr uint32_t TEAM_CLOSED = 1u << 16;

// Arrivals at a team are numbered from 0.  The launch and the dealing of its
// workgroups keep them at about 32; a team has room for TEAM_MAX whoever
// comes, so the bound does not rest on them.
constexpr __host__ __device__ bool team_admits(uint32_t arrival) { return arrival < TEAM_MAX; }
constexpr __host__ __device__ uint32_t team_size(uint32_t arrivals) {
  return arrivals < TEAM_MAX ? arrivals : TEAM_MAX;
}

// Everything a kernel needs, passed by value.
struct Dev {
  const uint32_t* orp;  // the caller's row_ptr [n+1]
  const uint32_t* oci;  // the caller's col_idx [2m]
  // The adjacency that everything after the validation works on: the
  // caller's, or (perm set) the same graph with its vertices renumbered by
  // descending degree.
  const uint32_t* rp;   // row_ptr [n+1]
  const uint32_t* ci;   // col_idx [2m] (as built; see cix)
  uint32_t* perm;       // renumbering: caller's vertex -> vertex [n], or null
  uint32_t* inv;        // ... and back [n]
  // Renumbered graphs have their own edge numbers too (see place_slot): own
  // number -> caller's [m], and back.  The outputs are written by the caller's.
  uint32_t* oe;
  uint32_t* ne;
  uint32_t n, m, h, W;  // W: 64-bit words per bitset row (padded)
  uint32_t nnz;
  uint32_t evcap;       // capacity of each level>=2 event list
  uint32_t itcap;       // capacity of each work item list
  uint32_t nminpart;    // blocks of the level-jump minimum kernel
  uint32_t serial;      // testing: bit 2 forces the windowed re-run of every level step,
                        // bit 3 of every support step, bit 4 compacts rows at every chance
  uint32_t* eid;        // caller's slot -> edge id   [2m]
  uint32_t* eu;         // edge id -> lower endpoint  [m]
  uint32_t* ev;         // edge id -> upper endpoint  [m]
  uint32_t* s1;         // edge id -> slot in row eu  [m]
  uint32_t* s2;         // edge id -> slot in row ev  [m]
  uint32_t* srem;       // slot -> round its edge was peeled, ALIVE if in S [2m]
  // Round kernels read the adjacency through a private copy whose rows are
  // compacted now and then (live slots first, in order): row x's active
  // slots are [rp[x], rp[x] + len[x]); slots past len[x] are dead.
  uint32_t* cix;        // private column ids [2m]
  uint32_t* len;        // active slots per row [n]
  // The support update's view of a slot, one 8-byte load: low word the
  // neighbour id with SLOT_GONE set once the edge is peeled, high word the
  // edge id [2m] (same row layout as cix)
  uint64_t* ce;
  uint32_t* up_cnt;     // per row: neighbours above the row vertex [n]
  uint32_t* up_off;     // exclusive prefix sum of up_cnt [n]
  uint32_t* scan_tmp;   // block sums for the scan
  uint32_t* minpart;    // per-block minima of the level-jump reduction
  uint32_t* sup;        // current h-support of every edge [m]
  uint32_t* t;          // trussness [m]
  uint32_t* rho;        // peel round [m]
  uint32_t* out_t;      // the caller's outputs (renumbered graphs: written at the end)
  uint32_t* out_rho;    // (may be null)
  uint32_t* R[2];       // peel lists by round parity [m]
  uint64_t* L[HMAX + 1];   // L[j]: closed j-hop balls, n rows of W words
  uint64_t* Dm[HMAX + 1];  // Dm[j]: pairs that left the j-ball this round
  uint64_t* evl[HMAX + 1][2];  // event lists (x<<32|w) per level and parity
  Item* itl[HMAX + 2];     // work items per level; index h+1: support items
  Ctl* ctl;
  struct Team* team;    // the team kernel's meeting point for this slot
  Dev* self;               // device-resident copy of this struct (round kernels read it)
  uint32_t* spart;         // stats mode: per-workgroup counters [NSTAT][STAT_GRID], else null
  uint32_t* status;        // this slot's {done, halt, live, -} words in the engine's status
                           // array (done: 1 finished, 2 malformed CSR; live: edges left)
  // stats mode, method-level work count: per vertex |N(x,h)|, live degree,
  // round stamps (h-ball changed, ball build counted) and this round's lists
  uint32_t* acct_ball;
  uint32_t* acct_deg;
  uint32_t* acct_stamp;
  uint32_t* acct_vstamp;
  uint32_t* acct_list;
  uint32_t* acct_vlist;
};

// Compact again once a tenth of the live edges have been peeled since the
// last compaction (a compaction reads and writes the active slots once).
__host__ __device__ inline uint32_t compact_next(uint32_t live) { return live - live / 10; }

// Load of a word that another workgroup of the same launch may have written
// (TEAM): a relaxed device-scope load is served by the L2 that the team's
// workgroups share, never by this CU's own L1, which nothing keeps current.
template <bool TEAM, class T>
__device__ __forceinline__ T ld(const T* p) {
  if constexpr (TEAM) return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  else return *p;
}

template <bool TEAM>
__device__ __forceinline__ Item ld_item(const Item* p) {
  if constexpr (TEAM) {
    const uint64_t* q = reinterpret_cast<const uint64_t*>(p);
    const uint64_t a = ld<true>(q), b = ld<true>(q + 1);
    return Item{(uint32_t)a, (uint32_t)(a >> 32), (uint32_t)b, (uint32_t)(b >> 32)};
  } else {
    return *p;
  }
}

// Atomics on words shared by the workgroups of a launch.  Device-scope ones go
// to memory, past every L2.  A team's workgroups share one L2, where atomics of
// workgroup scope are done: the same result for them, and the words stay there.
template <bool TEAM, class T>
__device__ __forceinline__ T at_add(T* p, T v) {
  return __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, TEAM ? __HIP_MEMORY_SCOPE_WORKGROUP : __HIP_MEMORY_SCOPE_AGENT);
}
template <bool TEAM, class T>
__device__ __forceinline__ T at_sub(T* p, T v) {
  return __hip_atomic_fetch_sub(p, v, __ATOMIC_RELAXED, TEAM ? __HIP_MEMORY_SCOPE_WORKGROUP : __HIP_MEMORY_SCOPE_AGENT);
}
template <bool TEAM, class T>
__device__ __forceinline__ T at_and(T* p, T v) {
  return __hip_atomic_fetch_and(p, v, __ATOMIC_RELAXED, TEAM ? __HIP_MEMORY_SCOPE_WORKGROUP : __HIP_MEMORY_SCOPE_AGENT);
}
template <bool TEAM, class T>
__device__ __forceinline__ T at_or(T* p, T v) {
  return __hip_atomic_fetch_or(p, v, __ATOMIC_RELAXED, TEAM ? __HIP_MEMORY_SCOPE_WORKGROUP : __HIP_MEMORY_SCOPE_AGENT);
}

// Workgroups are dealt to the eight XCDs in turn; this numbering gives each XCD
// consecutive numbers, so that neighbouring work items share an L2.
__device__ __forceinline__ uint32_t xcd_first(uint32_t b, uint32_t grid) {
  return grid % 8 == 0 ? (b & 7) * (grid / 8) + (b >> 3) : b;
}

__device__ __forceinline__ uint32_t lane_id() { return threadIdx.x & (WAVE - 1); }

__device__ __forceinline__ uint64_t slot_word(uint32_t e, uint32_t y, bool gone) {
  return ((uint64_t)e << 32) | y | (gone ? SLOT_GONE : 0u);
}

// End of row x's active slots (round kernels).
__device__ __forceinline__ uint32_t row_end(const Dev& d, uint32_t x) { return d.rp[x] + d.len[x]; }

__device__ __forceinline__ uint64_t* row(uint64_t* base, uint32_t W, uint32_t x) {
  return base + (size_t)x * W;
}
__device__ __forceinline__ const uint64_t* row(const uint64_t* base, uint32_t W, uint32_t x) {
  return base + (size_t)x * W;
}

// Wave-wide scans and reductions on DPP moves (row shifts inside the rows of
// 16 lanes, then row broadcasts 15 and 31): six VALU steps of a few cycles
// each, where a __shfl step goes through the LDS crossbar and takes over 50.
template <int CTRL, int ROWS>
__device__ __forceinline__ uint32_t dpp(uint32_t old, uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp((int)old, (int)v, CTRL, ROWS, 0xf, false);
}

// Inclusive prefix sum across the wave (all 64 lanes must call).
__device__ __forceinline__ uint32_t wave_incl_scan(uint32_t v) {
  v += dpp<0x111, 0xf>(0, v);  // row_shr:1, 2, 4, 8
  v += dpp<0x112, 0xf>(0, v);
  v += dpp<0x114, 0xf>(0, v);
  v += dpp<0x118, 0xf>(0, v);
  v += dpp<0x142, 0xa>(0, v);  // row_bcast:15 into rows 1 and 3
  v += dpp<0x143, 0xc>(0, v);  // row_bcast:31 into rows 2 and 3
  return v;
}

__device__ __forceinline__ uint32_t wave_last(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_readlane((int)v, WAVE - 1);
}

__device__ __forceinline__ uint32_t wave_sum(uint32_t v) { return wave_last(wave_incl_scan(v)); }

__device__ __forceinline__ uint32_t wave_min(uint32_t v) {
  constexpr uint32_t I = 0xffffffffu;
  v = min(v, dpp<0x111, 0xf>(I, v));
  v = min(v, dpp<0x112, 0xf>(I, v));
  v = min(v, dpp<0x114, 0xf>(I, v));
  v = min(v, dpp<0x118, 0xf>(I, v));
  v = min(v, dpp<0x142, 0xa>(I, v));
  v = min(v, dpp<0x143, 0xc>(I, v));
  return wave_last(v);
}

// Exclusive prefix sum across the wave (all 64 lanes must call).
__device__ __forceinline__ uint32_t wave_excl_scan(uint32_t v, uint32_t* total) {
  const uint32_t incl = wave_incl_scan(v);
  *total = wave_last(incl);
  return incl - v;
}

// Wave-aggregated reservation of `cnt` slots of a counter (all lanes call).
// Returns this lane's first slot.
template <bool TEAM>
__device__ __forceinline__ uint32_t wave_reserve(uint32_t* counter, uint32_t cnt) {
  uint32_t total;
  const uint32_t off = wave_excl_scan(cnt, &total);
  uint32_t base = 0;
  if (lane_id() == 0 && total) base = at_add<TEAM>(counter, total);
  base = __shfl(base, 0, WAVE);
  return base + off;
}

}  // namespace hotruss
