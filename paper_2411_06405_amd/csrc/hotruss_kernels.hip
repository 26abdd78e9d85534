// hotruss_kernels.hip -- CDNA4 (gfx950) kernels of the peeling method for
// higher-order truss decomposition (paper, Section 3, Algorithm 1), executed
// as bulk-synchronous rounds with exact incremental h-support maintenance.
//
// State per vertex x and level j = 1..h: L[j](x), the closed j-hop ball
// {y : dist_S(x,y) <= j} as a dense bitset row (x included).  The h-support
// of a live edge (u,v) is |L[h](u) & L[h](v)| - 2: u and v lie in both closed
// balls and are exactly the two members that the definition excludes.
//
// A peel round removes R (all live edges with sup <= k-2).  Ball members only
// ever leave.  A pair {x,w} leaves level j exactly when every path of length
// <= j between them in the old edge set used a removed edge, and its shortest
// such path starts either with a removed edge (x,z), with w in z's old
// (j-1)-ball, or with a surviving edge (x,z) (or x itself), where w left z's
// (j-1)-ball this round.  Those two families are the candidates tested at
// level j ("ball-change events" are the pairs that really left).  For the top
// level h, the support of a live edge (a,b) drops by
//     |D(a) & Bold(b)| + |D(b) & Bnew(a)|,
// D = pairs that left, Bold = Bnew + D; each top-level event (a -> w) is
// charged to every live edge (a,b) with w in Bold(b) when a < b and w in
// Bnew(b) when a > b, which counts every lost common neighbour exactly once.
// Edges whose support crosses k-2 form the next round's R.
#include "hotruss_dev.h"

namespace hotruss {

// ---------------------------------------------------------------- fills
__global__ void k_fill64(uint64_t* __restrict__ p, size_t cnt, uint64_t v) {
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < cnt;
       i += (size_t)gridDim.x * blockDim.x)
    p[i] = v;
}

__global__ void k_fill32(uint32_t* __restrict__ p, size_t cnt, uint32_t v) {
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < cnt;
       i += (size_t)gridDim.x * blockDim.x)
    p[i] = v;
}

__global__ void k_init_ctl(Ctl* ctl, uint32_t bytes, uint32_t n, uint32_t words, uint32_t m) {
  uint32_t* w = reinterpret_cast<uint32_t*>(ctl);
  for (uint32_t i = threadIdx.x; i < bytes / 4; i += blockDim.x) w[i] = 0;
  __syncthreads();
  if (threadIdx.x == 0) {
    ctl->nact = n;
    ctl->words = words;
    ctl->k = 2;
    ctl->jump = 1;  // nothing pushed yet: the first round jumps to min sup + 2
    ctl->live = m;
    ctl->phase = ROUND_CLOSED;
    ctl->compact_at = compact_next(m);
    ctl->levels = 0;
    ctl->done = (m == 0);
  }
}

// ---------------------------------------------------- CSR check, edge ids
// row_ptr must start at 0, never decrease and end at 2m.
__global__ void k_check_rowptr(Dev d) {
  for (uint32_t x = blockIdx.x * blockDim.x + threadIdx.x; x <= d.n;
       x += gridDim.x * blockDim.x) {
    uint32_t bad = 0;
    if (x == 0 && d.orp[0] != 0) bad |= ERR_ROWPTR;
    if (x == d.n && d.orp[d.n] != d.nnz) bad |= ERR_COUNT;
    if (x < d.n && d.orp[x] > d.orp[x + 1]) bad |= ERR_ROWPTR;
    if (bad) atomicOr(&d.ctl->err, bad);
  }
}

// Per row: ids in range, no self-loop, strictly ascending; count of
// neighbours above the row vertex.
__global__ void k_row_upper(Dev d) {
  if (d.ctl->err) return;
  const uint32_t lane = lane_id();
  const uint32_t wpb = blockDim.x / WAVE;
  for (uint32_t x = blockIdx.x * wpb + threadIdx.x / WAVE; x < d.n; x += gridDim.x * wpb) {
    const uint32_t beg = d.orp[x], end = d.orp[x + 1];
    uint32_t cnt = 0, bad = 0;
    for (uint32_t j = beg + lane; j < end; j += WAVE) {
      const uint32_t y = d.oci[j];
      if (y >= d.n) bad |= ERR_COL;
      if (y == x) bad |= ERR_LOOP;
      if (j > beg && d.oci[j - 1] >= y) bad |= ERR_ORDER;
      cnt += (y > x && y < d.n);
    }
    cnt = wave_sum(cnt);
    for (int o = WAVE / 2; o > 0; o >>= 1) bad |= __shfl_xor(bad, o, WAVE);
    if (lane == 0) {
      d.up_cnt[x] = cnt;
      if (bad) atomicOr(&d.ctl->err, bad);
    }
  }
}

// Exclusive scan of up_cnt into up_off: 1024 entries per block.
__global__ void __launch_bounds__(256) k_scan1(const uint32_t* __restrict__ in,
                                               uint32_t* __restrict__ out,
                                               uint32_t* __restrict__ bsum, uint32_t cnt) {
  __shared__ uint32_t ws[4];
  const uint32_t base = blockIdx.x * 1024 + threadIdx.x * 4;
  uint32_t v[4], s = 0;
  for (int i = 0; i < 4; ++i) {
    v[i] = (base + i < cnt) ? in[base + i] : 0u;
    s += v[i];
  }
  uint32_t incl = s;
  for (int o = 1; o < WAVE; o <<= 1) {
    uint32_t t = __shfl_up(incl, o, WAVE);
    if ((int)lane_id() >= o) incl += t;
  }
  if (lane_id() == WAVE - 1) ws[threadIdx.x / WAVE] = incl;
  __syncthreads();
  uint32_t woff = 0;
  for (uint32_t w = 0; w < threadIdx.x / WAVE; ++w) woff += ws[w];
  uint32_t run = woff + incl - s;
  for (int i = 0; i < 4; ++i) {
    if (base + i < cnt) out[base + i] = run;
    run += v[i];
  }
  if (threadIdx.x == 255) bsum[blockIdx.x] = woff + incl;
}

__global__ void __launch_bounds__(64) k_scan2(uint32_t* bsum, uint32_t nb) {
  uint32_t run = 0;
  for (uint32_t i0 = 0; i0 < nb; i0 += WAVE) {
    const uint32_t i = i0 + threadIdx.x, v = i < nb ? bsum[i] : 0u;
    uint32_t tot;
    const uint32_t ex = wave_excl_scan(v, &tot);
    if (i < nb) bsum[i] = run + ex;
    run += tot;
  }
}

__global__ void k_scan3(uint32_t* __restrict__ out, const uint32_t* __restrict__ bsum,
                        uint32_t cnt) {
  for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < cnt; i += gridDim.x * blockDim.x)
    out[i] += bsum[i / 1024];
}

// Canonical edge ids (upper-triangle CSR order), endpoints and slots; every
// lower slot (x,y), y < x, finds its partner (y,x) by binary search.  A graph
// that is renumbered gets its endpoints and slots from place_slot.
__global__ void k_edge_ids(Dev d) {
  if (d.ctl->err) return;
  const uint32_t lane = lane_id();
  const uint32_t wpb = blockDim.x / WAVE;
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    const uint32_t tot = d.n ? d.up_off[d.n - 1] + d.up_cnt[d.n - 1] : 0;
    if (tot != d.m) atomicOr(&d.ctl->err, ERR_COUNT);
  }
  for (uint32_t x = blockIdx.x * wpb + threadIdx.x / WAVE; x < d.n; x += gridDim.x * wpb) {
    const uint32_t beg = d.orp[x], end = d.orp[x + 1];
    const uint32_t fu = end - d.up_cnt[x];
    for (uint32_t j = beg + lane; j < end; j += WAVE) {
      const uint32_t y = d.oci[j];
      if (!d.perm) d.srem[j] = ALIVE;
      if (y > x) {
        const uint32_t e = d.up_off[x] + (j - fu);
        if (e >= d.m) { atomicOr(&d.ctl->err, ERR_COUNT); continue; }
        d.eid[j] = e;
        if (!d.perm) { d.eu[e] = x; d.ev[e] = y; d.s1[e] = j; }
      } else {
        uint32_t lo = d.orp[y + 1] - d.up_cnt[y], hi = d.orp[y + 1];
        const uint32_t first = lo;
        while (lo < hi) {
          const uint32_t mid = (lo + hi) >> 1;
          if (d.oci[mid] < x) lo = mid + 1; else hi = mid;
        }
        if (lo == d.orp[y + 1] || d.oci[lo] != x) { atomicOr(&d.ctl->err, ERR_ASYM); continue; }
        const uint32_t e = d.up_off[y] + (lo - first);
        if (e >= d.m) { atomicOr(&d.ctl->err, ERR_COUNT); continue; }
        d.eid[j] = e;
        if (!d.perm) d.s2[e] = j;
      }
    }
  }
}

// ---------------------------------------------- renumbering by degree
// A work item reads, for 64 neighbours b of one vertex, the word of some ball
// row that holds b: 8 of the row's n/8 bytes each, so what bounds it is how
// many cache lines the 64 lanes touch.  In most graphs a few vertices hold
// most of the edges; numbered first, and with each row's slots in ascending
// order, the 64 words of an item fall into a few lines at the row's start,
// and those lines stay in the caches from item to item.  Isolated vertices
// come last and get no rows (a quarter of an R-MAT graph's).  The order is by
// degree class, eight classes per octave; inside a class any order does.
// Results do not depend on the numbering: edge ids, and with them every
// output, come from the caller's CSR.
__device__ __forceinline__ uint32_t degree_bucket(uint32_t deg) {
  if (deg == 0) return DEG_BUCKETS - 1;
  const uint32_t e = 31u - (uint32_t)__clz(deg);
  return DEG_BUCKETS - 2 - min(DEG_BUCKETS - 2, e * 8 + (uint32_t)((((uint64_t)deg << 3) >> e) & 7u));
}

constexpr uint32_t DEG_TILE = 1024;  // vertices per workgroup of the two passes

__global__ void __launch_bounds__(256) k_degree_count(Dev d) {
  __shared__ uint32_t h[DEG_BUCKETS];
  if (d.ctl->err) return;
  h[threadIdx.x] = 0;
  __syncthreads();
  for (uint32_t i = 0; i < DEG_TILE; i += 256) {
    const uint32_t x = blockIdx.x * DEG_TILE + i + threadIdx.x;
    if (x < d.n) atomicAdd(&h[degree_bucket(d.orp[x + 1] - d.orp[x])], 1u);
  }
  __syncthreads();
  if (h[threadIdx.x]) atomicAdd(&d.ctl->bucket[threadIdx.x], h[threadIdx.x]);
}

// Where each class starts; rows and words in use.
__global__ void __launch_bounds__(256) k_degree_starts(Dev d) {
  __shared__ uint32_t ws[4];
  if (d.ctl->err) return;
  const uint32_t v = d.ctl->bucket[threadIdx.x], wave = threadIdx.x / WAVE;
  const uint32_t incl = wave_incl_scan(v);
  if (lane_id() == WAVE - 1) ws[wave] = incl;
  __syncthreads();
  uint32_t start = incl - v;
  for (uint32_t w = 0; w < wave; ++w) start += ws[w];
  d.ctl->bucket[threadIdx.x] = start;
  if (threadIdx.x == degree_bucket(63)) d.ctl->nlong = start;
  if (threadIdx.x == DEG_BUCKETS - 1) {
    d.ctl->nact = start;
    d.ctl->words = max(2u, (start + 127) / 128 * 2);
    const_cast<uint32_t*>(d.rp)[d.n] = d.nnz;
  }
}

// New ids, and the degrees in their order (into up_cnt, free by now).
__global__ void __launch_bounds__(256) k_degree_place(Dev d) {
  __shared__ uint32_t h[DEG_BUCKETS], base[DEG_BUCKETS];
  if (d.ctl->err) return;
  h[threadIdx.x] = 0;
  __syncthreads();
  uint32_t b[DEG_TILE / 256], r[DEG_TILE / 256], deg[DEG_TILE / 256];
#pragma unroll
  for (uint32_t i = 0; i < DEG_TILE / 256; ++i) {
    const uint32_t x = blockIdx.x * DEG_TILE + i * 256 + threadIdx.x;
    deg[i] = x < d.n ? d.orp[x + 1] - d.orp[x] : 0;
    b[i] = degree_bucket(deg[i]);
    r[i] = x < d.n ? atomicAdd(&h[b[i]], 1u) : 0;
  }
  __syncthreads();
  if (h[threadIdx.x]) base[threadIdx.x] = atomicAdd(&d.ctl->bucket[threadIdx.x], h[threadIdx.x]);
  __syncthreads();
#pragma unroll
  for (uint32_t i = 0; i < DEG_TILE / 256; ++i) {
    const uint32_t x = blockIdx.x * DEG_TILE + i * 256 + threadIdx.x;
    if (x >= d.n) continue;
    const uint32_t y = base[b[i]] + r[i];
    d.perm[x] = y;
    d.inv[y] = x;
    d.up_cnt[y] = deg[i];
    if (d.len) d.len[y] = deg[i];
  }
}

// Lower slots (neighbour below the row vertex) of every row in the new order.
__global__ void __launch_bounds__(256) k_rows_lower(Dev d) {
  if (d.ctl->err) return;
  const uint32_t lane = lane_id(), wpb = blockDim.x / WAVE, nact = d.ctl->nact;
  for (uint32_t x = blockIdx.x * wpb + threadIdx.x / WAVE; x < nact; x += gridDim.x * wpb) {
    const uint32_t o = d.inv[x], beg = d.orp[o], deg = d.orp[o + 1] - beg;
    uint32_t c = 0;
    for (uint32_t i = lane; i < deg; i += WAVE) c += d.perm[d.oci[beg + i]] < x;
    c = wave_sum(c);
    if (lane == 0) d.up_cnt[x] = c;
  }
}

// Slot `at` of row x holds neighbour y by the caller's edge e.  Edges are
// numbered along the lower slots of the rows: what the support update hits in
// a row is mostly its hub neighbours, which are below the row vertex, and the
// atomics of neighbouring lanes on neighbouring edges are one request
// (device-scope atomics all go to memory: 48,000 requests a round on R-MAT 16
// h = 2 by the caller's numbers, 290,000 numbered along the upper slots).
__device__ __forceinline__ void place_slot(const Dev& d, uint32_t x, uint32_t at, uint32_t y,
                                           uint32_t e) {
  const uint32_t q = d.rp[x] + at;
  d.cix[q] = y;
  if (y < x) {
    const uint32_t own = d.up_off[x] + at;
    d.ne[e] = own;
    d.oe[own] = e;
    d.eu[own] = y;
    d.ev[own] = x;
    if (d.ce) d.s2[own] = q;
  }
  if (d.ce) {
    d.ce[q] = slot_word(e, y, false);  // the caller's number, until k_rows_edges
    d.srem[q] = ALIVE;
  }
}

// Rows of fewer than 64 slots, one wave each: a lane's place is the number of
// lanes with a smaller neighbour.
__global__ void __launch_bounds__(256) k_rows_short(Dev d) {
  if (d.ctl->err) return;
  const uint32_t lane = lane_id(), wpb = blockDim.x / WAVE, nact = d.ctl->nact;
  for (uint32_t x = d.ctl->nlong + blockIdx.x * wpb + threadIdx.x / WAVE; x < nact;
       x += gridDim.x * wpb) {
    const uint32_t o = d.inv[x], beg = d.orp[o], deg = d.orp[o + 1] - beg;
    const uint32_t y = lane < deg ? d.perm[d.oci[beg + lane]] : 0xffffffffu;
    const uint32_t e = lane < deg ? d.eid[beg + lane] : 0;
    uint32_t at = 0;
    for (uint32_t i = 0; i < deg; ++i)
      at += (uint32_t)__builtin_amdgcn_readlane((int)y, (int)i) < y;
    if (lane < deg) place_slot(d, x, at, y, e);
  }
}

// Longer rows, one workgroup each: counted and placed by ranges of the
// neighbour id (1,024 of them: a ball row's word or a few), any order inside
// a range, the slots below x apart from those above.
__global__ void __launch_bounds__(1024) k_rows_long(Dev d) {
  __shared__ uint32_t h[1024], ws[16], mid;
  if (d.ctl->err) return;
  uint32_t shift = 0;
  while ((d.n - 1) >> shift >= 1024) ++shift;
  const uint32_t nlong = d.ctl->nlong, wave = threadIdx.x / WAVE;
  for (uint32_t x = blockIdx.x; x < nlong; x += gridDim.x) {
    const uint32_t o = d.inv[x], beg = d.orp[o], deg = d.orp[o + 1] - beg;
    const uint32_t low = d.up_cnt[x];
    h[threadIdx.x] = 0;
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < deg; i += 1024)
      atomicAdd(&h[d.perm[d.oci[beg + i]] >> shift], 1u);
    __syncthreads();
    const uint32_t v = h[threadIdx.x], incl = wave_incl_scan(v);
    if (lane_id() == WAVE - 1) ws[wave] = incl;
    __syncthreads();
    uint32_t start = incl - v;
    for (uint32_t w = 0; w < wave; ++w) start += ws[w];
    h[threadIdx.x] = start;
    if (threadIdx.x == 0) mid = low;  // slots above x of x's own range start here
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < deg; i += 1024) {
      const uint32_t y = d.perm[d.oci[beg + i]], r = y >> shift;
      const uint32_t at = atomicAdd(r == x >> shift && y > x ? &mid : &h[r], 1u);
      place_slot(d, x, at, y, d.eid[beg + i]);
    }
    __syncthreads();
  }
}

// Own edge numbers in place of the caller's; the lower endpoints' slots.  (Up to
// 2^32 - 2 slots: a 32-bit index would step past the last one and start again.)
__global__ void __launch_bounds__(256) k_rows_edges(Dev d) {
  if (d.ctl->err) return;
  for (size_t q = blockIdx.x * (size_t)blockDim.x + threadIdx.x; q < d.nnz;
       q += (size_t)gridDim.x * blockDim.x) {
    const uint64_t w = d.ce[q];
    const uint32_t y = (uint32_t)w, own = d.ne[(uint32_t)(w >> 32)];
    d.ce[q] = slot_word(own, y, false);
    if (d.ev[own] == y) d.s1[own] = (uint32_t)q;
  }
}

// ------------------------------------------------------------ ball build
// Level 1: closed neighbourhood N[x].  One workgroup per row, built in LDS
// and written out once (coalesced).
__global__ void __launch_bounds__(256) k_build_L1(Dev d) {
  extern __shared__ uint64_t srow[];
  if (d.ctl->err) return;
  const uint32_t nact = d.ctl->nact, words = d.ctl->words;
  uint64_t* L1 = d.L[1];
  for (uint32_t x = blockIdx.x; x < nact; x += gridDim.x) {
    for (uint32_t i = threadIdx.x; i < words; i += blockDim.x) srow[i] = 0;
    __syncthreads();
    if (threadIdx.x == 0) atomicOr(&srow[x >> 6], 1ull << (x & 63));
    for (uint32_t j = d.rp[x] + threadIdx.x; j < d.rp[x + 1]; j += blockDim.x) {
      const uint32_t y = d.ci[j];
      atomicOr(&srow[y >> 6], 1ull << (y & 63));
    }
    __syncthreads();
    uint64_t* out = row(L1, d.W, x);
    for (uint32_t i = threadIdx.x; i < words; i += blockDim.x) out[i] = srow[i];
    __syncthreads();
  }
}

// Level 2: B(x,2) is the union of N[z] over z in N[x].  The row is built in
// LDS, each z in the way that reads less: the adjacency of a short one is
// scattered into it, by 16 lanes (the chains of 16 rows run side by side) or
// by a wavefront, and the level-1 row of a long one is ORed, each thread owning
// words (long: more than dthr/16 entries a bitset word, and more than dmin).
// Hubs and short rows meet in most frontiers of a power-law graph; with one way
// for the whole frontier R-MAT 17 takes 5.28 ms, so 2.75 (a way for each, the
// line at 2 entries a word: 3.59; at a half: 2.75; at a quarter or an eighth
// 0.1 and 0.5 more).
constexpr uint32_t BALL_BATCH = 1024;  // frontier vertices per pass
constexpr uint32_t BALL_SHORT = 128;   // entries that 16 lanes scatter
__global__ void __launch_bounds__(256) k_build_L2(Dev d, uint32_t dthr, uint32_t dmin) {
  extern __shared__ uint64_t srow[];
  __shared__ uint32_t s_z[BALL_BATCH], s_mid, s_long;
  if (d.ctl->err) return;
  const uint32_t nact = d.ctl->nact, words = d.ctl->words;
  const uint32_t lane = lane_id(), wv = threadIdx.x / WAVE, nw = blockDim.x / WAVE;
  const uint32_t grp = threadIdx.x / 16, sub = threadIdx.x & 15, ngrp = blockDim.x / 16;
  const uint64_t* L1 = d.L[1];
  for (uint32_t x = blockIdx.x; x < nact; x += gridDim.x) {
    const uint32_t beg = d.rp[x], deg = d.rp[x + 1] - beg;
    for (uint32_t i = threadIdx.x; i < words; i += blockDim.x) srow[i] = 0;
    // z = x (index deg) and every neighbour z = ci[beg + q]
    for (uint32_t q0 = 0; q0 <= deg; q0 += BALL_BATCH) {
      const uint32_t q1 = min(q0 + BALL_BATCH, deg + 1);
      if (threadIdx.x == 0) s_mid = s_long = 0;
      __syncthreads();
      for (uint32_t q = q0 + grp; q < q1; q += ngrp) {
        const uint32_t z = (q == deg) ? x : d.ci[beg + q];
        const uint32_t zb = d.rp[z], zd = d.rp[z + 1] - zb;
        const bool dense = zd > dmin && (uint64_t)zd * 16 > (uint64_t)dthr * words;
        if (dense || zd > BALL_SHORT) {
          // mid-sized rows from the front of the list, long ones from its end
          if (sub == 0) {
            if (dense) s_z[BALL_BATCH - 1 - atomicAdd(&s_long, 1u)] = z;
            else s_z[atomicAdd(&s_mid, 1u)] = z;
          }
          continue;
        }
        if (sub == 0) atomicOr(&srow[z >> 6], 1ull << (z & 63));
        for (uint32_t k = sub; k < zd; k += 16) {
          const uint32_t y = d.ci[zb + k];
          atomicOr(&srow[y >> 6], 1ull << (y & 63));
        }
      }
      __syncthreads();
      const uint32_t nmid = s_mid, nlong = s_long;
      for (uint32_t l = wv; l < nmid; l += nw) {
        const uint32_t z = s_z[l], zb = d.rp[z], zd = d.rp[z + 1] - zb;
        if (lane == 0) atomicOr(&srow[z >> 6], 1ull << (z & 63));
        for (uint32_t k = lane; k < zd; k += WAVE) {
          const uint32_t y = d.ci[zb + k];
          atomicOr(&srow[y >> 6], 1ull << (y & 63));
        }
      }
      if (nlong) {
        if (nmid) __syncthreads();
        for (uint32_t i = threadIdx.x; i < words; i += blockDim.x) {
          uint64_t acc = srow[i];
#pragma unroll 8
          for (uint32_t l = 0; l < nlong; ++l) acc |= L1[(size_t)s_z[BALL_BATCH - 1 - l] * d.W + i];
          srow[i] = acc;
        }
      }
      __syncthreads();
    }
    uint64_t* out = row(d.L[2], d.W, x);
    for (uint32_t i = threadIdx.x; i < words; i += blockDim.x) out[i] = srow[i];
    __syncthreads();
  }
}

// Level j >= 3 by OR-ing the (j-1)-balls of x and its neighbours
// (B(x,j) = union over z in N[x] of B(z,j-1)); each thread owns a set of words.
__global__ void __launch_bounds__(256) k_build_Lj(Dev d, uint32_t j) {
  if (d.ctl->err) return;
  const uint32_t nact = d.ctl->nact, words = d.ctl->words;
  const uint64_t* P = d.L[j - 1];
  uint64_t* O = d.L[j];
  for (uint32_t x = blockIdx.x; x < nact; x += gridDim.x) {
    const uint32_t beg = d.rp[x], end = d.rp[x + 1];
    for (uint32_t i = threadIdx.x; i < words; i += blockDim.x) {
      uint64_t acc = P[(size_t)x * d.W + i];
#pragma unroll 8
      for (uint32_t q = beg; q < end; ++q) acc |= P[(size_t)d.ci[q] * d.W + i];
      O[(size_t)x * d.W + i] = acc;
    }
  }
}

// Change marks of every row in use, before the first round.
__global__ void k_clear_rows(Dev d, uint64_t* __restrict__ p) {
  const size_t cnt = (size_t)d.ctl->nact * d.W;
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < cnt;
       i += (size_t)gridDim.x * blockDim.x)
    p[i] = 0;
}

// Initial h-support of every edge: |L[h](u) & L[h](v)| - 2 (Def. 3).
// G lanes cooperate on one edge; each lane loads V 64-bit words at a time
// (V = 1: 64-bit loads, V = 2: 128-bit loads; rows are 64-byte aligned).
template <int G, int V>
__global__ void __launch_bounds__(256) k_support_init(Dev d, uint32_t* __restrict__ out, bool by_caller) {
  if (d.ctl->err) return;
  const uint64_t* Lh = d.L[d.h];
  const uint32_t sub = threadIdx.x & (G - 1);
  const uint32_t gpb = blockDim.x / G;
  const uint32_t nv = d.ctl->words / V;  // an even number of words
  for (uint32_t e = blockIdx.x * gpb + threadIdx.x / G; e < d.m; e += gridDim.x * gpb) {
    const uint64_t* a = Lh + (size_t)d.eu[e] * d.W;
    const uint64_t* b = Lh + (size_t)d.ev[e] * d.W;
    uint32_t c = 0;
    if constexpr (V == 2) {
      const ulonglong2* a2 = reinterpret_cast<const ulonglong2*>(a);
      const ulonglong2* b2 = reinterpret_cast<const ulonglong2*>(b);
      for (uint32_t i = sub; i < nv; i += G) {
        const ulonglong2 x = a2[i], y = b2[i];
        c += __popcll(x.x & y.x) + __popcll(x.y & y.y);
      }
    } else {
      for (uint32_t i = sub; i < nv; i += G) c += __popcll(a[i] & b[i]);
    }
    for (int o = G / 2; o > 0; o >>= 1) c += __shfl_xor(c, o, WAVE);
    if (sub == 0) out[by_caller && d.oe ? d.oe[e] : e] = c - 2;
  }
}

// The same for renumbered graphs, by slices of the words: blocks b with the
// same b mod 8 share an XCD, and take every edge's words of one eighth.  One
// wavefront an edge reads both rows whole, and is bound by the rows of the
// hubs, which most edges end at and no L2 holds (R-MAT 17 h = 2: 8.8 KB a row,
// 5.5 TB/s); an eighth of them, for the few thousand hubs that matter, stays in
// the XCD's L2 (2.70 ms before, 1.66 now; with 64-bit loads 2.44).  Uniform random
// 60,000 h = 2, all rows alike: 0.94 and 0.92 ms a call.  16 lanes take SLICE_EDGES consecutive edges, which share their
// upper endpoint in most cases, and add the eighth to each edge's support
// (sup: -2 before; own edge numbers, so that neighbouring edges' sums go to
// memory in one request).
constexpr int SLICE_EDGES = 4;
template <int V>
__global__ void __launch_bounds__(256) k_support_slices(Dev d, uint32_t* __restrict__ sup) {
  if (d.ctl->err) return;
  using Word = std::conditional_t<V == 2, ulonglong2, unsigned long long>;
  const Word* Lh = reinterpret_cast<const Word*>(d.L[d.h]);
  const uint32_t words = d.ctl->words, per = ((words + 7) / 8 + 7) & ~7u;
  const uint32_t lo = min(words, (blockIdx.x & 7) * per) / V, hi = min(words, lo * V + per) / V;
  if (lo >= hi) return;
  constexpr uint32_t G = 16, K = SLICE_EDGES;
  const uint32_t sub = threadIdx.x & (G - 1), gpb = blockDim.x / G;
  const uint32_t stride = (gridDim.x >> 3) * gpb * K;
  const size_t W = d.W / V;
  auto both = [](const Word& x, const Word& y) -> uint32_t {
    if constexpr (V == 2) return __popcll(x.x & y.x) + __popcll(x.y & y.y);
    else return __popcll(x & y);
  };
  for (uint32_t e0 = ((blockIdx.x >> 3) * gpb + threadIdx.x / G) * K; e0 < d.m; e0 += stride) {
    const Word *a[K], *b[K];
    uint32_t c[K] = {};
    bool one = true;
#pragma unroll
    for (uint32_t k = 0; k < K; ++k) {
      const uint32_t e = min(e0 + k, d.m - 1);
      a[k] = Lh + d.ev[e] * W;
      b[k] = Lh + d.eu[e] * W;
      one = one && a[k] == a[0];
    }
    if (one) {
#pragma unroll 2
      for (uint32_t i = lo + sub; i < hi; i += G) {
        const Word x = a[0][i];
#pragma unroll
        for (uint32_t k = 0; k < K; ++k) c[k] += both(x, b[k][i]);
      }
    } else {
      for (uint32_t i = lo + sub; i < hi; i += G)
#pragma unroll
        for (uint32_t k = 0; k < K; ++k) c[k] += both(a[k][i], b[k][i]);
    }
    uint32_t mine = 0;  // lane k of the group: edge e0 + k
#pragma unroll
    for (uint32_t k = 0; k < K; ++k) {
      for (int o = G / 2; o > 0; o >>= 1) c[k] += __shfl_xor(c[k], o, WAVE);
      if (sub == k) mine = c[k];
    }
    if (mine && e0 + sub < d.m) atomicAdd(&sup[e0 + sub], mine);
  }
}

// Supports by own edge number to the caller's (a malformed graph has no numbers).
__global__ void __launch_bounds__(256) k_support_out(Dev d, const uint32_t* __restrict__ sup,
                                                     uint32_t* __restrict__ out) {
  if (d.ctl->err) return;
  for (uint32_t e = blockIdx.x * blockDim.x + threadIdx.x; e < d.m; e += gridDim.x * blockDim.x)
    out[e] = sup[d.ne[e]];
}

// ============================================================ peel rounds
// A round of the whole chip is a fixed kernel sequence (captured into a HIP
// graph and replayed): k_mark, k_level(j) for j = 2..h, k_support, k_end.  Small
// rounds are run by the team kernel instead, with the same step functions; a
// round that it began goes on at the step that Ctl::phase names.  Every kernel
// reads the control block and returns at once when there is nothing for it to
// do, so a graph may run past the last round.

struct RoundCtx {
  uint32_t r, k, p;
  uint32_t edges;  // peeled in the round, where the marking goes by it (see word_chunk)
};

__device__ __forceinline__ RoundCtx round_ctx(const Ctl* c) { return RoundCtx{c->r, c->k, c->r & 1, 0}; }

// ---- work item emission (all 64 lanes call; per-lane counts may be 0) ----
// A lane's group of items covers one CSR row (or one ball row's words), CHUNK
// entries per item.  The wave reserves the items of all its lanes with one
// atomic and writes them cooperatively, consecutive lanes on consecutive list
// entries, so a lane whose row belongs to a hub (hundreds of items) does not
// write them alone.
//   ITEM_ROW    Item{x, y, base, meta(kind, extra, len, vstart)}: nv virtual
//               entries (the row's slots, plus the extra candidate at virtual
//               index 0 when extra = 1)
//   ITEM_SLOTS  Item{x, y, base + vstart, meta(0, 0, len, 0)}: support items
//   ITEM_WORDS  Item{x, y, vstart, meta(KIND_A_WORDS, 0, len, 0)}: ball words
enum { ITEM_ROW = 0, ITEM_SLOTS = 1, ITEM_WORDS = 2 };

__device__ __forceinline__ uint32_t chunks_of(uint32_t nv) { return (nv + CHUNK - 1) / CHUNK; }

// Ball words per item.  A word can hold 64 candidates, so on small graphs 64
// words would leave the few rows of a small round to a few waves (Chung-Lu 5,001
// h = 3: the slowest workgroup took 24 us over its items, the others 2), and 8
// are taken.  A round with enough items of 64 words takes those: eight times
// the items are that many more steps of mostly idle lanes, and more list space.
// `edges`: peeled in the round.  12 uniform graphs of 8,000 to 11,300 h = 3 in one
// batch: 8 words always 59.3 ms, 64 always 45.3, by this rule 52.6; 6 Chung-Lu
// of 12,000 to 16,500 h = 3: 984, 1,253, 988 ms; uniform 32,000 of degree 5 alone:
// 20.2 by 8 always, 14.7 by the rule.  (512 items: 50.2 and 1,001 ms; 8,192: 54.7
// and 992.)
constexpr uint32_t WORDS_FEW = 8, WORD_ITEMS = 2048;
__device__ __forceinline__ uint32_t word_chunk(uint32_t words, uint32_t edges) {
  return words > 512 || (uint64_t)edges * chunks_of(words) >= WORD_ITEMS / 2 ? CHUNK : WORDS_FEW;
}
// A level jump finds its edges as it marks them.  8 words, unless the list could
// run over by them.
__device__ __forceinline__ uint32_t word_chunk_edges(const Dev& d) {
  const uint64_t rows = 2ull * d.ctl->live;
  return rows * ((d.ctl->words + WORDS_FEW - 1) / WORDS_FEW) > d.itcap ? d.ctl->live : 0;
}

// Item number `chunk` of a group (nv entries, `size` an item).
template <int MODE>
__device__ __forceinline__ Item make_item(uint32_t kind, uint32_t extra, uint32_t x, uint32_t y,
                                          uint32_t base, uint32_t nv, uint32_t chunk,
                                          uint32_t size = CHUNK) {
  const uint32_t vs = chunk * size, len = min(size, nv - vs);
  if (MODE == ITEM_ROW) return Item{x, y, base, item_meta(kind, extra, len, vs)};
  if (MODE == ITEM_SLOTS) return Item{x, y, base + vs, item_meta(0, 0, len, 0)};
  return Item{x, y, vs, item_meta(KIND_A_WORDS, 0, len, 0)};
}

// Lane 0 reserves `total` entries of a counter for the whole wave.
template <bool TEAM>
__device__ __forceinline__ uint32_t reserve_wave(uint32_t* counter, uint32_t total) {
  uint32_t b = 0;
  if (lane_id() == 0 && total) b = at_add<TEAM>(counter, total);
  return __shfl(b, 0, WAVE);
}

// Write the wave's groups: this lane's items are entries [first + excl,
// first + excl + cnt) of list `list` (excl: exclusive prefix of cnt over the
// wave, total: the wave's sum; both from wave_excl_scan).
template <int MODE>
__device__ void emit_items_wave(const Dev& d, uint32_t p, uint32_t list, uint32_t first, uint32_t total,
                                uint32_t excl, uint32_t cnt, uint32_t kind, uint32_t extra,
                                uint32_t x, uint32_t y, uint32_t base, uint32_t nv,
                                uint32_t size = CHUNK) {
  if (!__ballot(cnt > 1)) {
    // at most one item per lane (most rows fit one chunk): no owner to look up
    const uint32_t idx = first + excl;
    if (cnt && idx < d.itcap) d.itl[list][idx] = make_item<MODE>(kind, extra, x, y, base, nv, 0, size);
    if (__ballot(cnt && idx >= d.itcap)) d.ctl->cnt[list][p].iovf = 1;
    return;
  }
  const uint32_t incl = excl + cnt;
  bool over = false;
  for (uint32_t t0 = 0; t0 < total; t0 += WAVE) {
    const uint32_t t = t0 + lane_id();
    // owner of entry t: the number of lanes whose groups end at or before t
    uint32_t own = 0;
#pragma unroll
    for (uint32_t step = 32; step > 0; step >>= 1) {
      const uint32_t v = (uint32_t)__shfl(incl, (int)(own + step - 1), WAVE);
      if (v <= t) own += step;
    }
    const uint32_t ox = __shfl(x, own, WAVE), oy = __shfl(y, own, WAVE);
    const uint32_t ob = __shfl(base, own, WAVE), onv = __shfl(nv, own, WAVE);
    const uint32_t oex = __shfl(excl, own, WAVE);
    if (t < total) {
      const uint32_t idx = first + t;
      if (idx < d.itcap)
        d.itl[list][idx] = make_item<MODE>(kind, extra, ox, oy, ob, onv, t - oex, size);
      else over = true;
    }
  }
  if (over) d.ctl->cnt[list][p].iovf = 1;
}

// One group per lane with its own reservation.
template <int MODE, bool TEAM>
__device__ void emit_group(const Dev& d, uint32_t p, uint32_t list, uint32_t kind, uint32_t extra,
                           uint32_t x, uint32_t y, uint32_t base, uint32_t nv,
                           uint32_t size = CHUNK) {
  const uint32_t cnt = (nv + size - 1) / size;
  uint32_t total;
  const uint32_t excl = wave_excl_scan(cnt, &total);
  if (!total) return;
  const uint32_t first = reserve_wave<TEAM>(&d.ctl->cnt[list][p].nit, total);
  emit_items_wave<MODE>(d, p, list, first, total, excl, cnt, kind, extra, x, y, base, nv, size);
}

// Support items of event (a -> w): the live edges (a,b), CHUNK slots per item.
template <bool TEAM>
__device__ void emit_support_items(const Dev& d, uint32_t p, bool active, uint32_t a, uint32_t w) {
  uint32_t base = 0, deg = 0;
  if (active) {
    base = d.rp[a];
    deg = row_end(d, a) - base;
  }
  emit_group<ITEM_SLOTS, TEAM>(d, p, d.h + 1, 0, 0, a, w, base, deg);
}

// Items over z's old (j-1)-ball words for candidates (x, w), j >= 3.
template <bool TEAM>
__device__ void emit_word_items(const Dev& d, uint32_t p, uint32_t j, bool active, uint32_t x, uint32_t z,
                                uint32_t size) {
  emit_group<ITEM_WORDS, TEAM>(d, p, j, 0, 0, x, z, 0, active ? d.ctl->words : 0u, size);
}

// ---- level-jump minimum ----------------------------------------------------
// Per-workgroup minima of the live edges' supports (read by k_mark of a round
// that starts with a level jump).  Computed by the end-of-round kernel of the
// previous round, when every support of that round is final, and once after
// the initial pass.
__device__ void jump_partials(const Dev& d) {
  __shared__ uint32_t smin[4];
  // eight edges per thread in flight; peeled edges hold SUP_GONE
  uint32_t mn = SUP_GONE;
  const uint32_t stride = gridDim.x * blockDim.x;
  uint32_t e = blockIdx.x * blockDim.x + threadIdx.x;
  for (; e + 7 * stride < d.m; e += 8 * stride) {
    uint32_t sv[8];
#pragma unroll
    for (uint32_t u = 0; u < 8; ++u) sv[u] = d.sup[e + u * stride];
#pragma unroll
    for (uint32_t u = 0; u < 8; ++u) mn = min(mn, sv[u]);
  }
  for (; e < d.m; e += stride) mn = min(mn, d.sup[e]);
  mn = wave_min(mn);
  if (lane_id() == 0) smin[threadIdx.x / WAVE] = mn;
  __syncthreads();
  if (threadIdx.x == 0)
    d.minpart[blockIdx.x] = min(min(smin[0], smin[1]), min(smin[2], smin[3]));
}

// After the initial pass: the first round starts with a level jump
// (host-driven rounds; the team kernel finds its own minimum).
__global__ void __launch_bounds__(256) k_first_min(const Dev* __restrict__ devs) {
  const Dev& d = devs[blockIdx.y];
  if (d.ctl->done || d.ctl->err) return;
  if (blockIdx.x == 0 && threadIdx.x == 0) d.ctl->phase = 0;
  jump_partials(d);
}

// One direction of a wave's pairs that leave a ball: bit `col` of row `row`, for
// the lanes with `drop`.  Neighbouring lanes hold neighbouring columns of one
// row (a work item's pairs share a vertex), so runs of lanes on the same word
// are merged into one atomic: atomics on one cache line serialise at about
// 11 ns each wherever they come from, and with the hubs numbered first a
// row's pairs share a few lines (R-MAT 16 h = 2, renumbered: k_level 39 us a
// round without the merge, 17 us with it and the eight-lane dealing below).
struct Run {
  uint64_t upto, bit;  // bits of the run up to this lane; this lane's own
  size_t o;            // the word
  uint32_t last;       // the run's last lane, which does its atomics
  bool twice;          // an earlier lane of the run has the same pair
};

__device__ __forceinline__ Run word_runs(uint32_t W, uint32_t row_, uint32_t col, bool drop) {
  const uint32_t lane = lane_id(), word = col >> 6;
  Run R;
  R.bit = drop ? 1ull << (col & 63) : 0ull;
  R.o = (size_t)row_ * W + word;
  // a lane starts a run unless it is on its left neighbour's word
  const uint32_t pr = dpp<0x138, 0xf>(~row_, row_), pw = dpp<0x138, 0xf>(~word, word);  // wave_shr:1
  const bool head = lane == 0 || pr != row_ || pw != word;
  // inclusive OR inside the runs
  uint32_t lo = (uint32_t)R.bit, hi = (uint32_t)(R.bit >> 32), fl = head;
  auto step = [&](uint32_t plo, uint32_t phi, uint32_t pf) {
    if (!fl) {
      lo |= plo;
      hi |= phi;
      fl = pf;
    }
  };
  step(dpp<0x111, 0xf>(0, lo), dpp<0x111, 0xf>(0, hi), dpp<0x111, 0xf>(0, fl));
  step(dpp<0x112, 0xf>(0, lo), dpp<0x112, 0xf>(0, hi), dpp<0x112, 0xf>(0, fl));
  step(dpp<0x114, 0xf>(0, lo), dpp<0x114, 0xf>(0, hi), dpp<0x114, 0xf>(0, fl));
  step(dpp<0x118, 0xf>(0, lo), dpp<0x118, 0xf>(0, hi), dpp<0x118, 0xf>(0, fl));
  step(dpp<0x142, 0xa>(0, lo), dpp<0x142, 0xa>(0, hi), dpp<0x142, 0xa>(0, fl));
  step(dpp<0x143, 0xc>(0, lo), dpp<0x143, 0xc>(0, hi), dpp<0x143, 0xc>(0, fl));
  R.upto = ((uint64_t)hi << 32) | lo;
  const uint64_t before =
      ((uint64_t)dpp<0x138, 0xf>(0, hi) << 32) | dpp<0x138, 0xf>(0, lo);
  R.twice = !head && (before & R.bit);
  const uint64_t heads = __ballot(head);
  const uint64_t later = lane == 63 ? 0ull : heads >> (lane + 1);
  R.last = later ? lane + (uint32_t)__ffsll((unsigned long long)later) - 1 : 63u;
  return R;
}

// Pairs {x, w} leave a ball, for the lanes with `drop`: both bits are cleared in
// L and set in D.  *xw, *wx: this lane cleared w in x's row, x in w's (one lane
// only, should two hold the same pair).  All lanes of the wave call it; the
// atomics of both directions are in flight together.  merge: by runs, for
// renumbered graphs.
template <bool TEAM>
__device__ __forceinline__ void clear_pairs(uint64_t* __restrict__ L, uint64_t* __restrict__ D,
                                            uint32_t W, uint32_t x, uint32_t w, bool drop,
                                            bool merge, bool* xw, bool* wx) {
  auto clear = [&](size_t o, uint64_t bits) -> uint64_t {
    return at_and<TEAM>(L + o, ~bits) & bits;
  };
  auto mark = [&](size_t o, uint64_t bits) {
    if (bits) at_or<TEAM>(D + o, bits);
  };
  if (!merge) {
    uint64_t oa = 0, ob = 0;
    if (drop) {
      const size_t pa = (size_t)x * W + (w >> 6), pb = (size_t)w * W + (x >> 6);
      oa = clear(pa, 1ull << (w & 63));
      ob = clear(pb, 1ull << (x & 63));
      mark(pa, oa);
      mark(pb, ob);
    }
    *xw = oa != 0;
    *wx = ob != 0;
    return;
  }
  const uint32_t lane = lane_id();
  const Run A = word_runs(W, x, w, drop), B = word_runs(W, w, x, drop);
  const bool da = A.last == lane && A.upto, db = B.last == lane && B.upto;
  uint64_t oa = 0, ob = 0;
  if (da) oa = clear(A.o, A.upto);
  if (db) ob = clear(B.o, B.upto);
  if (da) mark(A.o, oa);
  if (db) mark(B.o, ob);
  auto at = [&](uint64_t v, uint32_t l) {
    return ((uint64_t)(uint32_t)__shfl((uint32_t)(v >> 32), l, WAVE) << 32) |
           (uint32_t)__shfl((uint32_t)v, l, WAVE);
  };
  const uint64_t ra = at(oa, A.last), rb = at(ob, B.last);  // all lanes take part
  *xw = !A.twice && (ra & A.bit);
  *wx = !B.twice && (rb & B.bit);
}

// The same for peeled edges {x, w} and level 1, where every edge is listed once
// and nothing depends on what the atomics return (a marking kernel that waits
// for them takes 2.6 times as long in the largest rounds).  D: only at h = 1.
template <bool TEAM>
__device__ __forceinline__ void clear_edges(uint64_t* __restrict__ L, uint64_t* __restrict__ D,
                                            uint32_t W, uint32_t x, uint32_t w, bool valid,
                                            bool merge) {
  auto clear = [&](size_t o, uint64_t bits) {
    at_and<TEAM>(L + o, ~bits);
    if (D) at_or<TEAM>(D + o, bits);
  };
  if (merge) {
    const Run A = word_runs(W, x, w, valid), B = word_runs(W, w, x, valid);
    if (A.last == lane_id() && A.upto) clear(A.o, A.upto);
    if (B.last == lane_id() && B.upto) clear(B.o, B.upto);
  } else if (valid) {
    clear((size_t)x * W + (w >> 6), 1ull << (w & 63));
    clear((size_t)w * W + (x >> 6), 1ull << (x & 63));
  }
}

// ---- K2: peel R (level jump: collect it first), level-1 events, items ----
template <bool TEAM>
__device__ void mark_edge(const Dev& d, const RoundCtx& rc, bool valid, uint32_t e, uint32_t i) {
  uint32_t a = 0, b = 0;
  if (valid) {
    d.t[e] = rc.k;
    d.rho[e] = rc.r;
    d.sup[e] = SUP_GONE;  // the level-jump scans read only this array
    const uint32_t q1 = d.s1[e], q2 = d.s2[e];
    d.srem[q1] = rc.r;
    d.srem[q2] = rc.r;
    a = d.eu[e];
    b = d.ev[e];
    d.ce[q1] = slot_word(e, b, true);
    d.ce[q2] = slot_word(e, a, true);
    d.evl[1][rc.p][2 * i] = ((uint64_t)a << 32) | b;
    d.evl[1][rc.p][2 * i + 1] = ((uint64_t)b << 32) | a;
  }
  clear_edges<TEAM>(d.L[1], d.h == 1 ? d.Dm[1] : nullptr, d.W, a, b, valid, d.perm != nullptr);
  if (d.h == 1) {
    emit_support_items<TEAM>(d, rc.p, valid, a, b);
    emit_support_items<TEAM>(d, rc.p, valid, b, a);
    return;
  }
  // level 2: a lost neighbour b (candidates (a, y), y in b's old neighbourhood,
  // plus (a, b) itself) and symmetrically; level-1 events (a->b), (b->a):
  // candidates (y, b), y a live neighbour of a, and symmetrically.
  // (one reservation for the four item groups)
  uint32_t ba = 0, da = 0, bb = 0, db = 0;
  if (valid) {
    ba = d.rp[a];
    da = row_end(d, a) - ba;
    bb = d.rp[b];
    db = row_end(d, b) - bb;
  }
  // virtual entries per group: (a, y), y in N(b), plus (a, b); (b, y), y in
  // N(a), plus (b, a); (y, b), y in N(a); (y, a), y in N(b)
  const uint32_t v0 = valid ? db + 1 : 0, v1 = valid ? da + 1 : 0, v2 = valid ? da : 0,
                 v3 = valid ? db : 0;
  const uint32_t n0 = chunks_of(v0), n1 = chunks_of(v1), n2 = chunks_of(v2), n3 = chunks_of(v3);
  uint32_t t0, t1, t2, t3;
  const uint32_t e0 = wave_excl_scan(n0, &t0), e1 = wave_excl_scan(n1, &t1);
  const uint32_t e2 = wave_excl_scan(n2, &t2), e3 = wave_excl_scan(n3, &t3);
  const uint32_t first = reserve_wave<TEAM>(&d.ctl->cnt[2][rc.p].nit, t0 + t1 + t2 + t3);
  emit_items_wave<ITEM_ROW>(d, rc.p, 2, first, t0, e0, n0, KIND_A_SLOTS, 1, a, b, bb, v0);
  emit_items_wave<ITEM_ROW>(d, rc.p, 2, first + t0, t1, e1, n1, KIND_A_SLOTS, 1, b, a, ba, v1);
  emit_items_wave<ITEM_ROW>(d, rc.p, 2, first + t0 + t1, t2, e2, n2, KIND_B_SLOTS, 0, a, b, ba, v2);
  emit_items_wave<ITEM_ROW>(d, rc.p, 2, first + t0 + t1 + t2, t3, e3, n3, KIND_B_SLOTS, 0, b, a, bb,
                            v3);
  if (d.h < 3) return;
  const uint32_t wc = word_chunk(d.ctl->words, rc.edges);
  for (uint32_t j = 3; j <= d.h; ++j) {
    emit_word_items<TEAM>(d, rc.p, j, valid, a, b, wc);
    emit_word_items<TEAM>(d, rc.p, j, valid, b, a, wc);
  }
}

// One peeled edge, by a whole wave (e the same in all lanes): no lane waits for
// another's row, and the items need no owner search -- lane t writes item t.
// Small rounds are bound by this chain of dependent loads and atomics, not by
// bytes.
template <bool TEAM>
__device__ void mark_edge_wave(const Dev& d, const RoundCtx& rc, uint32_t e, uint32_t i) {
  const uint32_t lane = lane_id();
  const uint32_t a = d.eu[e], b = d.ev[e], q1 = d.s1[e], q2 = d.s2[e];
  const uint32_t ba = d.rp[a], da = d.len[a], bb = d.rp[b], db = d.len[b];
  if (lane == 0) {
    d.t[e] = rc.k;
    d.rho[e] = rc.r;
    d.sup[e] = SUP_GONE;
    d.srem[q1] = rc.r;
    d.srem[q2] = rc.r;
    d.ce[q1] = slot_word(e, b, true);
    d.ce[q2] = slot_word(e, a, true);
    at_and<TEAM>(&row(d.L[1], d.W, a)[b >> 6], ~((uint64_t)1 << (b & 63)));
    at_and<TEAM>(&row(d.L[1], d.W, b)[a >> 6], ~((uint64_t)1 << (a & 63)));
    if (d.h == 1) {
      at_or<TEAM>(&row(d.Dm[1], d.W, a)[b >> 6], (uint64_t)1 << (b & 63));
      at_or<TEAM>(&row(d.Dm[1], d.W, b)[a >> 6], (uint64_t)1 << (a & 63));
    }
    d.evl[1][rc.p][2 * i] = ((uint64_t)a << 32) | b;
    d.evl[1][rc.p][2 * i + 1] = ((uint64_t)b << 32) | a;
  }
  // the groups of mark_edge: at h = 1 the two support rows; else the four row
  // groups of level 2, and per level j >= 3 the two ball rows' words
  const uint32_t v0 = d.h == 1 ? da : db + 1, v1 = d.h == 1 ? db : da + 1;
  const uint32_t n0 = chunks_of(v0), n1 = chunks_of(v1);
  const uint32_t n2 = d.h == 1 ? 0 : chunks_of(da), n3 = d.h == 1 ? 0 : chunks_of(db);
  const uint32_t words = d.ctl->words, wc = word_chunk(words, rc.edges), nw = (words + wc - 1) / wc;
  const uint32_t rows = n0 + n1 + n2 + n3;
  uint32_t base = 0;
  if (lane == 0 || lane + 2 <= d.h)  // lane l reserves the items of list l + 2
    base = at_add<TEAM>(&d.ctl->cnt[lane + 2][rc.p].nit, lane == 0 ? rows : 2 * nw);
  const uint32_t first = (uint32_t)__builtin_amdgcn_readlane((int)base, 0);
  bool over = false;
  for (uint32_t t = lane; t < rows; t += WAVE) {
    Item it;
    if (d.h == 1)
      it = t < n0 ? make_item<ITEM_SLOTS>(0, 0, a, b, ba, v0, t)
                  : make_item<ITEM_SLOTS>(0, 0, b, a, bb, v1, t - n0);
    else if (t < n0) it = make_item<ITEM_ROW>(KIND_A_SLOTS, 1, a, b, bb, v0, t);
    else if (t < n0 + n1) it = make_item<ITEM_ROW>(KIND_A_SLOTS, 1, b, a, ba, v1, t - n0);
    else if (t < n0 + n1 + n2) it = make_item<ITEM_ROW>(KIND_B_SLOTS, 0, a, b, ba, da, t - n0 - n1);
    else it = make_item<ITEM_ROW>(KIND_B_SLOTS, 0, b, a, bb, db, t - n0 - n1 - n2);
    if (first + t < d.itcap) d.itl[2][first + t] = it;
    else over = true;
  }
  if (over) d.ctl->cnt[2][rc.p].iovf = 1;
  for (uint32_t j = 3; j <= d.h; ++j) {
    const uint32_t at = __shfl(base, j - 2, WAVE);
    over = false;
    for (uint32_t t = lane; t < 2 * nw; t += WAVE) {
      const Item it = t < nw ? make_item<ITEM_WORDS>(0, 0, a, b, 0, words, t, wc)
                             : make_item<ITEM_WORDS>(0, 0, b, a, 0, words, t - nw, wc);
      if (at + t < d.itcap) d.itl[j][at + t] = it;
      else over = true;
    }
    if (over) d.ctl->cnt[j][rc.p].iovf = 1;
  }
}

// Clear the change marks that the previous round (parity q) set at level j,
// from its event list.  At levels j >= 2 every bit set now is from the
// previous round (this round sets its own in the ball-change step, later), so
// whole words are zeroed with plain stores; level 1 (h = 1 only) gets this
// round's marks while this runs, so its old bits are cleared one by one.
template <bool TEAM>
__device__ void clear_marks(const Dev& d, uint32_t j, uint32_t q, uint32_t ne, uint32_t first,
                            uint32_t stride) {
  uint64_t* D = d.Dm[j];
  const uint64_t* E = d.evl[j][q];
  for (uint32_t i = first; i < ne; i += stride) {
    const uint64_t xw = ld<TEAM>(E + i);
    const uint32_t x = (uint32_t)(xw >> 32), w = (uint32_t)xw;
    if (j >= 2) row(D, d.W, x)[w >> 6] = 0;
    else at_and<TEAM>(&row(D, d.W, x)[w >> 6], ~((uint64_t)1 << (w & 63)));
  }
}

// At most 64 registers per lane (eight waves per SIMD): the launch's 2,048
// workgroups of 256 threads are then all resident at once on 256 CUs, so a
// level-jump scan runs in one pass instead of leaving a second batch waiting.
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(8)))
k_mark(const Dev* __restrict__ devs) {
  const Dev& d = devs[blockIdx.y];
  Ctl* c = d.ctl;
  if (c->done || c->halt || c->phase != 0) return;
  RoundCtx rc = round_ctx(c);
  if (blockIdx.x == 0 && threadIdx.x == 0) c->nPushc[rc.p].v = 0;
  const uint32_t q = rc.p ^ 1;
  const uint32_t lane = lane_id();
  const uint32_t wstride = gridDim.x * blockDim.x;
  const uint32_t wbase = blockIdx.x * blockDim.x + (threadIdx.x & ~(WAVE - 1));
  if (c->jump) {
    // level jump: k <- min live sup + 2 (Algorithm 1 moving to the next
    // non-empty bin); R <- every live edge with sup <= k-2
    uint32_t mn = 0xffffffffu;
    for (uint32_t i = lane; i < d.nminpart; i += WAVE) mn = min(mn, d.minpart[i]);
    mn = wave_min(mn);
    rc.k = mn + 2;
    if (d.h >= 3) rc.edges = word_chunk_edges(d);
    if (blockIdx.x == 0 && threadIdx.x == 0) {
      c->k = rc.k;
      c->levels += 1;
    }
    for (uint32_t base = wbase; base < d.m; base += wstride) {
      const uint32_t e = base + lane;
      const uint32_t sv = e < d.m ? d.sup[e] : SUP_GONE;
      const bool take = sv != SUP_GONE && sv <= rc.k - 2;
      if (!__ballot(take)) continue;  // nothing to peel in these 64 edges
      const uint32_t i = wave_reserve<false>(&c->nRc.v, take ? 1u : 0u);
      if (take) d.R[rc.p][i] = e;
      mark_edge<false>(d, rc, take, e, i);
    }
  } else {
    const uint32_t nR = rc.edges = c->nRc.v;
    if (nR <= wstride / WAVE) {
      // no more peeled edges than wavefronts: one edge per wavefront, so the
      // 64 lanes share the writing of its work items -- the rows of a hub
      // endpoint are hundreds of items
      const uint32_t i = wbase / WAVE;
      if (i < nR) mark_edge_wave<false>(d, rc, d.R[rc.p][i], i);
    } else {
      for (uint32_t base = wbase; base < nR; base += wstride) {
        const uint32_t i = base + lane;
        const bool valid = i < nR;
        mark_edge<false>(d, rc, valid, valid ? d.R[rc.p][i] : 0, i);
      }
    }
  }
  // the change marks of a level whose event list overflowed: its whole array
  for (uint32_t j = 2; j <= d.h; ++j) {
    if (!c->cnt[j][q].ovf) continue;
    uint64_t* D = d.Dm[j];
    const size_t cnt = (size_t)c->nact * d.W;
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < cnt;
         i += (size_t)gridDim.x * blockDim.x)
      D[i] = 0;
  }
  for (uint32_t j = 1; j <= d.h; ++j)
    if (d.Dm[j] && !c->cnt[j][q].ovf)
      clear_marks<false>(d, j, q, c->cnt[j][q].nev, blockIdx.x * blockDim.x + threadIdx.x, wstride);
}

// ---- K3: ball-change events at level j >= 2 ----------------------------
// Two workgroup shapes.  A single graph runs 16 wavefronts per workgroup,
// one workgroup per CU (its registers allow no second): the drop phase
// reserves list space once per workgroup on device-wide counters
// (same-address atomics serialise at about 11 ns each), so fewer, larger
// workgroups mean fewer of them, and a hub pair's witness probes spread over
// 1,024 threads.  Batched and served steps give every slot its own small
// grid, most of whose workgroups find nothing to do and return at once:
// there 256-thread workgroups pass through the CUs several at a time, where
// 1,024-thread ones would queue one per CU.
// The buffer holds the candidate pairs of a workgroup: a flush comes once
// another emission step (one candidate per thread at most) might not fit, so
// it holds at least two steps' worth -- bitset-word items at j >= 3 yield few
// candidates per step, and a flush per step would dominate their time.
constexpr uint32_t LV_WIDE_THREADS = 1024, LV_WIDE_CAP = 2048;    // single graph
constexpr uint32_t LV_NARROW_THREADS = 256, LV_NARROW_CAP = 1024; // batched slots
constexpr uint32_t LV_FIRST = 32;  // witness probes of a pair before it is looked at again
constexpr uint32_t LV_DENSE = 256; // of those, most tested on bitset rows per flush

// LDS of one workgroup of the ball-change step.  flag[] is all zero between
// steps.
template <uint32_t LV_THREADS, uint32_t LV_CAP>
struct LevelLds {
  // a candidate: the pair, the endpoint whose ball is probed, the other one's
  // row, its first probe's number, and whether a witness was found
  uint32_t x[LV_CAP], w[LV_CAP], b[LV_CAP], beg[LV_CAP], deg[LV_CAP], off[LV_CAP], flag[LV_CAP];
  uint16_t rest[LV_CAP];     // candidates with probes left after the first few
  uint32_t dense[LV_DENSE];  // candidates tested by bitset rows (see the flush)
  uint32_t ndense, longrow, busy[2];
  unsigned long long fill;    // candidates (low half) and their first probes (high half)
  unsigned long long more;    // rest[] (low half) and its probes (high half)
  unsigned long long res[2];  // a drop pass's items (low half) and events (high half)
  uint32_t bres[2];           // ... and where the workgroup's start
  uint32_t stat[5];  // stats mode: items, slots, candidates, probes, drops
};

// Level-j events.  Each workgroup turns its share of the nit work items into
// candidate pairs (quick filters: still in the j-ball, not directly
// reachable), buffers them in LDS, then tests every buffered pair at once:
// the pair's probes (the live neighbours y of its lower-degree endpoint a,
// each checked against the other endpoint's (j-1)-ball) are laid out flat
// over all threads of the workgroup.  Pairs with no witness leave the ball.
// Most rounds give a workgroup a handful of pairs, and their time is the chain
// of dependent loads and barriers, so a flush has as few of both as it can:
// append() numbers the probes as pairs come, so no scan over the buffer; a
// slot's liveness and neighbour are one word; list space is summed in LDS and
// reserved by two lanes at once.  With the marking step's changes: Chung-Lu
// 100k h = 2 287 -> 238 ms, R-MAT 16 h = 2 1,207 -> 1,003 ms, Chung-Lu 5,001
// h = 3 288 -> 192 ms (there mostly the word-wise candidates) a decomposition.
// wg of nwg workgroups call it together; TEAM: inside the team kernel, where
// other workgroups' writes of the same launch are read (see ld()).
template <uint32_t LV_THREADS, uint32_t LV_CAP, bool TEAM>
__device__ __forceinline__ void level_step(const Dev& d, const RoundCtx rc, uint32_t j, uint32_t nit, uint32_t wg,
                           uint32_t nwg, LevelLds<LV_THREADS, LV_CAP>& s) {
  static_assert(LV_CAP >= 2 * LV_THREADS && LV_CAP % LV_THREADS == 0, "two emission steps fit");
  constexpr uint32_t LV_WAVES = LV_THREADS / WAVE;
  uint32_t *cx = s.x, *cw = s.w, *cb = s.b, *cbeg = s.beg, *cdeg = s.deg, *coff = s.off;
  uint32_t *cflag = s.flag, *cdense = s.dense, *s_busy = s.busy;
  Ctl* c = d.ctl;
  const uint32_t wave = threadIdx.x / WAVE, lane = lane_id(), words = c->words;
  // items are dealt to workgroups first, then to their waves, so a round
  // with few items still spreads its candidates (and their probes) over as
  // many CUs as it has items
  const uint32_t stride = nwg * LV_WAVES;
  uint32_t it = wave * nwg + wg;
  const bool counting = !TEAM && d.spart != nullptr;
  if (wg >= nit) return;  // whole workgroup idle
  const uint64_t* Lj = d.L[j];
  const uint64_t* Lp = d.L[j - 1];
  const Item* items = d.itl[j];
  if (threadIdx.x == 0) {
    s.fill = 0;
    s.more = 0;
    s.longrow = 0;
    s.ndense = 0;
    s.res[0] = s.res[1] = 0;
    s_busy[0] = s_busy[1] = 0;
  }
  uint32_t par = 0, pass = 0;
  uint32_t next = wg;  // wave 0's next item
  const bool merge = d.perm != nullptr;
  // KIND_A_WORDS item in progress: this lane's word of candidates, their number
  // up to this lane's, in all and so far taken
  uint64_t wd = 0;
  uint32_t wincl = 0, wtotal = 0, wdone = 0;
  bool inword = false;
  uint32_t X = 0, Wv = 0;
  // Append this wave's candidates (X, Wv) to the buffer.  The witness probes
  // run over the endpoint with fewer active slots.  One LDS atomic per wave
  // reserves buffer entries (low half) and first-probe numbers (high half)
  // together, so both ascend in the same order and the flush needs no scan.
  auto append = [&](bool have, uint32_t bx, uint32_t dx, uint32_t bw, uint32_t dw) {
    const uint64_t bal = __ballot(have);
    if (!bal) return;
    const uint32_t deg = have ? min(dx, dw) : 0u;
    uint32_t psum;
    const uint32_t pex = wave_excl_scan(min(deg, LV_FIRST), &psum);
    if (__ballot(deg > LV_FIRST) && lane == 0) s.longrow = 1;
    unsigned long long at = 0;
    if (lane == 0)
      at = atomicAdd(&s.fill, ((unsigned long long)psum << 32) | (uint32_t)__popcll(bal));
    const uint32_t slot = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)at) +
                          (uint32_t)__popcll(bal & ((1ull << lane) - 1));
    const uint32_t p0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(at >> 32)) + pex;
    if (have) {
      cx[slot] = X;
      cw[slot] = Wv;
      cb[slot] = dx <= dw ? Wv : X;
      cbeg[slot] = dx <= dw ? bx : bw;
      cdeg[slot] = deg;
      coff[slot] = p0;
    }
  };
  __syncthreads();
  while (true) {
    // ---- one emission step per wave: at most 64 candidates ----
    uint32_t examined = 0;  // stats mode
    bool it_taken = false;
    uint32_t cands = 0;
    if (it < nit) {
      const Item I = ld_item<TEAM>(items + it);
      const uint32_t kind = meta_kind(I.meta), len = meta_len(I.meta);
      if (kind == KIND_A_WORDS) {
        // the candidates of a whole word at once: members of z's old
        // (j-1)-ball that are in x's j-ball and not within j-1 hops of x
        // (x itself is); four coalesced rows in place of two gathers per pair
        if (!inword) {
          wd = 0;
          if (lane < len) {
            const size_t o = (size_t)I.y * d.W + I.base + lane;
            const size_t ox = (size_t)I.x * d.W + I.base + lane;
            const uint64_t old = ld<TEAM>(Lp + o) | ld<TEAM>(d.Dm[j - 1] + o);
            wd = old & ld<TEAM>(Lj + ox) & ~ld<TEAM>(Lp + ox);
            if (counting) examined = (uint32_t)__popcll(old);
          }
          wincl = wave_incl_scan((uint32_t)__popcll(wd));
          wtotal = wave_last(wincl);
          wdone = 0;
          inword = true;
        }
        // lane l takes candidate wdone + l: the word that holds it, and its bit
        const uint32_t t = wdone + lane;
        const bool have = t < wtotal;
        uint32_t own = 0;
#pragma unroll
        for (uint32_t step = 32; step > 0; step >>= 1) {
          const uint32_t v = (uint32_t)__shfl(wincl, (int)(own + step - 1), WAVE);
          if (v <= t) own += step;
        }
        own = min(own, WAVE - 1u);
        uint64_t word = ((uint64_t)(uint32_t)__shfl((uint32_t)(wd >> 32), own, WAVE) << 32) |
                        (uint32_t)__shfl((uint32_t)wd, own, WAVE);
        uint32_t nth = t - ((uint32_t)__shfl(wincl, own, WAVE) - (uint32_t)__popcll(word));
        uint32_t bit = 0;
#pragma unroll
        for (uint32_t step = 32; step > 0; step >>= 1) {
          const uint32_t below = (uint32_t)__popcll(word & ((1ull << step) - 1));
          if (nth >= below) {
            nth -= below;
            word >>= step;
            bit += step;
          }
        }
        X = I.x;
        uint32_t bx = 0, dx = 0, bw = 0, dw = 0;
        if (have) {
          Wv = (I.base + own) * 64 + bit;
          bx = d.rp[X];
          dx = d.len[X];
          bw = d.rp[Wv];
          dw = d.len[Wv];
        }
        append(have, bx, dx, bw, dw);
        wdone += WAVE;
        cands = wdone <= wtotal ? WAVE : wtotal - (wdone - WAVE);
        if (wdone >= wtotal) {
          if (wtotal == 0) cands = 0;
          inword = false;
          it += stride;
          it_taken = true;
        }
      } else {
        const uint32_t extra = meta_extra(I.meta);
        const uint32_t v = meta_vstart(I.meta) + lane;
        bool have = false;
        if (lane < len) {
          if (extra && v == 0) {
            have = true;
            X = I.x;
            Wv = I.y;
          } else {
            const uint32_t q = I.base + v - extra;
            // live after this round, or (KIND_A) peeled in it
            const uint32_t sw = (uint32_t)ld<TEAM>(d.ce + q), y2 = sw & ~SLOT_GONE;
            if (!(sw & SLOT_GONE) || (kind == KIND_A_SLOTS && ld<TEAM>(d.srem + q) == rc.r)) {
              have = true;
              X = (kind == KIND_A_SLOTS) ? I.x : y2;
              Wv = (kind == KIND_A_SLOTS) ? y2 : I.y;
            }
          }
        }
        if (counting) examined = lane < len;
        it += stride;
        it_taken = true;
        // quick filters: a real pair, still in the j-ball, not within j-1
        // hops.  Balls are symmetric: both bits are read from the row of the
        // vertex that the item's pairs share, where the lanes' ascending
        // neighbours lie in few cache lines, together with the row extents.
        uint32_t bx = 0, dx = 0, bw = 0, dw = 0;
        have = have && X != Wv;
        if (have) {
          const uint32_t at = kind == KIND_A_SLOTS ? Wv : X;
          const size_t o = (size_t)(kind == KIND_A_SLOTS ? X : Wv) * d.W + (at >> 6);
          const uint64_t sh = at & 63;
          const uint64_t wj = ld<TEAM>(Lj + o), wp = ld<TEAM>(Lp + o);
          bx = d.rp[X];
          dx = d.len[X];
          bw = d.rp[Wv];
          dw = d.len[Wv];
          have = ((wj >> sh) & 1ull) && !((wp >> sh) & 1ull);
        }
        cands = (uint32_t)__popcll(__ballot(have));
        append(have, bx, dx, bw, dw);
      }
    }
    if (counting) {
      const uint32_t nex = wave_sum(examined);
      if (lane == 0) {
        if (it_taken) atomicAdd(&s.stat[0], 1u);
        atomicAdd(&s.stat[1], nex);
        atomicAdd(&s.stat[2], cands);
      }
    }
    // more to emit: at level 2 an item takes one step, so wave 0's next item
    // tells for the whole workgroup; above, the waves say so
    bool busy;
    next += stride;
    if (j == 2) {
      __syncthreads();  // appends visible
      busy = next < nit;
    } else {
      if (lane == 0 && (it < nit || inword)) s_busy[par] = 1u;
      __syncthreads();  // appends and flags visible
      busy = s_busy[par] != 0;
      par ^= 1;
      if (threadIdx.x == 0) s_busy[par] = 0;
    }
    const uint32_t n = (uint32_t)s.fill, total = (uint32_t)(s.fill >> 32);
    const bool longrow = s.longrow != 0;
    if (n == 0 && !busy) break;
    if (n + LV_THREADS <= LV_CAP && busy) {
      __syncthreads();  // everyone has read the counts before anyone appends
      continue;
    }
    // ---- flush: look for a witness of every buffered pair ----
    // The pairs' probes (a live neighbour y of the lower-degree endpoint,
    // checked against the other's (j-1)-ball) are laid out flat over all
    // threads of the workgroup: the first LV_FIRST of every pair, then the rest
    // of the pairs without a witness so far.  Rows have their hubs first, so
    // most pairs that have a witness show one early, and long rows are
    // scanned for few others.
    if (counting && threadIdx.x == 0) s.stat[3] += total;
    // four probes per thread in flight: owners found in LDS first, then all
    // slot loads, then all ball-word loads
    auto probe = [&](uint32_t cnt, uint32_t probes, uint32_t skip, auto&& who) {
      constexpr uint32_t PU = 4;
      for (uint32_t p0 = threadIdx.x; p0 < probes; p0 += PU * LV_THREADS) {
        uint32_t own[PU], q[PU], y[PU];
        bool act[PU];
#pragma unroll
        for (uint32_t u = 0; u < PU; ++u) {
          const uint32_t pidx = p0 + u * LV_THREADS;
          uint32_t lo = 0, hi = cnt;
          while (hi - lo > 1) {
            const uint32_t mid = (lo + hi) >> 1;
            if (coff[mid] <= pidx) lo = mid; else hi = mid;
          }
          own[u] = who(lo);
          act[u] = pidx < probes && !cflag[own[u]];
          q[u] = cbeg[own[u]] + skip + (pidx - coff[lo]);
        }
#pragma unroll
        for (uint32_t u = 0; u < PU; ++u)
          y[u] = act[u] ? (uint32_t)ld<TEAM>(d.ce + q[u]) : SLOT_GONE;
#pragma unroll
        for (uint32_t u = 0; u < PU; ++u)
          if (!(y[u] & SLOT_GONE)) {
            const uint64_t word = ld<TEAM>(row(Lp, d.W, cb[own[u]]) + (y[u] >> 6));
            if ((word >> (y[u] & 63)) & 1ull) cflag[own[u]] = 1;
          }
      }
    };
    probe(n, total, 0, [](uint32_t i) { return i; });
    __syncthreads();
    // Pairs with probes left.  Where that is many for the words of a ball row,
    // one wave ANDs two rows instead, to the first non-zero word: the
    // witnesses are exactly the members of L[1](low) & L[j-1](other) (L[1]
    // holds the live closed neighbourhood, and low itself is not within j-1
    // hops of the other endpoint).  A probe gathers one word, the rows come
    // 64 words a load: the AND pays from a quarter of the words on.
    if (longrow) {
      for (uint32_t b0 = 0; b0 < n; b0 += LV_THREADS) {
        const uint32_t i = b0 + threadIdx.x;
        uint32_t left = i < n && !cflag[i] && cdeg[i] > LV_FIRST ? cdeg[i] - LV_FIRST : 0u;
        if (!__ballot(left != 0)) continue;
        const bool big = left > words / 4;
        const uint64_t bd = __ballot(big);
        if (bd) {
          uint32_t at = 0;
          if (lane == 0) at = atomicAdd(&s.ndense, (uint32_t)__popcll(bd));
          at = (uint32_t)__builtin_amdgcn_readfirstlane((int)at) +
               (uint32_t)__popcll(bd & ((1ull << lane) - 1));
          if (big && at < LV_DENSE) {  // the others keep their neighbour probes
            cdense[at] = i;
            left = 0;
          }
        }
        const uint64_t bl = __ballot(left != 0);
        uint32_t psum;
        const uint32_t pex = wave_excl_scan(left, &psum);
        unsigned long long at = 0;
        if (lane == 0) at = atomicAdd(&s.more, ((unsigned long long)psum << 32) | (uint32_t)__popcll(bl));
        const uint32_t slot = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)at) +
                              (uint32_t)__popcll(bl & ((1ull << lane) - 1));
        const uint32_t p0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(at >> 32)) + pex;
        if (left) {
          s.rest[slot] = (uint16_t)i;
          coff[slot] = p0;
        }
      }
      __syncthreads();
      const uint32_t nrest = (uint32_t)s.more, left_total = (uint32_t)(s.more >> 32);
      const uint32_t ndense = min(s.ndense, LV_DENSE);
      if (counting && threadIdx.x == 0) s.stat[3] += left_total;
      probe(nrest, left_total, LV_FIRST, [&](uint32_t i) { return (uint32_t)s.rest[i]; });
      for (uint32_t k = wave; k < ndense; k += LV_WAVES) {
        const uint32_t i = cdense[k];
        const uint32_t hi = cb[i], lo = (hi == cx[i]) ? cw[i] : cx[i];
        const uint64_t* ra = row(d.L[1], d.W, lo);
        const uint64_t* rb = row(Lp, d.W, hi);
        uint32_t nread = 0;
        bool found = false;
        for (uint32_t w0 = 0; w0 < words && !found; w0 += 4 * WAVE) {
          uint64_t any = 0;
  #pragma unroll
          for (uint32_t u = 0; u < 4; ++u) {
            const uint32_t wi = w0 + u * WAVE + lane;
            if (wi < words) any |= ld<TEAM>(ra + wi) & ld<TEAM>(rb + wi);
          }
          nread += min(4 * WAVE, words - w0);
          found = __ballot(any != 0) != 0;
        }
        if (lane == 0) {
          if (found) cflag[i] = 1;
          if (counting) atomicAdd(&s.stat[3], nread);  // a word pair counts as one probe
        }
      }
      __syncthreads();
    }
    // ---- pairs without a witness leave the j-ball (both directions) ----
    // Eight neighbouring pairs to a wave, the next eight to the next wave: the
    // pairs of one item are often all hubs, with hundreds of follow-up items
    // that one wave would write alone, and eight are enough to merge atomics.
    for (uint32_t base = 0; base < n; base += LV_THREADS) {
      const uint32_t i =
          base + (merge ? ((lane >> 3) * LV_WAVES + wave) * 8 + (lane & 7) : threadIdx.x);
      const bool drop = i < n && !cflag[i];
      uint32_t x = 0, w = 0, bx = 0, dx = 0, bw = 0, dw = 0;
      if (i < n) {
        x = cx[i];
        w = cw[i];
      }
      if (drop) {
        bx = d.rp[x];
        dx = d.len[x];
        bw = d.rp[w];
        dw = d.len[w];
      }
      bool w1 = false, w2 = false;
      if (__ballot(drop)) clear_pairs<TEAM>(d.L[j], d.Dm[j], d.W, x, w, drop, merge, &w1, &w2);
      if (counting && (w1 || w2)) atomicAdd(&s.stat[4], (uint32_t)w1 + (uint32_t)w2);
      // Follow-up work of both events: the events themselves, and items over
      // the row of each event's source -- the support update (j == h), else
      // the next level's candidates (y, w) over that row plus (x, w) itself.
      // Both lists are reserved once per workgroup: device-scope atomics on
      // one address serialise, and a large round has thousands of wavefronts
      // with drops.
      const uint32_t extra = j == d.h ? 0u : 1u;
      const uint32_t list = j == d.h ? d.h + 1 : j + 1;
      const uint32_t nx = w1 ? dx + extra : 0, nw = w2 ? dw + extra : 0;
      const uint32_t c1 = chunks_of(nx), c2 = chunks_of(nw);
      const uint32_t ne = (uint32_t)w1 + (uint32_t)w2;
      uint32_t t1, t2, te;
      const uint32_t e1 = wave_excl_scan(c1, &t1), e2 = wave_excl_scan(c2, &t2);
      const uint32_t ee = wave_excl_scan(ne, &te);
      unsigned long long off = 0;
      if (lane == 0 && te)
        off = atomicAdd(&s.res[pass], ((unsigned long long)te << 32) | (t1 + t2));
      __syncthreads();
      if (wave == LV_WAVES - 1 && lane < 2) {
        // the last wave: in small rounds it has no pair, and so no atomics in
        // flight for the reservation to wait behind
        const unsigned long long sum = s.res[pass];
        const uint32_t v = lane ? (uint32_t)(sum >> 32) : (uint32_t)sum;
        uint32_t* at = lane ? &c->cnt[j][rc.p].nev : &c->cnt[list][rc.p].nit;
        s.bres[lane] = v ? at_add<TEAM>(at, v) : 0u;
        s.res[pass ^ 1] = 0;
      }
      pass ^= 1;
      __syncthreads();
      const uint32_t ifirst = s.bres[0] + (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)off);
      const uint32_t efirst =
          s.bres[1] + (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(off >> 32));
      {
        const uint64_t exw = ((uint64_t)x << 32) | w, ewx = ((uint64_t)w << 32) | x;
        const uint32_t slot = efirst + ee;
        bool over = false;
        for (uint32_t k = 0; k < ne; ++k) {
          if (slot + k < d.evcap) d.evl[j][rc.p][slot + k] = (k || !w1) ? ewx : exw;
          else over = true;
        }
        if (over) c->cnt[j][rc.p].ovf = 1;
      }
      if (j == d.h) {
        // support items carry the slot base of their chunk
        emit_items_wave<ITEM_SLOTS>(d, rc.p, list, ifirst, t1, e1, c1, 0, 0, x, w, bx, nx);
        emit_items_wave<ITEM_SLOTS>(d, rc.p, list, ifirst + t1, t2, e2, c2, 0, 0, w, x, bw, nw);
      } else {
        emit_items_wave<ITEM_ROW>(d, rc.p, list, ifirst, t1, e1, c1, KIND_B_SLOTS, 1, x, w, bx, nx);
        emit_items_wave<ITEM_ROW>(d, rc.p, list, ifirst + t1, t2, e2, c2, KIND_B_SLOTS, 1, w, x, bw,
                                  nw);
      }
    }
    for (uint32_t i = threadIdx.x; i < n; i += LV_THREADS) cflag[i] = 0;
    if (threadIdx.x == 0) {
      s.fill = 0;
      s.longrow = 0;
      s.more = 0;
      s.ndense = 0;
    }
    __syncthreads();
    if (!busy) break;
  }
}

template <uint32_t LV_THREADS, uint32_t LV_CAP>
__global__ void __launch_bounds__(LV_THREADS) k_level(const Dev* __restrict__ devs, uint32_t j) {
  __shared__ LevelLds<LV_THREADS, LV_CAP> s;
  const Dev& d = devs[blockIdx.y];
  if (j > d.h) return;  // this slot's graph has fewer levels
  Ctl* c = d.ctl;
  if (c->done) return;
  if (c->halt || c->phase > j) return;  // phase: earlier steps were done by the team kernel
  // a round that peels every remaining edge leaves no ball or support that
  // could matter: the decomposition ends with it
  if (c->nRc.v == c->live) return;
  const RoundCtx rc = round_ctx(c);
  if (!c->recovering && (c->cnt[j][rc.p].iovf || (d.serial & 4u))) {
    // work list overflowed (or forced): halt; the host re-runs this level in windows
    if (blockIdx.x == 0 && threadIdx.x == 0) {
      c->halt = 1;
      c->halt_step = j;
      d.status[1] = 1;
    }
    return;
  }
  for (uint32_t i = threadIdx.x; i < LV_CAP; i += LV_THREADS) s.flag[i] = 0;
  if (threadIdx.x < 5) s.stat[threadIdx.x] = 0;
  __syncthreads();
  level_step<LV_THREADS, LV_CAP, false>(d, rc, j, min(c->cnt[j][rc.p].nit, d.itcap), blockIdx.x,
                                        gridDim.x, s);
  if (d.spart) {
    __syncthreads();
    if (threadIdx.x < 5) d.spart[threadIdx.x * STAT_GRID + blockIdx.x] = s.stat[threadIdx.x];
  }
}


__device__ __forceinline__ void reset_team(const Dev& d) {
  if (d.team)
    for (uint32_t i = threadIdx.x; i < sizeof(Team) / 4; i += blockDim.x)
      reinterpret_cast<uint32_t*>(d.team)[i] = 0;
}

// ---- K4: support update --------------------------------------------------
// Top-level event (a -> w): every live edge (a,b) that had w as a common
// h-neighbour loses it.  Old/new rule: w counts against (a,b) if it was in
// b's old ball when a < b, and in b's new ball when a > b (see the header).
// wg of nwg workgroups of `wpb` waves call it together; stat: stats mode only.
template <bool TEAM, uint32_t U>
__device__ __forceinline__ void support_step(const Dev& d, const RoundCtx rc, uint32_t nit, uint32_t wg,
                             uint32_t nwg, uint32_t wpb, uint32_t* stat) {
  const uint32_t lane = lane_id();
  const uint64_t* Lh = d.L[d.h];
  const uint64_t* Dh = d.Dm[d.h];
  uint32_t* Rn = d.R[rc.p ^ 1];
  const Item* items = d.itl[d.h + 1];
  uint32_t* nPush = &d.ctl->nPushc[rc.p].v;
  // Items are dealt in blocks of up to four: neighbours in the list share the
  // event's target (whose ball row then stays in this CU's L1) or its source
  // row, and waves next to each other share an XCD's L2; longer blocks leave
  // waves with only long rows.  Rounds with fewer items than waves deal them
  // to workgroups first.
  const bool flip = d.perm != nullptr;
  const uint32_t waves = nwg * wpb, wave = threadIdx.x / WAVE;
  const uint32_t sh = nit <= waves ? 0 : nit <= 2 * waves ? 1 : 2;  // log2 of the block
  const uint32_t wid = sh == 0 ? wave * nwg + wg : (TEAM ? wg : xcd_first(wg, nwg)) * wpb + wave;
  // this wave's s-th item
  auto item_at = [&](uint32_t s) {
    return ((wid + (s >> sh) * waves) << sh) + (s & ((1u << sh) - 1));
  };
  // U items per step; the step's successors and their slots load while the
  // current items' ball words and support atomics are in flight: more memory
  // operations outstanding per wave than one item's dependent chain.
  // a slot is one 8-byte word: neighbour b (with SLOT_GONE once the edge is
  // peeled, i.e. not alive after this round) and edge id e
  struct Slot {
    Item I;
    uint32_t b, e;
  };
  auto fetch = [&](uint32_t s, Slot& S) {
    S.I = Item{0, 0, ~0u, 0};
    S.b = SLOT_GONE;
    S.e = 0;
    const uint32_t i = item_at(s);
    if (i < nit) {
      S.I = ld_item<TEAM>(items + i);
      if (lane < meta_len(S.I.meta)) {
        const uint64_t w = ld<TEAM>(d.ce + S.I.base + lane);
        S.b = (uint32_t)w;
        S.e = (uint32_t)(w >> 32);
      }
    }
  };
  // w in b's old ball when the event's source a < b, in its new ball when
  // a > b; the other way round in renumbered graphs: the long rows are the
  // hubs', which come first, and then need the new ball only (the other side
  // reads the change marks too)
  auto hit_of = [&](const Slot& S) -> bool {
    if (S.b & SLOT_GONE) return false;
    const size_t o = (size_t)S.I.y * d.W + (S.b >> 6);
    uint64_t word = ld<TEAM>(Lh + o);
    if ((S.I.x < S.b) != flip) word |= ld<TEAM>(Dh + o);
    return (word >> (S.b & 63)) & 1ull;
  };
  Slot A[U];
#pragma unroll
  for (uint32_t u = 0; u < U; ++u) fetch(u, A[u]);
  uint32_t acc = 0;  // lost by this lane's edge to the items so far of the same slots
  for (uint32_t it = 0; item_at(it) < nit; it += U) {
    bool hit[U];
    uint32_t e[U], base[U + 1], dec[U];
#pragma unroll
    for (uint32_t u = 0; u < U; ++u) {
      hit[u] = hit_of(A[u]);
      e[u] = A[u].e;
      base[u] = A[u].I.base;
    }
    if (!TEAM && stat) {
      uint32_t hits = 0, slots = 0, taken = 0;
      for (uint32_t u = 0; u < U; ++u) {
        taken += item_at(it + u) < nit;
        hits += (uint32_t)__popcll(__ballot(hit[u]));
        slots += meta_len(A[u].I.meta);
      }
      if (lane == 0) {
        atomicAdd(&stat[0], taken);
        atomicAdd(&stat[1], slots);
        atomicAdd(&stat[2], hits);
      }
    }
#pragma unroll
    for (uint32_t u = 0; u < U; ++u) fetch(it + U + u, A[u]);
    base[U] = A[0].I.base;
    // items over the same slots (events of one source) are charged together
#pragma unroll
    for (uint32_t u = 0; u < U; ++u) {
      acc += hit[u];
      dec[u] = base[u] == base[u + 1] ? 0u : acc;
      if (base[u] != base[u + 1]) acc = 0;
    }
    uint32_t push = 0;
#pragma unroll
    for (uint32_t u = 0; u < U; ++u)
      if (dec[u]) {
        const uint32_t old = at_sub<TEAM>(&d.sup[e[u]], dec[u]);
        push |= (uint32_t)(old > rc.k - 2 && old - dec[u] <= rc.k - 2) << u;
      }
    if (__ballot(push != 0)) {
      uint32_t slot = wave_reserve<TEAM>(nPush, (uint32_t)__popc(push));
#pragma unroll
      for (uint32_t u = 0; u < U; ++u)
        if ((push >> u) & 1u) Rn[slot++] = e[u];
    }
  }
}

__global__ void __launch_bounds__(256) k_support(const Dev* __restrict__ devs, uint32_t after_team) {
  const Dev& d = devs[blockIdx.y];
  Ctl* c = d.ctl;
  // the team of this graph step has gone; its meeting point is free again
  if (after_team && blockIdx.x == 0) reset_team(d);
  if (c->done) return;
  const uint32_t list = d.h + 1;
  if (c->halt || c->phase > list) return;
  if (c->nRc.v == c->live) return;  // the last round: nothing left to update
  const RoundCtx rc = round_ctx(c);
  if (!c->recovering && (c->cnt[list][rc.p].iovf || (d.serial & 8u))) {
    if (blockIdx.x == 0 && threadIdx.x == 0) {
      c->halt = 1;
      c->halt_step = list;
      d.status[1] = 1;
    }
    return;
  }
  __shared__ uint32_t s_stat[3];  // stats mode: items, slots, hits
  const bool counting = d.spart != nullptr;
  if (counting) {
    if (threadIdx.x < 3) s_stat[threadIdx.x] = 0;
    __syncthreads();
  }
  support_step<false, 2>(d, rc, min(c->cnt[list][rc.p].nit, d.itcap), blockIdx.x, gridDim.x,
                      blockDim.x / WAVE, counting ? s_stat : nullptr);
  if (counting) {
    __syncthreads();
    if (threadIdx.x < 3) d.spart[(5 + threadIdx.x) * STAT_GRID + blockIdx.x] = s_stat[threadIdx.x];
  }
}

// Stats mode: fold the per-workgroup counters of one launch into Ctl::stat.
__global__ void k_stats_fold(const Dev* __restrict__ dp, uint32_t first, uint32_t count,
                             uint32_t grid) {
  const Dev& d = *dp;
  __shared__ uint64_t acc[NSTAT];
  if (threadIdx.x < NSTAT) acc[threadIdx.x] = 0;
  __syncthreads();
  for (uint32_t c = first; c < first + count; ++c) {
    uint64_t s = 0;
    for (uint32_t b = threadIdx.x; b < grid; b += blockDim.x) {
      s += d.spart[c * STAT_GRID + b];
      d.spart[c * STAT_GRID + b] = 0;  // a launch that returns early leaves zeros
    }
    atomicAdd((unsigned long long*)&acc[c], (unsigned long long)s);
  }
  __syncthreads();
  if (threadIdx.x < NSTAT && threadIdx.x >= first && threadIdx.x < first + count)
    d.ctl->stat[threadIdx.x] += acc[threadIdx.x];
}

// ---- K5: end of round ------------------------------------------------------
// Ends a round that the whole chip ran (the team kernel ends the others
// itself); phase: what the next one starts with, 0 or ROUND_CLOSED.  One
// wavefront closes the round (counters, next round's peel set and level-jump
// flag).  When the round pushed no edge, the next round starts with a level
// jump, and every workgroup computes its share of the live minimum now (not
// for ROUND_CLOSED: the team kernel has its own).  A workgroup may look while
// the closing wavefront is at work, or after it, when the round number may
// have moved on: so it asks whether either parity's push count is zero.  Both
// stay as they are until the next round's marking, so a minimum is computed
// too often only in the round of a jump.
// Closing is a handful of words, each on a line of its own that the kernels
// before wrote in memory: lane j has level j's, so that all of them are in
// flight at once and the stores follow (R-MAT 16 h = 2: 4.0 us for one thread
// one after the other).
// compacted: rows were compacted, if due, before this round.
__global__ void __launch_bounds__(256) k_end(const Dev* __restrict__ devs, uint32_t phase,
                                             uint32_t compacted) {
  const Dev& d = devs[blockIdx.y];
  Ctl* c = d.ctl;
  // one decision per workgroup, taken before its closing wavefront (workgroup
  // 0) changes anything, so that every thread of it takes the same branch
  __shared__ uint32_t s_mode;  // 0 close only, 1 minimum and close, 2 nothing
  if (threadIdx.x == 0) {
    const uint32_t none = (c->done != 0) | (c->halt != 0) | (c->phase == ROUND_CLOSED);
    const uint32_t jump = (c->nPushc[0].v == 0) | (c->nPushc[1].v == 0);
    s_mode = none ? 2u : phase == ROUND_CLOSED ? 0u : jump;
  }
  __syncthreads();
  const uint32_t mode = s_mode;
  if (mode == 2) return;
  if (mode == 1) jump_partials(d);
  if (blockIdx.x != 0 || threadIdx.x >= WAVE) return;
  const uint32_t lane = threadIdx.x, h = d.h, r = c->r, p = r & 1, q = p ^ 1;
  const uint32_t nR = c->nRc.v, was = c->live, live = was - nR;
  const uint32_t pushed = p ? c->nPushc[1].v : c->nPushc[0].v;
  const bool level = lane >= 1 && lane <= h + 1;  // h + 1: the support items
  uint32_t over = 0, nev = 0;
  uint64_t levents = 0;
  if (level) {
    const Cnt& n = c->cnt[lane][p];
    over = n.ovf | n.iovf;
    nev = n.nev;
    if (lane <= h) levents = c->levents[lane];
  }
  if (lane == 1) nev = 2 * nR;  // level-1 events: both directions of every peeled edge
  const uint64_t events = c->events, overflows = c->overflows;
  const uint32_t top = __shfl(nev, (int)h, WAVE);
  const bool any = __ballot(over != 0) != 0;
  if (level) {
    // the other parity's counters, for the next round (this round's stay: the
    // next one clears the change marks they list and peels the edges it pushed)
    Cnt& n = c->cnt[lane][q];
    n.nit = n.iovf = n.nev = n.ovf = 0;
    if (lane <= h) c->levents[lane] = levents + nev;
  }
  if (lane == 1) c->cnt[1][p].nev = nev;
  if (lane == 0) {
    if (phase == ROUND_CLOSED) c->nPushc[q].v = 0;  // else the marking does it
    if (compacted && was <= c->compact_at) c->compact_at = compact_next(was);
    c->events = events + top;
    c->overflows = overflows + (any ? 1 : 0);
    c->live = live;
    c->r = r + 1;
    c->nRc.v = pushed;
    c->jump = pushed == 0;
    c->phase = phase;
    d.status[2] = live;
    d.status[3] = r + 1;
    if (live == 0) {
      c->done = 1;
      d.status[0] = 1;
    }
  }
}

// A finished graph's outputs in the caller's edge order (renumbered graphs).
// Written here and not as edges are peeled: neighbouring own numbers are far
// apart in the caller's order, and scattered stores to lines that other XCDs
// are writing too cost more than this pass (Chung-Lu 100k h = 1: the marking
// of the largest round 740 us with them, 274 us without).
__global__ void __launch_bounds__(256) k_outputs(Dev d) {
  if (d.ctl->err) return;
  for (uint32_t e = blockIdx.x * blockDim.x + threadIdx.x; e < d.m; e += gridDim.x * blockDim.x) {
    const uint32_t own = d.ne[e];
    d.out_t[e] = d.t[own];
    if (d.out_rho) d.out_rho[e] = d.rho[own];
  }
}

// After the initial pass of a newly admitted graph: publish its state
// (malformed CSR: finished with error).
__global__ void k_post_init(Dev d) {
  if (blockIdx.x != 0) return;
  reset_team(d);
  if (threadIdx.x != 0) return;
  Ctl* c = d.ctl;
  if (c->err) c->done = 1;
  d.status[0] = c->err ? 2u : (c->done ? 1u : 0u);
  d.status[1] = 0;
  d.status[2] = c->err ? 0u : c->live;
  d.status[3] = 0;
}

// ---- recovery of a round whose work list overflowed ----------------------
// The host re-creates the work items of the overflowed step from their
// sources, a window of sources at a time small enough for the list, and
// runs the ordinary step kernel on each window.  Re-testing a pair is
// harmless: pairs that already left fail the ball-bit filter.  Sources of
// level j: the directed removals x-lost-z of the round (index < 2|R|), then
// the level-(j-1) events from their list, or, when that list overflowed,
// the bits of the level-(j-1) change marks (row-major, 64 per word).

// Follow-up items of the event (x -> w) at list `list` (all lanes call).
__device__ __forceinline__ void fill_event_items(const Dev& d, uint32_t p, uint32_t list, bool support,
                                                 bool has, uint32_t x, uint32_t w) {
  uint32_t bx = 0, nx = 0;
  if (has) {
    bx = d.rp[x];
    nx = d.len[x] + (support ? 0u : 1u);
  }
  if (support) emit_group<ITEM_SLOTS, false>(d, p, list, 0, 0, x, w, bx, nx);
  else emit_group<ITEM_ROW, false>(d, p, list, KIND_B_SLOTS, 1, x, w, bx, nx);
}

// Change-mark bits [blo, bhi) of level jm as events (x -> w): follow-up
// items at `list` (support items when `support`).
__device__ void fill_from_marks(const Dev& d, uint32_t p, uint32_t jm, uint32_t list, bool support,
                                uint64_t blo, uint64_t bhi) {
  if (blo >= bhi) return;
  const uint64_t wlo = blo / 64, whi = (bhi + 63) / 64;
  const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
  for (uint64_t wb = wlo + blockIdx.x * (uint64_t)blockDim.x + (threadIdx.x & ~(WAVE - 1)); wb < whi;
       wb += stride) {
    const uint64_t kw = wb + lane_id();
    uint64_t wd = 0;
    uint32_t x = 0, word = 0;
    if (kw < whi) {
      x = (uint32_t)(kw / d.W);
      word = (uint32_t)(kw % d.W);
      wd = row(d.Dm[jm], d.W, x)[word];
      if (kw == wlo && (blo & 63)) wd &= ~0ull << (blo & 63);
      if (kw == whi - 1 && (bhi & 63)) wd &= (1ull << (bhi & 63)) - 1;
    }
    while (__ballot(wd != 0)) {
      const bool has = wd != 0;
      uint32_t w = 0;
      if (has) {
        w = word * 64 + (uint32_t)(__ffsll((unsigned long long)wd) - 1);
        wd &= wd - 1;
      }
      fill_event_items(d, p, list, support, has, x, w);
    }
  }
}

// Listed events [elo, ehi) of level je (or the directed removals when
// `removals`): follow-up items at `list`.
__device__ void fill_from_list(const Dev& d, uint32_t je, bool removals, uint32_t p,
                               uint32_t list, bool support, uint64_t elo, uint64_t ehi) {
  const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
  for (uint64_t b = elo + blockIdx.x * (uint64_t)blockDim.x + (threadIdx.x & ~(WAVE - 1)); b < ehi;
       b += stride) {
    const uint64_t i = b + lane_id();
    const bool has = i < ehi;
    uint32_t x = 0, w = 0;
    if (has) {
      if (removals) {
        const uint32_t e = d.R[p][i >> 1];
        x = (i & 1) ? d.ev[e] : d.eu[e];
        w = (i & 1) ? d.eu[e] : d.ev[e];
      } else {
        const uint64_t xw = d.evl[je][p][i];
        x = (uint32_t)(xw >> 32);
        w = (uint32_t)xw;
      }
    }
    fill_event_items(d, p, list, support, has, x, w);
  }
}

__global__ void __launch_bounds__(256) k_fill_level(const Dev* __restrict__ dp, uint32_t j,
                                                    uint64_t lo, uint64_t hi) {
  const Dev& d = *dp;
  const Ctl* c = d.ctl;
  const RoundCtx rc = round_ctx(c);
  const uint64_t nA = 2ull * c->nRc.v;
  // the directed removals x-lost-z
  const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
  const uint64_t ahi = min(hi, nA);
  for (uint64_t b = lo + blockIdx.x * (uint64_t)blockDim.x + (threadIdx.x & ~(WAVE - 1)); b < ahi;
       b += stride) {
    const uint64_t src = b + lane_id();
    const bool a = src < ahi;
    uint32_t x = 0, z = 0;
    if (a) {
      const uint32_t e = d.R[rc.p][src >> 1];
      x = (src & 1) ? d.ev[e] : d.eu[e];
      z = (src & 1) ? d.eu[e] : d.ev[e];
    }
    if (j == 2) {
      // (x, y), y an old neighbour of z, and (x, z); (y, z), y a live neighbour of x
      uint32_t bz = 0, dz = 0, bx = 0, dx = 0;
      if (a) {
        bz = d.rp[z];
        dz = d.len[z];
        bx = d.rp[x];
        dx = d.len[x];
      }
      const uint32_t v0 = a ? dz + 1 : 0, v1 = a ? dx : 0;
      const uint32_t n0 = chunks_of(v0), n1 = chunks_of(v1);
      uint32_t t0, t1;
      const uint32_t e0 = wave_excl_scan(n0, &t0), e1 = wave_excl_scan(n1, &t1);
      const uint32_t first = reserve_wave<false>(&d.ctl->cnt[2][rc.p].nit, t0 + t1);
      emit_items_wave<ITEM_ROW>(d, rc.p, 2, first, t0, e0, n0, KIND_A_SLOTS, 1, x, z, bz, v0);
      emit_items_wave<ITEM_ROW>(d, rc.p, 2, first + t0, t1, e1, n1, KIND_B_SLOTS, 0, x, z, bx, v1);
    } else {
      // (x, w), w in z's old (j-1)-ball
      emit_word_items<false>(d, rc.p, j, a, x, z, word_chunk(c->words, c->nRc.v));
    }
  }
  // the level-(j-1) events (x -> w): (y, w), y a live neighbour of x, and (x, w)
  if (j == 2 || hi <= nA) return;
  const uint64_t blo = lo > nA ? lo - nA : 0, bhi = hi - nA;
  if (c->cnt[j - 1][rc.p].ovf) fill_from_marks(d, rc.p, j - 1, j, false, blo, bhi);
  else fill_from_list(d, j - 1, false, rc.p, j, false, blo, bhi);
}

// Support items of the top-level events (listed, or the bits of the
// top-level change marks); for h = 1 the events are the directed removals.
__global__ void __launch_bounds__(256) k_fill_support(const Dev* __restrict__ dp, uint64_t lo,
                                                      uint64_t hi) {
  const Dev& d = *dp;
  const Ctl* c = d.ctl;
  const RoundCtx rc = round_ctx(c);
  if (c->cnt[d.h][rc.p].ovf) fill_from_marks(d, rc.p, d.h, d.h + 1, true, lo, hi);
  else fill_from_list(d, d.h, d.h == 1, rc.p, d.h + 1, true, lo, hi);
}

// Start of a recovery window: the step's work list is empty again.
__global__ void k_window_begin(const Dev* __restrict__ dp, uint32_t list) {
  if (blockIdx.x != 0 || threadIdx.x != 0) return;
  Ctl* c = dp->ctl;
  c->cnt[list][c->r & 1].nit = 0;
  c->cnt[list][c->r & 1].iovf = 0;
  c->halt = 0;
  c->recovering = 1;
  dp->status[1] = 0;
}

__global__ void k_recovery_end(const Dev* __restrict__ dp) {
  if (blockIdx.x != 0 || threadIdx.x != 0) return;
  dp->ctl->recovering = 0;
}

// ---- adjacency compaction (between rounds) -------------------------------
// Keep each row's live slots at its front, in order, so that later rounds
// scan only live ones.  Sixteen lanes per row, four rows per wave: most rows
// are short, and what bounds the step is the chain of dependent loads per row,
// not bytes.  In place: a chunk's slots are read before any is written, and
// slots only move to the front, never past a chunk still to be read.
template <bool TEAM>
__device__ void compact_rows(const Dev& d, uint32_t wave, uint32_t nwaves) {
  constexpr uint32_t G = 16;
  const uint32_t g = lane_id() / G, sub = lane_id() & (G - 1);
  for (uint32_t x0 = wave * (WAVE / G); x0 < d.n; x0 += nwaves * (WAVE / G)) {
    const uint32_t x = x0 + g;
    const uint32_t beg = x < d.n ? d.rp[x] : 0, n = x < d.n ? d.len[x] : 0;
    uint32_t kept = 0;
    for (uint32_t i0 = 0; __ballot(i0 < n); i0 += G) {
      const uint32_t i = i0 + sub, q = beg + i;
      uint64_t w = SLOT_GONE;
      uint32_t y = 0, e = 0;
      if (i < n) {
        w = ld<TEAM>(d.ce + q);
        y = d.cix[q];
        e = (uint32_t)(w >> 32);
      }
      const bool live = !((uint32_t)w & SLOT_GONE);
      const uint32_t bal = (uint32_t)(__ballot(live) >> (g * G)) & ((1u << G) - 1);
      const uint32_t at = kept + (uint32_t)__popc(bal & ((1u << sub) - 1));
      if (live && at != i) {
        const uint32_t z = beg + at;
        d.cix[z] = y;
        d.srem[z] = ALIVE;
        d.ce[z] = w;
        if (y > x) d.s1[e] = z;
        else d.s2[e] = z;
      }
      kept += (uint32_t)__popc(bal);
    }
    if (x < d.n && sub == 0 && kept != n) d.len[x] = kept;
  }
}

// At the head of a captured run of whole-chip rounds, where it is due.
__global__ void __launch_bounds__(256) k_compact_due(const Dev* __restrict__ devs) {
  const Dev& d = devs[blockIdx.y];
  Ctl* c = d.ctl;
  if (c->done || c->halt || !(c->live <= c->compact_at || (d.serial & 16u))) return;
  if (blockIdx.x == 0 && threadIdx.x == 0) c->compactions += 1;
  compact_rows<false>(d, blockIdx.x * (blockDim.x / WAVE) + threadIdx.x / WAVE,
                      gridDim.x * (blockDim.x / WAVE));
}

// Host-driven rounds: runs only at a round boundary of a running slot.
__global__ void __launch_bounds__(256) k_compact(Dev d) {
  Ctl* c = d.ctl;
  if (c->done || c->halt) return;
  if (blockIdx.x == 0 && threadIdx.x == 0) c->compactions += 1;
  compact_rows<false>(d, blockIdx.x * (blockDim.x / WAVE) + threadIdx.x / WAVE,
               gridDim.x * (blockDim.x / WAVE));
}

// Private adjacency copy and full rows, before the first round.
__global__ void k_init_rows(Dev d) {
  if (d.ctl->err) return;
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < d.nnz;
       i += (size_t)gridDim.x * blockDim.x) {
    d.cix[i] = d.ci[i];
    d.ce[i] = slot_word(d.eid[i], d.ci[i], false);
  }
  for (uint32_t x = blockIdx.x * blockDim.x + threadIdx.x; x < d.n; x += gridDim.x * blockDim.x)
    d.len[x] = d.rp[x + 1] - d.rp[x];
}

// ============================================ method-level work count
// Stats mode only.  On the bulk round schedule the kernels follow, count what
// the re-evaluating form of the peeling method (Section 3) would do:
//   evaluations  every edge once at the start, then in each round the live
//                edges with an endpoint whose h-ball changed (an endpoint with
//                a top-level ball-change event: h-support depends only on the
//                two endpoint balls, Def. 3);
//   bytes        per evaluation (u,v): s(u) + s(v) + 4, s(x) = min(4 |N(x,h)|,
//                ceil(n/8)) (the smaller exact encoding of a ball); per ball
//                build: min(frontier reads of a bounded BFS to depth h-1,
//                8 + 4 deg per vertex reached; h full scans of the CSR and a
//                bitset); builds: every non-isolated vertex at the start, then
//                in each round the vertices within h-1 hops (before the round)
//                of an endpoint of a removed edge.  A round that removes every
//                remaining edge evaluates and builds nothing.
// Per-vertex ball sizes and live degrees are kept from the round's top-level
// events and removals.

__device__ __forceinline__ uint64_t wave_sum64(uint64_t v) {
  for (int o = WAVE / 2; o > 0; o >>= 1) v += __shfl_xor(v, o, WAVE);
  return v;
}

__device__ __forceinline__ uint64_t acct_s(const Dev& d, uint32_t x) {
  return min((uint64_t)4 * d.acct_ball[x], (uint64_t)((d.n + 7) / 8));
}

// Cost of building x's ball in the live edge set after round r (all lanes
// call with the same x; every lane gets the wave total).  live_m: |S|.
__device__ uint64_t acct_build(const Dev& d, uint32_t x, uint32_t r, uint64_t live_m) {
  uint64_t f = 0;
  const uint32_t lane = lane_id();
  if (lane == 0) f = 8 + 4ull * d.acct_deg[x];
  if (d.h == 2) {
    for (uint32_t q = d.rp[x] + lane; q < row_end(d, x); q += WAVE)
      if (d.srem[q] > r) f += 8 + 4ull * d.acct_deg[d.cix[q]];
  } else if (d.h >= 3) {
    const uint64_t* B = row(d.L[d.h - 1], d.W, x);
    for (uint32_t i = lane; i < d.ctl->words; i += WAVE) {
      uint64_t wd = B[i];
      if (i == (x >> 6)) wd &= ~(1ull << (x & 63));  // x itself is counted above
      while (wd) {
        const uint32_t y = i * 64 + (uint32_t)(__ffsll((unsigned long long)wd) - 1);
        wd &= wd - 1;
        f += 8 + 4ull * d.acct_deg[y];
      }
    }
  }
  f = wave_sum64(f);
  const uint64_t scans = (uint64_t)d.h * (4ull * (d.n + 1) + 8 * live_m + (d.n + 7) / 8);
  return min(f, scans);
}

// Start: ball sizes and degrees in G (one wave per vertex), stamps cleared.
__global__ void __launch_bounds__(256) k_acct_init(const Dev* __restrict__ dp) {
  const Dev& d = *dp;
  if (d.ctl->err) return;
  const uint32_t lane = lane_id(), wpb = blockDim.x / WAVE;
  for (uint32_t x = blockIdx.x * wpb + threadIdx.x / WAVE; x < d.n; x += gridDim.x * wpb) {
    const uint64_t* B = row(d.L[d.h], d.W, x);
    uint32_t c = 0;
    if (x < d.ctl->nact)
      for (uint32_t i = lane; i < d.ctl->words; i += WAVE) c += (uint32_t)__popcll(B[i]);
    c = max(1u, wave_sum(c));  // an isolated vertex's ball holds itself
    if (lane == 0) {
      d.acct_ball[x] = c - 1;
      d.acct_deg[x] = d.rp[x + 1] - d.rp[x];
      d.acct_stamp[x] = 0;
      d.acct_vstamp[x] = 0;
    }
  }
}

// Start: the initial pass (every edge evaluated, every non-isolated vertex's
// ball built in G).
__global__ void __launch_bounds__(256) k_acct_start(const Dev* __restrict__ dp) {
  const Dev& d = *dp;
  if (d.ctl->err) return;
  uint64_t bytes = 0;
  for (uint32_t e = blockIdx.x * blockDim.x + threadIdx.x; e < d.m; e += gridDim.x * blockDim.x)
    bytes += acct_s(d, d.eu[e]) + acct_s(d, d.ev[e]) + 4;
  bytes = wave_sum64(bytes);
  const uint32_t wpb = blockDim.x / WAVE;
  uint64_t builds = 0;
  for (uint32_t x = blockIdx.x * wpb + threadIdx.x / WAVE; x < d.n; x += gridDim.x * wpb)
    if (d.acct_deg[x]) builds += acct_build(d, x, 0, d.m);
  if (lane_id() == 0) {
    atomicAdd((unsigned long long*)&d.ctl->acct_bytes, (unsigned long long)(bytes + builds));
    if (blockIdx.x == 0 && threadIdx.x == 0)
      atomicAdd((unsigned long long*)&d.ctl->acct_evals, (unsigned long long)d.m);
  }
}

// True when this round leaves edges for the count (not finished, not the
// round that removes everything).
__device__ __forceinline__ bool acct_round_counts(const Ctl* c) {
  return !c->done && !c->halt && !c->err && c->nRc.v < c->live;
}

// Round, step 1: degrees after the removals; vertices whose h-ball changed
// (sources of top-level events; at h = 1 the events are the removals), their
// ball sizes after the round, listed once each.
__global__ void __launch_bounds__(256) k_acct_round1(const Dev* __restrict__ dp) {
  const Dev& d = *dp;
  Ctl* c = d.ctl;
  if (!acct_round_counts(c)) return;
  const RoundCtx rc = round_ctx(c);
  const uint32_t stride = gridDim.x * blockDim.x, tid = blockIdx.x * blockDim.x + threadIdx.x;
  const uint32_t nR = c->nRc.v;
  for (uint32_t i = tid; i < 2 * nR; i += stride) {
    const uint32_t e = d.R[rc.p][i >> 1];
    atomicSub(&d.acct_deg[(i & 1) ? d.ev[e] : d.eu[e]], 1u);
  }
  const bool from_removals = d.h == 1;
  if (!from_removals && c->cnt[d.h][rc.p].ovf) {
    if (tid == 0) c->acct_incomplete = 1;
    return;
  }
  const uint32_t ne = from_removals ? 2 * nR : min(c->cnt[d.h][rc.p].nev, d.evcap);
  for (uint32_t i = tid; i < ne; i += stride) {
    uint32_t x;
    if (from_removals) {
      const uint32_t e = d.R[rc.p][i >> 1];
      x = (i & 1) ? d.ev[e] : d.eu[e];
    } else {
      x = (uint32_t)(d.evl[d.h][rc.p][i] >> 32);
    }
    atomicSub(&d.acct_ball[x], 1u);
    if (atomicExch(&d.acct_stamp[x], rc.r + 1) != rc.r + 1)
      d.acct_list[atomicAdd(&c->acct_nch, 1u)] = x;
  }
}

// Round, step 2: the evaluations (each live edge at a changed vertex once: by
// its smaller endpoint when both changed) and the ball builds, listed once
// each: the vertices within h-1 hops, before the round, of a removed edge's
// endpoint (at h-1 = 1 the endpoint and its neighbours then; above, the old
// (h-1)-ball = L[h-1] plus the pairs that left it this round).
__global__ void __launch_bounds__(256) k_acct_round2(const Dev* __restrict__ dp) {
  const Dev& d = *dp;
  Ctl* c = d.ctl;
  if (!acct_round_counts(c) || c->acct_incomplete) return;
  const RoundCtx rc = round_ctx(c);
  const uint32_t lane = lane_id(), wpb = blockDim.x / WAVE;
  const uint32_t wid = blockIdx.x * wpb + threadIdx.x / WAVE, nw = gridDim.x * wpb;
  uint64_t evals = 0, bytes = 0;
  const uint32_t nch = c->acct_nch;
  for (uint32_t k = wid; k < nch; k += nw) {
    const uint32_t x = d.acct_list[k];
    const uint64_t sx = acct_s(d, x);
    for (uint32_t q = d.rp[x] + lane; q < row_end(d, x); q += WAVE) {
      if (d.srem[q] <= rc.r) continue;
      const uint32_t b = d.cix[q];
      if (d.acct_stamp[b] == rc.r + 1 && b < x) continue;  // counted from b
      evals += 1;
      bytes += sx + acct_s(d, b) + 4;
    }
  }
  const uint32_t nR = c->nRc.v;
  for (uint32_t k = wid; k < 2 * nR; k += nw) {
    const uint32_t e = d.R[rc.p][k >> 1];
    const uint32_t z = (k & 1) ? d.ev[e] : d.eu[e];
    auto claim = [&](uint32_t x) {
      if (atomicExch(&d.acct_vstamp[x], rc.r + 1) != rc.r + 1)
        d.acct_vlist[atomicAdd(&c->acct_nv, 1u)] = x;
    };
    if (lane == 0) claim(z);
    if (d.h == 2) {
      for (uint32_t q = d.rp[z] + lane; q < row_end(d, z); q += WAVE)
        if (d.srem[q] >= rc.r) claim(d.cix[q]);
    } else if (d.h >= 3) {
      const uint64_t* B = row(d.L[d.h - 1], d.W, z);
      const uint64_t* D = row(d.Dm[d.h - 1], d.W, z);
      for (uint32_t i = lane; i < d.ctl->words; i += WAVE) {
        uint64_t wd = B[i] | D[i];
        while (wd) {
          claim(i * 64 + (uint32_t)(__ffsll((unsigned long long)wd) - 1));
          wd &= wd - 1;
        }
      }
    }
  }
  evals = wave_sum64(evals);
  bytes = wave_sum64(bytes);
  if (lane == 0) {
    if (evals) atomicAdd((unsigned long long*)&c->acct_evals, (unsigned long long)evals);
    if (bytes) atomicAdd((unsigned long long*)&c->acct_bytes, (unsigned long long)bytes);
  }
}

// Round, step 3: the listed ball builds, in the edge set after the round;
// the round's lists are emptied for the next round.
__global__ void __launch_bounds__(256) k_acct_round3(const Dev* __restrict__ dp) {
  const Dev& d = *dp;
  Ctl* c = d.ctl;
  if (!acct_round_counts(c) || c->acct_incomplete) return;
  const RoundCtx rc = round_ctx(c);
  const uint32_t wpb = blockDim.x / WAVE;
  const uint64_t live_m = c->live - c->nRc.v;
  uint64_t bytes = 0;
  const uint32_t nv = c->acct_nv;
  for (uint32_t k = blockIdx.x * wpb + threadIdx.x / WAVE; k < nv; k += gridDim.x * wpb)
    bytes += acct_build(d, d.acct_vlist[k], rc.r, live_m);
  if (lane_id() == 0 && bytes)
    atomicAdd((unsigned long long*)&c->acct_bytes, (unsigned long long)bytes);
}

// After step 3 (one thread): the round's lists are empty again.
__global__ void k_acct_reset(const Dev* __restrict__ dp) {
  if (blockIdx.x != 0 || threadIdx.x != 0) return;
  dp->ctl->acct_nch = 0;
  dp->ctl->acct_nv = 0;
}

// ============================================ (k,h)-truss extraction
// The (k,h)-truss is the edge set {e : t(e,h) >= k} (Def. 4: t(e,h) is the
// largest k whose truss holds e, and trusses are nested).  Its connected
// components come from a lock-free union-find over the vertices: a root is
// only ever linked below a smaller root, so parent[x] <= x throughout and
// every component's root is its smallest vertex.

__device__ __forceinline__ uint32_t cc_find(uint32_t* parent, uint32_t x) {
  uint32_t p = parent[x];
  while (p != x) {
    const uint32_t g = parent[p];
    if (g != p) parent[x] = g;  // path halving (any ancestor is a valid parent)
    x = p;
    p = g;
  }
  return x;
}

__global__ void k_cc_init(uint32_t* __restrict__ parent, uint32_t* __restrict__ touched,
                          uint32_t n) {
  for (uint32_t x = blockIdx.x * blockDim.x + threadIdx.x; x < n; x += gridDim.x * blockDim.x) {
    parent[x] = x;
    touched[x] = 0;
  }
}

__global__ void k_cc_hook(Dev d, const uint32_t* __restrict__ t, uint32_t k,
                          uint32_t* parent, uint32_t* __restrict__ touched) {
  if (d.ctl->err) return;
  for (uint32_t e = blockIdx.x * blockDim.x + threadIdx.x; e < d.m; e += gridDim.x * blockDim.x) {
    if (t[e] < k) continue;
    const uint32_t u = d.eu[e], v = d.ev[e];
    touched[u] = 1;
    touched[v] = 1;
    while (true) {
      uint32_t ru = cc_find(parent, u), rv = cc_find(parent, v);
      if (ru == rv) break;
      if (ru > rv) {
        const uint32_t tmp = ru;
        ru = rv;
        rv = tmp;
      }
      // link the larger root below the smaller one, if it is still a root
      if (atomicCAS(&parent[rv], rv, ru) == rv) break;
    }
  }
}

// Every vertex points at its root; edges of the truss take their component's
// root, the others UINT32_MAX; roots of touched vertices are counted.
__global__ void k_cc_label(Dev d, const uint32_t* __restrict__ t, uint32_t k, uint32_t* parent,
                           const uint32_t* __restrict__ touched, uint32_t* __restrict__ out,
                           uint32_t* __restrict__ count) {
  if (d.ctl->err) return;
  const uint32_t stride = gridDim.x * blockDim.x;
  for (uint32_t base = blockIdx.x * blockDim.x + (threadIdx.x & ~(WAVE - 1)); base < d.n;
       base += stride) {
    const uint32_t x = base + lane_id();
    const bool root = x < d.n && touched[x] && parent[x] == x;
    const uint32_t c = (uint32_t)__popcll(__ballot(root));
    if (lane_id() == 0 && c) atomicAdd(count, c);
  }
  for (uint32_t e = blockIdx.x * blockDim.x + threadIdx.x; e < d.m; e += stride)
    out[e] = t[e] >= k ? cc_find(parent, d.eu[e]) : 0xffffffffu;
}

}  // namespace hotruss
