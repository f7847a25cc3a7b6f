// vc_device.hip -- HIP kernels for gfx950 (MI355X) of the hybrid vertex-cover traversal.
//
// Method (paper §IV): a persistent grid; every workgroup walks a sub-tree of the
// branch-and-reduce search tree depth first with its own stack in device memory, and hands
// branches to a global worklist while the worklist holds fewer entries than a threshold
// (§IV-A). An intermediate graph is a degree array over one read-only CSR (§IV-B): one int32
// per vertex holding its degree, or a negative value once the vertex is in the cover, followed
// by the cover size s (the |S| counter of §IV-B) and a pending branch vertex (see below).
//
// gfx950 mapping:
//  - the node being worked on lives in LDS; every rule pass, the max-degree search and the
//    vertex removals read and update it there (LDS atomics for degree decrements); the row
//    pointers, and the column indices too when they fit, are staged in LDS after it. Where
//    each of them lives is a template parameter of the kernels, so every access compiles to
//    an LDS or a device-memory instruction, never a generic one;
//  - after each removal step one scan lists the vertices of degree one and two and finds the
//    largest degree; the rule passes work on those lists. A candidate's CSR row is walked by its
//    own lane when it is short, and in 64-entry pieces by the whole wavefront when it is long;
//  - the maximum-degree vertex and the degree sum come from one pass reduced with DPP row
//    operations inside each wavefront and one LDS step across wavefronts;
//  - a deferred child is stored as its parent's reduced degree array plus the vertex whose
//    neighbourhood it removes (the "pending" vertex); the removal is done in LDS by whoever
//    takes the child, so a branch costs one plain copy of the node out and one copy back in,
//    and no global-memory atomics touch node data;
//  - the worklist is a bounded ring of node slots with per-slot lap tickets; producers and
//    consumers synchronise through agent-scope atomics, so a node written on one XCD is seen
//    correctly by a workgroup on another;
//  - termination: a counter of outstanding sub-trees (queued, or held by a workgroup) is
//    raised before a node is published and lowered when a workgroup has finished the whole
//    sub-tree it took; the search is over when it reads zero (§IV-C).
//
// Rule semantics (paper §II-B, parallel tie-breaks §IV-D): each rule is one pass that decides
// from the degree array as it stood at the start of the pass (decisions are marked with a
// flag bit that leaves the degree bits untouched), then removes every marked vertex at once.
// The passes run degree-one, degree-two-triangle, high-degree, and repeat until a whole round
// changes nothing or s exceeds the bound.

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "vc_device_common.h"
#include "vc_internal.h"

namespace vc {

constexpr int32_t kFlag = 0x40000000;     // "decided this pass" mark on a live entry
// "degree two, and its two live neighbours are not adjacent" on a live entry. Along a path of
// the search tree vertices are only removed, so a vertex that still has degree two has the same
// two neighbours: the mark stays true in every descendant node (stored nodes keep it) and the
// triangle rule checks each degree-two vertex once per path instead of once per pass.
constexpr int32_t kNoTri = 0x20000000;
constexpr int32_t kDegMask = 0x1FFFFFFF;  // degree bits of a live entry

// ---- node operations on the LDS degree array -------------------------------------------------
// st[0..n) degrees (negative = in the cover), st[n] = s, st[n+1] = pending vertex (-1 = none).

// The node operations work on a node and three lists in LDS, rings of cap = mask + 1 entries
// (at least 32 per wavefront of the workgroup):
//  - rm: the vertices marked since the last removal step;
//  - one, two: the vertices of degree one, and of degree two not marked kNoTri, as the last
//    refresh_lists found them.
// After each removal step one scan of the node (refresh_lists) finds the candidates of both rules
// and the largest degree; the rule passes then work on packed candidates, and a rule without a
// candidate costs nothing. A list that overflows is not used: that pass scans for itself.
struct Node {
  int32_t* st;
  int n;
  const int32_t* __restrict__ rp;
  const int32_t* __restrict__ ci;
  int32_t* rm;    // cap entries; `one` and `two` follow
  uint32_t mask;
  bool spread;    // long rows: a removal step's rows go to the wavefronts in turn
  bool far;       // the node lives in device memory
  __device__ int32_t* one() const { return rm + mask + 1; }
  __device__ int32_t* two() const { return rm + 2 * (mask + 1); }
};

// Where the lists' current entries lie (their tails grow in Ctrl), and the largest degree at the
// last refresh, an upper bound until the next. The same in every thread of the workgroup.
struct Front {
  int32_t s;               // cover size of the node, as st[n] holds it
  uint32_t rm;             // marked vertices already removed end here
  uint32_t one, one_end;
  uint32_t two, two_end;
  int32_t most;
  uint32_t turn;           // refreshes so far
  // The instance has shown a degree above kLaneRow: removal steps spread their rows, also where the
  // average degree is small. In a planted graph of average degree 6 the removed vertices' rows have
  // 30 to 60 entries, and all fell to one or two wavefronts (greedy of 512 / 1,000 / 4,000 vertices
  // 46 -> 40.5, 50 -> 42.5, 63 -> 52 us).
  bool wide;
};

// Rows longer than this are walked in 64-entry pieces by the whole wavefront; shorter ones by
// their own lane.
constexpr int kLaneRow = 16;
// Entries a walk hands on at once, per lane.
constexpr int kWalk = 4;

// One batch of walked entries: entry u of this lane is xs[u], of the row with tag tags[u], where
// ok[u] (a valid vertex of some row otherwise).
struct Walked {
  int xs[kWalk];
  bool ok[kWalk];
  int tags[kWalk];
};

// Walk the CSR rows [beg, end) held by the lanes of a wavefront (empty where beg >= end; at least
// one lane holds an entry). fn(batch) runs, in uniform control flow, for batches of kWalk entries
// per lane, each with the `tag` of its row's owner lane. A batch's loads are issued before the
// first is used, and fn does the same with the accesses that depend on them. Rows of up to
// kLaneRow entries are read by their own lane, kWalk entries at a time; longer rows are cut into
// 64-entry pieces that the whole wavefront reads, kWalk pieces at a time, with the cursor (row
// bounds, tag, position) in scalar registers. So are all rows of more than kWalk entries where at
// most kWalk lanes hold one: by its own lane a lone row of 16 entries is a chain of four batches
// (greedy of G(300, 8/300), a vertex a step: 735 -> 683 us).
// A root's reduction runs on one CU, whose four SIMDs issue one wavefront instruction a cycle
// between them, and a large root walks 10^5 entries: the walk is bound by instructions per entry
// (and, in small frontiers, by the latency of its chain). So loads are unconditional, with the
// index clamped into the row, a piece's address is a scalar base plus the lane, and nothing is
// looked up per entry.
template <typename Fn>
__device__ __forceinline__ void walk_rows(const int32_t* __restrict__ ci, int beg, int end, int tag,
                                          Fn fn) {
  const int lane = lane_id();
  const bool few = __popcll(__builtin_amdgcn_ballot_w64(beg < end)) <= kWalk;
  const bool longrow = end - beg > (few ? kWalk : kLaneRow);
  uint64_t longs = __builtin_amdgcn_ballot_w64(longrow);
  const int stop = longrow ? beg : max(beg, end);
  const int last = max(stop - 1, 0);
  int at = beg;
  while (__builtin_amdgcn_ballot_w64(at < stop)) {
    Walked w;
#pragma unroll
    for (int u = 0; u < kWalk; ++u) {
      w.ok[u] = at + u < stop;
      w.tags[u] = tag;
      w.xs[u] = ci[min(at + u, last)];
    }
    at += kWalk;
    fn(w);
  }
  int rb = 0, re = 0, rt = 0;  // the piece cursor: next entry, end and tag of the current row
  while (longs || rb < re) {
    Walked w;
#pragma unroll
    for (int u = 0; u < kWalk; ++u) {
      if (rb >= re && longs) {
        const int o = first_lane(longs);
        longs &= longs - 1;
        rb = __builtin_amdgcn_readlane(beg, o);
        re = __builtin_amdgcn_readlane(end, o);
        rt = __builtin_amdgcn_readlane(tag, o);
      }
      const int left = re - rb;  // <= 0 once the rows have run out: entry 0 of the last one, unused
      const int32_t* piece = ci + (left > 0 ? rb : re - 1);
      w.ok[u] = lane < left;
      w.tags[u] = rt;
      w.xs[u] = piece[static_cast<uint32_t>(max(min(lane, left - 1), 0))];
      rb += 64;
    }
    fn(w);
  }
}

__device__ __forceinline__ uint32_t lanes_below(uint64_t m) {
  return __builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(m >> 32),
                                   __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(m), 0));
}

// Append this lane's values v[u], where its bit of m[u] is set, to a list at `at` (its tail before
// the wavefront raised it by count_bits(m)). Uniform control flow.
__device__ __forceinline__ void list_write(int32_t* list, uint32_t mask, uint32_t at,
                                           const uint64_t (&m)[kWalk], const int (&v)[kWalk]) {
#pragma unroll
  for (int u = 0; u < kWalk; ++u) {
    if (__builtin_amdgcn_inverse_ballot_w64(m[u])) list[(at + lanes_below(m[u])) & mask] = v[u];
    at += __popcll(m[u]);
  }
}

__device__ __forceinline__ int count_bits(const uint64_t (&m)[kWalk]) {
  int count = 0;
#pragma unroll
  for (int u = 0; u < kWalk; ++u) count += __popcll(m[u]);
  return count;
}

// Hand the candidates, the vertices with pred(d), to process(cand): one per lane, -1 where a lane
// has none. They are the list entries [from, to), which hold exactly these vertices, or, if the list
// has overflowed, they are found among all vertices. Whole workgroup; the control flow is uniform in
// each wavefront. With `spread`, list entry i goes to wavefront i mod waves, so that a few candidates
// with long rows do not all fall to one; otherwise the list goes out 64 entries at a time, so that a
// short list leaves the other wavefronts out of a step's instructions (every wavefront's cost issue
// slots of the four SIMDs, whether or not its lanes hold a candidate). The scan stages its finds in
// the wavefront's share of the overflowed list; a chunk with more finds than that goes out as it is.
template <typename Pred, typename Proc>
__device__ __forceinline__ void for_candidates(const Node& nd, int32_t* list, uint32_t from,
                                               uint32_t to, bool spread, Pred pred,
                                               Proc process) {
  const int lane = lane_id();
  const int wave = wave_id();
  const int waves = blockDim.x >> 6;
  const int total = static_cast<int>(to - from);
  const bool scan = to - from > nd.mask + 1;
  const int room = min(64, static_cast<int>(nd.mask + 1) / waves);
  int32_t* staged = list + room * wave;
  int base = wave * 64;                // scan: next chunk
  int i0 = spread ? wave : wave * 64;  // list: first entry of the next batch
  for (;;) {
    int held = -1;
    if (!scan) {
      if (i0 >= total) break;
      const int i = spread ? i0 + waves * lane : i0 + lane;
      if (i < total) held = list[(from + static_cast<uint32_t>(i)) & nd.mask];
      i0 += waves * 64;
    } else {
      int count = 0;
      for (; base < nd.n; base += blockDim.x) {
        const int v = base + lane;
        const bool take = v < nd.n && pred(nd.st[v]);
        const uint64_t m = __builtin_amdgcn_ballot_w64(take);
        const int cnt = __popcll(m);
        if (count + cnt > room) {  // this chunk starts the next batch, or is one by itself
          if (count == 0) {
            held = take ? v : -1;
            base += blockDim.x;
            count = -1;
          }
          break;
        }
        if (take) staged[count + lanes_below(m)] = v;
        count += cnt;
      }
      if (count == 0) break;
      __builtin_amdgcn_wave_barrier();
      if (lane < count) held = staged[lane];
      __builtin_amdgcn_wave_barrier();
    }
    process(held);
  }
}

// Is an entry live and not marked?
__device__ __forceinline__ bool unmarked(int32_t d) {
  return static_cast<uint32_t>(d) < static_cast<uint32_t>(kFlag);
}

// The largest of the wavefronts' values in `part` (one per wavefront, kMaxWaves long): one LDS
// read and a reduction inside each wavefront.
__device__ __forceinline__ int32_t block_part_max(const int32_t* part) {
  const int waves = blockDim.x >> 6;
  const int32_t x = lane_id() < waves ? part[lane_id() & (kMaxWaves - 1)] : 0;
  return static_cast<int32_t>(wave_max32(static_cast<uint32_t>(x)));
}

// The neighbours in a batch of walked entries lose one degree each (see apply_marks).
__device__ __forceinline__ void drop_degrees(const Node& nd, const Walked& w) {
  int32_t* st = nd.st;
  if (nd.far) {
#pragma unroll
    for (int u = 0; u < kWalk; ++u)
      if (w.ok[u]) atomicSub(&st[w.xs[u]], 1);
    return;
  }
  int32_t d[kWalk];
#pragma unroll
  for (int u = 0; u < kWalk; ++u) d[u] = st[w.xs[u]];
#pragma unroll
  for (int u = 0; u < kWalk; ++u)
    if (w.ok[u] && unmarked(d[u])) atomicSub(&st[w.xs[u]], 1);
}

// Remove every marked vertex (paper §IV-B): marked vertices become kSent and s grows by their
// number; each live unmarked neighbour of a marked vertex loses one degree per marked neighbour.
// The walks only decrement entries that are live and unmarked (a marked vertex may turn kSent
// meanwhile: either way it is left alone), which also keeps the LDS atomics off the entries of
// vertices already removed. A node in device memory is decremented without the look first: 64
// scattered reads cost the CU's memory pipe as much as the 64 atomics, nothing waits for the
// atomics, and a removed entry that goes further below zero, or a marked one whose degree bits
// fall (by at most its degree) before it turns kSent, stays what it was (one planted root of
// 50,021 vertices: 457 -> 353 us). Called right after a barrier that ends a decide step (or a mark
// step); ends with a barrier.
__device__ __forceinline__ void apply_marks(const Node& nd, Ctrl& c, Front& f) {
  int32_t* st = nd.st;
  const uint32_t tail = c.rm_tail;
  for_candidates(
      nd, nd.rm, f.rm, tail, nd.spread || f.wide, [](int32_t d) { return d >= 0 && (d & kFlag); },
      [&](int v) {
        const bool mine = v >= 0;
        if (mine) st[v] = kSent;
        walk_rows(nd.ci, mine ? nd.rp[v] : 0, mine ? nd.rp[v + 1] : 0, v,
                  [&](const Walked& w) { drop_degrees(nd, w); });
      });
  f.s += static_cast<int32_t>(tail - f.rm);
  if (threadIdx.x == 0) st[nd.n] = f.s;
  f.rm = tail;
  __syncthreads();
}

// The four entries from vertex v0 on (a multiple of four), kSent past the last vertex.
__device__ __forceinline__ void four_entries(const Node& nd, int v0, bool whole,
                                             int32_t (&d)[kWalk]) {
  const int4* st4 = reinterpret_cast<const int4*>(nd.st);
  const int4 x = whole || v0 < nd.n ? st4[v0 >> 2] : int4{kSent, kSent, kSent, kSent};
  d[0] = x.x, d[1] = x.y, d[2] = x.z, d[3] = x.w;
  if (!whole) {
#pragma unroll
    for (int u = 0; u < kWalk; ++u) d[u] = v0 + u < nd.n ? d[u] : kSent;
  }
}

// The candidates of the degree-one and triangle rules and the largest degree of the node as it
// stands (nothing marked), by one scan, four consecutive vertices per thread and step: four
// vector instructions per 64 vertices where there is no candidate. Holds one barrier. (red_max is
// used in turn: the barrier of the next refresh lies between the reads of this one and the next
// write of the same half.)
__device__ __forceinline__ void refresh_lists(const Node& nd, Ctrl& c, Front& f) {
  f.one = f.one_end;
  f.two = f.two_end;
  int32_t most = 0;
  for (int base = wave_id() * 256; base < nd.n; base += 4 * blockDim.x) {
    const int v0 = base + 4 * lane_id();
    int32_t d[kWalk];
    four_entries(nd, v0, base + 256 <= nd.n, d);
    uint64_t one[kWalk], two[kWalk];
    uint64_t any = 0;
    int v[kWalk];
#pragma unroll
    for (int u = 0; u < kWalk; ++u) {
      const int32_t e = d[u] & ~kNoTri;  // the degree, negative where the vertex is in the cover
      most = max(most, e);
      one[u] = __builtin_amdgcn_ballot_w64(e == 1);
      two[u] = __builtin_amdgcn_ballot_w64(d[u] == 2);
      any |= one[u] | two[u];
      v[u] = v0 + u;
    }
    if (any) {
      const int n1 = count_bits(one), n2 = count_bits(two);
      uint32_t at1 = 0, at2 = 0;
      if (lane_id() == 0) {
        at1 = atomicAdd(&c.one_tail, static_cast<uint32_t>(n1));
        at2 = atomicAdd(&c.two_tail, static_cast<uint32_t>(n2));
      }
      if (n1) list_write(nd.one(), nd.mask, __builtin_amdgcn_readfirstlane(at1), one, v);
      if (n2) list_write(nd.two(), nd.mask, __builtin_amdgcn_readfirstlane(at2), two, v);
    }
  }
  int32_t* part = c.red_max[f.turn++ & 1u];
  most = static_cast<int32_t>(wave_max32(static_cast<uint32_t>(most)));
  if (lane_id() == 0) part[wave_id()] = most;
  __syncthreads();
  f.one_end = c.one_tail;
  f.two_end = c.two_tail;
  f.most = block_part_max(part);
  f.wide |= f.most > kLaneRow;
}

// Degree-one rule (§II-B): v with one live neighbour u puts u in the cover; of two adjacent
// degree-one vertices only the smaller id is removed, and a shared neighbour once (§IV-D).
// The rows of all degree-one vertices are walked together; the one live entry of a row names
// u, and the lane that reads it makes the decision for that row's owner.
__device__ __forceinline__ void decide_degree_one(const Node& nd, Ctrl& c, const Front& f) {
  int32_t* st = nd.st;
  for_candidates(
      nd, nd.one(), f.one, f.one_end, false,
      [](int32_t d) { return d >= 0 && (d & kDegMask) == 1; },
      [&](int cv) {
        const bool mine = cv >= 0;
        walk_rows(nd.ci, mine ? nd.rp[cv] : 0, mine ? nd.rp[cv + 1] : 0, cv, [&](const Walked& w) {
          int32_t d[kWalk];
#pragma unroll
          for (int u = 0; u < kWalk; ++u) d[u] = st[w.xs[u]];
          // the live neighbour of the row's owner, if it is to go and no other lane has marked it
          bool hit[kWalk];
          bool any = false;
#pragma unroll
          for (int u = 0; u < kWalk; ++u) {
            hit[u] = w.ok[u] && unmarked(d[u]);
            any |= hit[u];
          }
          if (!__builtin_amdgcn_ballot_w64(any)) return;
          uint64_t m[kWalk];
          int32_t was[kWalk];  // all marks are issued before the first one's answer is waited for
#pragma unroll
          for (int u = 0; u < kWalk; ++u) {
            was[u] = kFlag;
            if (hit[u] && ((d[u] & kDegMask) != 1 || w.xs[u] < w.tags[u]))
              was[u] = atomicOr(&st[w.xs[u]], kFlag);
          }
#pragma unroll
          for (int u = 0; u < kWalk; ++u) m[u] = __builtin_amdgcn_ballot_w64(!(was[u] & kFlag));
          const int count = count_bits(m);
          if (count == 0) return;
          uint32_t at = 0;
          if (lane_id() == 0) at = atomicAdd(&c.rm_tail, static_cast<uint32_t>(count));
          list_write(nd.rm, nd.mask, __builtin_amdgcn_readfirstlane(at), m, w.xs);
        });
      });
}

// Mark v for the next removal step.
__device__ __forceinline__ void mark(const Node& nd, Ctrl& c, int v) {
  if (!(atomicOr(&nd.st[v], kFlag) & kFlag))
    nd.rm[atomicAdd(&c.rm_tail, 1u) & nd.mask] = v;
}

// Is `key` in the sorted CSR segment ci[lo, hi)? An 8-ary search: each round reads seven
// evenly spaced entries at once and keeps the part that can hold the key, so a row of 125
// entries takes three rounds of independent loads instead of seven dependent ones.
__device__ __forceinline__ bool row_contains(const int32_t* __restrict__ ci, int lo, int hi,
                                             int key) {
  while (hi - lo > 8) {
    const int step = (hi - lo + 7) >> 3;
    int probe[7];
#pragma unroll
    for (int i = 0; i < 7; ++i) {
      const int at = lo + (i + 1) * step;
      probe[i] = at < hi ? ci[at] : 0x7FFFFFFF;
    }
    int below = 0;  // probes that are <= key
#pragma unroll
    for (int i = 0; i < 7; ++i) below += probe[i] <= key;
    const int nlo = lo + below * step;
    const int nhi = nlo + step < hi ? nlo + step : hi;
    lo = nlo;
    hi = nhi;
  }
  bool hit = false;
#pragma unroll
  for (int i = 0; i < 8; ++i) hit |= lo + i < hi && ci[lo + i] == key;
  return hit;
}

// Degree-two-triangle rule (§II-B): v with live neighbours u, w and uw an edge puts u and w in
// the cover; among degree-two vertices of one triangle only the smallest id fires (§IV-D).
// Each lane takes one degree-two vertex: it finds the two live neighbours in its own row (rows
// longer than kLaneRow are searched by the whole wavefront), then searches the shorter of the
// two neighbours' rows for the other.
__device__ __forceinline__ void decide_triangle(const Node& nd, Ctrl& c, const Front& f) {
  constexpr int kLaneRow = 32;
  int32_t* st = nd.st;
  const int lane = lane_id();
  for_candidates(nd, nd.two(), f.two, f.two_end, false,
                 [](int32_t d) { return d >= 0 && (d & kDegMask) == 2 && !(d & kNoTri); },
                 [&](int cv) {
                   const bool mine = cv >= 0;
                   const int beg = mine ? nd.rp[cv] : 0, end = mine ? nd.rp[cv + 1] : 0;
                   int a = -1, b = -1;
                   if (mine && end - beg <= kLaneRow) {
                     for (int j = beg; j < end && b < 0; j += 8) {
                       int x[8];
#pragma unroll
                       for (int u = 0; u < 8; ++u) x[u] = j + u < end ? nd.ci[j + u] : -1;
#pragma unroll
                       for (int u = 0; u < 8; ++u) {
                         if (x[u] >= 0 && b < 0 && st[x[u]] >= 0) {
                           if (a < 0) a = x[u]; else b = x[u];
                         }
                       }
                     }
                   }
                   // long rows: the whole wavefront scans one row at a time
                   uint64_t longs = __builtin_amdgcn_ballot_w64(mine && end - beg > kLaneRow);
                   while (longs) {
                     const int owner = first_lane(longs);
                     longs &= longs - 1;
                     const int rb = __builtin_amdgcn_readlane(beg, owner);
                     const int re = __builtin_amdgcn_readlane(end, owner);
                     int fa = -1, fb = -1;
                     for (int j = rb; j < re && fb < 0; j += 64) {
                       const int x = j + lane < re ? nd.ci[j + lane] : -1;
                       uint64_t live = __builtin_amdgcn_ballot_w64(x >= 0 && st[x] >= 0);
                       while (live && fb < 0) {
                         const int y = bcast(x, first_lane(live));
                         live &= live - 1;
                         if (fa < 0) fa = y; else fb = y;
                       }
                     }
                     if (lane == owner) {
                       a = fa;
                       b = fb;
                     }
                   }
                   if (b < 0) return;  // no candidate in this lane
                   // is b in row a? search the shorter of the two sorted rows
                   const int ab = nd.rp[a], ae = nd.rp[a + 1];
                   const int bb = nd.rp[b], be = nd.rp[b + 1];
                   const bool in_a = ae - ab <= be - bb;
                   if (!row_contains(nd.ci, in_a ? ab : bb, in_a ? ae : be, in_a ? b : a)) {
                     // no triangle through cv: no other lane flags cv in this pass (a firing
                     // vertex flags only the two vertices of its own triangle)
                     atomicOr(&st[cv], kNoTri);
                     return;
                   }
                   const int32_t da = st[a] & kDegMask, db = st[b] & kDegMask;
                   if ((da == 2 && a < cv) || (db == 2 && b < cv)) return;
                   mark(nd, c, a);
                   mark(nd, c, b);
                 });
}

// High-degree rule (§II-B): a vertex whose degree exceeds r = bound - s is in every cover of
// size <= bound (bound = best - 1 for MVC, k for PVC).
__device__ __forceinline__ void decide_high_degree(const Node& nd, Ctrl& c, int64_t r) {
  int32_t* st = nd.st;
  for (int v = threadIdx.x; v < nd.n; v += blockDim.x) {
    const int32_t d = st[v];
    if (d >= 0 && static_cast<int64_t>(d & kDegMask) > r) {
      st[v] = d | kFlag;
      nd.rm[atomicAdd(&c.rm_tail, 1u) & nd.mask] = v;
    }
  }
}

// No-op activity clock for the uninstrumented callers.
struct NoClock {
  __device__ void charge(int) {}
};

// The reduction rules until the graph stops changing (§II-B, §IV-D), or until s > bound.
// Precondition: the node is visible to the whole workgroup and f.s is its cover size. With `marked`,
// the vertices that mark_neighbourhood flagged (a stored child's pending removal) are removed first.
// The three rules take turns through one loop, so that the removal step is compiled once per kernel.
// On small graphs a step is a chain of LDS latencies: the cover size is kept in a register (f.s),
// listed candidates are not looked at again, and a batch's marks are waited for together (greedy of
// G(512, 2.5/512): 117 -> 104 us, of a path of 1,000 vertices: 946 -> 798).
template <typename Clock>
__device__ __forceinline__ void reduce_node(const Node& nd, Ctrl& c, Front& f, int64_t bound,
                                            int rules, Clock& clk, bool marked) {
  // A rule pass is skipped when nothing has been removed since it last found nothing, and when it
  // has no candidate: its list is empty, or (high-degree rule) no degree exceeds r. It would find
  // nothing: this drops empty passes, not any decision.
  int changes = 0;                   // removal steps applied by the rules in this call
  int quiet[3] = {-1, -1, -1};       // `changes` when each rule last found nothing
  int32_t s0 = 0;                    // s at the start of the current round
  int rule = -1;
  for (;;) {
    if (rule >= 0) {
      if (rule == 0) {
        if (changes > 0 && f.s == s0) return;  // a round that removed nothing
        s0 = f.s;
      }
      bool skip = !(rules & (kRuleDeg1 << rule)) || quiet[rule] == changes;
      if (rule == 0) skip |= f.one_end == f.one;
      else if (rule == 1) skip |= f.two_end == f.two;
      else skip |= f.most <= bound - f.s;
      if (!skip) {
        if (rule == 0) decide_degree_one(nd, c, f);
        else if (rule == 1) decide_triangle(nd, c, f);
        else decide_high_degree(nd, c, bound - f.s);
        __syncthreads();
        if (rule == 0) clk.charge(kActDeg1);
        else if (rule == 1) clk.charge(kActTri);
        else clk.charge(kActHigh);
        skip = c.rm_tail == f.rm;
        if (skip) quiet[rule] = changes;
      }
      if (skip) {
        if (rule == 2 && changes == 0) return;  // a first round that found nothing
        rule = rule == 2 ? 0 : rule + 1;
        continue;
      }
    }
    if (rule >= 0 || marked) apply_marks(nd, c, f);
    if (f.s > bound) return;
    refresh_lists(nd, c, f);
    if (rule < 0) {
      clk.charge(kActBranch);
    } else {
      ++changes;
      clk.charge(kActApply);
    }
    rule = rule == 2 ? 0 : rule + 1;
  }
}

__device__ __forceinline__ void reduce_node(const Node& nd, Ctrl& c, Front& f, int64_t bound,
                                            int rules, bool marked = false) {
  NoClock none;
  reduce_node(nd, c, f, bound, rules, none, marked);
}

// The sum of live degrees (= 2|E|) and the live vertex of maximum degree, smallest id on ties
// (§IV-B), of a node that reduce_node has just left: its largest degree is known. No scan when
// there is no edge left. Results are the same in every thread.
__device__ __forceinline__ void max_degree_and_sum(const Node& nd, Ctrl& c, const Front& f,
                                                   int& vmax, int32_t& degsum) {
  vmax = -1;
  degsum = 0;
  if (f.most <= 0) return;
  uint32_t key = 0;  // largest ~id of a vertex of the largest degree
  int32_t sum = 0;
  for (int base = wave_id() * 256; base < nd.n; base += 4 * blockDim.x) {
    const int v0 = base + 4 * lane_id();
    int32_t d[kWalk];
    four_entries(nd, v0, base + 256 <= nd.n, d);
#pragma unroll
    for (int u = 0; u < kWalk; ++u) {
      const int32_t e = d[u] & ~kNoTri;
      sum += max(e, 0);
      key = max(key, e == f.most ? ~static_cast<uint32_t>(v0 + u) : 0u);
    }
  }
  key = wave_max32(key);
  sum = wave_sum(sum);
  if (lane_id() == 0) {
    c.red_key[wave_id()] = key;
    c.red_sum[wave_id()] = sum;
  }
  __syncthreads();
  const int waves = blockDim.x >> 6;
  const bool mine = lane_id() < waves;
  const int at = lane_id() & (kMaxWaves - 1);
  vmax = static_cast<int>(~wave_max32(mine ? c.red_key[at] : 0u));
  degsum = wave_sum(mine ? c.red_sum[at] : 0);
}

// The cover of the node, one byte per vertex: four to a store where the output is aligned to four
// bytes (a packed batch's covers start anywhere).
__device__ __forceinline__ void store_cover(uint8_t* cov, const Node& nd) {
  if ((reinterpret_cast<uintptr_t>(cov) & 3u) == 0) {
    for (int v0 = 4 * threadIdx.x; v0 < nd.n; v0 += 4 * blockDim.x) {
      int32_t d[kWalk];
      four_entries(nd, v0, v0 + 4 <= nd.n, d);
      if (v0 + 4 <= nd.n) {
        uint32_t x = 0;
#pragma unroll
        for (int u = 0; u < kWalk; ++u) x |= (static_cast<uint32_t>(d[u]) >> 31) << (8 * u);
        *reinterpret_cast<uint32_t*>(cov + v0) = x;
      } else {
        for (int v = v0; v < nd.n; ++v) cov[v] = nd.st[v] < 0;
      }
    }
  } else {
    for (int v = threadIdx.x; v < nd.n; v += blockDim.x) cov[v] = nd.st[v] < 0;
  }
}

// Flag every live neighbour of v (the "N(v) in the cover" child, §II-B); the next reduce_node
// (marked = true) removes them. Ends with a barrier.
__device__ __forceinline__ void mark_neighbourhood(const Node& nd, Ctrl& c, int v) {
  int32_t* st = nd.st;
  const int beg = nd.rp[v], end = nd.rp[v + 1];
  for (int j = beg + static_cast<int>(threadIdx.x); j < end; j += blockDim.x) {
    const int x = nd.ci[j];
    const int32_t d = st[x];  // distinct x per thread: plain read-modify-write
    if (d >= 0) {
      st[x] = d | kFlag;
      nd.rm[atomicAdd(&c.rm_tail, 1u) & nd.mask] = x;
    }
  }
  __syncthreads();
}

// Remove v alone, a live vertex that every thread names, from a node with nothing marked (the "v in
// the cover" child, §II-B). One wavefront walks its row: no list to go through, and one barrier, at
// the end (greedy of G(1000, 8/1000), a vertex a step: 2,201 -> 2,053 us).
__device__ __forceinline__ void remove_vertex(const Node& nd, Front& f, int v) {
  f.s += 1;
  if (wave_id() == 0) {
    const bool mine = lane_id() == 0;
    if (mine) {
      nd.st[v] = kSent;
      nd.st[nd.n] = f.s;
    }
    walk_rows(nd.ci, mine ? nd.rp[v] : 0, mine ? nd.rp[v + 1] : 0, v,
              [&](const Walked& w) { drop_degrees(nd, w); });
  }
  __syncthreads();
}

// Copy a node between LDS and device memory, 16 bytes per thread per step. The same thread
// always handles the same words, so a node written to the workgroup's own stack is read back
// by the threads that wrote it. `pending` replaces word n+1 on the way out.
__device__ __forceinline__ void node_store(int32_t* __restrict__ dst, const int32_t* st, int stride,
                                           int n,
                           int pending) {
  const int4* s4 = reinterpret_cast<const int4*>(st);
  int4* d4 = reinterpret_cast<int4*>(dst);
  const int q = (n + 1) >> 2, r = (n + 1) & 3;
  for (int i = threadIdx.x; i < (stride >> 2); i += blockDim.x) {
    int4 x = s4[i];
    if (i == q) {
      if (r == 0) x.x = pending;
      else if (r == 1) x.y = pending;
      else if (r == 2) x.z = pending;
      else x.w = pending;
    }
    d4[i] = x;
  }
}


// Copy a stored node between two device-memory slots with the same thread-to-word mapping as
// node_store / node_load, so each thread reads back words it wrote itself.
__device__ __forceinline__ void node_copy(int32_t* __restrict__ dst, const int32_t* __restrict__ src,
                                          int stride) {
  const int4* s4 = reinterpret_cast<const int4*>(src);
  int4* d4 = reinterpret_cast<int4*>(dst);
  for (int i = threadIdx.x; i < (stride >> 2); i += blockDim.x) d4[i] = s4[i];
}

__device__ __forceinline__ void node_load(int32_t* st, const int32_t* __restrict__ src,
                                          int stride) {
  const int4* s4 = reinterpret_cast<const int4*>(src);
  int4* d4 = reinterpret_cast<int4*>(st);
  for (int i = threadIdx.x; i < (stride >> 2); i += blockDim.x) d4[i] = s4[i];
}

// The node a workgroup works on: in LDS (dynamic shared memory, followed by the staged row
// pointers), or, for graphs whose node does not fit there, in slot `slot` of the device-memory
// node array. The node operations take a plain pointer, so one body serves both; in device
// memory their reads, writes and atomics are global-memory accesses, ordered inside the
// workgroup by the same barriers.
// Where a launch keeps the node being worked on and the CSR it reads. Fixed per kernel
// instantiation, so that every access compiles to an LDS (ds_*) or a device-memory (global_*)
// instruction rather than a generic one that has to test its address.
enum MemMode : int {
  kMemGlobal = 0,  // node in device memory (graphs too large for LDS); CSR in device memory
  kMemLds = 1,     // node in LDS; CSR in device memory
  kMemLdsRp = 2,   // node and row pointers in LDS; column indices in device memory
  kMemLdsCsr = 3,  // node and the whole CSR in LDS
};

// The dynamic LDS: the lists, then (node in LDS) the node and the staged CSR.
__device__ __forceinline__ int32_t* lists_base() {
  extern __shared__ int4 lds4[];
  return reinterpret_cast<int32_t*>(lds4);
}

template <int MEM>
__device__ __forceinline__ int32_t* node_base(const Params& p, int slot) {
  if constexpr (MEM == kMemGlobal) {
    return p.gnodes + static_cast<size_t>(slot) * p.stride;
  } else {
    return lists_base() + list_lds_words(p.list_cap);
  }
}

// ---- instances -------------------------------------------------------------------------------

// Whole workgroup: make instance j the one the node operations work on. Its row pointers are
// copied into LDS right after the node when the launch has room for them (one LDS access
// instead of an L2 round trip at the head of every row walk), and its column indices after
// them when the launch has room for those too (every row walk of a rule pass is then a chain
// of LDS accesses); the copy ends with a barrier. The copies read only the instance's own
// n + 1 row pointers and nnz entries, so they stay in bounds whatever the graph holds.
// Graphs whose column indices stay in device memory (up to 1 MB of them) are first touched
// once per 128-byte line, with independent loads, so that the dependent row walks of the rule
// passes find them in this XCD's L2.
constexpr int32_t kTouchMaxEntries = 1 << 18;

// Average degree from which a removal step spreads its rows over the wavefronts.
constexpr int32_t kSpreadDegree = 8;

template <int MEM>
__device__ __forceinline__ Node make_node(const Params& p, int32_t* st, const Instance& in,
                                          const int32_t* rp, const int32_t* ci) {
  return Node{st, in.n, rp, ci, lists_base(), static_cast<uint32_t>(p.list_cap) - 1u,
              in.nnz / kSpreadDegree >= in.n, MEM == kMemGlobal};
}

// Copy `count` words into LDS, eight independent loads per thread and step (one at a time, a
// root's 16,000 row pointers took sixteen device-memory latencies).
__device__ __forceinline__ void stage(int32_t* dst, const int32_t* __restrict__ src, int count) {
  constexpr int kAhead = 8;
  for (int i0 = threadIdx.x; i0 < count; i0 += kAhead * blockDim.x) {
    int32_t x[kAhead];
#pragma unroll
    for (int u = 0; u < kAhead; ++u) {
      const int i = i0 + u * static_cast<int>(blockDim.x);
      x[u] = src[i < count ? i : count - 1];
    }
#pragma unroll
    for (int u = 0; u < kAhead; ++u) {
      const int i = i0 + u * static_cast<int>(blockDim.x);
      if (i < count) dst[i] = x[u];
    }
  }
}

template <int MEM>
__device__ __forceinline__ Node load_instance(const Params& p, int j, int32_t* st) {
  const Instance in = p.inst[j];
  const int32_t* rp = p.rp_all + in.rp_off;
  const int32_t* ci = p.ci_all + in.ci_off;
  int32_t acc = 0;
  if constexpr (MEM == kMemLds || MEM == kMemLdsRp) {
    if (in.nnz <= kTouchMaxEntries)
      for (int i = threadIdx.x * 32; i < in.nnz; i += blockDim.x * 32) acc ^= ci[i];
  }
  if constexpr (MEM >= kMemLdsRp) {
    int32_t* dst = st + p.stride;
    stage(dst, rp, in.n + 1);
    if constexpr (MEM == kMemLdsCsr) {
      int32_t* dci = dst + rp_lds_words(p.n_max);
      stage(dci, ci, in.nnz);
      ci = dci;
    }
    __syncthreads();
    rp = dst;
  }
  asm volatile("" ::"v"(acc));  // the touches are waited for last
  return make_node<MEM>(p, st, in, rp, ci);
}

// A node with no instance yet, whose CSR pointers already point where this memory mode keeps
// them (so that the compiler sees one kind of memory behind each pointer).
template <int MEM>
__device__ __forceinline__ Node empty_node(const Params& p, int32_t* st) {
  const int32_t* rp = p.rp_all;
  const int32_t* ci = p.ci_all;
  if constexpr (MEM >= kMemLdsRp) rp = st + p.stride;
  if constexpr (MEM == kMemLdsCsr) ci = st + p.stride + rp_lds_words(p.n_max);
  return make_node<MEM>(p, st, Instance{}, rp, ci);
}

// Whole workgroup: the root of instance j in LDS -- the input's degree array, s = 0, nothing
// pending, the instance in the last word. Ends with a barrier.
__device__ __forceinline__ void build_root(const Params& p, const Node& nd, int j) {
  for (int v = threadIdx.x; v < p.stride; v += blockDim.x) {
    int32_t x = 0;
    if (v < nd.n) x = nd.rp[v + 1] - nd.rp[v];
    else if (v == nd.n + 1) x = -1;
    else if (v == p.stride - 1) x = j;
    nd.st[v] = x;
  }
  __syncthreads();
}

// Launch-local instance holding packed vertex i (or CSR entry i): the last instance whose
// first index is <= i. Instances with no vertices (entries) share their first index with the
// next one, so the search lands on the instance that owns i.
__device__ __forceinline__ int instance_of_vertex(const Params& p, int64_t i) {
  int lo = 0, hi = p.num_inst - 1;
  while (lo < hi) {
    const int mid = lo + ((hi - lo + 1) >> 1);
    if (p.inst[mid].vtx_first <= i) lo = mid; else hi = mid - 1;
  }
  return lo;
}
__device__ __forceinline__ int instance_of_entry(const Params& p, int64_t i) {
  int lo = 0, hi = p.num_inst - 1;
  while (lo < hi) {
    const int mid = lo + ((hi - lo + 1) >> 1);
    if (p.inst[mid].ent_first <= i) lo = mid; else hi = mid - 1;
  }
  return lo;
}

// ---- worklist ---------------------------------------------------------------------------------

// Whole workgroup: donate a deferred child of instance `inst` to the worklist; true if the
// worklist took it. The child is the stored node at `oldest` (the bottom of this workgroup's
// stack) when that is not null, else the node in LDS with `pending` as its branch vertex.
__device__ __forceinline__ bool try_enqueue(const Params& p, const Node nd, Ctrl& c, int pending,
                            const int32_t* oldest, int inst) {
  if (!enqueue_begin(p, c, inst)) return false;
  int32_t* dst = p.payload + static_cast<size_t>(c.slot) * p.stride;
  if (oldest) node_copy(dst, oldest, p.stride);
  else node_store(dst, nd.st, p.stride, nd.n, pending);
  enqueue_publish(p, c);
  return true;
}

// ---- kernels ---------------------------------------------------------------------------------


// Row v of a CSR: are its bounds wrong?
__device__ __forceinline__ bool row_bad(const int32_t* __restrict__ rp, int n, int nnz, int v) {
  const int beg = rp[v], end = rp[v + 1];
  return (v == 0 && beg != 0) || (v == n - 1 && end != nnz) || beg < 0 || end < beg || end > nnz;
}

// Row v (of good bounds) as adjacency words.
__device__ __forceinline__ void pack_row(const int32_t* __restrict__ rp,
                                         const int32_t* __restrict__ ci, int n, int v, int words,
                                         uint64_t* __restrict__ dst) {
  uint64_t row[kMaxBitsetWords] = {};
  for (int e = rp[v]; e < rp[v + 1]; ++e) {
    const int u = ci[e];
    if (u >= 0 && u < n) row[u >> 6] |= 1ull << (u & 63);
  }
  for (int w = 0; w < words; ++w) dst[w] = row[w];
}

// CSR entry e: the row it makes the graph invalid in (out of range, a self-loop, not above the
// entry before it, or not present in reverse), kNoRow if none. Every read is bounds-checked
// before it is made.
__device__ __forceinline__ int32_t entry_bad_row(const int32_t* __restrict__ rp,
                                                 const int32_t* __restrict__ ci, int n, int nnz,
                                                 int e) {
  const int v = owner_row(rp, n, e);
  const int beg = rp[v], end = rp[v + 1];
  if (!(beg <= e && e < end && beg >= 0 && end <= nnz)) return kNoRow;  // row_bad finds it
  const int u = ci[e];
  bool bad = u < 0 || u >= n || u == v || (e > beg && ci[e - 1] >= u);
  if (!bad) {
    const int ub = rp[u], ue = rp[u + 1];
    bad = ub < 0 || ue < ub || ue > nnz;
    if (!bad) {
      int lo = ub, hi = ue;
      while (lo < hi) {
        const int mid = lo + ((hi - lo) >> 1);
        if (ci[mid] < v) lo = mid + 1; else hi = mid;
      }
      bad = lo >= ue || ci[lo] != v;
    }
  }
  return bad ? v : kNoRow;
}

// Whole workgroup: the launch's control lines and result block.
__device__ __forceinline__ void reset_launch(const Params& p, DevResult* res) {
  for (int i = threadIdx.x; i < kNumCounters * kCounterStride; i += blockDim.x) p.ctr[i] = 0;
  char* r = reinterpret_cast<char*>(res);
  for (int i = threadIdx.x; i < static_cast<int>(sizeof(DevResult)); i += blockDim.x) r[i] = 0;
  __syncthreads();
  if (threadIdx.x == 0) {
    *ctr_i32(p, kWork) = p.num_inst;
    *ctr_i32(p, kOpen) = p.num_inst;
    res->wg_nodes_min = INT64_MAX;
  }
}

// Check every graph of the launch (simple undirected, §II-A). Index i < vertices checks row
// i's bounds (and, for the bitset kernels, packs the row into adjacency words); index i <
// entries checks one CSR entry. A malformed input cannot send a thread out of its instance's
// arrays. Each instance keeps the smallest offending row.
//
// The same launch first resets the launch's control lines and result block and marks every
// worklist slot free (the host uploads the fresh per-instance state with the instance table);
// every instance's root is handed out by the root ticket counter, so the worklist starts empty.
// Nothing in the validation reads what the reset writes.
__global__ void prepare_kernel(Params p, DevResult* res, int64_t vertices, int64_t entries) {
  const int64_t total = vertices > entries ? vertices : entries;
  const int64_t gsize = static_cast<int64_t>(gridDim.x) * blockDim.x;
  if (blockIdx.x == 0) reset_launch(p, res);
  for (int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < p.q_cap;
       i += gsize)
    p.seq[i] = 0u;
  for (int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < total;
       i += gsize) {
    if (i < vertices) {
      const int j = instance_of_vertex(p, i);
      const Instance in = p.inst[j];
      const int v = static_cast<int>(i - in.vtx_first);
      const int32_t* rp = p.rp_all + in.rp_off;
      const int32_t* ci = p.ci_all + in.ci_off;
      const bool bad = row_bad(rp, in.n, in.nnz, v);
      if (bad) atomicMin(&p.ist[j].err_row, v);
      if (p.words && !bad)
        pack_row(rp, ci, in.n, v, p.words,
                 p.bits + (static_cast<int64_t>(in.vtx_first) + v) * p.words);
    }
    if (i < entries) {
      const int j = instance_of_entry(p, i);
      const Instance in = p.inst[j];
      const int32_t bad = entry_bad_row(p.rp_all + in.rp_off, p.ci_all + in.ci_off, in.n, in.nnz,
                                        static_cast<int>(i - in.ent_first));
      if (bad != kNoRow) atomicMin(&p.ist[j].err_row, bad);
    }
  }
}

// prepare_kernel for a launch of one small graph (see kSmallEntries). Block 0 copies the CSR into
// LDS, where the searches of an entry's check cost a tenth of what they cost in L2, and writes the
// instance table, state and work counter itself, so that the call needs no copy command before its
// first kernel (G(60, 0.1): a copy, a gap and a validation of 25 us became one launch); the other
// blocks free the worklist's slots.
__global__ void __launch_bounds__(1024) prepare_small_kernel(Params p, DevResult* res, Instance in) {
  extern __shared__ int32_t csr[];
  __shared__ int32_t err;
  if (blockIdx.x > 0) {
    for (uint32_t i = (blockIdx.x - 1) * blockDim.x + threadIdx.x; i < p.q_cap;
         i += (gridDim.x - 1) * blockDim.x)
      p.seq[i] = 0u;
    return;
  }
  int32_t* rp = csr;
  int32_t* ci = csr + in.n + 1;
  stage(rp, p.rp_all + in.rp_off, in.n + 1);
  if (in.nnz > 0) stage(ci, p.ci_all + in.ci_off, in.nnz);
  if (threadIdx.x == 0) err = kNoRow;
  reset_launch(p, res);  // holds a barrier
  for (int v = threadIdx.x; v < in.n; v += blockDim.x) {
    if (row_bad(rp, in.n, in.nnz, v)) atomicMin(&err, v);
    else if (p.words) pack_row(rp, ci, in.n, v, p.words, p.bits + static_cast<int64_t>(v) * p.words);
  }
  for (int e = threadIdx.x; e < in.nnz; e += blockDim.x) {
    const int32_t bad = entry_bad_row(rp, ci, in.n, in.nnz, e);
    if (bad != kNoRow) atomicMin(&err, bad);
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    InstState s{};
    s.best = kNoBest;
    s.err_row = err;
    s.greedy = -1;
    *const_cast<Instance*>(p.inst) = in;
    *p.ist = s;
    *p.work = 1;
  }
}

// Greedy approximation (§II-B, used as an instance's first best and for the stack depth bound,
// §IV-E): degree-one and degree-two-triangle rules, then a maximum-degree vertex into the
// cover, until no edge is left. One workgroup per instance (a grid-stride loop over the
// launch's instances); the cover goes to the instance's cover output.
template <int MEM>
__global__ void __launch_bounds__(1024) greedy_kernel(Params p) {
  __shared__ Ctrl c;
  int32_t* st = node_base<MEM>(p, blockIdx.x);
  if (threadIdx.x == 0) {
    c.rm_tail = c.one_tail = c.two_tail = 0;
    if (blockIdx.x == 0) p.res->t_greedy = realtime();
  }
  Front f{};
  for (int j = blockIdx.x; j < p.num_inst; j += gridDim.x) {
    if (threadIdx.x == 0) c.err = load_relaxed(&p.ist[j].err_row) != kNoRow;
    __syncthreads();
    const bool skip = c.err;
    __syncthreads();  // every thread has read c.err before thread 0 writes it again
    if (skip) continue;
    const Node nd = load_instance<MEM>(p, j, st);
    build_root(p, nd, j);
    f.s = 0;
    f.wide = false;
    const int64_t unbounded = 0x3FFFFFFFFFFFFFFFll;
    for (;;) {
      reduce_node(nd, c, f, unbounded, kRuleDeg1 | kRuleTri);
      int vmax;
      int32_t degsum;
      max_degree_and_sum(nd, c, f, vmax, degsum);
      if (degsum == 0) break;
      remove_vertex(nd, f, vmax);
    }
    const int s = f.s;
    uint8_t* cov = p.covers + p.inst[j].vtx_off;
    store_cover(cov, nd);
    if (threadIdx.x == 0) {
      p.ist[j].best = s;
      p.ist[j].greedy = s;
    }
    __syncthreads();  // the node and row pointers in LDS are read before the next instance
  }
}

// Thread 0: claim the right to record a cover of size s for instance j (§IV-A: atomic best /
// found). PVC: the first cover found wins. MVC: a cover wins if it lowers the instance's best;
// the winner then takes the instance's lock, and keeps it only if no smaller cover has been
// claimed meanwhile, so the last cover written under the lock is one of the final best size.
template <bool PVC>
__device__ __forceinline__ int claim_solution(const Params& p, int j, int32_t s) {
  InstState* is = p.ist + j;
  if (PVC) return (atomicOr(&is->state, kInstFound) & kInstFound) == 0;
  if (atomicMin(&is->best, s) <= s) return 0;
  lock_acquire(&is->lock);
  if (load_relaxed(&is->best) == s) return 1;
  store_release(&is->lock, 0);
  return 0;
}

// Thread 0, after the whole workgroup has written the cover and fenced it: finish the claim.
template <bool PVC>
__device__ __forceinline__ void publish_solution(const Params& p, int j, int32_t s) {
  InstState* is = p.ist + j;
  if (PVC) {
    store_relaxed(&is->best, s);
    fetch_add(ctr_i32(p, kOpen), -1);
  } else {
    store_release(&is->lock, 0);
  }
}

// Thread 0: add this workgroup's nodes on instance j to the instance's counter, and mark the
// instance out of budget once the counter reaches the per-instance budget.
__device__ __forceinline__ void report_nodes(const Params& p, int j, int64_t count) {
  if (count <= 0) return;
  unsigned long long* total = reinterpret_cast<unsigned long long*>(&p.ist[j].nodes);
  const unsigned long long before = fetch_add(total, static_cast<unsigned long long>(count));
  if (p.node_budget > 0 && static_cast<int64_t>(before) + count >= p.node_budget)
    atomicOr(&p.ist[j].state, kInstOutOfBudget);
}

// The hybrid traversal (§IV-A, Fig. 4; PVC differences in §IV-A, termination §IV-C) over every
// instance of the launch. A workgroup takes the root of an unstarted instance or a node from
// the worklist, walks that node's sub-tree depth first with its stack, and loads an instance
// (row pointers) only when the node it takes belongs to another one than the last.
template <bool PVC, bool PROF, int MEM, bool SO>
__global__ void __launch_bounds__(1024) traverse_kernel(Params args) {
  __shared__ Ctrl c;
  int32_t* st = node_base<MEM>(args, blockIdx.x);
  const int rules = args.rules;
  const int wg = blockIdx.x;
  const int tid = threadIdx.x;
  if (tid == 0) {
    c.stop = 0;
    c.rm_tail = c.one_tail = c.two_tail = 0;
  }
  __syncthreads();
  ActivityClock<PROF> clk;
  clk.begin();
  if (tid == 0) watch_begin(args, c);
  uint32_t headers = 0;  // thread 0: node headers read so far
  uint64_t root_header = 0;   // thread 0: a root's header, loaded when the root was taken
  bool header_ready = false;
  bool first = true;          // the workgroup has not looked for work yet

  const auto stack_slot = [&](const Params& p, int at) -> int32_t* {
    return p.stacks +
           (static_cast<size_t>(wg) * p.depth_cap + static_cast<size_t>(at % p.depth_cap)) * p.stride;
  };
  // The stack is a ring of depth_cap entries holding [bot, top): pops take the top, donations
  // take the bottom (the oldest deferred child, nearest its sub-tree root). Every entry belongs
  // to the instance of the sub-tree being walked.
  int top = 0, bot = 0;
  bool have = false;      // a node is in LDS and still to be visited
  bool holding = false;   // this workgroup holds a sub-tree (a root or a worklist node)
  bool marked = false;    // the node in LDS has flagged vertices still to be removed
  int cur = -1;           // instance of the node in LDS
  int32_t cur_k = 0, cur_vtx = 0;
  Node nd = empty_node<MEM>(args, st);
  Front f{};
  int64_t nodes = 0, pushes = 0, pops = 0, enqueues = 0, dequeues = 0, insts = 0;
  int64_t unreported = 0;  // nodes on `cur` not yet added to its counter
  int max_depth = 0;
  uint32_t so_path = 0;    // StackOnly: the current path index

  for (;;) {
    if (!have) {
      const Params& p = cold_params();
      marked = false;   // whatever node comes next replaces the one in LDS
      f.rm = c.rm_tail;  // (what a dropped node still had marked is no longer to be removed)
      __syncthreads();  // every thread has read the last broadcast before thread 0 writes
      if (top > bot) {
        --top;
        node_load(st, stack_slot(p, top), p.stride);
        ++pops;
        __syncthreads();
        clk.charge(kActAcquire);
      } else if constexpr (SO) {
        // StackOnly (the comparison method of §V-A), as in bitset_traverse_kernel: walk this
        // workgroup's next path down from the root, then take the node at the start depth.
        if (cur < 0) {
          nd = load_instance<MEM>(p, 0, st);
          const Instance in = p.inst[0];
          cur = 0;
          cur_k = in.k;
          cur_vtx = in.vtx_off;
          ++insts;
          so_path = static_cast<uint32_t>(wg);
        } else {
          so_path += static_cast<uint32_t>(p.num_wg);
        }
        if (tid == 0) c.err = load_relaxed(&p.ist[0].err_row) != kNoRow;
        __syncthreads();
        if (so_path >= (1u << p.start_depth) || c.err) {
          clk.charge(kActAcquire);
          break;
        }
        build_root(p, nd, 0);
        f.s = 0;
        bool reached = true;
        for (int d = 0; d < p.start_depth && reached; ++d) {
          const bool owner = (so_path >> d) == 0;
          if (tid == 0) {
            const uint64_t h = inst_header(p, cur);
            const int32_t state = static_cast<int32_t>(h >> 32);
            c.drop = (state & kInstOutOfBudget) | (PVC ? (state & kInstFound) : 0);
            c.best = static_cast<int32_t>(static_cast<uint32_t>(h));
          }
          __syncthreads();
          if (c.drop) {
            reached = false;
            break;
          }
          const int64_t bound = PVC ? static_cast<int64_t>(cur_k) : static_cast<int64_t>(c.best) - 1;
          ++nodes;
          if (owner) ++unreported;
          reduce_node(nd, c, f, bound, rules, clk, marked);
          marked = false;
          const int32_t s = f.s;
          const int64_t r = bound - s;
          int vmax = 0;
          int32_t degsum = 0;
          if (r >= 0) max_degree_and_sum(nd, c, f, vmax, degsum);
          const int64_t edges = degsum / 2;
          if (r < 0 || ((rules & kPruneEdges) && (rules & kRuleHigh) && edges > r * r)) {
            reached = false;
          } else if (edges == 0) {  // a cover: recorded once, on the owning path
            if (owner) {
              if (tid == 0) c.status = claim_solution<PVC>(p, cur, s);
              __syncthreads();
              if (c.status) {
                uint8_t* cov = p.covers + cur_vtx;
                store_cover(cov, nd);
                __threadfence();
                __syncthreads();
                if (tid == 0) publish_solution<PVC>(p, cur, s);
              }
            }
            reached = false;
          } else {
            marked = (so_path >> d) & 1u;
            if (marked) mark_neighbourhood(nd, c, vmax);
            else remove_vertex(nd, f, vmax);
          }
          __syncthreads();  // every thread has read c.* before thread 0 writes it again
        }
        clk.charge(kActAcquire);
        if (!reached) continue;
      } else {
        if (holding) {
          if (tid == 0) release_work(p, cur);
          holding = false;
        }
        const int got = dequeue_begin(p, c, first);
        if (got != 1 && got != 2) {
          clk.charge(kActAcquire);
          break;
        }
        int j;
        if (got == 1) {
          node_load(st, p.payload + static_cast<size_t>(c.slot) * p.stride, p.stride);
          dequeue_finish(p, c);  // ends with a barrier: the node is visible to every thread
          j = st[p.stride - 1];
          ++dequeues;
          if (j < 0 || j >= p.num_inst) {  // cannot happen: every stored node names its instance
            if (tid == 0) {
              atomicMax(ctr_i32(p, kError), 2);
              store_relaxed(ctr_i32(p, kAbort), 1);
            }
            break;
          }
        } else {
          j = static_cast<int>(c.slot);  // an unstarted instance: its root
        }
        holding = true;
        clk.charge(kActAcquire);
        // a root: its input check and its first header are loaded now, while the instance is
        // being staged, instead of one after the other once it is
        int32_t err_row = kNoRow;
        if (got == 2 && tid == 0) {
          err_row = load_relaxed(&p.ist[j].err_row);
          root_header = inst_header(p, j);
          header_ready = true;
        }
        if (j != cur) {
          if (tid == 0 && cur >= 0) report_nodes(p, cur, unreported);
          unreported = 0;
          nd = load_instance<MEM>(p, j, st);
          f.wide = false;
          const Instance in = p.inst[j];
          cur = j;
          cur_k = in.k;
          cur_vtx = in.vtx_off;
          ++insts;
        }
        if (got == 2) {
          // c.err, not c.status: slow waves may still be reading the dequeue status
          if (tid == 0) c.err = err_row != kNoRow;
          __syncthreads();
          if (c.err) {  // rejected input: no search (PVC: the instance is settled)
            if (PVC && tid == 0) fetch_add(ctr_i32(p, kOpen), -1);
            header_ready = false;
            continue;
          }
          build_root(p, nd, j);
        }
        clk.charge(kActOther);
      }
      f.s = st[nd.n];
      const int pending = st[nd.n + 1];
      if (pending >= 0) {
        __syncthreads();  // every thread has read the pending vertex
        if (tid == 0) st[nd.n + 1] = -1;
        mark_neighbourhood(nd, c, pending);
        marked = true;
      }
      clk.charge(kActBranch);
      have = true;
    }

    // node header: the instance's flags and current best (one load), and every 16 nodes
    // the launch-wide stop (idle workgroups also look at it while they wait for work)
    if (tid == 0) {
      const Params& p = cold_params();
      const uint64_t h = header_ready ? root_header : inst_header(p, cur);
      header_ready = false;
      const int32_t state = static_cast<int32_t>(h >> 32);
      if ((headers++ & 15) == 0) c.stop = search_stopped(p, c);
      c.drop = (state & kInstOutOfBudget) | (PVC ? (state & kInstFound) : 0);
      c.best = static_cast<int32_t>(static_cast<uint32_t>(h));
    }
    __syncthreads();
    clk.charge(kActOther);
    if (c.stop) break;
    if (c.drop) {  // answered or out of budget: drop this node and the rest of the sub-tree
      have = false;
      top = bot;
      continue;
    }

    ++nodes;
    ++unreported;
    {
      const Params& p = cold_params();
      if (p.node_budget > 0 && unreported >= p.budget_chunk) {
        if (tid == 0) report_nodes(p, cur, unreported);
        unreported = 0;
      }
    }

    const int64_t bound = PVC ? static_cast<int64_t>(cur_k) : static_cast<int64_t>(c.best) - 1;
    reduce_node(nd, c, f, bound, rules, clk, marked);
    marked = false;
    clk.charge(kActReduce);

    // stopping condition (§II-B): no cover of size <= bound below this node if r < 0 or
    // |E| > r^2 (every remaining degree is <= r once the high-degree rule has run)
    const int n = nd.n;
    const int32_t s = f.s;
    const int64_t r = bound - s;
    if (r < 0) {
      have = false;
      continue;
    }
    int vmax;
    int32_t degsum;
    max_degree_and_sum(nd, c, f, vmax, degsum);
    clk.charge(kActBranch);
    const int64_t edges = degsum / 2;
    if ((rules & kPruneEdges) && (rules & kRuleHigh) && edges > r * r) {
      have = false;
      continue;
    }
    const Params& p = cold_params();
    if (edges == 0) {  // a vertex cover of size s
      if (tid == 0) c.status = claim_solution<PVC>(p, cur, s);
      __syncthreads();
      if (c.status) {
        uint8_t* cov = p.covers + cur_vtx;
        store_cover(cov, nd);
        __threadfence();
        __syncthreads();
        if (tid == 0) publish_solution<PVC>(p, cur, s);
      }
      clk.charge(kActOther);
      have = false;
      continue;
    }

    // branch on v_max (§II-B): defer the N(v_max) child, continue with the v_max child. While
    // the worklist is below its threshold a deferred child is donated (§IV-A): the oldest one on
    // this workgroup's stack if there is one (the largest sub-tree it holds), else this one.
    bool kept_local = true;
    if (p.q_threshold > 0) {
      const bool from_stack = top > bot;
      const int32_t* oldest =
          from_stack ? stack_slot(p, bot) : nullptr;
      if (try_enqueue(p, nd, c, vmax, oldest, cur)) {
        ++enqueues;
        if (from_stack) ++bot;
        else kept_local = false;
      }
    }
    if (kept_local) {
      if (top - bot >= p.depth_cap) {  // cannot happen: the depth bound of §IV-E holds
        if (tid == 0) {
          atomicMax(ctr_i32(p, kError), 1);
          store_relaxed(ctr_i32(p, kAbort), 1);
        }
        break;
      }
      node_store(stack_slot(p, top), st, p.stride, n, vmax);
      ++top;
      ++pushes;
      if (top - bot > max_depth) max_depth = top - bot;
      __syncthreads();  // the copy has read the node before it changes below
    }
    clk.charge(kActDonate);
    remove_vertex(nd, f, vmax);
    clk.charge(kActBranch);
  }
  clk.end();

  if (tid == 0) {
    const Params& p = cold_params();
    if (cur >= 0) report_nodes(p, cur, unreported);
    WgStats w{};
    w.nodes = nodes;
    w.pushes = pushes;
    w.pops = pops;
    w.enqueues = enqueues;
    w.dequeues = dequeues;
    w.max_depth = max_depth;
    w.instances = static_cast<int32_t>(insts);
    for (int a = 0; a < kNumActivities; ++a) w.cycles[a] = static_cast<int64_t>(clk.cycles[a]);
    publish_wg_stats(p, wg, w);
  }
}

// Add each lane's x to *dst (dst may differ between lanes, or be null): one atomic per distinct
// destination in the wavefront. Whole wavefront, uniform control flow.
__device__ void add_grouped(int32_t* dst, int32_t x) {
  bool pending = dst != nullptr && x != 0;
  const uint64_t mine_addr = reinterpret_cast<uint64_t>(dst);
  for (;;) {
    const uint64_t m = __builtin_amdgcn_ballot_w64(pending);
    if (!m) break;
    const int leader = first_lane(m);
    const uint64_t target = readlane64(mine_addr, leader);
    const bool mine = pending && mine_addr == target;
    const int32_t sum = wave_sum(mine ? x : 0);
    if (lane_id() == leader) atomicAdd(reinterpret_cast<int32_t*>(target), sum);
    if (mine) pending = false;
  }
}

// After the traversal (256-thread blocks, any grid): check each recorded cover edge by edge
// and count its vertices. One wavefront per 64 consecutive vertices of the launch: a vertex in
// the cover covers its whole row, so only the rows of vertices outside it are walked (as one
// list, one lane per entry), and each entry of such a row must lead into the cover; an
// uncovered edge is counted from each end. Clear the cover output of instances without an
// answer (rejected, out of budget, PVC no). (The traversal's workgroups add their statistics
// to the result block themselves.) Packed entry offsets must fit in int32.
// With ist_host, the last block to finish writes the instances' states and the result block to
// host memory, which saves the call a copy command after its last kernel.
__global__ void __launch_bounds__(256) finalize_kernel(Params p, int64_t vertices, DevResult* res,
                                                       InstState* ist_host, DevResult* res_host) {
  if (blockIdx.x == 0 && threadIdx.x == 0) res->t_end = realtime();
  const int64_t waves = static_cast<int64_t>(gridDim.x) * (blockDim.x >> 6);
  for (int64_t w = static_cast<int64_t>(blockIdx.x) * (blockDim.x >> 6) + wave_id();
       w * 64 < vertices; w += waves) {
    const int64_t i = w * 64 + lane_id();
    int32_t* ones_dst = nullptr;
    int32_t one = 0;
    int beg = 0, end = 0, j = 0;
    if (i < vertices) {
      j = instance_of_vertex(p, i);
      const Instance in = p.inst[j];
      const InstState is = p.ist[j];
      const bool answer = is.err_row == kNoRow && !(is.state & kInstOutOfBudget) &&
                          (!p.pvc || (is.state & kInstFound));
      uint8_t* cov = p.covers + in.vtx_off;
      const int v = static_cast<int>(i - in.vtx_first);
      if (answer) {
        one = cov[v] != 0;
        if (!one) {
          const int32_t* rp = p.rp_all + in.rp_off;
          beg = static_cast<int>(in.ci_off) + rp[v];
          end = static_cast<int>(in.ci_off) + rp[v + 1];
        }
      } else {
        cov[v] = 0;
      }
      ones_dst = &p.ist[j].cover_count;
    }
    add_grouped(ones_dst, one);
    walk_rows(p.ci_all, beg, end, j, [&](const Walked& w) {
      uint8_t c[kWalk];
#pragma unroll
      for (int u = 0; u < kWalk; ++u)
        c[u] = w.ok[u] ? p.covers[p.inst[w.tags[u]].vtx_off + w.xs[u]] : 1;
#pragma unroll
      for (int u = 0; u < kWalk; ++u)
        if (c[u] == 0) atomicAdd(&p.ist[w.tags[u]].uncovered, 1);
    });
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    res->aborted = *ctr_i32(p, kAbort);
    res->error = *ctr_i32(p, kError);
    res->stop_reason = *ctr_i32(p, kStopReason);
  }
  if (ist_host == nullptr) return;
  __shared__ int last;
  __threadfence();  // this thread's counts and result fields, before its block counts as done
  __syncthreads();
  if (threadIdx.x == 0)
    last = fetch_add(ctr_i32(p, kDone), 1) == static_cast<int32_t>(gridDim.x) - 1;
  __syncthreads();
  if (!last) return;
  __threadfence();
  // agent-scope loads: other blocks' counts and fields may sit in other XCDs' caches
  using ull = unsigned long long;
  const int states = p.num_inst * static_cast<int>(sizeof(InstState) / sizeof(ull));
  constexpr int kRes = static_cast<int>(sizeof(DevResult) / sizeof(ull));
  for (int i = threadIdx.x; i < states + kRes; i += blockDim.x) {
    if (i < states)
      reinterpret_cast<ull*>(ist_host)[i] = load_relaxed(reinterpret_cast<ull*>(p.ist) + i);
    else
      reinterpret_cast<ull*>(res_host)[i - states] =
          load_relaxed(reinterpret_cast<ull*>(res) + (i - states));
  }
}
static_assert(sizeof(InstState) % 8 == 0 && sizeof(DevResult) % 8 == 0, "copied in 8-byte words");

// The reduction rules of one node, alone, on a degree array in device memory (instance 0 of
// the launch, one workgroup). A rejected input leaves the degree array alone.
template <int MEM>
__global__ void __launch_bounds__(1024) reduce_kernel(Params p, int32_t* deg, int32_t* s,
                                                      int64_t bound) {
  __shared__ Ctrl c;
  int32_t* st = node_base<MEM>(p, 0);
  if (threadIdx.x == 0) {
    c.err = load_relaxed(&p.ist[0].err_row) != kNoRow;
    c.rm_tail = c.one_tail = c.two_tail = 0;
  }
  __syncthreads();
  if (c.err) return;
  const Node nd = load_instance<MEM>(p, 0, st);
  const int n = nd.n;
  for (int v = threadIdx.x; v < p.stride; v += blockDim.x)
    st[v] = v < n ? deg[v] : (v == n ? *s : (v == n + 1 ? -1 : 0));
  __syncthreads();
  Front f{};
  f.s = st[n];
  reduce_node(nd, c, f, bound, p.rules);
  for (int v = threadIdx.x; v < n; v += blockDim.x) deg[v] = st[v] < 0 ? kSent : (st[v] & kDegMask);
  if (threadIdx.x == 0) *s = st[n];
}

// Largest greedy cover size over the launch's instances (the stack depth bound of MVC).
__global__ void __launch_bounds__(256) max_greedy_kernel(Params p, int32_t* out) {
  if (threadIdx.x == 0) p.res->t_greedy_end = realtime();
  int32_t m = 0;
  for (int j = threadIdx.x; j < p.num_inst; j += blockDim.x) {
    const int32_t g = p.ist[j].greedy;
    m = g > m ? g : m;
  }
  m = static_cast<int32_t>(wave_max(static_cast<uint64_t>(static_cast<uint32_t>(m))));
  __shared__ int32_t part[4];
  if (lane_id() == 0) part[wave_id()] = m;
  __syncthreads();
  if (threadIdx.x == 0) {
    int32_t r = part[0];
    for (int w = 1; w < static_cast<int>(blockDim.x >> 6); ++w) r = part[w] > r ? part[w] : r;
    *out = r;
  }
}

// ---- launchers ---------------------------------------------------------------------------------

static int grid_for(int64_t items, int threads, int cap) {
  int64_t blocks = (items + threads - 1) / threads;
  if (blocks < 1) blocks = 1;
  if (blocks > cap) blocks = cap;
  return static_cast<int>(blocks);
}

hipError_t launch_prepare(const Params& p, DevResult* res, int64_t vertices, int64_t entries,
                          hipStream_t stream) {
  const int64_t items = vertices > entries ? vertices : entries;
  const int blocks = std::max(grid_for(items, 256, 4096), grid_for(p.q_cap, 256, 1024));
  hipLaunchKernelGGL(prepare_kernel, dim3(blocks), dim3(256), 0, stream, p, res, vertices,
                     entries);
  return hipGetLastError();
}

// Grid of the greedy launch (one workgroup per instance, at most 65,535); the device-memory
// node array needs this many slots.
int greedy_grid(const Params& p) { return p.num_inst < 65535 ? p.num_inst : 65535; }

// Memory mode of a launch: node in device memory, else in LDS with the row pointers (rp_lds 1)
// or the whole CSR (rp_lds 2) staged after it.
static int mem_mode(bool global_node, int32_t rp_lds) {
  if (global_node) return kMemGlobal;
  return rp_lds >= 2 ? kMemLdsCsr : (rp_lds == 1 ? kMemLdsRp : kMemLds);
}

template <int MEM>
static size_t launch_lds(const Params& p) {
  return 4 * list_lds_words(p.list_cap) +
         (MEM == kMemGlobal ? 0 : node_lds_bytes(p.stride, p.n_max, p.rp_lds, p.nnz_max));
}

template <int MEM>
static void greedy_on(const Params& p, int32_t wg_size, hipStream_t stream) {
  hipLaunchKernelGGL(greedy_kernel<MEM>, dim3(greedy_grid(p)), dim3(wg_size),
                     launch_lds<MEM>(p), stream, p);
}

hipError_t launch_greedy(const Params& p, int32_t wg_size, hipStream_t stream) {
  switch (mem_mode(p.gnodes != nullptr, p.rp_lds)) {
    case kMemGlobal: greedy_on<kMemGlobal>(p, wg_size, stream); break;
    case kMemLds: greedy_on<kMemLds>(p, wg_size, stream); break;
    case kMemLdsRp: greedy_on<kMemLdsRp>(p, wg_size, stream); break;
    default: greedy_on<kMemLdsCsr>(p, wg_size, stream); break;
  }
  return hipGetLastError();
}

template <int MEM, bool SO>
static const void* traverse_fn_m(bool pvc, bool prof) {
  if (pvc) return prof ? reinterpret_cast<const void*>(&traverse_kernel<true, true, MEM, SO>)
                       : reinterpret_cast<const void*>(&traverse_kernel<true, false, MEM, SO>);
  return prof ? reinterpret_cast<const void*>(&traverse_kernel<false, true, MEM, SO>)
              : reinterpret_cast<const void*>(&traverse_kernel<false, false, MEM, SO>);
}

// The StackOnly walk-down is a separate instantiation, so the hybrid kernels carry none of its
// registers.
template <bool SO>
static const void* traverse_fn_s(bool pvc, bool prof, int mem) {
  switch (mem) {
    case kMemGlobal: return traverse_fn_m<kMemGlobal, SO>(pvc, prof);
    case kMemLds: return traverse_fn_m<kMemLds, SO>(pvc, prof);
    case kMemLdsRp: return traverse_fn_m<kMemLdsRp, SO>(pvc, prof);
    default: return traverse_fn_m<kMemLdsCsr, SO>(pvc, prof);
  }
}
static const void* traverse_fn(bool pvc, bool prof, int mem, bool stack_only = false) {
  return stack_only ? traverse_fn_s<true>(pvc, prof, mem) : traverse_fn_s<false>(pvc, prof, mem);
}

// A plain launch: the grid is sized by the occupancy API so that all workgroups are normally
// resident together, but the search does not depend on it. A workgroup only ever waits for
// workgroups that have already taken a worklist ticket or an instance's lock (and are
// therefore running); one that starts late finds either work or a zero outstanding-work
// counter.
hipError_t launch_traverse(bool pvc, bool prof, const Params& p, int32_t wg_size,
                           hipStream_t stream) {
  const bool global_node = p.gnodes != nullptr;
  const size_t lds =
      4 * list_lds_words(p.list_cap) +
      (global_node ? 0 : node_lds_bytes(p.stride, p.n_max, p.rp_lds, p.nnz_max));
  Params args = p;
  void* kargs[] = {&args};
  return hipLaunchKernel(traverse_fn(pvc, prof, mem_mode(global_node, p.rp_lds), p.start_depth > 0),
                         dim3(p.num_wg), dim3(wg_size), kargs, lds, stream);
}

hipError_t launch_prepare_small(const Params& p, DevResult* res, const Instance& in,
                                hipStream_t stream) {
  const size_t lds = 4 * (static_cast<size_t>(in.n) + 1 + static_cast<size_t>(in.nnz));
  hipLaunchKernelGGL(prepare_small_kernel, dim3(1 + grid_for(p.q_cap, 4096, 16)), dim3(1024), lds,
                     stream, p, res, in);
  return hipGetLastError();
}

hipError_t launch_finalize(const Params& p, int64_t vertices, DevResult* res, InstState* ist_host,
                           DevResult* res_host, hipStream_t stream) {
  hipLaunchKernelGGL(finalize_kernel, dim3(grid_for(vertices, 256, 1024)), dim3(256), 0, stream, p,
                     vertices, res, ist_host, res_host);
  return hipGetLastError();
}

template <int MEM>
static void reduce_on(const Params& p, int32_t wg_size, int32_t* deg, int32_t* s, int64_t bound,
                      hipStream_t stream) {
  hipLaunchKernelGGL(reduce_kernel<MEM>, dim3(1), dim3(wg_size), launch_lds<MEM>(p),
                     stream, p, deg, s, bound);
}

hipError_t launch_reduce(const Params& p, int32_t wg_size, int32_t* deg, int32_t* s,
                         int64_t bound, hipStream_t stream) {
  switch (mem_mode(p.gnodes != nullptr, p.rp_lds)) {
    case kMemGlobal: reduce_on<kMemGlobal>(p, wg_size, deg, s, bound, stream); break;
    case kMemLds: reduce_on<kMemLds>(p, wg_size, deg, s, bound, stream); break;
    case kMemLdsRp: reduce_on<kMemLdsRp>(p, wg_size, deg, s, bound, stream); break;
    default: reduce_on<kMemLdsCsr>(p, wg_size, deg, s, bound, stream); break;
  }
  return hipGetLastError();
}

hipError_t launch_max_greedy(const Params& p, int32_t* out, hipStream_t stream) {
  hipLaunchKernelGGL(max_greedy_kernel, dim3(1), dim3(256), 0, stream, p, out);
  return hipGetLastError();
}

hipError_t traverse_occupancy(bool pvc, bool prof, bool global_node, int32_t rp_lds,
                              int32_t wg_size, size_t lds_bytes, int* blocks_per_cu) {
  const void* fn = traverse_fn(pvc, prof, mem_mode(global_node, rp_lds));
  return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks_per_cu, fn, wg_size, lds_bytes);
}

// Every degree-array kernel: with the node in device memory too, the lists alone take up to 96 KB.
hipError_t set_lds_limit(size_t lds_bytes) {
  for (int mem = kMemGlobal; mem <= kMemLdsCsr; ++mem) {
    const void* fns[] = {traverse_fn(true, false, mem), traverse_fn(false, false, mem),
                         traverse_fn(true, true, mem), traverse_fn(false, true, mem),
                         traverse_fn(true, false, mem, true), traverse_fn(false, false, mem, true),
                         traverse_fn(true, true, mem, true), traverse_fn(false, true, mem, true)};
    for (const void* fn : fns) {
      hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize,
                                         static_cast<int>(lds_bytes));
      if (e != hipSuccess) return e;
    }
  }
  const void* others[] = {
      reinterpret_cast<const void*>(&greedy_kernel<kMemGlobal>),
      reinterpret_cast<const void*>(&greedy_kernel<kMemLds>),
      reinterpret_cast<const void*>(&greedy_kernel<kMemLdsRp>),
      reinterpret_cast<const void*>(&greedy_kernel<kMemLdsCsr>),
      reinterpret_cast<const void*>(&reduce_kernel<kMemGlobal>),
      reinterpret_cast<const void*>(&reduce_kernel<kMemLds>),
      reinterpret_cast<const void*>(&reduce_kernel<kMemLdsRp>),
      reinterpret_cast<const void*>(&reduce_kernel<kMemLdsCsr>)};
  for (const void* fn : others) {
    hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize,
                                       static_cast<int>(lds_bytes));
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace vc
