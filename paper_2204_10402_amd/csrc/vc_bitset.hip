// vc_bitset.hip -- the vertex-cover search for graphs of at most 512 vertices, with a search
// node held as a bitset of live vertices (gfx950).
//
// Same method and same rules as the degree-array kernels in vc_device.hip (paper §II-B, §IV):
// the same passes in the same order with the same tie-breaks, the same branching vertex, the
// same child order, the same stack / worklist protocol. Only the representation of an
// intermediate graph differs: instead of a degree array (§IV-B) a node is the set L of live
// vertices (W = ceil(n/64) 64-bit words, held in scalar registers) plus |S|. It is just as
// self-contained, given the read-only adjacency, and W*8 + 8 bytes instead of 4(n+2). A degree
// is recomputed as popcount(adj[v] & L).
//
// One wavefront per node, several to a workgroup (a team, which shares the adjacency matrix and
// hands sub-trees over inside the workgroup; see Team). Lane l holds vertices l, 64+l, ...,
// (W-1)*64+l and their W adjacency words each in vector registers; the whole adjacency matrix also
// sits in LDS for random access (the triangle test). A rule pass is a handful of ballots and bit
// operations; the main loop has no barriers except where a team looks for work.

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "vc_device_common.h"
#include "vc_internal.h"

namespace vc {

template <int W>
struct Rows {  // this lane's vertices (w*64 + lane) and their adjacency words
  uint64_t adj[W][W];
};

template <int W>
struct Live {  // a search node, uniform across the wavefront
  uint64_t bits[W];
  int32_t s;
};

// After a branch that only some lanes take, and before a jump: keeps the lanes' meeting point a
// block of its own. Folded into the jump's target, it makes every value that meets there look
// different from lane to lane to the compiler, the loop's exit included, and the node, the stack
// positions and all masks move from scalar to vector registers.
__device__ __forceinline__ void rejoin() { __builtin_amdgcn_wave_barrier(); }

__device__ __forceinline__ uint64_t ballot(bool b) { return __builtin_amdgcn_ballot_w64(b); }

__device__ __forceinline__ uint64_t uniform64(uint64_t x) {
  const uint32_t lo = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(x));
  const uint32_t hi = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(x >> 32));
  return (static_cast<uint64_t>(hi) << 32) | lo;
}

// Lane mask test: bit `lane` of a wavefront-uniform 64-bit mask, used directly as the lane's
// condition (the mask becomes the lane mask of one v_cndmask; no shift per lane).
__device__ __forceinline__ bool lane_in(uint64_t m) { return __builtin_amdgcn_inverse_ballot_w64(m); }

// Is this lane's vertex of word wv live?
template <int W>
__device__ __forceinline__ bool held_live(const Live<W>& L, int wv) {
  return lane_in(L.bits[wv]);
}

// Bit x of a W-word mask (x < 64 W), without indexing the register array at run time.
template <int W>
__device__ __forceinline__ bool bit_of(const uint64_t (&M)[W], int x) {
  uint64_t word = 0;
#pragma unroll
  for (int w = 0; w < W; ++w) word = (x >> 6) == w ? M[w] : word;
  return (word >> (x & 63)) & 1ull;
}

// Per-lane cached degrees of the held vertices, and per-lane marks of held degree-two vertices
// already known to lie in no triangle (bit wv of no_tri: the lane's vertex of word wv; kept in
// a vector register rather than as W uniform masks, which would add to the scalar registers
// the traversal loop holds). Invariant at every rule pass: for each live held vertex v,
// deg = |N(v) ∩ L| (entries of removed vertices are stale; every use masks them with L). Along
// one root-to-leaf path vertices are only ever removed, so a vertex that still has degree two
// still has the same two neighbours, and if they were not adjacent they still are not: the
// marks stay valid down a path and are cleared whenever the node is replaced by one that is
// not its descendant (a pop, a dequeue, a root).
template <int W>
struct Degrees {
  int32_t deg[W];
  uint32_t no_tri;
};

// All degrees from scratch: deg(v) = popcount(adj(v) & L) over W words.
template <int W>
__device__ __forceinline__ void degrees_full(const Rows<W>& r, const Live<W>& L, Degrees<W>& D) {
#pragma unroll
  for (int wv = 0; wv < W; ++wv) {
    int d = 0;
#pragma unroll
    for (int w = 0; w < W; ++w) d += __popcll(r.adj[wv][w] & L.bits[w]);
    D.deg[wv] = d;
  }
}

// The held vertices adjacent to vertex w*64 + b lose one degree. W is a compile-time word of
// the caller's unrolled loop; b is uniform, so the half select is a scalar condition.
template <int W>
__device__ __forceinline__ void drop_neighbour(const Rows<W>& r, int w, int b, Degrees<W>& D) {
#pragma unroll
  for (int wv = 0; wv < W; ++wv) {
    const uint64_t a = r.adj[wv][w];
    const uint32_t half = (b & 32) ? static_cast<uint32_t>(a >> 32) : static_cast<uint32_t>(a);
    D.deg[wv] -= static_cast<int32_t>(__builtin_amdgcn_ubfe(half, static_cast<uint32_t>(b & 31), 1u));
  }
}

// Remove the set F from the node: |S| grows by the number of live vertices in F (§IV-B, with
// the |S| counter) and the degrees follow, one removed vertex at a time for fewer than W of
// them, from scratch for more.
template <int W>
__device__ __forceinline__ int remove_set(const Rows<W>& r, Live<W>& L, const uint64_t (&F)[W],
                                          Degrees<W>& D) {
  uint64_t R[W];
  int removed = 0;
#pragma unroll
  for (int w = 0; w < W; ++w) {
    R[w] = F[w] & L.bits[w];
    removed += __popcll(R[w]);
    L.bits[w] &= ~R[w];
  }
  L.s += removed;
  // one removed vertex costs 3W VALU and about 7 scalar instructions, a full count 4W^2 VALU
  if (removed >= W) {
    degrees_full(r, L, D);
  } else if (removed > 0) {
#pragma unroll
    for (int w = 0; w < W; ++w) {
      uint64_t m = R[w];
      while (m) {
        const int b = __ffsll(static_cast<long long>(m)) - 1;
        m &= m - 1;
        drop_neighbour(r, w, b, D);
      }
    }
  }
  return removed;
}

// Degree-one rule (§II-B, tie-breaks §IV-D). A live u is removed if it has a degree-one live
// neighbour c and either deg(u) != 1 or u < c (for deg(u) = 1, c is its only neighbour).
// With H the live vertices next to a degree-one vertex: every u in H of degree other than
// one goes; a u in H of degree one forms a mutual pair with its only neighbour, and only the
// smaller of the two goes.
template <int W>
__device__ __forceinline__ int pass_degree_one(const Rows<W>& r, Live<W>& L, Degrees<W>& D) {
  uint64_t D1[W];
  uint64_t any = 0;
#pragma unroll
  for (int w = 0; w < W; ++w) {
    D1[w] = ballot(D.deg[w] == 1) & L.bits[w];
    any |= D1[w];
  }
  if (!any) return 0;
  uint64_t F[W], M[W];
  uint64_t mutual = 0;
#pragma unroll
  for (int wv = 0; wv < W; ++wv) {
    uint32_t near = 0;
#pragma unroll
    for (int w = 0; w < W; ++w) {
      const uint64_t m = r.adj[wv][w] & D1[w];
      near |= static_cast<uint32_t>(m) | static_cast<uint32_t>(m >> 32);
    }
    const uint64_t H = ballot(near != 0) & L.bits[wv];
    F[wv] = H & ~D1[wv];
    M[wv] = H & D1[wv];
    mutual |= M[wv];
  }
  if (mutual) {
    const int lane = lane_id();
#pragma unroll
    for (int wv = 0; wv < W; ++wv) {
      bool bigger = false;
#pragma unroll
      for (int w = 0; w < W; ++w) {
        const uint64_t m = r.adj[wv][w] & D1[w];
        if (w > wv) bigger |= m != 0;
        if (w == wv) bigger |= ((m >> lane) >> 1) != 0;  // a neighbour with a larger id
      }
      F[wv] |= ballot(lane_in(M[wv]) && bigger);
    }
  }
  return remove_set(r, L, F, D);
}

// Lowest set bit of a W-word mask (the mask is not empty): the minimum over its 32-bit halves
// of (first set bit | 32 * half index), where an empty half gives 0xFFFFFFFF.
template <int W>
__device__ __forceinline__ int lowest_bit(const uint64_t (&N)[W]) {
  uint32_t best = 0xFFFFFFFFu;
#pragma unroll
  for (int w = 0; w < W; ++w) {
    const uint32_t lo = static_cast<uint32_t>(N[w]), hi = static_cast<uint32_t>(N[w] >> 32);
    // (the search of an empty half gives all ones, which the or leaves: no test of its own)
    const uint32_t flo = (lo ? static_cast<uint32_t>(__builtin_ctz(lo)) : 0xFFFFFFFFu) | (64u * w);
    const uint32_t fhi = (hi ? static_cast<uint32_t>(__builtin_ctz(hi)) : 0xFFFFFFFFu) | (64u * w + 32u);
    best = min(best, min(flo, fhi));
  }
  return static_cast<int>(best);
}

// Degree-two-triangle rule (§II-B, tie-break §IV-D). A live v of degree two whose neighbours
// a < b are adjacent fires unless a or b is a degree-two vertex with a smaller id; the live
// neighbours of firing vertices (exactly their a and b) are removed. Degree-two vertices not
// yet marked in D.no_tri are checked (row a of the adjacency matrix against {a, b}); the pass ends
// there unless one of them lies in a triangle.
template <int W>
__device__ __forceinline__ int pass_triangle(const Rows<W>& r, Live<W>& L, Degrees<W>& D,
                                             const uint64_t* __restrict__ adj_lds) {
  uint64_t C[W], A[W];
  uint64_t any = 0;
#pragma unroll
  for (int w = 0; w < W; ++w) {
    C[w] = ballot(D.deg[w] == 2 && !((D.no_tri >> w) & 1u)) & L.bits[w];
    any |= C[w];
  }
  if (!any) return 0;
  uint64_t anytri = 0;
#pragma unroll
  for (int wv = 0; wv < W; ++wv) {
    const uint64_t check = C[wv];
    A[wv] = 0;
    if (check) {
      bool adjacent = false;
      if (lane_in(check)) {
        uint64_t N[W];
#pragma unroll
        for (int w = 0; w < W; ++w) N[w] = r.adj[wv][w] & L.bits[w];
        const int a = min(lowest_bit<W>(N), 64 * W - 1);  // N holds exactly two bits
        uint32_t hit = 0;
#pragma unroll
        for (int w = 0; w < W; ++w) {
          const uint64_t x = adj_lds[a * W + w] & N[w];
          hit |= static_cast<uint32_t>(x) | static_cast<uint32_t>(x >> 32);
        }
        adjacent = hit != 0;
      }
      A[wv] = ballot(adjacent) & check;
      if (lane_in(check & ~A[wv])) D.no_tri |= 1u << wv;
      anytri |= A[wv];
    }
  }
  if (!anytri) return 0;
  // A degree-two vertex lies in a triangle: the firing decisions with their tie-breaks.
  uint64_t D2[W];
#pragma unroll
  for (int w = 0; w < W; ++w) D2[w] = ballot(D.deg[w] == 2) & L.bits[w];
  const int lane = lane_id();
  uint64_t Fire[W];
#pragma unroll
  for (int wv = 0; wv < W; ++wv) {
    bool fires = false;
    if (lane_in(A[wv])) {
      const int v = wv * 64 + lane;
      int a = -1, b = -1;
#pragma unroll
      for (int w = 0; w < W; ++w) {
        uint64_t m = r.adj[wv][w] & L.bits[w];
        while (m && b < 0) {
          const int x = w * 64 + (__ffsll(static_cast<long long>(m)) - 1);
          m &= m - 1;
          if (a < 0) a = x; else b = x;
        }
      }
      const bool a2 = bit_of<W>(D2, a);
      const bool b2 = bit_of<W>(D2, b);
      fires = !((a2 && a < v) || (b2 && b < v));
    }
    Fire[wv] = ballot(fires);
  }
  uint64_t F[W];
#pragma unroll
  for (int wu = 0; wu < W; ++wu) {
    bool near = false;
#pragma unroll
    for (int w = 0; w < W; ++w) near |= (r.adj[wu][w] & L.bits[w] & Fire[w]) != 0;
    F[wu] = ballot(near) & L.bits[wu];
  }
  return remove_set(r, L, F, D);
}

// High-degree rule (§II-B): degree above r = bound - |S| (r >= 0 here).
template <int W>
__device__ __forceinline__ int pass_high_degree(const Rows<W>& r, Live<W>& L, Degrees<W>& D,
                                                int32_t rr) {
  uint64_t F[W];
#pragma unroll
  for (int w = 0; w < W; ++w) F[w] = ballot(D.deg[w] > rr) & L.bits[w];
  return remove_set(r, L, F, D);
}

// The rules until the graph stops changing or |S| exceeds bound (same order as the
// degree-array kernels). Callers clamp bound to [-1, n]: a larger bound (PVC with k >= n)
// removes and prunes exactly as n does, since no live degree reaches n - |S|.
template <int W>
__device__ __forceinline__ void reduce_bits(const Rows<W>& r, Live<W>& L, Degrees<W>& D,
                                            const uint64_t* adj_lds, int32_t bound, int rules) {
  // A pass is skipped when nothing has been removed since it last found nothing (its inputs
  // are unchanged), as in the degree-array kernels.
  int changes = 0, quiet1 = -1, quiet2 = -1, quiet3 = -1;
  for (;;) {
    const int32_t s0 = L.s;
    if (s0 > bound) return;
    if ((rules & kRuleDeg1) && quiet1 != changes) {
      if (pass_degree_one(r, L, D)) {
        ++changes;
        if (L.s > bound) return;
      } else {
        quiet1 = changes;
      }
    }
    if ((rules & kRuleTri) && quiet2 != changes) {
      if (pass_triangle(r, L, D, adj_lds)) {
        ++changes;
        if (L.s > bound) return;
      } else {
        quiet2 = changes;
      }
    }
    if ((rules & kRuleHigh) && quiet3 != changes) {
      if (pass_high_degree(r, L, D, bound - L.s)) ++changes;
      else quiet3 = changes;
    }
    if (L.s == s0) return;
  }
}

// Live vertex of maximum degree (smallest id on ties) and that degree, from the cached degrees: one
// 32-bit key (degree << 16 | 0xFFFF - id) per vertex, reduced with DPP.
template <int W>
__device__ __forceinline__ void bits_max_degree(const Live<W>& L, const Degrees<W>& D, int& vmax,
                                                int32_t& dmax) {
  uint32_t key = 0;
  const int lane = lane_id();
#pragma unroll
  for (int wv = 0; wv < W; ++wv) {
    const uint32_t k = (static_cast<uint32_t>(D.deg[wv]) << 16) |
                       (0xFFFFu - static_cast<uint32_t>(wv * 64 + lane));
    key = max(key, held_live(L, wv) ? k : 0u);
  }
  key = wave_max32(key);
  vmax = static_cast<int>(0xFFFFu - (key & 0xFFFFu));
  dmax = static_cast<int32_t>(key >> 16);
}

// The stop test's |E| > limit (§II-B), limit >= 0. The degrees are added up only where the live
// vertices could reach the limit at all, each with the largest degree.
template <int W>
__device__ __forceinline__ bool bits_more_edges(const Live<W>& L, const Degrees<W>& D, int32_t dmax,
                                                int32_t limit) {
  int32_t live = 0;
#pragma unroll
  for (int w = 0; w < W; ++w) live += __popcll(L.bits[w]);
  if (live * dmax <= 2 * limit) return false;
  int32_t sum = 0;
#pragma unroll
  for (int wv = 0; wv < W; ++wv) sum += held_live(L, wv) ? D.deg[wv] : 0;
  return wave_sum(sum) / 2 > limit;
}

// The v_max child: v joins the cover.
template <int W>
__device__ __forceinline__ void remove_vertex_bits(const Rows<W>& r, Live<W>& L, Degrees<W>& D,
                                                   int v) {
  const int wv = v >> 6, b = v & 63;
#pragma unroll
  for (int w = 0; w < W; ++w) {
    if (w == wv) {
      L.bits[w] &= ~(1ull << b);
      drop_neighbour(r, w, b, D);
    }
  }
  L.s += 1;
}

// The N(v) child: every live neighbour of v joins the cover.
template <int W>
__device__ __forceinline__ void remove_neighbourhood_bits(const Rows<W>& r, Live<W>& L,
                                                          Degrees<W>& D, int v,
                                                          const uint64_t* adj_lds) {
  uint64_t F[W];
#pragma unroll
  for (int w = 0; w < W; ++w) F[w] = uniform64(adj_lds[v * W + w]);
  remove_set(r, L, F, D);
}

// A node taken from a stack or the worklist (or a root): its removal of N(pending) goes to
// the live set first, then the degrees are computed once.
template <int W>
__device__ __forceinline__ void enter_node(const Rows<W>& r, Live<W>& L, Degrees<W>& D,
                                           int pending, const uint64_t* adj_lds) {
  if (pending >= 0) {
    int removed = 0;
#pragma unroll
    for (int w = 0; w < W; ++w) {
      const uint64_t f = uniform64(adj_lds[pending * W + w]) & L.bits[w];
      removed += __popcll(f);
      L.bits[w] &= ~f;
    }
    L.s += removed;
  }
  degrees_full(r, L, D);
  D.no_tri = 0;
}


// A stored node: W words of live bits (lo/hi 32-bit halves), |S|, then one word packing the
// pending vertex plus one (10 bits, n <= 512) with the instance (launch-local index below
// 2^22, shifted left 10), padding to a multiple of four words. Lane 0 writes and reads every
// stored node, so a node pushed on the workgroup's stack is read back in program order, and
// the worklist publishes it with one release store.
template <int W>
constexpr int bits_stride() {
  return ((2 * W + 2) + 3) & ~3;
}
constexpr int kPendingBits = 10;

template <int W>
__device__ __forceinline__ void bits_pack(uint32_t (&x)[2 * W + 2], const Live<W>& L, int pending,
                                          int inst) {
#pragma unroll
  for (int w = 0; w < W; ++w) {
    x[2 * w] = static_cast<uint32_t>(L.bits[w]);
    x[2 * w + 1] = static_cast<uint32_t>(L.bits[w] >> 32);
  }
  x[2 * W] = static_cast<uint32_t>(L.s);
  x[2 * W + 1] = static_cast<uint32_t>(pending + 1) | (static_cast<uint32_t>(inst) << kPendingBits);
}

template <int W>
__device__ __forceinline__ void bits_store(int32_t* dst, const Live<W>& L, int pending, int inst) {
  if (lane_id() == 0) {
    uint32_t x[2 * W + 2];
    bits_pack<W>(x, L, pending, inst);
#pragma unroll
    for (int i = 0; i < 2 * W + 2; ++i) dst[i] = static_cast<int32_t>(x[i]);
  }
}

// Node words read by lane 0 into (uniform) L, pending vertex and instance.
template <int W>
__device__ __forceinline__ void bits_unpack(const uint32_t (&x)[2 * W + 2], Live<W>& L,
                                            int& pending, int& inst) {
#pragma unroll
  for (int w = 0; w < W; ++w) {
    const uint32_t lo = __builtin_amdgcn_readfirstlane(x[2 * w]);
    const uint32_t hi = __builtin_amdgcn_readfirstlane(x[2 * w + 1]);
    L.bits[w] = (static_cast<uint64_t>(hi) << 32) | lo;
  }
  L.s = __builtin_amdgcn_readfirstlane(x[2 * W]);
  const uint32_t tag = __builtin_amdgcn_readfirstlane(x[2 * W + 1]);
  pending = static_cast<int>(tag & ((1u << kPendingBits) - 1u)) - 1;
  inst = static_cast<int>(tag >> kPendingBits);
}

template <int W>
__device__ __forceinline__ void bits_load(const int32_t* src, Live<W>& L, int& pending, int& inst) {
  uint32_t x[2 * W + 2];
  if (lane_id() == 0) {
#pragma unroll
    for (int i = 0; i < 2 * W + 2; ++i) x[i] = static_cast<uint32_t>(src[i]);
  }
  bits_unpack<W>(x, L, pending, inst);
}

// The same from an LDS stack entry: every lane reads the same words (an LDS broadcast, no
// exec mask to set up), and the reads are LDS instructions that wait only for LDS.
template <int W>
__device__ __forceinline__ void bits_load_lds(const int32_t* src, Live<W>& L, int& pending,
                                              int& inst) {
  uint32_t x[2 * W + 2];
#pragma unroll
  for (int i = 0; i < 2 * W + 2; ++i) x[i] = static_cast<uint32_t>(src[i]);
  bits_unpack<W>(x, L, pending, inst);
}

// Instance j: its adjacency rows into LDS (all rows) and this lane's rows into registers.
template <int W>
__device__ __forceinline__ int load_adjacency(const Params& p, int j, uint64_t* adj_lds,
                                              Rows<W>& r) {
  const Instance in = p.inst[j];
  const uint64_t* rows = p.bits + static_cast<int64_t>(in.vtx_first) * W;
  __syncthreads();  // the previous instance's rows are no longer read
  for (int i = threadIdx.x; i < in.n * W; i += blockDim.x) adj_lds[i] = rows[i];
#pragma unroll
  for (int wv = 0; wv < W; ++wv) {
    const int v = wv * 64 + lane_id();
#pragma unroll
    for (int w = 0; w < W; ++w) r.adj[wv][w] = v < in.n ? rows[v * W + w] : 0ull;
  }
  __syncthreads();
  return in.n;
}

// The root of an instance with n vertices: every vertex live, |S| = 0.
template <int W>
__device__ __forceinline__ void root_bits(Live<W>& L, int n) {
#pragma unroll
  for (int w = 0; w < W; ++w) {
    const int lo = w * 64, cnt = n - lo;
    L.bits[w] = cnt <= 0 ? 0ull : (cnt >= 64 ? ~0ull : ((1ull << cnt) - 1ull));
  }
  L.s = 0;
}

template <int W>
__device__ __forceinline__ void write_cover(uint8_t* cov, const Live<W>& L, int n) {
#pragma unroll
  for (int wv = 0; wv < W; ++wv) {
    const int v = wv * 64 + lane_id();
    if (v < n) cov[v] = !held_live(L, wv);
  }
}

// ---- worklist protocol -----------------------------------------------------------------------
// One lane runs the whole protocol (reservation, the node copy, the release / acquire of the slot
// ticket), so one agent-scope release store orders the node's words before the ticket and one
// acquire load orders them after it.

// Ring slot `at` entries after `from` in a ring of `cap` (at <= cap).
__device__ __forceinline__ int ring_slot(int from, int at, int cap) {
  const int x = from + at;
  return x >= cap ? x - cap : x;
}

// Word i of stack entry `slot`: from the ring in LDS or in device memory.
template <int W>
__device__ __forceinline__ void bits_copy_entry(int32_t* __restrict__ dst, const int32_t* lstack,
                                                const int32_t* gstack, bool stack_lds, int slot) {
  constexpr int kStride = bits_stride<W>();
  uint32_t x[2 * W + 2];
  if (stack_lds) {
#pragma unroll
    for (int i = 0; i < 2 * W + 2; ++i) x[i] = static_cast<uint32_t>(lstack[slot * kStride + i]);
  } else {
#pragma unroll
    for (int i = 0; i < 2 * W + 2; ++i)
      x[i] = static_cast<uint32_t>(gstack[static_cast<size_t>(slot) * kStride + i]);
  }
#pragma unroll
  for (int i = 0; i < 2 * W + 2; ++i) dst[i] = static_cast<int32_t>(x[i]);
}

// Donate the `m` (at most 64) oldest entries of this wavefront's stack, nodes of instance `inst`,
// to the worklist; false if the worklist is at its threshold. Whole wavefront: lane 0 reserves m
// consecutive tickets with one set of atomics, lane i copies entry i into ticket i's slot.
template <int W>
__device__ __forceinline__ bool bits_enqueue(const Params& p, Ctrl& c, int inst, int m,
                                             const int32_t* lstack, const int32_t* gstack,
                                             bool stack_lds, int bot_slot) {
  const int lane = lane_id();
  uint32_t t_lo = 0, t_hi = 0;
  int ok = 0;
  if (lane == 0) {
    int32_t* count = ctr_i32(p, kQCount);
    if (load_relaxed(count) < static_cast<int32_t>(p.q_threshold)) {
      fetch_add(p.work + inst, m);
      fetch_add(ctr_i32(p, kWork), m);
      fetch_add(count, m);  // stays below cap: threshold + producers * (kDonateMost + 1) <= cap
      const unsigned long long t =
          fetch_add(ctr_u64(p, kQTail), static_cast<unsigned long long>(m));
      t_lo = static_cast<uint32_t>(t);
      t_hi = static_cast<uint32_t>(t >> 32);
      ok = 1;
    }
  }
  if (!__builtin_amdgcn_readfirstlane(ok)) return false;
  const uint64_t t = ((static_cast<uint64_t>(__builtin_amdgcn_readfirstlane(t_hi)) << 32) |
                      static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(t_lo))) + lane;
  if (lane < m) {
    const uint32_t slot = static_cast<uint32_t>(t) & (p.q_cap - 1);
    const uint32_t lap = static_cast<uint32_t>(t / p.q_cap);
    int spins = 0;
    bool lost = false;
    while (load_acquire(p.seq + slot) != 2u * lap) {
      if (search_stopped(p, c)) {  // the launch is ending: the node no longer matters
        lost = true;
        break;
      }
      backoff(spins);
    }
    if (!lost) {
      bits_copy_entry<W>(p.payload + static_cast<size_t>(slot) * p.stride, lstack, gstack,
                         stack_lds, ring_slot(bot_slot, lane, p.depth_cap));
      store_release(p.seq + slot, 2u * lap + 1u);
    }
  }
  rejoin();
  return true;
}

// What the wavefronts of one workgroup (a team) share, in LDS. They all work on one instance, the
// one whose adjacency matrix the workgroup holds, and pass sub-trees to each other through one
// mailbox per wavefront:
//  - a wavefront that has finished its sub-tree lowers `active` and sets its bit of `idle`;
//  - one that has a deferred child and sees an idle bit clears it (the claim), raises `active`,
//    writes the child into that wavefront's box and sets its mail flag.
// `active` counts the sub-trees the team holds, handed-over ones included, so it reaches zero
// only when the team has finished everything it took; thread 0 then looks for more work in the
// worklist. A handover costs a few LDS operations, where a donation through the worklist is a
// chain of six device-scope memory operations (several microseconds, and far more when thousands
// of workgroups contend for its counters).
template <int W>
struct Team {
  int32_t active;
  uint32_t idle;
  uint32_t best;   // MVC: smallest cover size any wavefront of the team has seen
  int32_t status;  // thread 0's look for work: 1 a node in words, 2 the root of `inst`, <= 0 end
  int32_t inst;
  uint32_t nodes;  // nodes not yet reported to the instance, gathered when it is left
  uint32_t words[2 * W + 2];
  int32_t mail[bitset_max_team(W)];
  alignas(16) int32_t box[bitset_max_team(W)][bits_stride<W>()];
};

__device__ __forceinline__ int32_t team_load(int32_t* a) {
  return __hip_atomic_load(a, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP);
}
__device__ __forceinline__ uint32_t team_load(uint32_t* a) {
  return __hip_atomic_load(a, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// This wavefront has no work: wait for a sub-tree from another wavefront of the team. True with
// its box filled, false once the whole team has finished. `held`: it has just finished a sub-tree.
template <int W>
__device__ __forceinline__ bool team_wait(Team<W>& t, int wave, bool held) {
  int got = 0;
  if (lane_id() == 0) {
    const bool last =
        held && __hip_atomic_fetch_add(&t.active, -1, __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_WORKGROUP) == 1;
    if (!last) {
      // (release: the last box's flag is lowered before the bit shows)
      __hip_atomic_fetch_or(&t.idle, 1u << wave, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
      for (;;) {
        // the flag first: `active` stays positive from before the flag is set until the sub-tree
        // in the box is finished, so reading it as zero means that no box is being filled
        if (team_load(&t.mail[wave])) {
          got = 1;
          break;
        }
        if (team_load(&t.active) == 0) break;
        __builtin_amdgcn_s_sleep(2);
      }
      if (got) t.mail[wave] = 0;
    }
  }
  return __builtin_amdgcn_readfirstlane(got);
}

// Hand the oldest entries of this wavefront's stack (`avail` of them) to idle wavefronts of the
// team, one each; returns how many were handed over. Lane i serves wavefront i.
template <int W>
__device__ __forceinline__ int team_give(Team<W>& t, uint32_t idle, int avail,
                                         const int32_t* lstack, const int32_t* gstack,
                                         bool stack_lds, int bot_slot, int cap) {
  const int lane = lane_id();
  const uint32_t bit = lane < 32 ? 1u << lane : 0u;
  bool claim = (idle & bit) && __popc(idle & (bit - 1u)) < avail;
  if (claim)
    // (acquire: the receiver's reads of its box's last content come before the writes below)
    claim = __hip_atomic_fetch_and(&t.idle, ~bit, __ATOMIC_ACQUIRE,
                                   __HIP_MEMORY_SCOPE_WORKGROUP) & bit;
  const uint64_t mask = ballot(claim);
  const int given = __popcll(mask);
  if (given == 0) return 0;
  if (lane == 0)
    __hip_atomic_fetch_add(&t.active, given, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  if (claim) {
    const int e = __popc(static_cast<uint32_t>(mask) & (bit - 1u));
    bits_copy_entry<W>(t.box[lane], lstack, gstack, stack_lds, ring_slot(bot_slot, e, cap));
    __hip_atomic_store(&t.mail[lane], 1, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
  }
  rejoin();
  return given;
}

// Thread 0: take work for the team. Returns 1 with the node's words in `words`, 2 with *root set
// to an unstarted instance (its root), 0 when the launch is over, -1 when it is being stopped.
// Queued nodes go first, then roots in instance order; an idle team looks again with exponential
// back-off.
template <int W>
__device__ __forceinline__ int bits_dequeue(const Params& p, Ctrl& c, bool first,
                                            uint32_t* words, int* root) {
  int status = 3;
  int polls = 0;
  while (status == 3) {
    uint32_t slot = 0, lap = 0;
    status = first ? first_take(p, root)
                   : worklist_take(p, c, (polls & 3) == 0, &slot, &lap, root);
    if (status == 1) {
      int wait = 0;
      while (load_acquire(p.seq + slot) != 2u * lap + 1u) {
        if (search_stopped(p, c)) {
          status = -1;
          break;
        }
        backoff(wait);
      }
      if (status == 1) {
        const int32_t* src = p.payload + static_cast<size_t>(slot) * p.stride;
#pragma unroll
        for (int i = 0; i < 2 * W + 2; ++i) words[i] = static_cast<uint32_t>(src[i]);
        store_release(p.seq + slot, 2u * (lap + 1u));
      }
    } else if (status == 3) {
      idle_sleep(p, polls);
      if (!first) ++polls;
      first = false;
    }
  }
  return status;
}

// ---- kernels -----------------------------------------------------------------------------------

// Greedy approximation (§II-B), as greedy_kernel, on bitset nodes: one workgroup per instance
// (grid-stride loop over the launch's instances).
template <int W>
__global__ void __launch_bounds__(64) bitset_greedy_kernel(Params p) {
  extern __shared__ uint64_t adj_lds[];
  if (blockIdx.x == 0 && threadIdx.x == 0) p.res->t_greedy = realtime();
  for (int j = blockIdx.x; j < p.num_inst; j += gridDim.x) {
    if (__builtin_amdgcn_readfirstlane(load_relaxed(&p.ist[j].err_row)) != kNoRow) continue;
    Rows<W> r;
    const int n = load_adjacency<W>(p, j, adj_lds, r);
    Live<W> L;
    Degrees<W> D;
    root_bits<W>(L, n);
    enter_node<W>(r, L, D, -1, adj_lds);
    const int32_t unbounded = 0x3FFFFFFF;
    for (;;) {
      reduce_bits<W>(r, L, D, adj_lds, unbounded, kRuleDeg1 | kRuleTri);
      int vmax;
      int32_t dmax;
      bits_max_degree<W>(L, D, vmax, dmax);
      if (dmax == 0) break;
      remove_vertex_bits<W>(r, L, D, vmax);
    }
    write_cover<W>(p.covers + p.inst[j].vtx_off, L, n);
    if (threadIdx.x == 0) {
      p.ist[j].best = L.s;
      p.ist[j].greedy = L.s;
    }
  }
}

// Lane 0: claim / publish a cover of size s for instance j (see claim_solution in the
// degree-array kernels; the same protocol).
template <bool PVC>
__device__ __forceinline__ int bits_claim(const Params& p, int j, int32_t s) {
  InstState* is = p.ist + j;
  if (PVC) return (atomicOr(&is->state, kInstFound) & kInstFound) == 0;
  if (atomicMin(&is->best, s) <= s) return 0;
  lock_acquire(&is->lock);
  if (load_relaxed(&is->best) == s) return 1;
  store_release(&is->lock, 0);
  return 0;
}

template <bool PVC>
__device__ __forceinline__ void bits_publish(const Params& p, int j, int32_t s) {
  InstState* is = p.ist + j;
  if (PVC) {
    store_relaxed(&is->best, s);
    fetch_add(ctr_i32(p, kOpen), -1);
  } else {
    store_release(&is->lock, 0);
  }
}

// Lane 0: add `count` nodes to instance j; returns 1 if that used up the instance's budget.
__device__ __forceinline__ int bits_report_nodes(const Params& p, int j, uint32_t count) {
  if (count == 0) return 0;
  unsigned long long* total = reinterpret_cast<unsigned long long*>(&p.ist[j].nodes);
  const unsigned long long before = fetch_add(total, static_cast<unsigned long long>(count));
  if (p.node_budget > 0 && static_cast<int64_t>(before + count) >= p.node_budget) {
    atomicOr(&p.ist[j].state, kInstOutOfBudget);
    return 1;
  }
  return 0;
}

// Without a node budget a wavefront reports its nodes to the instance every kFlushNodes of them, so
// that what all wavefronts of a team have not reported (at most this many each) fits in Team::nodes.
constexpr uint32_t kFlushNodes = 1u << 27;
static_assert(uint64_t{kMaxWaves} * kFlushNodes <= 0xFFFFFFFFu, "a team's unreported nodes wrap");

// Nodes between two reads of the node header (a power of two).
constexpr uint32_t kPollNodes = 16;
// In a team of more than one, nodes a wavefront visits between two donations to the worklist:
// the team's own idle wavefronts are served first (team_give), and a donation costs the donor the
// time of a few nodes. Up to kDonateMost entries go out at once, so that a tree whose side
// branches are small still spreads. Measured (one 5-regular graph of 120 vertices / a G(200, 0.5)
// search of 85,000 nodes), entries x interval: 1 x 8: 5.4 / 5.1 ms, 2 x 8: 4.4 / 3.7,
// 4 x 8: 3.9 / 2.4, 4 x 2: 4.1 / 3.9, 4 x 32: 4.2 / 4.0 (with the node in scalar registers 4 x 8
// takes 3.4 / 1.7). A node of five words or more takes several times as long, so that a donation
// costs less of one and a small tree waits longer for its nodes to spread: every 4 nodes there (PVC
// no, one G(500, 3.1/500) / one G(400, 3.1/400) / eight graphs of 257-512 vertices, average degree
// 2.6: 8 nodes 532 / 280 / 295 us, 4 nodes 384 / 228 / 228, 2 nodes 333 / 199 / 208; but 16 graphs
// G(390, 3.5/390), 750,000 nodes: 1.71, 1.73 and 1.80 ms).
template <int W>
constexpr uint32_t kDonateNodes = W >= 5 ? 4 : 8;

// The hybrid traversal (§IV-A, Fig. 4; termination §IV-C) on bitset nodes, over every instance
// of the launch (as traverse_kernel). Each wavefront of a workgroup walks its own sub-trees with
// its own stack; the wavefronts of a workgroup (a team) share the instance's adjacency matrix and
// pass sub-trees to each other in LDS, and the workgroup as a whole takes nodes and roots from
// the launch's worklist when all of its wavefronts have run out.
// Registers: a lane's adjacency rows take 2 W^2 of them. Up to seven words the kernel is held to two
// wavefronts per SIMD; at seven that spills about 40 registers to scratch, which costs less than half
// the wavefronts do (16 graphs G(390, 3.5/390): 1.76 ms, with one wavefront per SIMD and no spill
// 2.37; planted batch of 40-400 vertices level). Eight words take about 400 registers and one
// wavefront per SIMD.
template <int W, bool PVC, bool PROF, bool SO>
__global__ void __launch_bounds__(64 * bitset_max_team(W), W <= 7 ? 2 : 1)
    bitset_traverse_kernel(Params args) {
  const int rules = args.rules;
  const int32_t threshold = static_cast<int32_t>(args.q_threshold);
  extern __shared__ uint64_t adj_lds[];
  __shared__ Ctrl c;
  __shared__ Team<W> team;
  // 64-bit statistics in LDS: the loop's scalar registers hold only the 32-bit counts since the
  // last flush
  __shared__ WgStats tally;
  const int wg = blockIdx.x;
  const int tid = threadIdx.x;
  const int lane = lane_id();
  const int wave = __builtin_amdgcn_readfirstlane(wave_id());
  const int waves = args.team;
  Rows<W> r;
  ActivityClock<PROF> clk;
  clk.begin();
  if (tid == 0) {
    watch_begin(args, c);
    tally = WgStats{};
    team.nodes = 0;
  }
  if (lane == 0) team.mail[wave] = 0;
  auto add_tally = [](int64_t* dst, int64_t x) {
    __hip_atomic_fetch_add(dst, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  };

  constexpr int kStride = bits_stride<W>();
  // Lane 0 alone writes and reads a wavefront's stack entries, in program order, so the ring
  // needs no barrier in LDS either.
  // The rings live in LDS after the adjacency matrix (stack_lds) or in device memory. The two
  // are addressed through separate pointers, each access under a uniform branch, so that LDS
  // entries are read and written with LDS instructions rather than flat ones (a flat access
  // waits for every outstanding memory operation, the node header's load included).
  const bool stack_lds = args.stack_lds != 0;
  int32_t* const lstack = reinterpret_cast<int32_t*>(adj_lds + static_cast<size_t>(args.n_max) * W) +
                          static_cast<size_t>(wave) * args.depth_cap * kStride;
  const auto gstack = [&]() -> int32_t* {
    const Params& p = cold_params();
    return p.stacks + (static_cast<size_t>(wg) * waves + wave) * p.depth_cap * kStride;
  };
  // The stack is a ring of depth_cap entries holding [bot, top): pops take the top, handovers and
  // donations take the bottom (the oldest deferred child, nearest its sub-tree root). Every entry
  // belongs to the team's instance.
  int top = 0, bot = 0;
  // ring slots of top and bot, kept reduced modulo depth_cap (no division per push or pop)
  int top_slot = 0, bot_slot = 0;
  const int cap = args.depth_cap;
  bool have = false;
  bool held = false;     // this wavefront holds a sub-tree (counted in team.active)
  bool holding = false;  // thread 0: the team holds a sub-tree of the launch (a root, a queued node)
  bool first = true;     // the team has not looked for work yet
  int cur = -1, cur_n = 0;
  int32_t cur_k = 0, cur_vtx = 0;
  // Statistics: nodes and stack traffic are counted in 32 bits since the last flush (instance
  // switch, budget report, or every kFlushNodes nodes) and folded into `tally` there.
  uint32_t unreported = 0, pushes32 = 0, pops32 = 0;  // since the last flush
  const uint32_t flush_at = args.node_budget > 0 ? static_cast<uint32_t>(args.budget_chunk) : kFlushNodes;
  int max_depth = 0;
  uint32_t headers = 0;  // nodes since the last header, and so on (see kPollNodes)
  uint32_t so_path = 0;  // StackOnly: the current path index
  uint32_t quiet = 0;    // nodes since this wavefront's last donation to the worklist
  int32_t seen_best = 0; // MVC: the instance's best as this wavefront last saw it
  bool inst_done = false;  // it is answered (PVC) or out of budget
  int32_t seen_count = 0;  // worklist count at the last header
  int stop = 0;            // the launch is being stopped
  Live<W> L;
  Degrees<W> D;

  for (;;) {
    if (!have) {
      int pending, inst;
      if (top > bot) {
        --top;
        top_slot = top_slot == 0 ? cap - 1 : top_slot - 1;
        if (stack_lds) bits_load_lds<W>(lstack + top_slot * kStride, L, pending, inst);
        else bits_load<W>(gstack() + static_cast<size_t>(top_slot) * kStride, L, pending, inst);
        ++pops32;
        clk.charge(kActAcquire);
      } else if constexpr (SO) {
        // StackOnly (the comparison method of §V-A): no worklist, one wavefront per workgroup.
        // This workgroup's sub-trees are the paths wg, wg + num_wg, ... < 2^start_depth (bit d:
        // which child at depth d); it walks each path down from the root, then walks the sub-tree
        // with its stack. A node above the start depth counts for the instance only on the path
        // whose remaining bits are zero, so the instance's node count is the tree's.
        const Params& p = cold_params();
        if (cur < 0) {
          cur_n = load_adjacency<W>(p, 0, adj_lds, r);
          const Instance in = p.inst[0];
          cur = 0;
          cur_k = min(in.k, cur_n);  // a k beyond n acts as n (see reduce_bits)
          cur_vtx = in.vtx_off;
          seen_best = 0x7FFFFFFF;
          if (tid == 0) {
            ++tally.instances;
            team.best = 0x7FFFFFFF;
          }
          so_path = static_cast<uint32_t>(wg);
        } else {
          so_path += static_cast<uint32_t>(p.num_wg);
        }
        const int rejected =
            __builtin_amdgcn_readfirstlane(load_relaxed(&p.ist[0].err_row) != kNoRow);
        if (so_path >= (1u << p.start_depth) || rejected) {
          clk.charge(kActAcquire);
          break;
        }
        root_bits<W>(L, cur_n);
        enter_node<W>(r, L, D, -1, adj_lds);
        pending = -1;
        bool reached = true;
        for (int d = 0; d < p.start_depth && reached; ++d) {
          const bool owner = (so_path >> d) == 0;
          const uint64_t h = uniform64(inst_header(p, cur));
          const int32_t state = static_cast<int32_t>(h >> 32);
          if ((state & kInstOutOfBudget) || (PVC && (state & kInstFound))) {
            reached = false;
            break;
          }
          if (!PVC) seen_best = min(seen_best, static_cast<int32_t>(h));
          const int32_t bound = PVC ? cur_k : static_cast<int32_t>(h) - 1;
          if (owner) ++unreported;  // counted for the instance (and the workgroup) at the flush
          else if (tid == 0) ++tally.nodes;  // a walk through a node another path owns
          reduce_bits<W>(r, L, D, adj_lds, bound, p.rules);
          const int32_t rr = bound - L.s;
          int vmax = 0;
          int32_t dmax = 0;
          if (rr >= 0) bits_max_degree<W>(L, D, vmax, dmax);
          if (rr < 0 || ((p.rules & kPruneEdges) && (p.rules & kRuleHigh) && rr < cur_n &&
                         bits_more_edges<W>(L, D, dmax, rr * rr))) {
            reached = false;
          } else if (dmax == 0) {  // a cover: recorded once, on the owning path
            if (owner) {
              int won = 0;
              if (tid == 0) won = bits_claim<PVC>(p, cur, L.s);
              if (__builtin_amdgcn_readfirstlane(won)) {
                write_cover<W>(p.covers + cur_vtx, L, cur_n);
                __threadfence();
                if (tid == 0) bits_publish<PVC>(p, cur, L.s);
              }
            }
            reached = false;
          } else if ((so_path >> d) & 1u) {
            remove_neighbourhood_bits<W>(r, L, D, vmax, adj_lds);
          } else {
            remove_vertex_bits<W>(r, L, D, vmax);
          }
        }
        clk.charge(kActAcquire);
        if (!reached) continue;
      } else if (waves > 1 && !first && team_wait<W>(team, wave, held)) {
        // a sub-tree from another wavefront of the team
        held = true;
        bits_load_lds<W>(team.box[wave], L, pending, inst);
        clk.charge(kActAcquire);
      } else {
        // the whole team is out of work: every wavefront of the workgroup comes here
        held = false;
        const Params& p = cold_params();
        __syncthreads();
        if (tid == 0) {
          if (holding) release_work(p, cur);
          uint32_t words[2 * W + 2];
          int root = 0;
          const int got = bits_dequeue<W>(p, c, first, words, &root);
          holding = got > 0;
          team.status = got;
          team.inst = got == 1 ? static_cast<int32_t>(words[2 * W + 1] >> kPendingBits) : root;
          if (got == 1) {
            ++tally.dequeues;
#pragma unroll
            for (int i = 0; i < 2 * W + 2; ++i) team.words[i] = words[i];
          }
          team.active = 1;
          team.idle = 0;
        }
        __syncthreads();
        first = false;
        const int got = __builtin_amdgcn_readfirstlane(team.status);
        inst = __builtin_amdgcn_readfirstlane(team.inst);
        clk.charge(kActAcquire);
        if (got != 1 && got != 2) break;
        if (inst < 0 || inst >= p.num_inst) {  // cannot happen: every stored node names its instance
          if (tid == 0) {
            atomicMax(ctr_i32(p, kError), 2);
            store_relaxed(ctr_i32(p, kAbort), 1);
          }
          rejoin();
          break;
        }
        // a root's input check and the instance's header are loaded now, while the instance is
        // being staged
        const int32_t err_row = got == 2 ? load_relaxed(&p.ist[inst].err_row) : kNoRow;
        const uint64_t hraw = inst_header(p, inst);
        if (inst != cur) {
          if (lane == 0) {
            if (unreported) {
              __hip_atomic_fetch_add(&team.nodes, unreported, __ATOMIC_RELAXED,
                                     __HIP_MEMORY_SCOPE_WORKGROUP);
              add_tally(&tally.nodes, unreported);
              add_tally(&tally.pushes, pushes32);
              add_tally(&tally.pops, pops32);
            }
          }
          unreported = pushes32 = pops32 = 0;
          const int left = cur;
          cur_n = load_adjacency<W>(p, inst, adj_lds, r);  // begins and ends with a barrier
          if (tid == 0) {
            if (left >= 0) bits_report_nodes(p, left, team.nodes);
            team.nodes = 0;
            ++tally.instances;
          }
          const Instance in = p.inst[inst];
          cur = inst;
          cur_k = min(in.k, cur_n);  // a k beyond n acts as n (see reduce_bits)
          cur_vtx = in.vtx_off;
          seen_best = 0x7FFFFFFF;
          inst_done = false;
          if (!PVC) {
            if (tid == 0) team.best = 0x7FFFFFFF;
            __syncthreads();
          }
        }
        const uint64_t h = uniform64(hraw);
        const int32_t state = static_cast<int32_t>(h >> 32);
        if ((state & kInstOutOfBudget) || (PVC && (state & kInstFound))) inst_done = true;
        if (!PVC) seen_best = min(seen_best, static_cast<int32_t>(static_cast<uint32_t>(h)));
        headers = 1;
        if (wave != 0) {  // the other wavefronts wait for sub-trees of this one
          clk.charge(kActOther);
          continue;
        }
        held = true;
        if (got == 2) {
          const int rejected = __builtin_amdgcn_readfirstlane(err_row != kNoRow);
          if (rejected) {  // rejected input: no search (PVC: the instance is settled)
            if (PVC && tid == 0) fetch_add(ctr_i32(p, kOpen), -1);
            rejoin();
            continue;
          }
          root_bits<W>(L, cur_n);
          pending = -1;
        } else {
          uint32_t words[2 * W + 2];
#pragma unroll
          for (int i = 0; i < 2 * W + 2; ++i) words[i] = team.words[i];
          bits_unpack<W>(words, L, pending, inst);
        }
        clk.charge(kActOther);
      }
      enter_node<W>(r, L, D, pending, adj_lds);
      clk.charge(kActBranch);
      have = true;
    }

    // Node header, read every kPollNodes nodes (and when the team takes work): the instance's
    // flags and current best (one load), the worklist count for the donation test, and the
    // launch-wide stop. These are agent-scope loads of lines every workgroup reads, so they are
    // kept off most nodes: a stale best is only a weaker bound (MVC), a stale count only a stale
    // filter (the reservation re-reads it), and a wavefront that answers its instance or exhausts
    // its budget knows it at once (inst_done). The loads are issued here and waited for after the
    // reduction, which runs meanwhile with the bound known before them: k (PVC), or the best the
    // team saw last, lowered by the covers it found since (MVC); it then continues under the
    // fresh best. With one wavefront in the grid the two bounds always agree.
    const bool poll = (headers++ & (kPollNodes - 1)) == 0;
    uint64_t hraw = 0;
    int32_t qraw = 0, abort_raw = 0, open_raw = 1;
    if (poll) {
      const Params& p = cold_params();
      hraw = inst_header(p, cur);
      if (p.q_threshold > 0) qraw = load_relaxed(ctr_i32(p, kQCount));
      abort_raw = load_relaxed(ctr_i32(p, kAbort));
      if (PVC) open_raw = load_relaxed(ctr_i32(p, kOpen));
      if (lane == 0 && watchdog(p, c)) abort_raw = 1;
    }
    // the team's idle wavefronts and its best, read from LDS while the reduction runs
    uint32_t idle_raw = 0;
    if (waves > 1) {
      idle_raw = team_load(&team.idle);
      if (!PVC)
        seen_best = min(seen_best, __builtin_amdgcn_readfirstlane(
                                       static_cast<int>(team_load(&team.best))));
    }
    int32_t bound = PVC ? cur_k : seen_best - 1;
    for (bool looked = !poll;;) {
      reduce_bits<W>(r, L, D, adj_lds, bound, rules);
      if (!looked) {
        looked = true;
        const uint64_t h = uniform64(hraw);
        const int32_t state = static_cast<int32_t>(h >> 32);
        if ((state & kInstOutOfBudget) || (PVC && (state & kInstFound))) inst_done = true;
        if (!PVC) seen_best = min(seen_best, static_cast<int32_t>(static_cast<uint32_t>(h)));
        seen_count = __builtin_amdgcn_readfirstlane(qraw);
        stop |= __builtin_amdgcn_readfirstlane((abort_raw != 0 || open_raw == 0) ? 1 : 0);
        if (!PVC && seen_best - 1 < bound) {  // continue under the fresh best
          bound = seen_best - 1;
          continue;
        }
      }
      break;
    }
    clk.charge(kActReduce);
    if (stop | static_cast<int>(inst_done)) {
      // stopped, answered or out of budget: drop this node and the rest of the sub-tree (a
      // stopped team ends in its next look for work, once all of its wavefronts have dropped
      // theirs)
      if constexpr (SO) {
        if (stop) break;
      }
      have = false;
      top = bot;
      top_slot = bot_slot;
      continue;
    }

    if (++unreported >= flush_at) {
      int spent = 0;
      if (lane == 0) {
        const Params& p = cold_params();
        spent = bits_report_nodes(p, cur, unreported);
        add_tally(&tally.nodes, unreported);
        add_tally(&tally.pushes, pushes32);
        add_tally(&tally.pops, pops32);
      }
      unreported = pushes32 = pops32 = 0;
      if (__builtin_amdgcn_readfirstlane(spent)) inst_done = true;
    }

    const int32_t rr = bound - L.s;
    if (rr < 0) {
      have = false;
      continue;
    }
    int vmax;
    int32_t dmax;
    bits_max_degree<W>(L, D, vmax, dmax);
    clk.charge(kActBranch);
    // (rr >= n - |S| leaves no room for the prune: |E| < (n - |S|)^2 / 2)
    if ((rules & kPruneEdges) && (rules & kRuleHigh) && rr < cur_n &&
        bits_more_edges<W>(L, D, dmax, rr * rr)) {
      have = false;
      continue;
    }
    if (dmax == 0) {  // a vertex cover of size |S|
      if (!PVC && L.s < seen_best) {
        seen_best = L.s;
        if (lane == 0)
          __hip_atomic_fetch_min(&team.best, static_cast<uint32_t>(L.s), __ATOMIC_RELAXED,
                                 __HIP_MEMORY_SCOPE_WORKGROUP);
        rejoin();
      }
      const Params& p = cold_params();
      int won = 0;
      if (lane == 0) won = bits_claim<PVC>(p, cur, L.s);
      if (__builtin_amdgcn_readfirstlane(won)) {
        write_cover<W>(p.covers + cur_vtx, L, cur_n);
        __threadfence();
        if (lane == 0) bits_publish<PVC>(p, cur, L.s);
        rejoin();
      }
      // PVC: a cover of size <= k is recorded now, by this wavefront or another one
      if (PVC) inst_done = true;
      clk.charge(kActOther);
      have = false;
      continue;
    }

    // branch on v_max: defer the N(v_max) child on this wavefront's stack, continue with the v_max
    // child. Idle wavefronts of the team take the oldest entries of the stack (the largest
    // sub-trees it holds) first; else, while the worklist is below its threshold, some are donated.
    // A ring that is full (only one of the caller's size: the depth bound of §IV-E holds else) makes
    // room that way before the child is deferred.
    const bool full = top - bot >= cap;
    const auto defer = [&]() {
      if (stack_lds) bits_store<W>(lstack + top_slot * kStride, L, vmax, cur);
      else bits_store<W>(gstack() + static_cast<size_t>(top_slot) * kStride, L, vmax, cur);
      ++top;
      top_slot = top_slot + 1 == cap ? 0 : top_slot + 1;
    };
    if (!full) defer();
    int given = 0;
    const uint32_t idle = waves > 1 ? __builtin_amdgcn_readfirstlane(idle_raw) : 0u;
    ++quiet;
    if (idle) {
      if (!stack_lds) __threadfence_block();  // lane 0's entry, about to be read by other lanes
      given = team_give<W>(team, idle, top - bot, lstack, stack_lds ? nullptr : gstack(), stack_lds,
                           bot_slot, cap);
    }
    if (given == 0 && seen_count < threshold &&
        (full || (!idle && (waves == 1 || (top - bot > 1 && quiet >= kDonateNodes<W>))))) {
      const int m = min(kDonateMost, (top - bot + 1) / 2);
      if (!stack_lds) __threadfence_block();
      const Params& p = cold_params();
      if (bits_enqueue<W>(p, c, cur, m, lstack, stack_lds ? nullptr : gstack(), stack_lds, bot_slot)) {
        given = m;
        if (lane == 0) add_tally(&tally.enqueues, m);
        rejoin();
      }
      quiet = 0;
    }
    bot += given;
    bot_slot = ring_slot(bot_slot, given, cap);
    if (full) {
      if (given == 0) {  // no room: the stack overflows
        if (lane == 0) {
          const Params& p = cold_params();
          atomicMax(ctr_i32(p, kError), 1);
          store_relaxed(ctr_i32(p, kAbort), 1);
        }
        rejoin();
        if constexpr (SO) break;
        stop = 1;
        have = false;
        top = bot;
        top_slot = bot_slot;
        continue;
      }
      defer();
    }
    if (given == 0 || top > bot) ++pushes32;
    if (top - bot > max_depth) max_depth = top - bot;
    clk.charge(kActDonate);
    remove_vertex_bits<W>(r, L, D, vmax);
    clk.charge(kActBranch);
  }
  clk.end();

  if (lane == 0) {
    __hip_atomic_fetch_add(&team.nodes, unreported, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    add_tally(&tally.nodes, unreported);
    add_tally(&tally.pushes, pushes32);
    add_tally(&tally.pops, pops32);
    __hip_atomic_fetch_max(&tally.max_depth, max_depth, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_WORKGROUP);
    if (PROF)
      for (int a = 0; a < kNumActivities; ++a)
        add_tally(&tally.cycles[a], static_cast<int64_t>(clk.cycles[a]));
  }
  __syncthreads();
  if (tid == 0) {
    const Params& p = cold_params();
    if (cur >= 0) bits_report_nodes(p, cur, team.nodes);
    publish_wg_stats(p, wg, tally);
  }
}

// The reduction rules of one node on a degree array in device memory (-1 = in the cover),
// instance 0 of the launch.
template <int W>
__global__ void __launch_bounds__(64) bitset_reduce_kernel(Params p, int32_t* deg, int32_t* s,
                                                           int64_t bound) {
  extern __shared__ uint64_t adj_lds[];
  if (__builtin_amdgcn_readfirstlane(load_relaxed(&p.ist[0].err_row)) != kNoRow) return;
  Rows<W> r;
  const int n = load_adjacency<W>(p, 0, adj_lds, r);
  Live<W> L;
#pragma unroll
  for (int w = 0; w < W; ++w) {
    const int v = w * 64 + lane_id();
    L.bits[w] = ballot(v < n && deg[v] >= 0);
  }
  L.s = __builtin_amdgcn_readfirstlane(*s);
  Degrees<W> D;
  enter_node<W>(r, L, D, -1, adj_lds);
  // a bound beyond n removes and prunes exactly as n does (see reduce_bits)
  const int32_t b32 = bound < -1 ? -1 : (bound > n ? n : static_cast<int32_t>(bound));
  reduce_bits<W>(r, L, D, adj_lds, b32, p.rules);
#pragma unroll
  for (int w = 0; w < W; ++w) {
    const int v = w * 64 + lane_id();
    if (v < n) deg[v] = held_live(L, w) ? D.deg[w] : -1;
  }
  if (threadIdx.x == 0) *s = L.s;
}

// ---- launchers ---------------------------------------------------------------------------------

template <int W, bool SO>
static const void* bitset_traverse_fn(bool pvc, bool prof) {
  if (pvc) return prof ? reinterpret_cast<const void*>(&bitset_traverse_kernel<W, true, true, SO>)
                       : reinterpret_cast<const void*>(&bitset_traverse_kernel<W, true, false, SO>);
  return prof ? reinterpret_cast<const void*>(&bitset_traverse_kernel<W, false, true, SO>)
              : reinterpret_cast<const void*>(&bitset_traverse_kernel<W, false, false, SO>);
}

// The StackOnly walk-down is a separate instantiation, so the hybrid kernels carry none of its
// registers.
static const void* bitset_fn(int words, bool pvc, bool prof, bool stack_only = false) {
#define VC_BITSET_CASE(WW) \
  case WW: return stack_only ? bitset_traverse_fn<WW, true>(pvc, prof) : bitset_traverse_fn<WW, false>(pvc, prof);
  switch (words) {
    VC_BITSET_CASE(1)
    VC_BITSET_CASE(2)
    VC_BITSET_CASE(3)
    VC_BITSET_CASE(4)
    VC_BITSET_CASE(5)
    VC_BITSET_CASE(6)
    VC_BITSET_CASE(7)
    default: return stack_only ? bitset_traverse_fn<8, true>(pvc, prof) : bitset_traverse_fn<8, false>(pvc, prof);
  }
#undef VC_BITSET_CASE
}

size_t bitset_lds_bytes(int n_max, int words) { return static_cast<size_t>(n_max) * words * 8; }

int bitset_stride(int words) { return ((2 * words + 2) + 3) & ~3; }

size_t bitset_traverse_lds_bytes(const Params& p) {
  const size_t stack = p.stack_lds
      ? static_cast<size_t>(p.team) * p.depth_cap * bitset_stride(p.words) * 4 : 0;
  return bitset_lds_bytes(p.n_max, p.words) + stack;
}

hipError_t launch_bitset_greedy(const Params& p, hipStream_t stream) {
  const size_t lds = bitset_lds_bytes(p.n_max, p.words);
  const dim3 grid(p.num_inst < 65535 ? p.num_inst : 65535);
  switch (p.words) {
    case 1: hipLaunchKernelGGL(bitset_greedy_kernel<1>, grid, dim3(64), lds, stream, p); break;
    case 2: hipLaunchKernelGGL(bitset_greedy_kernel<2>, grid, dim3(64), lds, stream, p); break;
    case 3: hipLaunchKernelGGL(bitset_greedy_kernel<3>, grid, dim3(64), lds, stream, p); break;
    case 4: hipLaunchKernelGGL(bitset_greedy_kernel<4>, grid, dim3(64), lds, stream, p); break;
    case 5: hipLaunchKernelGGL(bitset_greedy_kernel<5>, grid, dim3(64), lds, stream, p); break;
    case 6: hipLaunchKernelGGL(bitset_greedy_kernel<6>, grid, dim3(64), lds, stream, p); break;
    case 7: hipLaunchKernelGGL(bitset_greedy_kernel<7>, grid, dim3(64), lds, stream, p); break;
    default: hipLaunchKernelGGL(bitset_greedy_kernel<8>, grid, dim3(64), lds, stream, p); break;
  }
  return hipGetLastError();
}

hipError_t launch_bitset_traverse(bool pvc, bool prof, const Params& p, hipStream_t stream) {
  Params args = p;
  void* kargs[] = {&args};
  // plain launch; see launch_traverse for why co-residency is not required
  return hipLaunchKernel(bitset_fn(p.words, pvc, prof, p.start_depth > 0), dim3(p.num_wg),
                         dim3(64 * p.team), kargs, bitset_traverse_lds_bytes(p), stream);
}

hipError_t launch_bitset_reduce(const Params& p, int32_t* deg, int32_t* s, int64_t bound,
                                hipStream_t stream) {
  const size_t lds = bitset_lds_bytes(p.n_max, p.words);
  switch (p.words) {
    case 1: hipLaunchKernelGGL(bitset_reduce_kernel<1>, dim3(1), dim3(64), lds, stream, p, deg, s, bound); break;
    case 2: hipLaunchKernelGGL(bitset_reduce_kernel<2>, dim3(1), dim3(64), lds, stream, p, deg, s, bound); break;
    case 3: hipLaunchKernelGGL(bitset_reduce_kernel<3>, dim3(1), dim3(64), lds, stream, p, deg, s, bound); break;
    case 4: hipLaunchKernelGGL(bitset_reduce_kernel<4>, dim3(1), dim3(64), lds, stream, p, deg, s, bound); break;
    case 5: hipLaunchKernelGGL(bitset_reduce_kernel<5>, dim3(1), dim3(64), lds, stream, p, deg, s, bound); break;
    case 6: hipLaunchKernelGGL(bitset_reduce_kernel<6>, dim3(1), dim3(64), lds, stream, p, deg, s, bound); break;
    case 7: hipLaunchKernelGGL(bitset_reduce_kernel<7>, dim3(1), dim3(64), lds, stream, p, deg, s, bound); break;
    default: hipLaunchKernelGGL(bitset_reduce_kernel<8>, dim3(1), dim3(64), lds, stream, p, deg, s, bound); break;
  }
  return hipGetLastError();
}

hipError_t bitset_lds_limit(int words, bool pvc, bool prof, bool stack_only, size_t lds) {
  return hipFuncSetAttribute(bitset_fn(words, pvc, prof, stack_only),
                             hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds));
}

hipError_t bitset_occupancy(int words, bool pvc, bool prof, int team, size_t lds,
                            int* blocks_per_cu) {
  return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks_per_cu, bitset_fn(words, pvc, prof),
                                                      64 * team, lds);
}

}  // namespace vc
