// Bridges by the Tarjan-Vishkin method (Section 4.1) on a symmetric CSR.
//
//  1. Spanning forest (the paper uses the connectivity code of Jaiganesh and
//     Burtscher, which yields a spanning tree as a by-product): union-find
//     hooking where a successful compare-and-swap of a root joins two
//     different trees, so its edge is a forest edge. A root is hooked at most
//     once, so the hooked root's id numbers the edge: half-edges 2e and 2e+1
//     are its two directions, twins by numbering. Parallel copies of an edge
//     are never forest edges and self-loops are skipped. Every vertex is
//     linked along its first edge and hooks its second; then the most
//     frequent root of a sample names the big component, and only rows of
//     vertices outside it hook all their edges (an edge inside the big
//     component joins nothing new).
//  2. Euler tour of the forest as the paper's DCEL (Section 2.1): succ(h) =
//     next(twin(h)), next() cyclic over the half-edges that leave a vertex.
//     Any cyclic order gives a tour and the bridges do not depend on it, so
//     the half-edges of a vertex are kept as a linked list in the order they
//     were found instead of being sorted. The tours of all components are
//     chained into one list.
//  3. One list ranking; a half-edge goes down iff it precedes its twin
//     (Section 2), which gives every vertex its parent edge and subtree
//     size. The preorder comes from an array scan over tour order of
//     (down + starts-a-component) weights (Section 2.2).
//  4. For every vertex the minimum and maximum preorder over itself and its
//     neighbours other than along its parent edge (the paper's segreduce
//     leaves out all forest edges; a child's preorder lies inside the subtree
//     interval of every vertex it could count for, so it changes no test);
//     stored by preorder.
//  5. low(v) / high(v) = range minimum / maximum of those over v's subtree
//     interval, with a sparse table over 32-element blocks and per-position
//     suffix-extreme bitmasks inside a block (the paper uses a segment tree).
//  6. The forest edge above v is a bridge iff low(v) and high(v) both lie
//     inside [pre(v), pre(v) + size(v)) (Tarjan 1974; including pre(v)
//     itself makes the test two equalities). Both slots get their bit.
#include "et_internal.hpp"

namespace et {
namespace {

constexpr int kB = 256;
constexpr int kRowsPerBlock = 256;
constexpr int32_t kTinySlots = 1 << 13;         // slots up to which a sparse graph hooks all its edges at once
constexpr int32_t kLabelNodes = (1 << 20) + 1;  // vertices from which k_hook_rest gathers labels
constexpr int kMaxGrid = 1 << 20;  // workgroups of a grid-stride launch (a dispatch holds < 2^32 work-items)

__global__ void k_fill_i32(int32_t* __restrict__ p, int64_t n, int32_t v) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    p[i] = v;
}

__device__ __forceinline__ void st(int32_t* p, int32_t v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// scalars of a forest
enum {
  FS_BIG = 0,    // the big component's root, -1 if none is named
  FS_HEAD = 1,   // first half-edge of the chained tour, -1 if there is none
  FS_LEN = 2,    // forest half-edges
  FS_ROOTS = 3,  // components with an edge
  FS_LABELS = 4,  // the vertices have labels
};

// Union-find over cc[]: roots satisfy cc[r] == r. A link always hangs the
// root with the larger key under the node with the smaller key, where the
// key is the vertex id except that the designated big component's root (if
// any) counts as smallest; keys therefore strictly decrease towards the
// root, so the forest stays acyclic under concurrent links, and every
// successful compare-and-swap joins two different trees: its edge is a
// spanning-forest edge.
//
// Loads are ordinary cached loads, which may return an out-of-date parent
// (each XCD has its own L2); an out-of-date parent is still an ancestor.
// Only the device-scope compare-and-swap decides a link, and when it fails
// it returns the node's current parent, from which the link continues.
__device__ __forceinline__ int32_t ldc(const int32_t* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
__device__ __forceinline__ void stc(int32_t* p, int32_t v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// an ancestor-or-self of x that looked like a root; halves the path on the way
__device__ int32_t cc_find(int32_t* cc, int32_t x) {
  int32_t cur = x;
  for (;;) {
    const int32_t p = ldc(cc + cur);
    if (p == cur) return cur;
    const int32_t gp = ldc(cc + p);
    if (gp != p) stc(cc + cur, gp);
    cur = gp;
  }
}

__device__ __forceinline__ int64_t cc_key(int32_t v, int32_t big) { return v == big ? -1 : (int64_t)v; }

// Climbing link of the trees of u and w: keep one ancestor of each, and at
// every step try to hang the one with the larger key (if it is a root)
// under the other, else move it up to its grandparent and the other one up
// to its parent. A node of one tree is never hung under a node of the same
// tree: the larger key of two such nodes is never that tree's root. Every
// step moves the larger-key side strictly up, so the loop ends.
// Returns the root this call hung under another tree (the id of the forest
// edge {u, w}), or -1 if it linked nothing.
__device__ int32_t cc_hook(int32_t* cc, int32_t u, int32_t w, int32_t big, bool* over) {
  int32_t p1 = ldc(cc + u), p2 = ldc(cc + w);
  for (int it = 0; it < (1 << 22); ++it) {
    if (p1 == p2) return -1;
    const bool up1 = cc_key(p1, big) > cc_key(p2, big);
    const int32_t hi = up1 ? p1 : p2, lo = up1 ? p2 : p1;
    int32_t ph = ldc(cc + hi);
    if (ph == lo) return -1;
    if (ph == hi) {
      const int32_t old = atomicCAS(cc + hi, hi, lo);
      if (old == hi) return hi;
      ph = old;  // linked meanwhile: continue from its current parent
    }
    p1 = ldc(cc + ph);
    p2 = ldc(cc + lo);
  }
  *over = true;
  return -1;
}

// slot of the twin of (u, w): the first (w, u) slot of row w (-1, flagged, if
// there is none)
__device__ int32_t twin_slot(const int32_t* __restrict__ row_ptr, const int32_t* __restrict__ col, int32_t nnz,
                             int32_t u, int32_t w, bool* bad) {
  const int32_t wbeg = min(max(row_ptr[w], 0), nnz);
  const int32_t wend = min(max(row_ptr[w + 1], wbeg), nnz);
  int32_t lo = wbeg, hi = wend;
  while (lo < hi) {
    const int32_t mid = lo + ((hi - lo) >> 1);
    if (col[mid] < u) lo = mid + 1;
    else hi = mid;
  }
  if (lo < wend && col[lo] == u) return lo;
  *bad = true;
  return -1;
}

__device__ __forceinline__ int32_t clampi(int32_t x, int32_t lo, int32_t hi) { return min(max(x, lo), hi); }

// Start of a forest, and its first round of links, one for the first neighbour
// of every vertex. A vertex whose first neighbour w has a smaller id hangs
// below it. A local minimum v hangs below the first neighbour x of its first
// neighbour w, if x < v: w hangs below x by its own link, so the edge {v, w}
// joins v's tree to that one (and if x is v, w hangs below v). Every vertex
// decides for itself and ids strictly decrease upwards, so all these links are
// edges of one forest and need no compare-and-swap (a device-scope one per
// vertex, at 24 G/s, and its dependent climb made this round 316 us at 2^22
// vertices and 2^25 edges; with plain stores it takes 86 us). The trees are
// chains as long as the graph where ids follow its shape, which a later link
// would climb step by step: a full compression comes before any. row_ptr must
// be monotone from 0 to nnz, anything else is flagged.
// EDGES: keep the forest: a linked edge's record {u, w, slot (u, w), -} and
// its half-edge out of u as u's list so far. Also clears the forest's scalars
// and, where given, the mask and the bridge count.
template <bool EDGES>
__global__ void k_forest_init(const int32_t* __restrict__ row_ptr, const int32_t* __restrict__ col, int32_t n,
                              int32_t nnz, int32_t* __restrict__ cc, int4* __restrict__ erec,
                              int32_t* __restrict__ first, int32_t* __restrict__ next, int32_t* __restrict__ sc,
                              uint32_t* __restrict__ mask, int32_t words, int64_t* __restrict__ count,
                              uint32_t* __restrict__ status) {
  const int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (mask)
    for (int64_t i = v; i < words; i += (int64_t)gridDim.x * blockDim.x) mask[i] = 0u;
  if (v == 0) {
    sc[FS_BIG] = -1;
    sc[FS_HEAD] = -1;
    sc[FS_LEN] = 0;
    sc[FS_ROOTS] = 0;
    sc[FS_LABELS] = 0;
    if (count) *count = 0;
  }
  if (v >= n) return;
  const int32_t a0 = row_ptr[v], b0 = row_ptr[v + 1];
  bool bad = a0 > b0 || a0 < 0 || b0 > nnz;
  if (v == 0 && a0 != 0) bad = true;
  if (v == n - 1 && b0 != nnz) bad = true;
  const int32_t a = clampi(a0, 0, nnz), b = clampi(b0, a, nnz);
  int32_t k = a, w = (int32_t)v, up = (int32_t)v;
  while (k < b && (w = col[k]) == (int32_t)v) ++k;  // self-loops
  // rows are sorted: no later slot has a smaller neighbour
  if (k < b) {
    if ((uint32_t)w >= (uint32_t)n) {
      bad = true;
    } else if (w < (int32_t)v) {
      up = w;
    } else {
      const int32_t wa = clampi(row_ptr[w], 0, nnz), wb = clampi(row_ptr[w + 1], wa, nnz);
      const int32_t x = wa < wb ? col[wa] : (int32_t)v;
      if (x >= 0 && x < (int32_t)v) up = x;
    }
  }
  const bool link = up != (int32_t)v;
  cc[v] = up;
  if (EDGES) {
    first[v] = link ? (int32_t)(2 * v) : -1;
    if (link) {
      erec[v] = make_int4((int32_t)v, w, k, -1);
      next[2 * v] = -1;
    }
  }
  if (bad) flag(status, ST_BAD_CSR);
}

// rows [b*256, b*256+256) of the CSR; lane-strided over their slots
__device__ __forceinline__ int row_of(const int32_t* rp_lds, int cnt, int32_t k) {
  int lo = 0, hi = cnt;  // largest i in [0, cnt) with rp[i] <= k
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (rp_lds[mid] <= k) lo = mid;
    else hi = mid;
  }
  return lo;
}

// Second round: every vertex hooks its second distinct neighbour. Both rounds
// end with a full path compression.
// EDGES: only the lane of u touches u's list here, so the insertion of the
// half-edge out of u needs no atomics; those out of the other ends follow in
// k_link_in.
template <bool EDGES>
__global__ void k_hook_sample(const int32_t* __restrict__ row_ptr, const int32_t* __restrict__ col, int32_t n,
                              int32_t nnz, int32_t* cc, int4* __restrict__ erec, int32_t* __restrict__ first,
                              int32_t* __restrict__ next, uint32_t* __restrict__ status) {
  const int64_t u = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (u >= n) return;
  const int32_t a = clampi(row_ptr[u], 0, nnz), b = clampi(row_ptr[u + 1], a, nnz);
  bool bad = false, over = false;
  int taken = 0;
  for (int32_t k = a; k < b && taken < 2; ++k) {
    const int32_t w = col[k];
    if ((uint32_t)w >= (uint32_t)n) {
      bad = true;
      continue;
    }
    if (w == u || (k > a && col[k - 1] == w)) continue;  // self-loop or a parallel copy
    if (taken++ == 0) continue;                          // the first round's
    const int32_t e = cc_hook(cc, (int32_t)u, w, -1, &over);
    if (EDGES && e >= 0) {
      erec[e] = make_int4((int32_t)u, w, k, -1);
      next[2 * e] = first[u];
      first[u] = 2 * e;
    }
  }
  if (bad) flag(status, ST_BAD_CSR);
  if (over) flag(status, ST_OVERFLOW);
}

// The big component: the most frequent root among 1024 sampled vertices.
// With a table (where labels follow, below) also the roots that the most
// samples have, ascending: their places are the labels. A root that has `least`
// samples is in, the smallest number for which they fit.
constexpr int kBigSample = 1024;
constexpr int kLabelMax = 255;                             // labels; also "none of them"
constexpr int kLabelRuns = kBigSample / (kLabelMax + 1);  // so many samples and they fit, but for one

__global__ __launch_bounds__(kBigSample) void k_big_component(const int32_t* __restrict__ cc, int32_t n, int32_t* __restrict__ sc,
                                                             int32_t* __restrict__ table) {
  __shared__ int32_t r[kBigSample];
  __shared__ int32_t best, best_count, in, all[kLabelRuns], wsum[kLabelRuns][kBigSample / 64];
  const int t = threadIdx.x;
  const uint32_t v = mix32(0x2545f491u + (uint32_t)t) % (uint32_t)n;
  r[t] = cc[v];
  if (t == 0) {
    best = INT32_MAX;
    best_count = 0;
    in = 0;
    for (int l = 0; l < kLabelRuns; ++l) all[l] = 0;
  }
  __syncthreads();
  for (int k = 2; k <= kBigSample; k <<= 1) {  // bitonic sort
    for (int j = k >> 1; j > 0; j >>= 1) {
      const int o = t ^ j;
      if (o > t) {
        const bool up = (t & k) == 0;
        const int32_t x = r[t], y = r[o];
        if ((x > y) == up) {
          r[t] = y;
          r[o] = x;
        }
      }
      __syncthreads();
    }
  }
  // the longest run of equal roots wins (smallest root on a tie)
  int len = 0;
  if (t == 0 || r[t - 1] != r[t]) {
    // the run's end by a binary search in the sorted samples (walking it
    // took one LDS read per member: ~1000 in a row when one component
    // holds nearly every sample)
    const int32_t x = r[t];
    int lo = t + 1, hi = kBigSample;
    while (lo < hi) {
      const int mid = (lo + hi) >> 1;
      if (r[mid] == x) lo = mid + 1;
      else hi = mid;
    }
    len = lo - t;
    atomicMax(&best_count, len);
  }
#pragma unroll
  for (int l = 0; l < kLabelRuns; ++l) {
    const uint64_t runs = __ballot(len > l);
    if ((t & 63) == 0) {
      wsum[l][t >> 6] = __popcll(runs);
      atomicAdd(all + l, __popcll(runs));
    }
  }
  __syncthreads();
  if (len > 0 && len == best_count) atomicMin(&best, r[t]);
  __syncthreads();
  if (t == 0) sc[FS_BIG] = best;
  if (!table) return;
  int least = 1;
  while (least < kLabelRuns && all[least - 1] > kLabelMax) ++least;
  const uint64_t runs = __ballot(len >= least);
  int at = __popcll(runs & ((1ull << (t & 63)) - 1));
#pragma unroll
  for (int i = 0; i < kBigSample / 64; ++i) at += i < (t >> 6) ? wsum[least - 1][i] : 0;
  if (t <= kLabelMax) table[t] = INT32_MAX;
  __syncthreads();  // (one workgroup: the roots come after the fill)
  if (len >= least && at < kLabelMax) {
    table[at] = r[t];
    atomicAdd(&in, len);
  }
  __syncthreads();
  // no labels if too many samples outside the big component have none
  if (t == 0) sc[FS_LABELS] = (kBigSample - in) * 4 <= kBigSample - best_count;
}

// Full path compression. LABEL: also the label of every vertex, the place of
// its root in the table of k_big_component, kLabelMax if it is not there.
// Vertices of one label below kLabelMax are in one tree.
template <bool LABEL>
__global__ __launch_bounds__(kB) void k_cc_compress(int32_t* cc, int32_t n, const int32_t* __restrict__ sc,
                                                   const int32_t* __restrict__ table, uint8_t* __restrict__ label) {
  __shared__ int32_t tab[LABEL ? kLabelMax + 1 : 1];
  const int64_t v = (int64_t)blockIdx.x * kB + threadIdx.x;
  const bool named = LABEL && sc[FS_LABELS];
  if (LABEL) {
    static_assert(kB == kLabelMax + 1, "one table entry a lane");
    tab[threadIdx.x] = table[threadIdx.x];
    __syncthreads();
  }
  if (v >= n) return;
  const int32_t r = cc_find(cc, (int32_t)v);
  st(cc + v, r);
  if (named) {
    int at = 0;  // first entry of at least r; the last one is INT32_MAX
#pragma unroll
    for (int h = (kLabelMax + 1) / 2; h > 0; h >>= 1)
      if (tab[at + h - 1] < r) at += h;
    label[v] = (uint8_t)(tab[at] == r ? at : kLabelMax);
  }
}

// Remaining phase: rows of vertices outside the big component hook every
// distinct neighbour. An edge between two vertices of the big component is
// already inside one tree; any other edge is seen from an endpoint outside.
// The lanes of one row run side by side here, so the list insertion is an
// exchange.
// A workgroup closes up its rows that are left and deals
// their slots to the lanes, PER neighbouring ones at a time. Nearly all slots
// are inside one tree; bound by the gathers that find this out: of the label
// where there are labels (a byte a vertex, so that the table of a graph of
// 2^22 vertices stays in a 4 MiB L2), else of the parent. At 2^22 vertices and
// 2^26 slots in 513 components 433 us with labels, 675 without; a connected
// graph of 2^21 vertices and 2^25 slots 16 us (67 when the slots of all rows
// were dealt out and dropped one by one).
// ALL: no second round and no big component came before; every row is left.
template <bool EDGES, bool ALL, int PER>
__global__ __launch_bounds__(kB) void k_hook_rest(const int32_t* __restrict__ row_ptr, const int32_t* __restrict__ col,
                                                 int32_t n, int32_t nnz, int32_t* cc, const int32_t* __restrict__ sc,
                                                 const uint8_t* __restrict__ label, int rows,
                                                 int4* __restrict__ erec, int32_t* first, int32_t* __restrict__ next,
                                                 uint32_t* __restrict__ status) {
  __shared__ int32_t start[kRowsPerBlock + 1];  // of the rows left: first slot in their numbering,
  __shared__ int32_t slot[kRowsPerBlock];       // first slot in col,
  __shared__ int32_t vert[kRowsPerBlock];       // vertex,
  __shared__ int32_t tree[kRowsPerBlock];       // label, or -1 - an ancestor
  __shared__ int32_t wdeg[kB / 64], wcnt[kB / 64];
  static_assert(kRowsPerBlock == kB, "a lane per row");
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
  const int32_t r0 = blockIdx.x * rows;
  const int32_t big = ALL ? -1 : sc[FS_BIG];
  const bool named = !ALL && sc[FS_LABELS];
  int32_t a = 0, b = 0, mine = 0;
  bool keep = false, bad = false, over = false;
  if (t < rows && r0 + t < n) {
    a = row_ptr[r0 + t];
    b = row_ptr[r0 + t + 1];
    bad = a < 0 || a > b || b > nnz;
    const int32_t root = cc_find(cc, r0 + t);
    mine = named ? (int32_t)label[r0 + t] : kLabelMax;
    if (mine == kLabelMax) mine = -1 - root;
    keep = a < b && root != big;
  }
  if (__syncthreads_or(bad)) return;  // flagged at the start of the forest
  const uint64_t kept = __ballot(keep);
  const int32_t deg = keep ? b - a : 0;
  int32_t inc = deg;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int32_t x = __shfl_up(inc, o, 64);
    if (lane >= o) inc += x;
  }
  if (lane == 63) {
    wdeg[wv] = inc;
    wcnt[wv] = __popcll(kept);
  }
  __syncthreads();
  int32_t total = 0, cnt = 0, at = __popcll(kept & ((1ull << lane) - 1)), from = inc - deg;
#pragma unroll
  for (int i = 0; i < kB / 64; ++i) {
    if (i < wv) {
      from += wdeg[i];
      at += wcnt[i];
    }
    total += wdeg[i];
    cnt += wcnt[i];
  }
  if (keep) {
    start[at] = from;
    slot[at] = a;
    vert[at] = r0 + t;
    tree[at] = mine;
  }
  if (t == 0) start[cnt] = total;
  __syncthreads();
  // 64-bit counter: total may lie within one stride of 2^31
  for (int64_t base = (int64_t)t * PER; base < total; base += kB * PER) {
    int j = row_of(start, cnt, (int32_t)base);
    int32_t row[PER], k[PER], w[PER], other[PER];
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int64_t x = base + i;
      if (i > 0 && x < total && (int32_t)x >= start[j + 1]) ++j;  // (rows that are left have slots)
      row[i] = j;
      k[i] = x < total ? slot[j] + ((int32_t)x - start[j]) : -1;
      w[i] = k[i] >= 0 ? col[k[i]] : 0;
      if ((uint32_t)w[i] >= (uint32_t)n) {
        bad = true;
        k[i] = -1;
        w[i] = 0;
      }
    }
#pragma unroll
    for (int i = 0; i < PER; ++i) other[i] = named ? (int32_t)label[w[i]] : -1 - ldc(cc + w[i]);
    if (named) {
#pragma unroll
      for (int i = 0; i < PER; ++i)
        if (other[i] == kLabelMax) other[i] = -1 - ldc(cc + w[i]);
    }
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      if (k[i] < 0 || other[i] == tree[row[i]]) continue;
      const int32_t u = vert[row[i]];
      if (w[i] == u || (k[i] > slot[row[i]] && col[k[i] - 1] == w[i])) continue;
      const int32_t e = cc_hook(cc, u, w[i], big, &over);
      if (EDGES && e >= 0) {
        erec[e] = make_int4(u, w[i], k[i], -1);
        next[2 * e] = atomicExch(first + u, 2 * e);
      }
    }
  }
  if (bad) flag(status, ST_BAD_CSR);
  if (over) flag(status, ST_OVERFLOW);
}

// The other half-edge of every forest edge in front of its vertex's list
// (cc[e] != e: root e was hooked, so edge e exists), and the slot of that
// half-edge. The search is made here, one lane per edge, not in the hooking
// kernels, whose lanes already climb. Bound by random accesses: an exchange
// (25 G/s) and two or three lines of the twin's row per edge; 339 us at 2^22
// vertices. It stands in place of sorted forest rows (both slots of every
// edge marked by atomics, degrees, a scan, the fill and a twin search per
// half-edge: 0.97 ms).
__global__ void k_link_in(const int32_t* __restrict__ row_ptr, const int32_t* __restrict__ col,
                          const int32_t* __restrict__ cc, int4* __restrict__ erec, int32_t n, int32_t nnz,
                          int32_t* first, int32_t* __restrict__ next, uint32_t* __restrict__ status) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= n || cc[e] == (int32_t)e) return;
  const int4 r = erec[e];
  const int32_t before = atomicExch(first + r.y, (int32_t)(2 * e + 1));
  bool bad = false;
  const int32_t t = twin_slot(row_ptr, col, nnz, r.x, r.y, &bad);
  next[2 * e + 1] = before;
  erec[e].w = t;
  if (bad) flag(status, ST_BAD_CSR);
}

// The roots of the components that have an edge and the first half-edge of
// each, in any order, and the number of forest half-edges. A workgroup takes
// kRootPer vertices per lane, so the shared counters see one update of each
// per 4096 vertices.
constexpr int kRootPer = 16;

__global__ __launch_bounds__(kB) void k_roots(const int32_t* __restrict__ cc, const int32_t* __restrict__ first,
                                             int32_t n, int32_t* __restrict__ roots, int32_t* __restrict__ heads,
                                             int32_t* __restrict__ sc) {
  __shared__ int32_t cnt[2], base;  // roots of this workgroup, its linked vertices; where its roots go
  if (threadIdx.x < 2) cnt[threadIdx.x] = 0;
  __syncthreads();
  const int64_t v0 = (int64_t)blockIdx.x * (kB * kRootPer) + threadIdx.x;
  uint32_t is = 0;
  int32_t linked = 0, at = 0;
#pragma unroll
  for (int i = 0; i < kRootPer; ++i) {
    const int64_t v = v0 + i * kB;
    if (v >= n) break;
    if (cc[v] != (int32_t)v) ++linked;
    else if (first[v] >= 0) is |= 1u << i;
  }
  for (int d = 32; d >= 1; d >>= 1) linked += __shfl_xor(linked, d, 64);
  if (__lane_id() == 0 && linked) atomicAdd(&cnt[1], linked);
  if (is) at = atomicAdd(&cnt[0], __popc(is));
  __syncthreads();
  if (threadIdx.x == 0) {
    if (cnt[0]) base = atomicAdd(sc + FS_ROOTS, cnt[0]);
    if (cnt[1]) atomicAdd(sc + FS_LEN, 2 * cnt[1]);
  }
  __syncthreads();
  for (int i = 0; is != 0; ++i, is >>= 1) {
    if (!(is & 1u)) continue;
    const int64_t v = v0 + i * kB;
    roots[base + at] = (int32_t)v;
    heads[base + at] = first[v];
    ++at;
  }
}

// The list of component i's root ends by going on to component i + 1 instead
// of wrapping: its list head becomes -3 - (that component's first half-edge,
// -1 after the last), below -1. The component's own first half-edge is kept
// in the root's edge record (a root is not hooked, so it has no edge).
__global__ void k_chain(const int32_t* __restrict__ roots, const int32_t* __restrict__ heads,
                        int32_t* __restrict__ sc, int32_t* __restrict__ first, int4* __restrict__ erec) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int32_t nroots = sc[FS_ROOTS];
  if (i >= nroots) return;
  if (i == 0) sc[FS_HEAD] = heads[0];
  erec[roots[i]].x = heads[i];
  first[roots[i]] = -3 - (i + 1 < nroots ? heads[i + 1] : -1);
}

// successors of both half-edges of edge e (one lane each edge, so the list
// pointers and the successors move as pairs), tour weights cleared and every
// vertex without a preorder. Each vertex's list wraps once, so of the 2n
// successors n gather a list head; otherwise bound by streaming (44 us at
// 2^22 vertices).
__global__ void k_forest_succ(const int32_t* __restrict__ cc, const int4* __restrict__ erec,
                              const int32_t* __restrict__ next, const int32_t* __restrict__ first, int32_t n,
                              int32_t* __restrict__ succ, uint32_t* __restrict__ dw, int32_t* __restrict__ pre) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= n) return;
  int32_t s0 = -2, s1 = -2;
  if (cc[e] != (int32_t)e) {
    const int2 nx = reinterpret_cast<const int2*>(next)[e];
    s0 = nx.y;  // succ(2e) = next(2e + 1), around the list of w
    s1 = nx.x;
    if (s0 < 0 || s1 < 0) {
      const int4 r = erec[e];
      if (s0 < 0) {
        const int32_t f = first[r.y];
        s0 = f >= 0 ? f : -3 - f;
      }
      if (s1 < 0) {
        const int32_t f = first[r.x];
        s1 = f >= 0 ? f : -3 - f;
      }
    }
  }
  reinterpret_cast<int2*>(succ)[e] = make_int2(s0, s1);
  reinterpret_cast<uint2*>(dw)[e] = make_uint2(0u, 0u);
  pre[e] = -1;
}

__device__ __forceinline__ int32_t rank_at(uint64_t pk, OffWord off, int32_t nsub, bool* bad) {
  uint32_t s = (uint32_t)pk;
  if (s >= (uint32_t)nsub) {
    *bad = true;
    s = 0;
  }
  return off.at(s) + (int32_t)((pk >> 32) & 0xffffu);
}

// Per forest edge: the rank of its half-edge that goes down (the earlier
// one), the child's subtree size (negative if the child is u, the first end)
// and the weight 1 at that rank. The twins are neighbours, so two sublist
// offsets are gathered and one weight scattered per edge (125 us at 2^22
// vertices; with twins apart and a record scattered to every vertex, 384 us
// and 67 us for the ranks before it). HYBRID: +1 / -1 at both ranks, whose
// prefix sum is the depth (component tours are balanced).
// A component's root, whose id numbers no edge: -2 - the rank at which the
// component starts, and its size. It counts in the preorder of what follows,
// so it puts a weight 1 on the half-edge before its start (the last one of the
// component before it, which goes up), the first component none.
template <bool HYBRID>
__global__ void k_direction(const uint64_t* __restrict__ packed, OffWord off, int32_t nsub,
                            const int32_t* __restrict__ cc, const int32_t* __restrict__ first,
                            const int4* __restrict__ erec, int32_t n, const int32_t* __restrict__ sc,
                            int2* __restrict__ ds, uint32_t* __restrict__ dw, uint32_t* __restrict__ status) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= n) return;
  const int32_t L = sc[FS_LEN];
  bool bad = false;
  int2 d = make_int2(-1, 0);
  if (cc[e] != (int32_t)e) {
    const ulonglong2 pk = reinterpret_cast<const ulonglong2*>(packed)[e];
    const int32_t r0 = rank_at(pk.x, off, nsub, &bad), r1 = rank_at(pk.y, off, nsub, &bad);
    if (bad || (uint32_t)r0 >= (uint32_t)L || (uint32_t)r1 >= (uint32_t)L) {
      bad = true;
    } else {
      const int32_t rd = min(r0, r1), ru = max(r0, r1);
      const int32_t size = (ru - rd + 1) >> 1;
      d = make_int2(rd, r0 < r1 ? size : -size);
      dw[rd] = 1u;
      if (HYBRID) dw[ru] = 0xffffffffu;
    }
  } else if (first[e] < -1) {
    const int32_t after = -3 - first[e];
    const int32_t r = rank_at(packed[erec[e].x], off, nsub, &bad);
    const int32_t end = after < 0 ? L : rank_at(packed[after], off, nsub, &bad);
    if (bad || (uint32_t)r >= (uint32_t)L || end <= r || end > L) {
      bad = true;
    } else {
      d = make_int2(-2 - r, ((end - r) >> 1) + 1);
      if (!HYBRID && r > 0) dw[r - 1] = 1u;
    }
  }
  if (bad) flag(status, ST_BAD_INDEX);
  ds[e] = d;
}

// preorder of every vertex from the scanned weights, its slot of the parent
// edge (-1 at a root), and by preorder {subtree size, the parent edge's slot
// at the parent, the slot at the child}. Bound by its scatters (4, 4 and 16
// bytes per edge, which cost the same) and the gathered weight: 170 us at 2^22
// vertices.
__global__ void k_preorder(const int2* __restrict__ ds, const int4* __restrict__ erec,
                           const uint32_t* __restrict__ I, int32_t n, int32_t* __restrict__ pre,
                           int32_t* __restrict__ uslot, int4* __restrict__ byp) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= n) return;
  const int2 d = ds[e];
  if (d.x == -1) return;  // an isolated vertex
  int32_t v = (int32_t)e, ps = -1, us = -1, p = 0;
  if (d.x >= 0) {
    const int4 r = erec[e];
    const bool down = d.y > 0;  // u is the parent
    v = down ? r.y : r.x;
    ps = down ? r.z : r.w;
    us = down ? r.w : r.z;
    p = (int32_t)I[d.x];
  } else if (d.x < -2) {
    p = (int32_t)I[-3 - d.x];  // the weight before the component's start
  }
  if ((uint32_t)p >= (uint32_t)n) return;  // only after a flagged error
  pre[v] = p;
  uslot[v] = us;
  byp[p] = make_int4(abs(d.y), ps, us, 0);
}

// Range passes over the slots of all rows, for a kernel that gathers a word
// per neighbour. Such gathers run at 73 G/s from a 16 MiB array but at 190
// G/s from 4 MiB, what one XCD's L2 holds. So a pass takes only the
// neighbours with ids in [lo, hi), all workgroups the same ones, and the next
// pass reads the columns again. A pass must then cost little besides its
// gathers: a workgroup's rows are staged in LDS with coalesced loads, and
// 2^glog lanes scan a row (its part in [lo, hi), found by binary search: rows
// are sorted). Workgroups whose rows do not fit the stage read their slots
// directly, all lanes together for the long rows.
constexpr int kRowStage = 6144;   // staged slots of a workgroup's rows
constexpr int kRowLoads = 8;      // column loads a lane issues together
constexpr int kRowHeavy = 512;    // longer rows of an unstaged workgroup are taken by all its lanes
constexpr int kRowLanesLog = 4;   // at most 16 lanes a row

__device__ __forceinline__ void stage_slots(const int32_t* __restrict__ col, int32_t m, int32_t* st) {
  for (int32_t i0 = threadIdx.x; i0 < m; i0 += kRowLoads * kB) {
    int32_t x[kRowLoads];  // a lane's loads first, then their stores
#pragma unroll
    for (int j = 0; j < kRowLoads; ++j) x[j] = i0 + j * kB < m ? col[i0 + j * kB] : 0;
#pragma unroll
    for (int j = 0; j < kRowLoads; ++j)
      if (i0 + j * kB < m) st[i0 + j * kB] = x[j];
  }
}

// first staged slot of [x, e) with a neighbour of at least lo
__device__ __forceinline__ int32_t range_start(const int32_t* st, int32_t x, int32_t e, int32_t lo) {
  if (lo <= 0) return x;
  while (x < e) {
    const int32_t mid = (x + e) >> 1;
    if (st[mid] < lo) x = mid + 1;
    else e = mid;
  }
  return x;
}

// One pass per 1.5 * 2^20 vertices (6 MiB of words), at most three: the
// extremes took, with 1 / 2 / 3 / 4 passes, 267 / 248 / 272 / 301 us at 2^21
// vertices and 2^25 slots, 794 / 667 / 650 / 700 at 2^22 and 2^26, 1105 /
// 1028 / 1001 / 1025 at 2^23 and 2^26, 2407 / 2336 / 2313 / 2365 at 2^24 and
// 2^27; below 6 slots a row reading the rows again costs what the gathers
// gain (253 / 256 / 270 at 2^22 and 2^24).
int range_passes(int32_t n, int32_t nnz) {
  constexpr int64_t kRangeVerts = 3 << 19;
  if (nnz < 6 * (int64_t)n) return 1;
  return (int)std::min<int64_t>(3, (n + kRangeVerts - 1) / kRangeVerts);
}

// lanes per row: one per 16 slots of an average row, more on a small graph,
// whose rows are then spread over the compute units
int row_lanes_log(int32_t n, int32_t nnz) {
  int g = 0;
  while (g < kRowLanesLog && (((int64_t)n << g) * 16 < nnz || ceil_div(n, kB >> g) < 512)) ++g;
  return g;
}

// per vertex: min / max preorder over itself and its neighbours, the parent
// edge's own slot left out (the paper's segreduce), stored at its preorder
// position as one 8-byte store.
// Rows are scanned in range passes (above): `acc` carries a row's extremes
// from pass to pass by vertex, and the last pass stores them by preorder. At
// 2^22 vertices and 2^26 slots three passes take 650 us, one pass 795, and
// one pass with 16 lanes a row combined by shuffles 891 (with passes that
// version was issue-bound, 350 us for each further one).
template <bool FIRST, bool LAST>
__global__ __launch_bounds__(kB) void k_minmax(const int32_t* __restrict__ row_ptr, const int32_t* __restrict__ col,
                                              const int32_t* __restrict__ uslot, const int32_t* __restrict__ pre,
                                              int32_t n, int32_t nnz, int32_t lo, int32_t hi, int glog,
                                              int2* __restrict__ acc, int2* __restrict__ amm) {
  __shared__ int32_t st[kRowStage];
  __shared__ int32_t heavy[kB], nheavy;
  __shared__ int2 wmm[kB / 64];
  const int g = 1 << glog, rows = kB >> glog, sub = threadIdx.x & (g - 1);
  const int64_t nblk = ((int64_t)n + rows - 1) / rows;
  // row blocks stride over the grid (a dispatch holds < 2^32 work-items)
  for (int64_t rb = blockIdx.x; rb < nblk; rb += gridDim.x) {
    const int32_t r0 = (int32_t)(rb * rows);
    const int cnt = min(rows, n - r0);
    const int32_t A = clampi(row_ptr[r0], 0, nnz), B = clampi(row_ptr[r0 + cnt], A, nnz);
    const bool staged = B - A <= kRowStage;  // the same for every lane
    const int ri = threadIdx.x >> glog;
    const int32_t u = r0 + min(ri, cnt - 1);
    const int32_t a = clampi(row_ptr[u], 0, nnz), b = clampi(row_ptr[u + 1], a, nnz);
    const int32_t up = uslot[u];
    int32_t p = (FIRST || LAST) ? pre[u] : 0, mn = p, mx = p;
    if (!FIRST) {
      const int2 x = acc[u];
      mn = x.x;
      mx = x.y;
    }
    const bool own = ri < cnt && p >= 0 && p < n;  // not past the end, not isolated
    if (threadIdx.x == 0) nheavy = 0;
    if (staged) stage_slots(col + A, B - A, st);
    __syncthreads();
    if (own && staged && a >= A && b <= B) {
      const int32_t e = b - A, ups = up - A;
      for (int32_t x = range_start(st, a - A, e, lo) + sub; x < e; x += g) {
        const int32_t w = st[x];
        if (w >= hi) break;
        if (x == ups || w < lo) continue;
        const int32_t pw = pre[w];
        mn = min(mn, pw);
        mx = max(mx, pw);
      }
    } else if (own && b - a <= kRowHeavy) {
      for (int64_t k = (int64_t)a + sub; k < b; k += g) {  // b may lie within one stride of 2^31
        const int32_t w = col[k];
        if (k == up || w < lo || w >= hi) continue;
        const int32_t pw = pre[w];
        mn = min(mn, pw);
        mx = max(mx, pw);
      }
    } else if (own && sub == 0) {
      heavy[atomicAdd(&nheavy, 1)] = ri;
    }
    for (int o = g >> 1; o > 0; o >>= 1) {
      mn = min(mn, __shfl_xor(mn, o, 64));
      mx = max(mx, __shfl_xor(mx, o, 64));
    }
    __syncthreads();
    for (int h = 0; h < nheavy; ++h) {
      const int hr = heavy[h];
      const int32_t ha = clampi(row_ptr[r0 + hr], 0, nnz), hb = clampi(row_ptr[r0 + hr + 1], ha, nnz);
      const int32_t hup = uslot[r0 + hr];
      int32_t m0 = INT32_MAX, m1 = INT32_MIN;
      for (int64_t k = (int64_t)ha + threadIdx.x; k < hb; k += kB) {
        const int32_t w = col[k];
        if (k == hup || w < lo || w >= hi) continue;
        const int32_t pw = pre[w];
        m0 = min(m0, pw);
        m1 = max(m1, pw);
      }
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) {
        m0 = min(m0, __shfl_xor(m0, o, 64));
        m1 = max(m1, __shfl_xor(m1, o, 64));
      }
      if (__lane_id() == 0) wmm[threadIdx.x >> 6] = make_int2(m0, m1);
      __syncthreads();
      if (ri == hr)
        for (int w = 0; w < kB / 64; ++w) {
          mn = min(mn, wmm[w].x);
          mx = max(mx, wmm[w].y);
        }
      __syncthreads();
    }
    if (own && sub == 0) {
      if (LAST) amm[p] = make_int2(mn, mx);
      else acc[u] = make_int2(mn, mx);
    }
    __syncthreads();  // the stage and the heavy list are rewritten by the next row block
  }
}

// In-block RMQ by suffix-extreme bitmasks: for position o of a block of
// B = 2^LOG elements, bit j <= o of mmin[o] is set iff element j is smaller
// than every element after it up to o. The minimum of [l, o] is then the
// element at the lowest set bit at or above l: that element is a suffix
// minimum and no suffix minimum between l and it can be smaller. Likewise
// for maxima. Lane o of each B-lane group builds its two masks; lane B-1
// also yields the block's extremes (level 0 of the sparse table).
template <int LOG>
__global__ __launch_bounds__(kB) void k_rmq_blocks(const int2* __restrict__ amm, int32_t n, typename RmqMask<LOG>::type* __restrict__ mmin,
                                                  typename RmqMask<LOG>::type* __restrict__ mmax,
                                                  int32_t* __restrict__ bmin, int32_t* __restrict__ bmax) {
  using M = typename RmqMask<LOG>::type;
  constexpr int B = 1 << LOG;
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const bool ok = i < n;
  const int2 v = ok ? amm[i] : make_int2(INT32_MAX, INT32_MIN);
  const int32_t vmin = v.x, vmax = v.y;
  const int o = __lane_id() & (B - 1);
  M fmin = 0, fmax = 0;
  int32_t rmin = INT32_MAX, rmax = INT32_MIN;
#pragma unroll
  for (int j = B - 1; j >= 0; --j) {
    const int32_t x = __shfl(vmin, j, B);
    const int32_t y = __shfl(vmax, j, B);
    if (j <= o) {
      if (x < rmin) {
        fmin |= (M)1 << j;
        rmin = x;
      }
      if (y > rmax) {
        fmax |= (M)1 << j;
        rmax = y;
      }
    }
  }
  if (ok) {
    mmin[i] = fmin;
    mmax[i] = fmax;
  }
  if (o == B - 1 && (i >> LOG) < (((int64_t)n + B - 1) >> LOG)) {
    bmin[i >> LOG] = rmin;
    bmax[i >> LOG] = rmax;
  }
}

// Levels base + 1 .. base + count of the sparse table (level k at k * nb: the
// extremes of blocks b .. b + 2^k - 1, as far as they exist) in one launch:
// level base + m at b is the extreme over 2^m entries of level `base`, 2^base
// apart, so one running extreme over 2^count entries passes all of them. At
// 2^17 blocks 3 launches take 27 us where one per level took 17 and 107, at
// 157 blocks 2 launches in place of 7.
constexpr int kSparseStep = 6;

__global__ __launch_bounds__(kB) void k_sparse_levels(int32_t* stmin, int32_t* stmax, int32_t nb, int base,
                                                     int count) {
  const int64_t b = (int64_t)blockIdx.x * kB + threadIdx.x;
  if (b >= nb) return;
  const int32_t* mn = stmin + (int64_t)base * nb;
  const int32_t* mx = stmax + (int64_t)base * nb;
  int32_t lo = mn[b], hi = mx[b];
  for (int m = 1; m <= count; ++m) {
    const int h = 1 << (m - 1);
#pragma unroll 8
    for (int j = h; j < 2 * h; ++j) {
      const int64_t o = b + ((int64_t)j << base);
      if (o < nb) {
        lo = min(lo, mn[o]);
        hi = max(hi, mx[o]);
      }
    }
    stmin[(int64_t)(base + m) * nb + b] = lo;
    stmax[(int64_t)(base + m) * nb + b] = hi;
  }
}

template <int LOG>
struct Rmq {
  const int2* amm;
  const typename RmqMask<LOG>::type *mmin, *mmax;
  const int32_t* stmin;  // sparse table levels concatenated: level k at k * nb
  const int32_t* stmax;
  int32_t nb;
};

// extremes of [l, r] inside one block, r's block
template <int LOG>
__device__ __forceinline__ void rmq_in_block(const Rmq<LOG>& q, int32_t l, int32_t r, int32_t* mn, int32_t* mx) {
  using M = typename RmqMask<LOG>::type;
  const int32_t base = r & ~((1 << LOG) - 1);
  const M keep = ~(M)0 << (l - base);
  *mn = q.amm[base + RmqMask<LOG>::ctz(q.mmin[r] & keep)].x;
  *mx = q.amm[base + RmqMask<LOG>::ctz(q.mmax[r] & keep)].y;
}

template <int LOG>
__device__ __forceinline__ void rmq(const Rmq<LOG>& q, int32_t l, int32_t r, int32_t* lo, int32_t* hi) {
  const int32_t bl = l >> LOG, br = r >> LOG;
  int32_t mn, mx;
  if (bl == br) {
    rmq_in_block(q, l, r, &mn, &mx);
  } else {
    int32_t a0, a1, b0, b1;
    rmq_in_block(q, l, (bl << LOG) + (1 << LOG) - 1, &a0, &a1);
    rmq_in_block(q, br << LOG, r, &b0, &b1);
    mn = min(a0, b0);
    mx = max(a1, b1);
    if (bl + 1 <= br - 1) {
      const int32_t a = bl + 1, b = br - 1;
      const int k = msb32((uint32_t)(b - a + 1));
      const int64_t base = (int64_t)k * q.nb;
      mn = min(mn, min(q.stmin[base + a], q.stmin[base + b - (1 << k) + 1]));
      mx = max(mx, max(q.stmax[base + a], q.stmax[base + b - (1 << k) + 1]));
    }
  }
  *lo = mn;
  *hi = mx;
}

// workgroups of the bridge test at most
constexpr int kTestBlocks = 2048;

// one lane per preorder position i < (number of non-isolated vertices, one
// more than the last value of the preorder scan), in a grid-stride loop: the subtree
// interval starts at i, so neighbouring lanes read neighbouring RMQ entries
template <int LOG>
__global__ __launch_bounds__(kB) void k_bridge_test(const int4* __restrict__ byp, const uint32_t* __restrict__ I,
                                                   const int32_t* __restrict__ sc, int32_t Lcap, int32_t n, Rmq<LOG> q,
                                                   uint32_t* __restrict__ mask,
                                                   int64_t* __restrict__ count) {
  const int32_t npre = sc[FS_LEN] == 0 ? 0 : min((int32_t)I[Lcap - 1] + 1, n);
  uint32_t found = 0;
  for (int64_t i = (int64_t)blockIdx.x * kB + threadIdx.x; i < npre; i += (int64_t)gridDim.x * kB) {
    const int4 b = byp[i];
    const int32_t l = (int32_t)i, r = l + b.x - 1;
    if (b.y >= 0 && r >= l && r < npre) {
      int32_t lo, hi;
      rmq(q, l, r, &lo, &hi);
      if (lo == l && hi == r) {
        ++found;
        atomicOr(mask + (b.y >> 5), 1u << (b.y & 31));
        if (b.z >= 0) atomicOr(mask + (b.z >> 5), 1u << (b.z & 31));
      }
    }
  }
  // one count update per workgroup: every wavefront adding its own to the
  // one counter serialised some 65K same-address atomics at 2^22 vertices
  __shared__ uint32_t wsum[kB / 64];
  uint32_t t = found;
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) t += __shfl_xor(t, o, 64);
  if (__lane_id() == 0) wsum[threadIdx.x >> 6] = t;
  __syncthreads();
  if (threadIdx.x == 0) {
    uint32_t tot = 0;
    for (int w = 0; w < kB / 64; ++w) tot += wsum[w];
    if (tot) atomicAdd((unsigned long long*)count, (unsigned long long)tot);
  }
}

__global__ void k_zero_i64(int64_t* p) { *p = 0; }

// hybrid: parent, level and the two slots of the parent edge of every vertex
// from the direction records and the depth prefix sums, and both slots of
// every forest edge in a bitmask. Isolated vertices keep -1 everywhere.
__global__ void k_hybrid_fill(int32_t n, int32_t words, int32_t* __restrict__ par, int32_t* __restrict__ lvl,
                              int32_t* __restrict__ pslot, int32_t* __restrict__ uslot,
                              uint32_t* __restrict__ tbits) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < max(n, words);
       i += (int64_t)gridDim.x * blockDim.x) {
    if (i < n) par[i] = lvl[i] = pslot[i] = uslot[i] = -1;
    if (i < words) tbits[i] = 0u;
  }
}

__global__ void k_hybrid_nodes(const int2* __restrict__ ds, const int4* __restrict__ erec,
                               const uint32_t* __restrict__ depth_at, int32_t n, int32_t nnz,
                               int32_t* __restrict__ par, int32_t* __restrict__ lvl, int32_t* __restrict__ pslot,
                               int32_t* __restrict__ uslot, uint32_t* __restrict__ tbits) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= n) return;
  const int2 d = ds[e];
  if (d.x < -1) {  // a component's root
    par[e] = -2;
    lvl[e] = 0;
  }
  if (d.x < 0) return;
  const int4 r = erec[e];
  const bool down = d.y > 0;
  const int32_t child = down ? r.y : r.x;
  par[child] = down ? r.x : r.y;
  lvl[child] = (int32_t)depth_at[d.x];
  pslot[child] = down ? r.z : r.w;
  uslot[child] = down ? r.w : r.z;
  if ((uint32_t)r.z < (uint32_t)nnz) atomicOr(tbits + (r.z >> 5), 1u << (r.z & 31));
  if ((uint32_t)r.w < (uint32_t)nnz) atomicOr(tbits + (r.w >> 5), 1u << (r.w & 31));
}

}  // namespace

// Connectivity labels (cc[v] == v at one root per component) and, with erec,
// a spanning forest: sampled hooking rounds, then the rows outside the
// largest sampled component. Edge e exists iff cc[e] != e; erec[e] = {u, w,
// slot (u, w), -}, and first / next hold the half-edges 2e out of u
// (k_link_in adds those out of w, and the slot (w, u)). sc: 8 scalars (FS_*).
// mask and count (optional) are cleared on the way. work: n words of scratch.
int spanning_forest(Ctx* c, const int32_t* row_ptr, const int32_t* col, int32_t n, int32_t nnz, int32_t* cc,
                    int32_t* sc, int4* erec, int32_t* first, int32_t* next, uint32_t* mask, int64_t* count,
                    int32_t* work, hipStream_t s) {
  const int32_t words = (int32_t)(((int64_t)nnz + 31) >> 5);
  const int gn = ceil_div(n, kB);
  // rows of a workgroup: fewer on a small graph, so that its rows are spread
  // over the compute units (5000 vertices at 16 slots, whole call: 135 us with
  // 256 rows a workgroup, 111 with 16)
  int rows = kRowsPerBlock;
  while (rows > 16 && ceil_div(n, rows) < 512) rows >>= 1;
  const int grows = ceil_div(n, rows);
  const bool edges = erec != nullptr;
  {
    ET_PROF(c, s, "k_forest_init");
    const auto kern = edges ? k_forest_init<true> : k_forest_init<false>;
    hipLaunchKernelGGL(kern, dim3(gn), dim3(kB), 0, s, row_ptr, col, n, nnz, cc, erec, first, next, sc, mask,
                       words, count, c->d_status);
  }
  // Labels where the parents (4 bytes a vertex) are more than an XCD's 4 MiB
  // L2 holds. Whole call without / with them, us: 2^20 vertices 870 / 885 (4
  // slots a vertex, connected), 949 / 939 (16), 951 / 952 (16, many
  // components); 2^21 1332 / 1330, 1431 / 1448, 1609 / 1575; 2^22 2287 / 2281,
  // 3088 / 2872, 3362 / 3134; 2^23 4210 / 4208, 5737 / 5674, 6842 / 6860 (there
  // too many components to name). They cost one more pass over the parents.
  const bool labels = nnz > kTinySlots && n >= kLabelNodes;
  int32_t* table = labels ? work : nullptr;
  uint8_t* label = reinterpret_cast<uint8_t*>(work + kLabelMax + 1);
  const auto compress = [&](bool named) {
    ET_PROF(c, s, "k_cc_compress");
    const auto kern = named ? k_cc_compress<true> : k_cc_compress<false>;
    hipLaunchKernelGGL(kern, dim3(gn), dim3(kB), 0, s, cc, n, sc, table, label);
  };
  compress(false);
  // A tiny sparse graph is bound by its launches, and the second round, its
  // compression and the pick are three. Whole call without / with them, us: at 8
  // slots a vertex 78 / 86 (200 vertices), 94 / 95 (500), 101 / 102 (1000), 122 /
  // 111 (2000); vertices joined to the next ones by id 90 / 102 (1000) and 154 /
  // 123 (2000); cycles 85 / 98 (1000), 119 / 130 (4000). Beyond, and with longer
  // rows, the hooks of all rows meet at too few roots.
  const bool sample = nnz > kTinySlots || nnz > 8 * (int64_t)n;
  if (sample) {
    {
      ET_PROF(c, s, "k_hook_sample");
      const auto kern = edges ? k_hook_sample<true> : k_hook_sample<false>;
      hipLaunchKernelGGL(kern, dim3(gn), dim3(kB), 0, s, row_ptr, col, n, nnz, cc, erec, first, next, c->d_status);
    }
    compress(false);  // (the pick climbs for its samples one by one)
    {
      ET_PROF(c, s, "k_big_component");
      hipLaunchKernelGGL(k_big_component, dim3(1), dim3(kBigSample), 0, s, cc, n, sc, table);
    }
    if (labels) compress(true);
  }
  {
    ET_PROF(c, s, "k_hook_rest");
    const auto kern = !sample                 ? (edges ? k_hook_rest<true, true, 1> : k_hook_rest<false, true, 1>)
                      : rows == kRowsPerBlock ? (edges ? k_hook_rest<true, false, 4> : k_hook_rest<false, false, 4>)
                                              : (edges ? k_hook_rest<true, false, 1> : k_hook_rest<false, false, 1>);
    hipLaunchKernelGGL(kern, dim3(grows), dim3(kB), 0, s, row_ptr, col, n, nnz, cc, sc, label, rows, erec, first,
                       next, c->d_status);
  }
  return hipGetLastError() == hipSuccess ? ET_OK : ET_EHIP;
}

// Scratch of the Tarjan-Vishkin path of bridges_run: every array below, the
// ranking's buffers (same scope) and the partials of its scan.
size_t bridges_scratch_bytes(const Ctx* c, int32_t n, int32_t nnz) {
  if (n <= 1 || nnz == 0) return 0;
  const size_t N = (size_t)n;
  const int rlog = c ? c->qs.rmq_log : QueryShape{}.rmq_log;
  const size_t nb = (N + (1u << rlog) - 1) >> rlog;
  size_t levels = 1;
  while (((size_t)1 << levels) <= nb) ++levels;
  size_t b = 6 * scratch_block<int32_t>(N) + 4 * scratch_block<int2>(N) + 2 * scratch_block<int4>(N) +
             2 * scratch_block<uint32_t>(N << (rlog - 5)) + 2 * scratch_block<int32_t>(levels * nb) +
             scratch_block<int32_t>(8);
  b += list_rank_plan_bytes(c, (int32_t)(2 * N), 1, 0, true);  // (a union's, the larger one)
  return b + scan_scratch_bytes((int64_t)(2 * N));
}

int bridges_run(Ctx* c, const int32_t* row_ptr, const int32_t* col, int32_t n, int32_t nnz, uint32_t* mask,
                hipStream_t s, int algo, int32_t graphs) {
  if (algo == kAlgoCK) return bridges_ck_bfs(c, row_ptr, col, n, nnz, mask, s);
  const int32_t words = (int32_t)(((int64_t)nnz + 31) >> 5);
  if (n <= 1 || nnz == 0) {  // no bridge
    hipLaunchKernelGGL(k_zero_i64, dim3(1), dim3(1), 0, s, c->d_bcount);
    if (words > 0)
      hipLaunchKernelGGL(k_fill_i32, dim3(std::min(ceil_div(words, kB), 4096)), dim3(kB), 0, s,
                         reinterpret_cast<int32_t*>(mask), (int64_t)words, 0);
    return hipGetLastError() == hipSuccess ? ET_OK : ET_EHIP;
  }

  const int32_t L2 = 2 * n;  // half-edge ids; edge ids are the vertices hooked as roots
  Scratch sc(c, s);
  int32_t* cc = sc.get<int32_t>(n);
  int32_t* first = sc.get<int32_t>(n);
  int2* next = sc.get<int2>(n);
  int4* erec = sc.get<int4>(n);
  int32_t* roots = sc.get<int32_t>(n);
  int32_t* heads = sc.get<int32_t>(n);
  int2* succ = sc.get<int2>(n);
  int2* dwp = sc.get<int2>(n);
  int32_t* pre = sc.get<int32_t>(n);
  int32_t* uslot = sc.get<int32_t>(n);
  int4* byp = sc.get<int4>(n);
  int2* amm = sc.get<int2>(n);
  const int rlog = c->qs.rmq_log;                        // range-minimum blocks of 2^rlog vertices
  uint32_t* mmin = sc.get<uint32_t>((size_t)n << (rlog - 5));
  uint32_t* mmax = sc.get<uint32_t>((size_t)n << (rlog - 5));
  const int32_t nb = (int32_t)(((int64_t)n + (1 << rlog) - 1) >> rlog);
  int levels = 1;
  while ((1 << levels) <= nb) ++levels;
  int32_t* stmin = sc.get<int32_t>((size_t)levels * nb);
  int32_t* stmax = sc.get<int32_t>((size_t)levels * nb);
  int32_t* scal = sc.get<int32_t>(8);
  if (sc.failed) return ET_ENOMEM;
  uint32_t* dw = reinterpret_cast<uint32_t*>(dwp);

  const int gn = ceil_div(n, kB);
  // 1. spanning forest
  ET_PROF(c, s, "phase:bridges");
  int rc = spanning_forest(c, row_ptr, col, n, nnz, cc, scal, erec, first, reinterpret_cast<int32_t*>(next), mask,
                           c->d_bcount, pre, s);
  if (rc) return rc;
  // 2. half-edge lists, component chaining, successors
  {
    ET_PROF(c, s, "k_link_in");
    hipLaunchKernelGGL(k_link_in, dim3(gn), dim3(kB), 0, s, row_ptr, col, cc, erec, n, nnz, first,
                       reinterpret_cast<int32_t*>(next), c->d_status);
  }
  {
    ET_PROF(c, s, "k_roots");
    hipLaunchKernelGGL(k_roots, dim3(ceil_div(n, kB * kRootPer)), dim3(kB), 0, s, cc, first, n, roots, heads, scal);
  }
  {
    ET_PROF(c, s, "k_chain");
    hipLaunchKernelGGL(k_chain, dim3(gn), dim3(kB), 0, s, roots, heads, scal, first, erec);
  }
  {
    ET_PROF(c, s, "k_forest_succ");
    hipLaunchKernelGGL(k_forest_succ, dim3(gn), dim3(kB), 0, s, cc, erec, reinterpret_cast<int32_t*>(next), first, n,
                       reinterpret_cast<int32_t*>(succ), dw, pre);
  }
  // 3. one list ranking, directions, preorder
  LRResult lr;
  rc = list_rank_core(c, sc, reinterpret_cast<int32_t*>(succ), L2, scal + FS_HEAD, 1, false, scal + FS_LEN, &lr, s,
                      true, 0, graphs > 1 ? L2 / graphs : 0);
  if (rc) return rc;
  int2* ds = next;  // the list pointers are dead
  {
    ET_PROF(c, s, "k_direction");
    const auto kern = algo == kAlgoHybrid ? k_direction<true> : k_direction<false>;
    hipLaunchKernelGGL(kern, dim3(gn), dim3(kB), 0, s, lr.packed, lr.word, lr.nsub, cc, first, erec, n, scal,
                       ds, dw, c->d_status);
  }
  if (algo == kAlgoHybrid) {
    // the hybrid of Section 4.1: this rooted forest, levels from the tour,
    // then Chaitanya-Kothapalli marking instead of low / high
    rc = scan_u32(c, dw, dw, L2, ScanOp::Add, false, s);
    if (rc) return rc;
    int32_t* par = first;                                 // per-vertex arrays of the other phases are unused
    int32_t* lvl = reinterpret_cast<int32_t*>(amm);
    int32_t* pslot = pre;
    uint32_t* tbits = sc.get<uint32_t>(words);
    if (sc.failed) return ET_ENOMEM;
    hipLaunchKernelGGL(k_hybrid_fill, dim3(std::min(ceil_div(std::max(n, words), kB), 4096)), dim3(kB), 0, s, n, words,
                       par, lvl, pslot, uslot, tbits);
    {
      ET_PROF(c, s, "k_hybrid_nodes");
      hipLaunchKernelGGL(k_hybrid_nodes, dim3(gn), dim3(kB), 0, s, ds, erec, dw, n, nnz, par, lvl, pslot, uslot,
                         tbits);
    }
    return ck_mark(c, row_ptr, col, n, nnz, tbits, par, lvl, pslot, uslot, mask, s);
  }
  rc = scan_u32(c, dw, dw, L2, ScanOp::Add, false, s);
  if (rc) return rc;
  {
    ET_PROF(c, s, "k_preorder");
    hipLaunchKernelGGL(k_preorder, dim3(gn), dim3(kB), 0, s, ds, erec, dw, n, pre, uslot, byp);
  }
  // 4. extremes over the neighbours, by preorder
  {
    ET_PROF(c, s, "k_minmax");
    const int passes = range_passes(n, nnz), glog = row_lanes_log(n, nnz);
    const int64_t step = ((int64_t)n + passes - 1) / passes;
    const dim3 g(std::min(ceil_div(n, kB >> glog), kMaxGrid));
    int2* acc = succ;  // the successors are dead
    for (int p = 0; p < passes; ++p) {
      const auto kern = passes == 1       ? k_minmax<true, true>
                        : p == 0          ? k_minmax<true, false>
                        : p == passes - 1 ? k_minmax<false, true>
                                          : k_minmax<false, false>;
      const int32_t lo = (int32_t)std::min<int64_t>(p * step, n), hi = (int32_t)std::min<int64_t>((p + 1) * step, n);
      hipLaunchKernelGGL(kern, g, dim3(kB), 0, s, row_ptr, col, uslot, pre, n, nnz, lo, hi, glog, acc, amm);
    }
  }
  // 5. range extremes
  {
    ET_PROF(c, s, "k_rmq_blocks");
    if (rlog == 6)
      hipLaunchKernelGGL(k_rmq_blocks<6>, dim3(gn), dim3(kB), 0, s, amm, n, reinterpret_cast<uint64_t*>(mmin),
                         reinterpret_cast<uint64_t*>(mmax), stmin, stmax);
    else
      hipLaunchKernelGGL(k_rmq_blocks<5>, dim3(gn), dim3(kB), 0, s, amm, n, mmin, mmax, stmin, stmax);
  }
  for (int k = 0; k + 1 < levels; k += kSparseStep) {
    ET_PROF(c, s, "k_sparse_levels");
    hipLaunchKernelGGL(k_sparse_levels, dim3(ceil_div(nb, kB)), dim3(kB), 0, s, stmin, stmax, nb, k,
                       std::min(kSparseStep, levels - 1 - k));
  }
  // 6. test
  {
    ET_PROF(c, s, "k_bridge_test");
    if (rlog == 6) {
      Rmq<6> q{amm, reinterpret_cast<const uint64_t*>(mmin), reinterpret_cast<const uint64_t*>(mmax), stmin, stmax,
               nb};
      hipLaunchKernelGGL(k_bridge_test<6>, dim3(std::min(gn, kTestBlocks)), dim3(kB), 0, s, byp, dw, scal, L2, n, q, mask,
                         c->d_bcount);
    } else {
      Rmq<5> q{amm, mmin, mmax, stmin, stmax, nb};
      hipLaunchKernelGGL(k_bridge_test<5>, dim3(std::min(gn, kTestBlocks)), dim3(kB), 0, s, byp, dw, scal, L2, n, q, mask,
                         c->d_bcount);
    }
  }
  return hipGetLastError() == hipSuccess ? ET_OK : ET_EHIP;
}

}  // namespace et
