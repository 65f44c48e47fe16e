// Euler tour of a rooted tree, node statistics and the Inlabel tables
// (Sections 2.1, 2.2 and 3.1), and the LCA query kernel (Section 3.1).
//
// Build, for a parent array of n nodes:
//   1. group_by_parent: children of every node, ascending (radix.hip).
//   2. k_succ: over the grouped order, succ(2c+1) = 2 * next sibling of c,
//      or 2 * parent(c) + 1 after the last sibling (-1 below the root), and
//      succ(2p) = 2 * first child of p; leaves keep succ(2c) = 2c+1. This is
//      next(twin(e)) of the paper's DCEL with the children of a node in
//      ascending order and the tour split before the root's first child.
//   3. one list ranking of the 2n half-edges, carrying the number of down
//      half-edges (Section 2: weights on the tour give preorder and level).
//   4. k_node: rank(2c) = R0, number of down half-edges up to it = D; then
//      pre(c) = D, depth(c) = 2D - R0 - 1, size(c) = (rank(2c+1) - R0 + 1)/2,
//      and inlabel(c) = the member of [pre+1, pre+size] with the most
//      trailing zeros, in closed form (j >> k) << k with j = pre + size and
//      k the highest bit in which pre and j differ.
//   5. k_head: a node is the top of its inlabel path iff it is the root or
//      its parent's inlabel differs; head[inlabel] = {parent, depth - 1},
//      and the label of the parent's path is recorded per label.
//   6. ascendant(v) (the OR of 2^h over the labels of v's ancestors) only
//      depends on v's path: it is the ascendant of the path above plus the
//      path's own level bit. Labels on a root path have strictly decreasing
//      levels, so k_asc_label walks each label's chain of parent path labels
//      (at most one link per level) into a table by label; k_record
//      writes the node records with it.
#include "et_internal.hpp"

namespace et {
namespace {

constexpr int kB = 256;

enum { SC_ROOT = 0, SC_NROOTS = 1, SC_HEAD = 2, SC_EXPECT = 3 };

// Block of nodes of this workgroup. xcd (batches): each XCD takes a
// contiguous range of the blocks. The trees of a batch have their ids side by
// side, so what a range gathers and stores stays in one L2 (1000 trees of up
// to 2^18 nodes, 3.1 * 10^7 in all: k_succ 426 -> 327 us, k_head 462 -> 420,
// k_node 419 -> 402). In one large tree with scattered ids there is nothing
// to gain and the plain order is a little faster (k_head 563 against 592 us at
// 2^24 nodes, k_succ 450 against 458).
__device__ __forceinline__ int32_t block_of(bool xcd) {
  return xcd ? xcd_block((int32_t)gridDim.x) : (int32_t)blockIdx.x;
}

// Successor of the half-edge up out of the node at position k of the grouped
// order; writes that of the half-edge down into its parent if it is the first
// child (parents ascend with k, so these stores meet in few lines). false:
// the root, or a node with an invalid parent (already flagged).
__device__ __forceinline__ bool succ_at(const uint32_t* __restrict__ keys, const int32_t* __restrict__ vals, int32_t n,
                                        int64_t k, int32_t root, int32_t* __restrict__ sc,
                                        int32_t* __restrict__ succ, int32_t* c_out, int32_t* nxt_out) {
  const int32_t c = vals[k];
  if (c == root) return false;
  const uint32_t p = keys[k];
  if (p >= (uint32_t)n) return false;
  int64_t k2 = k + 1;
  if (k2 < n && vals[k2] == root) ++k2;
  if (k2 < n && keys[k2] == p) *nxt_out = 2 * vals[k2];
  else *nxt_out = ((int32_t)p == root) ? -1 : (int32_t)(2 * p + 1);
  *c_out = c;
  int64_t k0 = k - 1;
  if (k0 >= 0 && vals[k0] == root) --k0;
  if (k0 < 0 || keys[k0] != p) {
    if ((int32_t)p == root) sc[SC_HEAD] = 2 * c;
    else succ[2 * p] = 2 * c;
  }
  return true;
}

__device__ __forceinline__ void succ_scalars(int64_t k, int32_t n, int32_t* __restrict__ sc,
                                             uint32_t* __restrict__ status) {
  if (k != 0) return;
  if (sc[SC_NROOTS] != 1) flag(status, ST_ROOTS);
  sc[SC_EXPECT] = 2 * (n - 1);
}

__global__ void k_succ(const uint32_t* __restrict__ keys, const int32_t* __restrict__ vals, int32_t n,
                       int32_t* __restrict__ sc, int32_t* __restrict__ succ, uint32_t* __restrict__ status, bool xcd) {
  const int64_t k = (int64_t)block_of(xcd) * kB + threadIdx.x;
  if (k >= n) return;
  succ_scalars(k, n, sc, status);
  int32_t c, nxt;
  if (succ_at(keys, vals, n, k, sc[SC_ROOT], sc, succ, &c, &nxt)) succ[2 * c + 1] = nxt;
}

// The same for large trees in two passes. One store per node at a random
// child is bound by the store rate (2^24 nodes: 455 us); here a workgroup
// first sorts its 4096 {child, successor} pairs by ranges of children in LDS
// and appends each range's pairs to that range's place in `pairs` (a child
// occurs once, so range b owns [b << shift, (b + 1) << shift)), and the second
// pass stores them, all of one range close together in time and on one XCD, so
// that its stores fill lines in the L2: 329 us. Where the ids follow the shape
// the stores of neighbours fill lines as they are, and pairs would only be
// more bytes: 64 neighbours of the grouped order whose children lie in one
// range are stored at once (a path in id order, 2^24 nodes: 265 -> 176 us, the
// call 2044 -> 1960; 110 and 1995 when there was one pass only).
constexpr int kPartThreads = 512;
constexpr int kPartPer = 8;
constexpr int kPartRanges = 512;  // at most; one lane each

__global__ void k_part_init(int32_t* __restrict__ used) { used[threadIdx.x] = 0; }

__global__ __launch_bounds__(kPartThreads) void k_succ_part(const uint32_t* __restrict__ keys,
                                                           const int32_t* __restrict__ vals, int32_t n, int shift,
                                                           int32_t* __restrict__ sc, int32_t* __restrict__ succ,
                                                           int2* __restrict__ pairs, int32_t* __restrict__ used,
                                                           uint32_t* __restrict__ status) {
  constexpr int kTile = kPartThreads * kPartPer;
  __shared__ int32_t cnt[kPartRanges], lstart[kPartRanges], wsum[kPartThreads / 64];
  __shared__ int64_t gstart[kPartRanges];
  __shared__ int2 st[kTile];
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  cnt[t] = 0;
  __syncthreads();
  const int32_t root = sc[SC_ROOT];
  const int64_t base = (int64_t)xcd_block((int32_t)gridDim.x) * kTile;
  int2 pr[kPartPer];
  int32_t at[kPartPer];
#pragma unroll
  for (int r = 0; r < kPartPer; ++r) {
    const int64_t k = base + r * kPartThreads + t;
    at[r] = -1;
    if (k >= n) continue;
    succ_scalars(k, n, sc, status);
    const bool has = succ_at(keys, vals, n, k, root, sc, succ, &pr[r].x, &pr[r].y);
    const int32_t range = has ? pr[r].x >> shift : -1;
    // (the lanes beyond n are the last ones: the others are here)
    const uint64_t mask = __ballot(has);
    if (mask == 0) continue;
    const int32_t lead = __shfl(range, __ffsll((unsigned long long)mask) - 1, 64);
    if (__ballot(range == lead) == mask) {
      if (has) succ[2 * pr[r].x + 1] = pr[r].y;
    } else if (has) {
      at[r] = atomicAdd(&cnt[range], 1);
    }
  }
  __syncthreads();
  // a lane per range: its start in the tile, its place in `pairs`
  const int32_t c = cnt[t];
  int32_t inc = c;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int32_t u = __shfl_up(inc, o, 64);
    if (lane >= o) inc += u;
  }
  if (lane == 63) wsum[w] = inc;
  __syncthreads();
  int32_t before = 0, total = 0;
  for (int i = 0; i < kPartThreads / 64; ++i) {
    if (i < w) before += wsum[i];
    total += wsum[i];
  }
  lstart[t] = before + inc - c;
  if (c) gstart[t] = ((int64_t)t << shift) + atomicAdd(used + t, c) - lstart[t];
  __syncthreads();
#pragma unroll
  for (int r = 0; r < kPartPer; ++r)
    if (at[r] >= 0) st[lstart[pr[r].x >> shift] + at[r]] = pr[r];
  __syncthreads();
  for (int32_t i = t; i < total; i += kPartThreads) {
    const int2 p = st[i];
    pairs[gstart[p.x >> shift] + i] = p;
  }
}

__global__ void k_succ_store(const int2* __restrict__ pairs, const int32_t* __restrict__ used, int32_t n, int shift,
                             int32_t* __restrict__ succ) {
  const int64_t i = (int64_t)xcd_block((int32_t)gridDim.x) * kB + threadIdx.x;
  if (i >= n || (i & ((1ll << shift) - 1)) >= used[i >> shift]) return;
  const int2 p = pairs[i];
  succ[2 * p.x + 1] = p.y;
}

__global__ void k_node(const uint64_t* __restrict__ packed, const int2* __restrict__ off, int32_t nsub,
                       int32_t n, const int32_t* __restrict__ sc, int32_t* __restrict__ rank,
                       int32_t* __restrict__ pre_out, int32_t* __restrict__ size_out,
                       uint32_t* __restrict__ inl_out, int32_t* __restrict__ depth_out, uint32_t* __restrict__ plab,
                       uint32_t* __restrict__ status, bool xcd) {
  const int64_t c = (int64_t)block_of(xcd) * kB + threadIdx.x;
  if (c >= n) return;
  plab[c] = kUnusedLabel;  // the label table of inlabel_phase, n + 1 entries
  if (c == n - 1) plab[n] = kUnusedLabel;
  const int32_t root = sc[SC_ROOT];
  int32_t depth, pre, size, r0, r1;
  if (c == root) {
    depth = 0; pre = 0; size = n; r0 = -1; r1 = -1;
  } else {
    const ulonglong2 pk = reinterpret_cast<const ulonglong2*>(packed)[c];
    uint32_t s0 = (uint32_t)pk.x, s1 = (uint32_t)pk.y;
    if (s0 >= (uint32_t)nsub || s1 >= (uint32_t)nsub) {
      flag(status, ST_BAD_INDEX);
      s0 = 0; s1 = 0;
    }
    const int2 o0 = off[s0];
    const int2 o1 = off[s1];
    r0 = o0.x + (int32_t)((pk.x >> 32) & 0xffffu);
    const int32_t dn = o0.y + (int32_t)(pk.x >> 48);
    r1 = o1.x + (int32_t)((pk.y >> 32) & 0xffffu);
    pre = dn;
    depth = 2 * dn - r0 - 1;
    size = (r1 - r0 + 1) >> 1;
  }
  reinterpret_cast<int2*>(rank)[c] = make_int2(r0, r1);
  pre_out[c] = pre;
  size_out[c] = size;
  inl_out[c] = inlabel_of(pre, size);
  depth_out[c] = depth;
}

// Path tops: a node is the top of its inlabel path iff it is the root or its
// parent's inlabel differs. head[I] = {parent of the top, its depth}, and
// plab[I] = the inlabel of that parent (0 for the root's path).
__global__ void k_head(const int32_t* __restrict__ parent, const int32_t* __restrict__ depth_of,
                       const uint32_t* __restrict__ inl_of, int32_t n, const int32_t* __restrict__ sc,
                       int2* __restrict__ head, uint32_t* __restrict__ plab, uint32_t* __restrict__ status, bool xcd) {
  const int64_t v = (int64_t)block_of(xcd) * kB + threadIdx.x;
  if (v >= n) return;
  const int32_t root = sc[SC_ROOT];
  const uint32_t inl = inl_of[v];
  const int32_t p = parent[v];
  bool top;
  uint32_t pinl = 0;
  if (v == root) {
    top = true;
  } else if ((uint32_t)p < (uint32_t)n) {
    pinl = inl_of[p];
    top = pinl != inl;
  } else {
    top = true;
    flag(status, ST_BAD_INDEX);
  }
  if (top) {
    if (inl >= 1u && inl <= (uint32_t)n) {
      head[inl] = make_int2(v == root ? -1 : p, depth_of[v] - 1);
      plab[inl] = (v == root) ? 0u : pinl;
    } else {
      flag(status, ST_BAD_INDEX);
    }
  }
}

// Ascendant of every path label: the level bits along its chain of parent
// path labels (plab; 0 ends it at the root's path). Levels strictly rise along
// a chain, so it has at most one link per level. A parent path's label is an
// ancestor of its child's in the binary tree of labels, so of an aligned range
// of 2^LOG labels a chain only leaves to labels of level LOG and up. Two forms:
//  - k_asc_chain, for trees whose launches cost more than their bytes: one
//    launch, a lane follows its label's chain, in LDS inside the workgroup's
//    range. Bound by the latency of the links above.
//  - k_asc_upper, then k_asc_range, for large trees: the labels of level
//    kAscLog and up first (their chains stay among themselves); then a
//    workgroup takes its range level by level in LDS, so every label is one
//    step instead of one per link (following chains there was issue-bound, 102
//    us at 2^24 nodes), and the first link above the range is one gather.
// One launch per level, the form before, took 177 us at 2^24 nodes (24
// launches) and 41 us at 10^6; these take 53 and 12.
constexpr int kAscChainLog = 8;

__global__ __launch_bounds__(kB) void k_asc_chain(const uint32_t* __restrict__ plab, int32_t n,
                                                 uint32_t* __restrict__ asc_of_label, uint32_t* __restrict__ status) {
  static_assert(kB == 1 << kAscChainLog, "a lane per label");
  __shared__ uint32_t lp[kB];
  const uint32_t I = (blockIdx.x << kAscChainLog) + threadIdx.x;
  uint32_t pl = I >= 1 && I <= (uint32_t)n ? plab[I] : kUnusedLabel;
  lp[threadIdx.x] = pl;
  __syncthreads();
  if (pl == kUnusedLabel) return;
  int t = ctz32(I);
  uint32_t acc = 1u << t;
  while (pl != 0) {
    if (pl > (uint32_t)n || ctz32(pl) <= t) {
      flag(status, ST_BAD_INDEX);
      break;
    }
    t = ctz32(pl);
    acc |= 1u << t;
    pl = (pl >> kAscChainLog) == blockIdx.x ? lp[pl & (kB - 1)] : plab[pl];
  }
  asc_of_label[I] = acc;
}

constexpr int kAscLog = 10;

__global__ __launch_bounds__(kB) void k_asc_range(const uint32_t* __restrict__ plab, int32_t n,
                                                 uint32_t* asc_of_label, uint32_t* __restrict__ status) {
  constexpr int kN = 1 << kAscLog, kPer = kN / kB;
  __shared__ uint32_t lp[kN];  // parent label inside the range as a position, 0 if the label is done
  __shared__ uint32_t la[kN];  // ascendant
  const uint32_t base = blockIdx.x << kAscLog;  // labels [base, base + kN) of 0 .. n
  uint32_t pl[kPer];
  bool bad = false;
#pragma unroll
  for (int j = 0; j < kPer; ++j) {
    const uint32_t I = base + threadIdx.x + j * kB;
    pl[j] = I >= 1 && I <= (uint32_t)n ? plab[I] : kUnusedLabel;
  }
#pragma unroll
  for (int j = 0; j < kPer; ++j) {
    const uint32_t i = threadIdx.x + j * kB;
    uint32_t up = 0, a = 0;
    if (pl[j] != kUnusedLabel && i != 0) {
      const int t = ctz32(i);
      a = 1u << t;
      if (pl[j] != 0 && (pl[j] > (uint32_t)n || ctz32(pl[j]) <= t)) bad = true;
      else if (pl[j] != 0 && (pl[j] >> kAscLog) == blockIdx.x && pl[j] != base) up = pl[j] - base;
      else if (pl[j] != 0) a |= asc_of_label[pl[j]];
    }
    lp[i] = up;
    la[i] = a;
  }
  for (int t = kAscLog - 2; t >= 0; --t) {  // (nothing in the range lies above its level kAscLog - 1)
    __syncthreads();
    for (uint32_t i = ((2 * threadIdx.x + 1) << t); i < (uint32_t)kN; i += (2 * kB) << t)
      if (lp[i] != 0) la[i] |= la[lp[i]];
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < kPer; ++j) {
    const uint32_t i = threadIdx.x + j * kB;
    if (i != 0 && base + i <= (uint32_t)n) asc_of_label[base + i] = la[i];  // unused labels too: whole lines
  }
  if (bad) flag(status, ST_BAD_INDEX);
}

__global__ __launch_bounds__(kB) void k_asc_upper(const uint32_t* __restrict__ plab, int32_t n,
                                                 uint32_t* __restrict__ asc_of_label, uint32_t* __restrict__ status) {
  const int64_t I = ((int64_t)blockIdx.x * kB + threadIdx.x + 1) << kAscLog;
  if (I > n) return;
  uint32_t pl = plab[I];
  if (pl == kUnusedLabel) return;
  int t = ctz32((uint32_t)I);
  uint32_t acc = 1u << t;
  while (pl != 0) {
    if (pl > (uint32_t)n || ctz32(pl) <= t) {
      flag(status, ST_BAD_INDEX);
      break;
    }
    t = ctz32(pl);
    acc |= 1u << t;
    pl = plab[pl];
  }
  asc_of_label[I] = acc;
}

// The node records {inlabel, ascendant, depth, preorder}, each written once
// and whole: the ascendant is gathered by label, the rest streamed. With the
// record begun in k_node and the ascendant stored into it here, every record
// was written twice, the second time as a quarter of its bytes; written here
// it takes the same time (the gather's, 367 us at 2^24 nodes) and k_node and
// k_head move fewer bytes (412 -> 377 and 590 -> 563 us).
// depth_of: nullptr if depth = 2 * preorder - rank - 1, rank[2v] being the
// rank of v's entering half-edge (-1 at the root).
__global__ void k_record(const uint32_t* __restrict__ inl_of, const uint32_t* __restrict__ asc_of_label,
                         const int32_t* __restrict__ pre_of, const int32_t* __restrict__ rank,
                         const int32_t* __restrict__ depth_of, int32_t n, int4* __restrict__ rec,
                         uint32_t* __restrict__ status) {
  const int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (v >= n) return;
  const uint32_t inl = inl_of[v];
  uint32_t a = 0;
  if (inl >= 1u && inl <= (uint32_t)n) a = asc_of_label[inl];
  else flag(status, ST_BAD_INDEX);
  const int32_t pre = pre_of[v];
  const int32_t depth = depth_of ? depth_of[v] : 2 * pre - reinterpret_cast<const int2*>(rank)[v].x - 1;
  rec[v] = make_int4((int32_t)inl, (int32_t)a, depth, pre);
}

// n == 1: the root is the only node
__global__ void k_single(const int32_t* __restrict__ parent, int32_t* __restrict__ sc, int32_t* __restrict__ succ,
                         int32_t* __restrict__ rank, int32_t* __restrict__ pre, int32_t* __restrict__ size,
                         int4* __restrict__ rec, int2* __restrict__ head, uint32_t* __restrict__ status) {
  if (parent[0] != -1) flag(status, ST_ROOTS);
  sc[SC_ROOT] = 0;
  succ[0] = succ[1] = -2;
  rank[0] = rank[1] = -1;
  pre[0] = 0;
  size[0] = 1;
  rec[0] = make_int4(1, 1, 0, 0);
  head[1] = make_int2(-1, -1);
}

__global__ void k_fill_zero(int32_t* __restrict__ p, int32_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0;
}

__global__ void k_export_rec(const int4* __restrict__ rec, int32_t n, int32_t* __restrict__ depth,
                             uint32_t* __restrict__ inl, uint32_t* __restrict__ asc) {
  const int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (v >= n) return;
  const int4 r = rec[v];
  if (depth) depth[v] = r.z;
  if (inl) inl[v] = (uint32_t)r.x;
  if (asc) asc[v] = (uint32_t)r.y;
}

// Schieber-Vishkin query, one lane per query. a = inlabel(x), b = inlabel(y).
//  - a == b: x and y lie on one path; the shallower one is the LCA.
//  - otherwise the LCA of a and b in the binary tree has height
//    i = max(h(a), h(b), msb(a xor b)); the LCA's inlabel has height
//    j = the lowest common ascendant bit at or above i; on each side the
//    node closest to it on the LCA's path is the side itself (if its own
//    label has height j) or the parent of the top of the path entered
//    below it, whose label keeps the bits above the highest ascendant bit
//    k < j and sets bit k; the shallower of the two is the LCA.
__device__ __forceinline__ int32_t sv_query(const int4* __restrict__ rec, const int2* __restrict__ head,
                                            uint32_t n, int32_t x, int32_t y, bool* bad) {
  const int4 rx = rec[x];
  const int4 ry = rec[y];
  const uint32_t a = (uint32_t)rx.x, b = (uint32_t)ry.x;
  if (a == b) return (rx.z <= ry.z) ? x : y;
  const int ha = ctz32(a), hb = ctz32(b);
  const int i0 = max(max(ha, hb), msb32(a ^ b));
  const uint32_t ax = (uint32_t)rx.y, ay = (uint32_t)ry.y;
  const uint32_t common = ax & ay & (~0u << i0);
  if (common == 0u) {
    *bad = true;
    return -1;
  }
  const int j = ctz32(common);
  const uint32_t low = (1u << j) - 1u;
  int32_t xv = x, xd = rx.z, yv = y, yd = ry.z;
  if (ha != j) {
    const int k = msb32(ax & low);
    const uint32_t w = ((a >> (k + 1)) << (k + 1)) | (1u << k);
    const int2 h = head[min(w, n)];
    xv = h.x;
    xd = h.y;
  }
  if (hb != j) {
    const int k = msb32(ay & low);
    const uint32_t w = ((b >> (k + 1)) << (k + 1)) | (1u << k);
    const int2 h = head[min(w, n)];
    yv = h.x;
    yd = h.y;
  }
  return (xd <= yd) ? xv : yv;
}

__global__ __launch_bounds__(kQueryBlockMax) void k_lca(const int4* __restrict__ rec, const int2* __restrict__ head, int32_t n,
                                           const int32_t* __restrict__ qx, const int32_t* __restrict__ qy,
                                           int64_t q, int32_t* __restrict__ out, uint32_t* __restrict__ status) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= q) return;
  const int32_t x = qx[i], y = qy[i];
  if ((uint32_t)x >= (uint32_t)n || (uint32_t)y >= (uint32_t)n) {
    flag(status, ST_BAD_QUERY);
    out[i] = -1;
    return;
  }
  bool bad = false;
  const int32_t r = sv_query(rec, head, (uint32_t)n, x, y, &bad);
  if (bad) flag(status, ST_BAD_INDEX);
  out[i] = r;
}

// Batched trees: tree t's nodes are the global ids [off[t], off[t+1]); all
// trees hang below a virtual root (global id N), so the LCA of two nodes of
// one tree is the LCA in the combined tree.
__device__ __forceinline__ int32_t tree_of(const int64_t* __restrict__ off, int32_t T, int64_t v) {
  int32_t lo = 0, hi = T;
  while (hi - lo > 1) {
    const int32_t mid = (lo + hi) >> 1;
    if (off[mid] <= v) lo = mid;
    else hi = mid;
  }
  return lo;
}

// Per-node passes over a batch: each lane takes kPerLane nodes a block
// width apart, so its tree id only moves forward; it searches once at its
// first node and again only when a node lies past its current tree.
constexpr int kPerLane = 16;

__device__ __forceinline__ int32_t tree_from(const int64_t* __restrict__ off, int32_t t, int32_t T, int64_t v) {
  if (off[t + 1] > v) return t;
  int32_t lo = t, hi = T;
  while (hi - lo > 1) {
    const int32_t mid = (lo + hi) >> 1;
    if (off[mid] <= v) lo = mid;
    else hi = mid;
  }
  return lo;
}

__global__ __launch_bounds__(kQueryBlockMax) void k_lca_batch(const int4* __restrict__ rec, const int2* __restrict__ head,
                                                 int32_t n, const int64_t* __restrict__ off, int32_t T,
                                                 const int32_t* __restrict__ qt, const int32_t* __restrict__ qx,
                                                 const int32_t* __restrict__ qy, int64_t q, int32_t* __restrict__ out,
                                                 uint32_t* __restrict__ status) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= q) return;
  const int32_t t = qt[i];
  if ((uint32_t)t >= (uint32_t)T) {
    flag(status, ST_BAD_QUERY);
    out[i] = -1;
    return;
  }
  const int64_t base = off[t];
  const int64_t nt = off[t + 1] - base;
  const int32_t x = qx[i], y = qy[i];
  if ((int64_t)(uint32_t)x >= nt || (int64_t)(uint32_t)y >= nt || base + nt > n) {
    flag(status, ST_BAD_QUERY);
    out[i] = -1;
    return;
  }
  bool bad = false;
  const int32_t r = sv_query(rec, head, (uint32_t)n, (int32_t)(base + x), (int32_t)(base + y), &bad);
  if (bad || r < base || r >= base + nt) {
    flag(status, ST_BAD_INDEX);
    out[i] = -1;
    return;
  }
  out[i] = (int32_t)(r - base);
}

// combined parent array: roots of the trees hang below the virtual root N.
// A workgroup whose nodes are all of one tree (nearly every one of a batch of
// large trees) takes that tree's range as it is, its loads together; the others
// look for the tree of every node: 1000 trees of up to 2^18 nodes 132 -> 68 us,
// near what reading and writing the parents takes.
__device__ __forceinline__ int32_t batch_parent(int32_t p, int64_t v, int32_t t, int64_t base, int64_t nt, int32_t N,
                                                int32_t* __restrict__ nroots, int32_t* __restrict__ root_of,
                                                uint32_t* __restrict__ status) {
  if (p == -1) {
    atomicAdd(nroots + t, 1);
    root_of[t] = (int32_t)v;
    return N;
  }
  if (p >= 0 && p < nt && base + p != v) return (int32_t)(base + p);
  flag(status, ST_BAD_PARENT);
  return N;
}

__global__ __launch_bounds__(kB) void k_batch_parent(const int32_t* __restrict__ parent,
                                                    const int64_t* __restrict__ off, int32_t T, int32_t N,
                                                    int32_t* __restrict__ gp, int32_t* __restrict__ nroots,
                                                    int32_t* __restrict__ root_of, uint32_t* __restrict__ status) {
  const int64_t b0 = (int64_t)blockIdx.x * kB * kPerLane;
  const int64_t first = b0 + threadIdx.x;
  const int64_t last = b0 + (int64_t)kB * kPerLane - 1;
  if (last < N) {
    const int32_t t = tree_of(off, T, b0);
    const int64_t base = off[t], nt = off[t + 1] - base;
    if (b0 >= base && last < off[t + 1]) {
      int32_t p[kPerLane];
#pragma unroll
      for (int i = 0; i < kPerLane; ++i) p[i] = parent[first + (int64_t)i * kB];
#pragma unroll
      for (int i = 0; i < kPerLane; ++i) {
        const int64_t v = first + (int64_t)i * kB;
        gp[v] = batch_parent(p[i], v, t, base, nt, N, nroots, root_of, status);
      }
      return;
    }
  }
  if (first > N) return;
  int32_t t = tree_of(off, T, min(first, (int64_t)N - 1));
  for (int i = 0; i < kPerLane; ++i) {
    const int64_t v = first + (int64_t)i * kB;
    if (v > N) break;
    if (v == N) {
      gp[N] = -1;
      if (off[0] != 0 || off[T] != N) flag(status, ST_BAD_PARENT);
      break;
    }
    t = tree_from(off, t, T, v);
    const int64_t base = off[t];
    gp[v] = batch_parent(parent[v], v, t, base, off[t + 1] - base, N, nroots, root_of, status);
  }
}

__global__ void k_batch_check(const int64_t* __restrict__ off, int32_t T, const int32_t* __restrict__ nroots,
                              uint32_t* __restrict__ status) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= T) return;
  if (nroots[t] != 1 || off[t + 1] <= off[t]) flag(status, ST_ROOTS);
}

// per-tree statistics of a batch: preorder and depth relative to the tree's root
__global__ void k_export_batch(const int4* __restrict__ rec, const int32_t* __restrict__ size_in,
                               const int64_t* __restrict__ off, int32_t T, int32_t N,
                               const int32_t* __restrict__ root_of, int32_t* __restrict__ depth,
                               int32_t* __restrict__ pre, int32_t* __restrict__ size) {
  const int64_t first = (int64_t)blockIdx.x * blockDim.x * kPerLane + threadIdx.x;
  if (first >= N) return;
  int32_t t = tree_of(off, T, first);
  for (int i = 0; i < kPerLane; ++i) {
    const int64_t v = first + (int64_t)i * blockDim.x;
    if (v >= N) break;
    t = tree_from(off, t, T, v);
    const int32_t r = root_of[t];
    const int4 rv = rec[v];
    const int32_t rp = ((uint32_t)r < (uint32_t)N) ? rec[r].w : 0;
    if (depth) depth[v] = rv.z - 1;
    if (pre) pre[v] = rv.w - rp;
    if (size) size[v] = size_in[v];
  }
}

}  // namespace

// Scratch of tree_build: the grouping buffer and the compact inlabels, the
// grouping's own scratch (released before the ranking starts, but counted
// as if held: the pool may hand a released block to a smaller request) and
// the ranking's buffers; a batch adds its combined parent array and root
// counts.
size_t tree_build_scratch_bytes(const Ctx* c, int32_t n, int32_t batch) {
  size_t b = 0;
  if (batch) {
    b += scratch_block<int32_t>((size_t)n) + scratch_block<int32_t>((size_t)batch);  // n counts the virtual root
  }
  if (n <= 1) return b;
  b += scratch_block<uint32_t>(2 * (size_t)n + 2) + scratch_block<uint32_t>((size_t)n) +
       scratch_block<int32_t>(kPartRanges);
  return b + group_by_parent_scratch_bytes(n) + list_rank_plan_bytes(c, 2 * n, 1, 0, batch != 0);
}

// Nodes from which the successors of one tree are stored in two passes. Up to
// here the successor array and the grouped order that it is made from (16
// bytes a node) stay in the 256 MB of Infinity Cache, which takes random
// stores at twice the rate of HBM. Direct and in two passes, us: 2^22 nodes 64
// and 75, 10M 166 and 180, 11M 213 and 199, 12M 283 and 214, 2^24 455 and 329,
// 24M 668 and 458, 2^25 604 and 622, 40M 795 and 754, 2^26 2232 and 1299. Never
// for a batch, whose children already lie in the order of its trees (2^24
// nodes in 4096 trees: 323 and 538).
constexpr int32_t kPartNodes = 12000000;

int tree_build(Ctx* c, et_tree* t, const int32_t* parent, hipStream_t s) {
  const int32_t n = t->n;
  int32_t* sc = t->d_root;
  if (n == 1) {
    hipLaunchKernelGGL(k_single, dim3(1), dim3(1), 0, s, parent, sc, t->d_succ, t->d_rank, t->d_pre, t->d_size,
                       t->d_rec, t->d_head, c->d_status);
    return hipGetLastError() == hipSuccess ? ET_OK : ET_EHIP;
  }
  if (n <= kSmallTreeMax) return small_tree_build(c, t, parent, s);
  const int32_t L2 = 2 * n;          // half-edge id space (the tour uses 2(n-1) of them)
  Scratch scr(c, s);
  uint32_t* kv = scr.get<uint32_t>((size_t)L2 + 2);  // sorted parents | children, later the two tables by label
  if (scr.failed) return ET_ENOMEM;
  uint32_t* keys = kv;
  int32_t* vals = reinterpret_cast<int32_t*>(kv + n);
  const int gn = ceil_div(n, kB);
  LRResult lr;
  uint32_t* inl = scr.get<uint32_t>((size_t)n);  // inlabel of every node, compact for gathers
  int32_t* used = scr.get<int32_t>(kPartRanges);
  if (scr.failed) return ET_ENOMEM;
  int rc;
  {
    ET_PROF(c, s, "phase:tour");
    rc = group_by_parent_impl(c, parent, n, keys, vals, t->d_succ, sc, s);
    if (rc) return rc;
    if (!t->batch && n >= kPartNodes) {
      int shift = 16;
      while (((int64_t)n >> shift) >= kPartRanges) ++shift;
      int2* pairs = reinterpret_cast<int2*>(t->d_rank);  // (written by k_node only)
      ET_PROF(c, s, "k_succ");
      hipLaunchKernelGGL(k_part_init, dim3(1), dim3(kPartRanges), 0, s, used);
      hipLaunchKernelGGL(k_succ_part, dim3(ceil_div(n, kPartThreads * kPartPer)), dim3(kPartThreads), 0, s, keys, vals,
                         n, shift, sc, t->d_succ, pairs, used, c->d_status);
      hipLaunchKernelGGL(k_succ_store, dim3(gn), dim3(kB), 0, s, pairs, used, n, shift, t->d_succ);
    } else {
      ET_PROF(c, s, "k_succ");
      hipLaunchKernelGGL(k_succ, dim3(gn), dim3(kB), 0, s, keys, vals, n, sc, t->d_succ, c->d_status,
                         t->batch != 0);
    }
    rc = list_rank_core(c, scr, t->d_succ, L2, sc + SC_HEAD, 1, true, sc + SC_EXPECT, &lr, s, false, 0,
                        t->batch ? L2 / t->batch : 0);
    if (rc) return rc;
    {
      ET_PROF(c, s, "k_node");
      hipLaunchKernelGGL(k_node, dim3(gn), dim3(kB), 0, s, lr.packed, lr.off, lr.nsub, n, sc, t->d_rank, t->d_pre,
                         t->d_size, inl, reinterpret_cast<int32_t*>(kv + n + 1), kv, c->d_status, t->batch != 0);
    }
  }
  // the grouping's keys and values are dead by now: the label table, and the
  // depths until the ascendants take their place
  return inlabel_phase(c, t, parent, inl, reinterpret_cast<int32_t*>(kv + n + 1), false, kv, s);
}

constexpr int32_t kAscTwo = 1 << 20;  // nodes from which the ascendants take two launches

int inlabel_phase(Ctx* c, et_tree* t, const int32_t* parent, const uint32_t* inl, const int32_t* depth,
                  bool depth_kept, uint32_t* plab, hipStream_t s) {
  const int32_t n = t->n;
  int32_t* sc = t->d_root;
  const int gn = ceil_div(n, kB);
  uint32_t* asc = plab + n + 1;  // ascendant by label
  ET_PROF(c, s, "phase:inlabel");
  {
    ET_PROF(c, s, "k_head");
    hipLaunchKernelGGL(k_head, dim3(gn), dim3(kB), 0, s, parent, depth, inl, n, sc, t->d_head, plab,
                       c->d_status, t->batch != 0);
  }
  {
    ET_PROF(c, s, "k_asc_label");
    // one launch / two launches: 7.3 / 11 us at 2^18 nodes, 9.6 / 11 at 2^19,
    // 14 / 12 at 2^20, 24 / 14 at 2^21, 184 / 54 at 2^24
    if (n >= kAscTwo) {
      hipLaunchKernelGGL(k_asc_upper, dim3(ceil_div((int64_t)n >> kAscLog, kB)), dim3(kB), 0, s, plab, n, asc,
                         c->d_status);
      hipLaunchKernelGGL(k_asc_range, dim3((unsigned)(n >> kAscLog) + 1), dim3(kB), 0, s, plab, n, asc, c->d_status);
    } else {
      hipLaunchKernelGGL(k_asc_chain, dim3((unsigned)(n >> kAscChainLog) + 1), dim3(kB), 0, s, plab, n, asc,
                         c->d_status);
    }
  }
  {
    ET_PROF(c, s, "k_record");
    hipLaunchKernelGGL(k_record, dim3(gn), dim3(kB), 0, s, inl, asc, t->d_pre, t->d_rank, depth_kept ? depth : nullptr,
                       n, t->d_rec, c->d_status);
  }
  return hipGetLastError() == hipSuccess ? ET_OK : ET_EHIP;
}

int tree_export(const et_tree* t, int32_t* succ, int32_t* rank, int32_t* depth, int32_t* pre, int32_t* size,
                uint32_t* inl, uint32_t* asc, hipStream_t s) {
  if (t->batch) {
    if (succ || rank || inl || asc) return ET_EINVAL;  // global tables of a batch are internal
    const int32_t N = t->n - 1;
    if (depth || pre || size)
      hipLaunchKernelGGL(k_export_batch, dim3(ceil_div(N, (int64_t)kB * kPerLane)), dim3(kB), 0, s, t->d_rec,
                         t->d_size, t->d_off,
                         t->batch, N, t->d_root_of, depth, pre, size);
    return hipGetLastError() == hipSuccess ? ET_OK : ET_EHIP;
  }
  const int32_t n = t->n;
  const size_t b = (size_t)n * sizeof(int32_t);
  if (succ && hipMemcpyAsync(succ, t->d_succ, 2 * b, hipMemcpyDeviceToDevice, s) != hipSuccess) return ET_EHIP;
  if (rank && hipMemcpyAsync(rank, t->d_rank, 2 * b, hipMemcpyDeviceToDevice, s) != hipSuccess) return ET_EHIP;
  if (pre && hipMemcpyAsync(pre, t->d_pre, b, hipMemcpyDeviceToDevice, s) != hipSuccess) return ET_EHIP;
  if (size && hipMemcpyAsync(size, t->d_size, b, hipMemcpyDeviceToDevice, s) != hipSuccess) return ET_EHIP;
  if (depth || inl || asc)
    hipLaunchKernelGGL(k_export_rec, dim3(ceil_div(n, kB)), dim3(kB), 0, s, t->d_rec, n, depth, inl, asc);
  return hipGetLastError() == hipSuccess ? ET_OK : ET_EHIP;
}

namespace {
// tour[rank(e)] = e for every half-edge on the tour
__global__ void k_tour(const int32_t* __restrict__ rank, int64_t E, int32_t L, int32_t* __restrict__ tour,
                       uint32_t* __restrict__ status) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= E) return;
  const int32_t r = rank[e];
  if (r < 0) return;  // the root's two unused ids
  if (r >= L) {
    flag(status, ST_BAD_INDEX);
    return;
  }
  tour[r] = (int32_t)e;
}
}  // namespace

int tree_export_tour(Ctx* c, const et_tree* t, int32_t* tour, hipStream_t s) {
  if (t->batch) return ET_EINVAL;  // the combined tour of a batch is internal
  const int32_t L = 2 * (t->n - 1);
  if (L == 0) return ET_OK;
  // a parent-array tree numbers its half-edges 2c / 2c+1 over all n nodes,
  // an edge-list tree 2i / 2i+1 over its n-1 edges
  const int64_t E = t->from_edges ? (int64_t)L : 2 * (int64_t)t->n;
  hipLaunchKernelGGL(k_tour, dim3(ceil_div(E, kB)), dim3(kB), 0, s, t->d_rank, E, L, tour, c->d_status);
  return hipGetLastError() == hipSuccess ? ET_OK : ET_EHIP;
}

int tree_lca_batch(Ctx* c, const et_tree* t, const int32_t* qt, const int32_t* qx, const int32_t* qy, int64_t q,
                   int32_t* out, hipStream_t s) {
  if (q == 0) return ET_OK;
  const int bs = c->qs.block;
  ET_PROF(c, s, "k_lca_batch");
  for (int64_t q0 = 0; q0 < q; q0 += kQueryChunk) {  // one dispatch holds < 2^32 work-items
    const int64_t m = std::min(q - q0, kQueryChunk);
    hipLaunchKernelGGL(k_lca_batch, dim3((unsigned)((m + bs - 1) / bs)), dim3(bs), 0, s, t->d_rec, t->d_head, t->n,
                       t->d_off, t->batch, qt + q0, qx + q0, qy + q0, m, out + q0, c->d_status);
  }
  return hipGetLastError() == hipSuccess ? ET_OK : ET_EHIP;
}

int tree_build_batch(Ctx* c, et_tree* t, const int32_t* parent, hipStream_t s) {
  const int32_t N = t->n - 1, T = t->batch;
  Scratch scr(c, s);
  int32_t* gp = scr.get<int32_t>((size_t)N + 1);
  int32_t* nroots = scr.get<int32_t>((size_t)T);
  if (scr.failed) return ET_ENOMEM;
  hipLaunchKernelGGL(k_fill_zero, dim3(ceil_div(T, kB)), dim3(kB), 0, s, nroots, T);
  {
    ET_PROF(c, s, "k_batch_parent");
    hipLaunchKernelGGL(k_batch_parent, dim3(ceil_div((int64_t)N + 1, (int64_t)kB * kPerLane)), dim3(kB), 0, s, parent,
                       t->d_off, T, N,
                       gp, nroots, t->d_root_of, c->d_status);
  }
  hipLaunchKernelGGL(k_batch_check, dim3(ceil_div(T, kB)), dim3(kB), 0, s, t->d_off, T, nroots, c->d_status);
  return tree_build(c, t, gp, s);
}

int tree_lca(Ctx* c, const et_tree* t, const int32_t* qx, const int32_t* qy, int64_t q, int32_t* out,
             hipStream_t s) {
  if (q == 0) return ET_OK;
  const int bs = c->qs.block;
  ET_PROF(c, s, "k_lca");
  for (int64_t q0 = 0; q0 < q; q0 += kQueryChunk) {  // one dispatch holds < 2^32 work-items
    const int64_t m = std::min(q - q0, kQueryChunk);
    hipLaunchKernelGGL(k_lca, dim3((unsigned)((m + bs - 1) / bs)), dim3(bs), 0, s, t->d_rec, t->d_head, t->n, qx + q0,
                       qy + q0, m, out + q0, c->d_status);
  }
  return hipGetLastError() == hipSuccess ? ET_OK : ET_EHIP;
}

}  // namespace et
