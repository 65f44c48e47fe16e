// List ranking and list prefix sums (Section 2.2).
//
// The paper ranks the tour with the GPU sublist algorithm of Wei and JaJa
// rather than pointer jumping. This is an MI355X design of the same idea:
//
//  level 1  Splitters: one pseudo-randomly placed element in every chunk of
//           K consecutive ids (plus every list head) starts a sublist. A
//           wavefront owns a contiguous range of sublist ids; its 64 lanes
//           each walk one sublist, and a lane whose sublist ends takes the
//           next id of the wave's range (ballot + popcount, no atomics), so
//           lanes stay busy even though sublist lengths are geometric. Each
//           visited element gets one 8-byte record {sublist, local rank,
//           local down-count}; each sublist gets {next sublist, length,
//           down-count}. Sublists longer than 65535 elements are split into
//           continuation sublists so the local fields fit 16 bits.
//  level k  The list of sublists is ranked the same way with the sublist
//           lengths as weights, until it has at most kLdsMax elements.
//  final    One workgroup ranks the last list in LDS, again by sublists (a
//           lane walks each, then predecessor pointers jump over them), and
//           checks that every used element is reached from a head; offsets
//           are then pushed back down the levels.
// A list of at most kLdsDirect elements goes to the final level at once.
//
// Every walk is bounded and every gathered index is range checked, so a
// malformed list (a cycle, a shared successor, an id out of range) sets a
// status bit instead of faulting or hanging.
#include "et_internal.hpp"

namespace et {
namespace {

constexpr int kCap = 65535;        // level-1 sublist length cap (16-bit local fields)
constexpr int kLdsMax = 12288;     // elements the final LDS kernel ranks (10 bytes of LDS each)
constexpr int kLdsDirect = 8192;   // elements of a list that goes to it whole
constexpr int kLdsHeads = 1024;    // heads it takes; beyond, the final level is k_final_lds
constexpr int kLdsMaxHeads = 4096; // elements k_final_lds ranks
constexpr int kWalkThreads = 256;
constexpr uint32_t kSalt = 0x9e3779b9u;

__device__ __forceinline__ bool is_splitter(int32_t e, int ks, uint32_t salt) {
  const uint32_t m = (1u << ks) - 1u;
  return ((uint32_t)e & m) == (mix32(((uint32_t)e >> ks) ^ salt) & m);
}

__device__ __forceinline__ int32_t splitter_of_chunk(int32_t i, int ks, uint32_t salt) {
  const uint32_t m = (1u << ks) - 1u;
  return (int32_t)(((uint32_t)i << ks) + (mix32((uint32_t)i ^ salt) & m));
}

__global__ void k_set_scalar(int32_t* __restrict__ p, int32_t v) { *p = v; }

// The second channel (down counts of a tour, or element weights) adds in
// 32-bit two's complement: weight sums wrap instead of overflowing.
__device__ __forceinline__ int32_t wadd(int32_t a, int32_t b) { return (int32_t)((uint32_t)a + (uint32_t)b); }
__device__ __forceinline__ int32_t wsub(int32_t a, int32_t b) { return (int32_t)((uint32_t)a - (uint32_t)b); }

// start of a ranking: the continuation counter and the counts of reached and
// of used elements at zero, the continuation records [begin, end) marked unused
__global__ void k_lr_init(int32_t* __restrict__ ctr, int4* __restrict__ rec, int32_t begin, int32_t end) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i == 0) {
    ctr[0] = 0;
    ctr[1] = 0;
    ctr[2] = 0;
  }
  if (begin + i < end) rec[begin + i] = make_int4(-3, 0, 0, 0);
}

// ------------------------------------------------------------------ level 1
// TREE: even ids count as "down" (tree half-edges) and a leaf's two
// half-edges share one load and one store. W > 0: succ holds {successor,
// weight} pairs (one 8-byte load per step) and the weights are summed
// instead (wrapping in 32 bits); the inclusive local sum does not fit the
// 16-bit field, so the record is {sublist, local sum} (W = 1, 8 bytes) or,
// when ranks are wanted too, {sublist | local rank << 32, local sum}
// (W = 2, 16 bytes).
// block: the workgroup's place in the order of the sublists.
template <bool TREE, int W>
__device__ __forceinline__ void walk1_body(
    const int32_t* __restrict__ succ, int32_t L, const int32_t* __restrict__ heads, int32_t H, int ks,
    uint32_t salt, int32_t S, int32_t per_wave, uint64_t* __restrict__ packed, int4* __restrict__ srec,
    int32_t* __restrict__ cont_ctr, int32_t cont_base, int32_t cont_max, bool empty_ok,
    uint32_t* __restrict__ status, int32_t block) {
  constexpr int kStride = W > 0 ? 2 : 1;  // int32 words per element in succ
  const int64_t wave = ((int64_t)block * blockDim.x + threadIdx.x) >> 6;
  const int32_t total = S + H;
  int32_t next_id = (int32_t)min<int64_t>(wave * per_wave, total);
  const int32_t end_id = (int32_t)min<int64_t>((int64_t)next_id + per_wave, total);
  int32_t cur = -1, sub = 0, j = 0, d = 0;
  int64_t steps = 0;
  for (;;) {
    const bool idle = cur < 0;
    const uint64_t idle_mask = __ballot(idle);
    if (idle_mask != 0ull && next_id < end_id) {
      if (idle) {
        const int32_t id = next_id + __popcll(idle_mask & lanemask_lt());
        if (id < end_id) {
          if (id < S) {
            const int32_t e = splitter_of_chunk(id, ks, salt);
            if (e >= L || succ[kStride * (int64_t)e] == -2) {
              srec[id] = make_int4(-3, 0, 0, 0);  // no element here
            } else {
              cur = e; sub = id; j = 0; d = 0;
            }
          } else {
            const int32_t e = heads[id - S];
            if (e == -1 && empty_ok) {
              srec[id] = make_int4(-1, 0, 0, 0);  // an empty list
            } else if (e < 0 || e >= L || succ[kStride * (int64_t)e] == -2) {
              flag(status, ST_BAD_HEAD);
              srec[id] = make_int4(-1, 0, 0, 0);
            } else if (is_splitter(e, ks, salt)) {
              srec[id] = make_int4(e >> ks, 0, 0, 0);  // the head's own chunk splitter walks it
            } else {
              cur = e; sub = id; j = 0; d = 0;
            }
          }
        }
      }
      next_id = min(end_id, next_id + (int32_t)__popcll(idle_mask));
    }
    if (__ballot(cur >= 0) == 0ull) {
      if (next_id >= end_id) break;
      continue;
    }
    if (cur >= 0) {
      int32_t nx;
      bool pair = false;
      if (TREE && (cur & 1) == 0) {
        // A leaf's down half-edge 2c is followed by its own up half-edge
        // 2c+1; both successors share one aligned 8-byte load and both
        // records one 16-byte store, unless 2c+1 starts a sublist or the
        // pair would reach the length cap.
        const int2 sp = *reinterpret_cast<const int2*>(succ + cur);
        nx = sp.x;
        if (nx == cur + 1 && j + 2 < kCap && !is_splitter(cur + 1, ks, salt)) {
          ++d;
          const uint64_t lo = (uint64_t)(uint32_t)sub | ((uint64_t)(uint32_t)d << 48);
          *reinterpret_cast<ulonglong2*>(packed + cur) =
              make_ulonglong2(lo | ((uint64_t)(uint32_t)j << 32), lo | ((uint64_t)(uint32_t)(j + 1) << 32));
          j += 2;
          steps += 2;
          nx = sp.y;
          pair = true;
        }
      } else if (W > 0) {
        const int2 sw = *reinterpret_cast<const int2*>(succ + 2 * (int64_t)cur);
        nx = sw.x;
        d = wadd(d, sw.y);
        if (W == 1)
          packed[cur] = (uint64_t)(uint32_t)sub | ((uint64_t)(uint32_t)d << 32);
        else
          *reinterpret_cast<ulonglong2*>(packed + 2 * (int64_t)cur) =
              make_ulonglong2((uint64_t)(uint32_t)sub | ((uint64_t)(uint32_t)j << 32), (uint64_t)(uint32_t)d);
        ++j;
        ++steps;
      } else {
        nx = succ[cur];
      }
      if (!pair && W == 0) {
        if (TREE) d += ((cur & 1) == 0);
        packed[cur] = (uint64_t)(uint32_t)sub | ((uint64_t)(uint32_t)j << 32) | ((uint64_t)(uint32_t)d << 48);
        ++j;
        ++steps;
      }
      bool stop = true;
      int32_t link = -1;
      if (nx == -1) {
        link = -1;
      } else if (nx < 0 || nx >= L) {
        flag(status, ST_BAD_SUCC);
      } else if (is_splitter(nx, ks, salt)) {
        link = nx >> ks;
      } else if (steps > L) {
        flag(status, ST_OVERFLOW);
      } else if (j == kCap) {
        const int32_t nid = atomicAdd(cont_ctr, 1);
        if (nid >= cont_max) {
          flag(status, ST_OVERFLOW);
        } else {
          srec[sub] = make_int4(cont_base + nid, j, d, 0);
          sub = cont_base + nid;
          j = 0;
          d = 0;
          stop = false;
        }
      } else {
        stop = false;
      }
      if (stop) {
        srec[sub] = make_int4(link, j, d, 0);
        cur = -1;
      } else {
        cur = nx;
      }
    }
  }
}

// Bound by random accesses, a load and a store per element (2^25 elements 1.2
// ms, 28 G/s; a random tree's 2^25 half-edges 930 us). Fewer wavefronts at a
// time are slower, and so are shorter runs of sublists per wavefront, unless
// the lists are local (see list_rank_launch): then xcd hands each XCD a
// contiguous range of the sublists.
template <bool TREE>
__global__ __launch_bounds__(kWalkThreads) void k_walk1(
    const int32_t* __restrict__ succ, int32_t L, const int32_t* __restrict__ heads, int32_t H, int ks,
    uint32_t salt, int32_t S, int32_t per_wave, uint64_t* __restrict__ packed, int4* __restrict__ srec,
    int32_t* __restrict__ cont_ctr, int32_t cont_base, int32_t cont_max, bool empty_ok,
    uint32_t* __restrict__ status, bool xcd) {
  walk1_body<TREE, 0>(succ, L, heads, H, ks, salt, S, per_wave, packed, srec, cont_ctr, cont_base, cont_max,
                      empty_ok, status, xcd ? xcd_block((int32_t)gridDim.x) : (int32_t)blockIdx.x);
}

// the same walk over {successor, weight} pairs, summing the weights; RANK:
// the records keep the local ranks too
template <bool RANK>
__global__ __launch_bounds__(kWalkThreads) void k_walk1w(
    const int32_t* __restrict__ sw, int32_t L, const int32_t* __restrict__ heads, int32_t H, int ks,
    uint32_t salt, int32_t S, int32_t per_wave, uint64_t* __restrict__ packed, int4* __restrict__ srec,
    int32_t* __restrict__ cont_ctr, int32_t cont_base, int32_t cont_max, bool empty_ok,
    uint32_t* __restrict__ status) {
  walk1_body<false, RANK ? 2 : 1>(sw, L, heads, H, ks, salt, S, per_wave, packed, srec, cont_ctr, cont_base,
                                  cont_max, empty_ok, status, (int32_t)blockIdx.x);
}

// ------------------------------------------------------------------ level k >= 2
// Input records rec[e] = {next, len, down}; next == -3 marks an unused element.
// Output per element: el[e] = {sublist, exclusive local len, exclusive local down}.
__global__ __launch_bounds__(kWalkThreads) void k_walkN(
    const int4* __restrict__ rec, int32_t T, int32_t hb, int32_t H, int ks, uint32_t salt, int32_t S,
    int32_t per_wave, int4* __restrict__ el, int4* __restrict__ srec, uint32_t* __restrict__ status) {
  const int64_t wave = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
  const int32_t total = S + H;
  int32_t next_id = (int32_t)min<int64_t>(wave * per_wave, total);
  const int32_t end_id = (int32_t)min<int64_t>((int64_t)next_id + per_wave, total);
  int32_t cur = -1, sub = 0, al = 0, ad = 0;
  int64_t steps = 0;
  for (;;) {
    const bool idle = cur < 0;
    const uint64_t idle_mask = __ballot(idle);
    if (idle_mask != 0ull && next_id < end_id) {
      if (idle) {
        const int32_t id = next_id + __popcll(idle_mask & lanemask_lt());
        if (id < end_id) {
          if (id < S) {
            const int32_t e = splitter_of_chunk(id, ks, salt);
            if (e >= T || rec[e].x == -3) {
              srec[id] = make_int4(-3, 0, 0, 0);
            } else {
              cur = e; sub = id; al = 0; ad = 0;
            }
          } else {
            const int32_t e = hb + (id - S);
            if (e < 0 || e >= T) {
              flag(status, ST_BAD_HEAD);
              srec[id] = make_int4(-1, 0, 0, 0);
            } else if (is_splitter(e, ks, salt)) {
              srec[id] = make_int4(e >> ks, 0, 0, 0);
            } else {
              cur = e; sub = id; al = 0; ad = 0;
            }
          }
        }
      }
      next_id = min(end_id, next_id + (int32_t)__popcll(idle_mask));
    }
    if (__ballot(cur >= 0) == 0ull) {
      if (next_id >= end_id) break;
      continue;
    }
    if (cur >= 0) {
      const int4 r = rec[cur];
      el[cur] = make_int4(sub, al, ad, 0);
      al += r.y;
      ad = wadd(ad, r.z);
      ++steps;
      const int32_t nx = r.x;
      bool stop = true;
      int32_t link = -1;
      if (nx == -1) {
        link = -1;
      } else if (nx < 0 || nx >= T) {
        flag(status, ST_BAD_SUCC);
      } else if (is_splitter(nx, ks, salt)) {
        link = nx >> ks;
      } else if (steps > T) {
        flag(status, ST_OVERFLOW);
      } else {
        stop = false;
      }
      if (stop) {
        srec[sub] = make_int4(link, al, ad, 0);
        cur = -1;
      } else {
        cur = nx;
      }
    }
  }
}

// ------------------------------------------------------------------ final level (LDS)
// Exclusive prefix (len, down) of every element of a short list from its
// list's head, by one workgroup: sublists once more, walked by a lane each at
// LDS latency (60 ns a step, where a step of k_walkN waits for memory: about
// 500 ns), then predecessor pointers jump over the at most 1024 + H sublists.
// Against jumping over every element, limited to 4096, a list of sublists
// needs one k_walkN and k_push_down level less: 10^6-node build 355 -> 345 us.
// Bound by LDS bandwidth: the wavefronts' steps until their longest sublists
// end. 20 us for 2000 elements, 30 for 8000.
//   IN_REC   level records {next, len, down} (next == -3 unused); the heads
//            are the H records from hb on
//   IN_SUCC, IN_PAIR   a whole list, as k_walk1's W = 0 (plain) and W > 0
//            inputs; the level-1 records are then one sublist per element
//            (PAIR2: with the 16-byte records), or, where `rank` is given, the
//            ranks are written themselves
// Elements whose predecessor chain does not start at a head are unreachable
// (malformed input), as are elements that no walk passes.
constexpr int kFinalThreads = 1024;
constexpr int kFinalSub = 2;  // sublists per lane: 1024 by chunks, kLdsHeads by heads
enum { IN_REC, IN_SUCC, IN_PAIR, IN_PAIR2 };

struct RankLds {  // bytes of the dynamic LDS of k_rank_lds
  uint32_t dn, acl, acd, nxt, pred, top, hb, total;
};

__host__ __device__ inline RankLds rank_lds_layout(uint32_t T, uint32_t SM) {
  RankLds l;
  l.dn = 4 * T;
  l.acl = 8 * T;
  l.acd = l.acl + 4 * SM;
  l.hb = l.acd + 4 * SM;
  l.nxt = l.hb + 4 * ((SM + 31) / 32) + 16;
  l.pred = l.nxt + 2 * ((T + 1) & ~1u);
  l.top = l.pred + 2 * ((SM + 1) & ~1u);
  l.total = l.top + 2 * ((SM + 1) & ~1u);
  return l;
}

// smallest spacing that leaves at most 1024 chunks
inline int rank_lds_ks(int32_t T) {
  int ks = 0;
  while (((T + (1 << ks) - 1) >> ks) > 1024) ++ks;
  return ks;
}

// dynamic LDS of k_rank_lds for T elements and H heads
inline uint32_t rank_lds_bytes(int32_t T, int32_t H) {
  const int ks = rank_lds_ks(T);
  return rank_lds_layout((uint32_t)T, (uint32_t)(((T + (1 << ks) - 1) >> ks) + H)).total;
}

template <int IN>
__global__ __launch_bounds__(kFinalThreads) void k_rank_lds(
    const int32_t* __restrict__ in, int32_t T, const int32_t* __restrict__ heads, int32_t hb, int32_t H,
    bool empty_ok, int ks, uint32_t salt, uint64_t* __restrict__ packed, int2* __restrict__ off,
    int32_t* __restrict__ rank, int32_t* __restrict__ reached_out, const int32_t* __restrict__ expected,
    uint32_t* __restrict__ status) {
  // NXT: the next element, kEnd or kUnused, kSplit set if the next element is
  // a splitter (decided here, not in the dependent walk); kWalked | sublist
  // once walked
  constexpr uint32_t kEnd = 0x3fffu, kUnused = 0x3ffeu, kSplit = 0x4000u, kWalked = 0x8000u;
  static_assert(kLdsMax <= 0x3ffe && 1024 + kLdsHeads <= 0x7fff, "the codes of NXT");
  constexpr uint32_t kNone = 0xffffu;
  constexpr bool kLen = IN == IN_REC;                    // element lengths other than 1
  constexpr bool kDn = IN != IN_SUCC;                    // element weights
  extern __shared__ __align__(16) unsigned char lds[];
  const int32_t S = (T + (1 << ks) - 1) >> ks, SM = S + H;
  const RankLds lay = rank_lds_layout((uint32_t)T, (uint32_t)SM);
  int32_t* LEN = reinterpret_cast<int32_t*>(lds);
  int32_t* DN = reinterpret_cast<int32_t*>(lds + lay.dn);
  int32_t* ACL = reinterpret_cast<int32_t*>(lds + lay.acl);
  int32_t* ACD = reinterpret_cast<int32_t*>(lds + lay.acd);
  uint32_t* HB = reinterpret_cast<uint32_t*>(lds + lay.hb);  // bit per sublist: starts at a head; then the reach
  uint16_t* NXT = reinterpret_cast<uint16_t*>(lds + lay.nxt);
  uint16_t* PRED = reinterpret_cast<uint16_t*>(lds + lay.pred);
  uint16_t* TOP = reinterpret_cast<uint16_t*>(lds + lay.top);
  const int hw = (SM + 31) / 32;
  const int t = threadIdx.x;
  bool bad = false, badhead = false;
  for (int s = t; s < SM; s += kFinalThreads) {
    PRED[s] = (uint16_t)kNone;
    TOP[s] = (uint16_t)s;
  }
  for (int i = t; i <= hw + 2; i += kFinalThreads) HB[i] = 0u;
#pragma unroll 4
  for (int32_t e = t; e < T; e += kFinalThreads) {
    int32_t nx, l = 1, d = 0;
    bool used;
    if (IN == IN_REC) {
      const int4 r = reinterpret_cast<const int4*>(in)[e];
      nx = r.x;
      used = nx != -3;
      l = r.y;
      d = r.z;
    } else if (IN == IN_PAIR || IN == IN_PAIR2) {
      const int2 r = reinterpret_cast<const int2*>(in)[e];
      nx = r.x;
      used = nx != -2;
      d = r.y;
    } else {
      nx = in[e];
      used = nx != -2;
    }
    uint32_t code = kUnused;
    if (used) {
      code = nx == -1 ? kEnd : (uint32_t)nx;
      if (nx < -1 || nx >= T) {
        bad = true;
        code = kEnd;
      }
      if (code != kEnd && is_splitter((int32_t)code, ks, salt)) code |= kSplit;
    }
    NXT[e] = (uint16_t)code;
    if (kLen) LEN[e] = l;
    if (kDn) DN[e] = d;
  }
  __syncthreads();
  int32_t wl[kFinalSub], wd[kFinalSub], to[kFinalSub], passed = 0;
#pragma unroll
  for (int k = 0; k < kFinalSub; ++k) {
    wl[k] = wd[k] = 0;
    to[k] = -1;
    const int32_t s = t + k * kFinalThreads;
    if (s >= SM) continue;
    int32_t e = -1;
    if (s < S) {
      e = splitter_of_chunk(s, ks, salt);
      if (e >= T || NXT[e] == kUnused) e = -1;
    } else {
      const int32_t h = IN == IN_REC ? hb + (s - S) : heads[s - S];
      if (!(h == -1 && empty_ok)) {
        if (h < 0 || h >= T) {
          badhead = true;
        } else if (NXT[h] == kUnused) {
          badhead = badhead || IN != IN_REC;
        } else if (is_splitter(h, ks, salt)) {
          // the head's own chunk walks it
          const uint32_t bit = 1u << ((h >> ks) & 31);
          if (atomicOr(&HB[(h >> ks) >> 5], bit) & bit) badhead = true;  // the same head twice
        } else {
          e = h;
          atomicOr(&HB[s >> 5], 1u << (s & 31));
        }
      }
    }
    if (e >= 0) {
      int32_t al = 0, ad = 0, after = -1;
      for (int32_t step = 0;; ++step) {
        const uint32_t nx = NXT[e];
        if ((nx & kWalked) || nx == kUnused || step >= T) {  // a second way into an element, or into no element
          bad = true;
          break;
        }
        NXT[e] = (uint16_t)(kWalked | (uint32_t)s);
        ++passed;
        const int32_t l = kLen ? LEN[e] : 1;
        const int32_t d = kDn ? DN[e] : 0;
        LEN[e] = al;
        if (kDn) DN[e] = ad;
        al += l;
        ad = wadd(ad, d);
        if (nx >= kEnd) {
          if (nx & kSplit) after = (int32_t)(nx & (kSplit - 1u));
          break;
        }
        e = (int32_t)nx;
      }
      if (after >= 0) {  // (out of the loop, whose lanes end one by one)
        if (NXT[after] == kUnused) bad = true;  // (the code of an unused slot never changes)
        to[k] = after >> ks;
        PRED[to[k]] = (uint16_t)s;
      }
      wl[k] = al;
      wd[k] = ad;
    }
    ACL[s] = wl[k];
    ACD[s] = wd[k];
  }
  if (bad) flag(status, ST_BAD_SUCC);
  if (badhead) flag(status, ST_BAD_HEAD);
  // at most clog2(SM) + 1 rounds; fewer once no pointer is left
  for (int it = 0; it < 13; ++it) {
    __syncthreads();
    int32_t nl[kFinalSub], nd[kFinalSub];
    uint32_t np[kFinalSub], nt[kFinalSub];
    bool more = false;
#pragma unroll
    for (int k = 0; k < kFinalSub; ++k) {
      const int32_t s = t + k * kFinalThreads;
      if (it == 0 && to[k] >= 0 && PRED[to[k]] != s) flag(status, ST_BAD_SUCC);  // two sublists lead into one
      np[k] = s < SM ? PRED[s] : kNone;
      if (np[k] != kNone) {
        if (it == 0 && ((HB[s >> 5] >> (s & 31)) & 1u)) flag(status, ST_BAD_HEAD);  // a head inside a list
        const uint32_t q = np[k];
        nl[k] = ACL[s] + ACL[q];
        nd[k] = wadd(ACD[s], ACD[q]);
        nt[k] = TOP[q];
        np[k] = PRED[q];
        more = true;
      } else {
        nt[k] = kNone;  // nothing to write
      }
    }
    if (!__syncthreads_or(more)) break;
#pragma unroll
    for (int k = 0; k < kFinalSub; ++k) {
      const int32_t s = t + k * kFinalThreads;
      if (nt[k] != kNone) {
        ACL[s] = nl[k];
        ACD[s] = nd[k];
        TOP[s] = (uint16_t)nt[k];
        PRED[s] = (uint16_t)np[k];
      }
    }
  }
  int32_t mine = 0;
  bool reached[kFinalSub];
#pragma unroll
  for (int k = 0; k < kFinalSub; ++k) {
    const int32_t s = t + k * kFinalThreads;
    reached[k] = false;
    if (s >= SM) continue;
    const uint32_t top = TOP[s];
    reached[k] = PRED[s] == kNone && ((HB[top >> 5] >> (top & 31)) & 1u);
    if (reached[k]) mine += wl[k];
    ACL[s] -= wl[k];
    ACD[s] = wsub(ACD[s], wd[k]);
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < kFinalSub; ++k) {
    const int32_t s = t + k * kFinalThreads;
    if (s < SM) PRED[s] = reached[k];
  }
  for (int dd = 32; dd >= 1; dd >>= 1) {
    mine += __shfl_xor(mine, dd, 64);
    passed += __shfl_xor(passed, dd, 64);
  }
  if (__lane_id() == 0) {  // (the slots after the bits)
    if (mine) atomicAdd(&HB[hw], (uint32_t)mine);
    if (passed) atomicAdd(&HB[hw + 1], (uint32_t)passed);
  }
  __syncthreads();
  if (t == 0 && reached_out) *reached_out = (int32_t)HB[hw];
  bool unreached = t == 0 && expected && (int32_t)HB[hw] != *expected;
  int32_t walked = 0;
#pragma unroll 4
  for (int32_t e = t; e < T; e += kFinalThreads) {
    const uint32_t c = NXT[e];  // kWalked | sublist, or never walked
    if (c == kUnused) {
      if (IN == IN_SUCC && rank) rank[e] = -1;
      continue;
    }
    int2 o = make_int2(0, 0);
    if (c & kWalked) {
      ++walked;
      const uint32_t s = c & (kWalked - 1u);
      o = make_int2(ACL[s] + LEN[e], kDn ? wadd(ACD[s], DN[e]) : 0);
      if (!PRED[s]) unreached = true;
    } else {
      unreached = true;
    }
    if (IN == IN_SUCC && rank) {
      rank[e] = o.x;
      continue;
    }
    off[e] = o;
    if (IN == IN_SUCC) packed[e] = (uint64_t)(uint32_t)e;
    if (IN == IN_PAIR) packed[e] = (uint64_t)(uint32_t)e | ((uint64_t)(uint32_t)in[2 * e + 1] << 32);
    if (IN == IN_PAIR2)
      reinterpret_cast<ulonglong2*>(packed)[e] =
          make_ulonglong2((uint64_t)(uint32_t)e, (uint64_t)(uint32_t)in[2 * e + 1]);
  }
  if (unreached) flag(status, ST_UNREACHED);
  // Two lanes may enter a shared element before either has marked it; then
  // they passed more elements than are marked.
  for (int dd = 32; dd >= 1; dd >>= 1) walked += __shfl_xor(walked, dd, 64);
  if (__lane_id() == 0 && walked) atomicAdd(&HB[hw + 2], (uint32_t)walked);
  __syncthreads();
  if (t == 0 && HB[hw + 1] != HB[hw + 2]) flag(status, ST_BAD_SUCC);
}

// The final level of lists with many heads (more sublists than the kernel
// above has lanes for): predecessor pointers jump over every element. T <=
// kLdsMaxHeads.
constexpr int kFinalPer = kLdsMaxHeads / kFinalThreads;

__global__ __launch_bounds__(kFinalThreads) void k_final_lds(const int4* __restrict__ rec, int32_t T,
                                                             int32_t hb, int32_t H, int2* __restrict__ off,
                                                             int32_t* __restrict__ reached,
                                                             const int32_t* __restrict__ expected,
                                                             uint32_t* __restrict__ status) {
  __shared__ int32_t pred[kLdsMaxHeads];
  __shared__ int32_t acl[kLdsMaxHeads];
  __shared__ int32_t acd[kLdsMaxHeads];
  __shared__ int32_t top[kLdsMaxHeads];
  const int t = threadIdx.x;
  int32_t wl[kFinalPer], wd[kFinalPer];
  bool used[kFinalPer];
  for (int k = 0; k < kFinalPer; ++k) pred[t + k * kFinalThreads] = -1;
  __syncthreads();
  bool bad = false;
  for (int k = 0; k < kFinalPer; ++k) {
    const int e = t + k * kFinalThreads;
    int4 r = (e < T) ? rec[e] : make_int4(-3, 0, 0, 0);
    used[k] = (r.x != -3);
    wl[k] = used[k] ? r.y : 0;
    wd[k] = used[k] ? r.z : 0;
    acl[e] = wl[k];
    acd[e] = wd[k];
    top[e] = e;
    if (used[k] && r.x >= 0) {
      if (r.x < T) pred[r.x] = e;
      if (r.x >= T || rec[r.x].x == -3) bad = true;
    }
  }
  __syncthreads();
  // two elements that lead into one: the other one's link is gone
  for (int k = 0; k < kFinalPer; ++k) {
    const int e = t + k * kFinalThreads;
    if (!used[k]) continue;
    const int32_t x = rec[e].x;
    if (x >= 0 && x < T && pred[x] != e) bad = true;
  }
  if (bad) flag(status, ST_BAD_SUCC);
  __syncthreads();
  int rounds = 1;
  while ((1 << (rounds - 1)) < T) ++rounds;
  for (int it = 0; it < rounds; ++it) {
    int32_t np[kFinalPer], nl[kFinalPer], nd[kFinalPer], nt[kFinalPer];
    for (int k = 0; k < kFinalPer; ++k) {
      const int e = t + k * kFinalThreads;
      const int32_t p = pred[e];
      if (p >= 0) {
        np[k] = pred[p];
        nl[k] = acl[e] + acl[p];
        nd[k] = wadd(acd[e], acd[p]);
        nt[k] = top[p];
      } else {
        np[k] = p; nl[k] = acl[e]; nd[k] = acd[e]; nt[k] = top[e];
      }
    }
    __syncthreads();
    for (int k = 0; k < kFinalPer; ++k) {
      const int e = t + k * kFinalThreads;
      pred[e] = np[k]; acl[e] = nl[k]; acd[e] = nd[k]; top[e] = nt[k];
    }
    __syncthreads();
  }
  int32_t mine = 0;
  bool unreached = false;
  for (int k = 0; k < kFinalPer; ++k) {
    const int e = t + k * kFinalThreads;
    if (e >= T) continue;
    const bool from_head = (top[e] >= hb && top[e] < hb + H && pred[e] < 0);
    if (used[k] && !from_head) unreached = true;
    if (from_head) mine += wl[k];
    off[e] = make_int2(acl[e] - wl[k], wsub(acd[e], wd[k]));
  }
  if (unreached) flag(status, ST_UNREACHED);
  for (int dd = 32; dd >= 1; dd >>= 1) mine += __shfl_xor(mine, dd, 64);
  if (__lane_id() == 0) atomicAdd(reached, mine);
  // every element must be reached from a head: the whole count is in once
  // all wavefronts have added theirs
  __syncthreads();
  if (threadIdx.x == 0 && expected && atomicAdd(reached, 0) != *expected) flag(status, ST_UNREACHED);
}

// Final level when many heads keep the list above kLdsMaxHeads: one lane per
// head walks its (short) list.
__global__ void k_final_walk(const int4* __restrict__ rec, int32_t T, int32_t hb, int32_t H,
                             int2* __restrict__ off, int32_t* __restrict__ reached,
                             uint32_t* __restrict__ status) {
  const int64_t h = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  int32_t al = 0, ad = 0;
  if (h < H) {
    int32_t e = hb + (int32_t)h;
    int64_t steps = 0;
    while (e != -1) {
      if (e < 0 || e >= T || ++steps > T) {
        flag(status, ST_BAD_SUCC);
        break;
      }
      const int4 r = rec[e];
      off[e] = make_int2(al, ad);
      al += r.y;
      ad = wadd(ad, r.z);
      e = r.x;
    }
  }
  // one add per wavefront to the shared count, not one per head
  for (int dd = 32; dd >= 1; dd >>= 1) al += __shfl_xor(al, dd, 64);
  if (__lane_id() == 0 && al) atomicAdd(reached, al);
}

__global__ void k_check_reached(const int32_t* __restrict__ reached, const int32_t* __restrict__ expected,
                                uint32_t* __restrict__ status) {
  if (expected && *reached != *expected) flag(status, ST_UNREACHED);
}

// off_k[e] = off_{k+1}[el[e].sub] + (el[e].len, el[e].down) for used elements.
// CH 1 / 2: store the first / second word alone, compact. The elements gather
// these offsets at random, and a plain ranking needs only the lengths, a scan
// without ranks only the sums: half the table, a faster gather (k_rank_fix at
// 2^25 elements, 2^21 sublists: 16 -> 8 MiB, 473 -> 365 us).
template <int CH>
__global__ void k_push_down(const int4* __restrict__ rec, const int4* __restrict__ el, int32_t T,
                            const int2* __restrict__ off_up, int32_t T_up, void* __restrict__ off,
                            uint32_t* __restrict__ status) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= T) return;
  if (rec[e].x == -3) return;
  const int4 x = el[e];
  int2 v = make_int2(0, 0);
  if ((uint32_t)x.x >= (uint32_t)T_up) {
    flag(status, ST_BAD_INDEX);
  } else {
    const int2 o = off_up[x.x];
    v = make_int2(o.x + x.y, wadd(o.y, x.z));
  }
  if (CH == 0) static_cast<int2*>(off)[e] = v;
  else static_cast<int32_t*>(off)[e] = CH == 1 ? v.x : v.y;
}

// weighted list prefix sums: sum[e] = the weight sum before e's sublist +
// the inclusive local sum; RANK: also rank as in k_rank_fix (16-byte
// records). Unused slots get rank -1 and sum 0.
template <bool RANK>
__global__ void k_scan_fix(const int2* __restrict__ sw, const uint64_t* __restrict__ packed, int32_t L,
                           const int2* __restrict__ off, OffWord offw, int32_t T1, int32_t* __restrict__ rank,
                           int32_t* __restrict__ sum, uint32_t* __restrict__ status) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= L) return;
  if (sw[e].x == -2) {
    if (RANK) rank[e] = -1;
    sum[e] = 0;
    return;
  }
  uint32_t sub, lsum, lrank = 0;
  if (RANK) {
    const ulonglong2 pk = reinterpret_cast<const ulonglong2*>(packed)[e];
    sub = (uint32_t)pk.x;
    lrank = (uint32_t)(pk.x >> 32) & 0xffffu;
    lsum = (uint32_t)pk.y;
  } else {
    const uint64_t p = packed[e];
    sub = (uint32_t)p;
    lsum = (uint32_t)(p >> 32);
  }
  if (sub >= (uint32_t)T1) {
    flag(status, ST_BAD_INDEX);
    if (RANK) rank[e] = -1;
    sum[e] = 0;
    return;
  }
  if (RANK) {
    const int2 o = off[sub];
    rank[e] = o.x + (int32_t)lrank;
    sum[e] = wadd(o.y, (int32_t)lsum);
  } else {
    sum[e] = wadd(offw.at(sub), (int32_t)lsum);
  }
}

// generic rank: rank[e] = off[sub] + local rank, -1 for unused slots. Counts
// the used elements on the way (a pass of its own over the successors took 57
// us at 2^25 elements), a workgroup per 256 * per elements so that the counter
// sees few updates; kFixTogether of a lane's loads go together. Bound by the
// gathered offsets.
constexpr int kFixTogether = 4;

__global__ __launch_bounds__(256) void k_rank_fix(const int32_t* __restrict__ succ, const uint64_t* __restrict__ packed,
                                                  int32_t L, int per, OffWord off, int32_t T1,
                                                  int32_t* __restrict__ rank, int32_t* __restrict__ used,
                                                  uint32_t* __restrict__ status) {
  __shared__ int32_t part[4];
  constexpr int kTogether = kFixTogether;
  const int64_t base = (int64_t)blockIdx.x * (256 * per) + threadIdx.x;
  int32_t count = 0;
  bool bad = false;
  for (int r0 = 0; r0 < per; r0 += kTogether) {
    int32_t nx[kTogether], v[kTogether];
    uint64_t pk[kTogether];
#pragma unroll
    for (int r = 0; r < kTogether; ++r) {
      const int64_t e = base + (int64_t)(r0 + r) * 256;
      nx[r] = e < L ? succ[e] : -2;
      pk[r] = e < L ? packed[e] : 0ull;
    }
#pragma unroll
    for (int r = 0; r < kTogether; ++r) {
      v[r] = -1;
      if (nx[r] == -2) continue;
      ++count;
      const uint32_t sub = (uint32_t)pk[r];
      if (sub >= (uint32_t)T1) bad = true;
      else v[r] = off.at(sub) + (int32_t)((pk[r] >> 32) & 0xffffu);
    }
#pragma unroll
    for (int r = 0; r < kTogether; ++r) {
      const int64_t e = base + (int64_t)(r0 + r) * 256;
      if (e < L) rank[e] = v[r];
    }
  }
  if (bad) flag(status, ST_BAD_INDEX);
  for (int d = 32; d >= 1; d >>= 1) count += __shfl_xor(count, d, 64);
  if (__lane_id() == 0) part[threadIdx.x >> 6] = count;
  __syncthreads();
  if (threadIdx.x == 0) atomicAdd(used, part[0] + part[1] + part[2] + part[3]);
}

// {successor, weight} pairs for the weighted walk, and the number of used
// elements (successor other than -2). The workgroups' updates of the one
// counter come at about 10 ns each, which bounded this kernel with one per 512
// elements (10^6 elements 30 us): at least 4096 elements a workgroup, on short
// lists 1024, where the lanes are too few otherwise (4 / 16 elements a lane:
// 10^5 elements 7 / 8 us, 10^6 18 / 11).
inline int pair_blocks(int32_t len) {
  const int32_t per = len < (1 << 18) ? 1024 : 4096;
  const int64_t b = ((int64_t)len + per - 1) / per;
  return (int)(b < 1024 ? b : 1024);
}

__global__ __launch_bounds__(256) void k_pair_count(const int32_t* __restrict__ succ, const int32_t* __restrict__ w,
                                                    int32_t L, int2* __restrict__ sw, int32_t* __restrict__ count) {
  constexpr int kTogether = kFixTogether;
  __shared__ int32_t part[4];
  int32_t c = 0;
  for (int64_t b = (int64_t)blockIdx.x * (256 * kTogether); b < L; b += (int64_t)gridDim.x * (256 * kTogether)) {
    int32_t x[kTogether], y[kTogether];
#pragma unroll
    for (int r = 0; r < kTogether; ++r) {
      const int64_t e = b + r * 256 + threadIdx.x;
      x[r] = e < L ? succ[e] : -2;
      y[r] = e < L ? w[e] : 0;
    }
#pragma unroll
    for (int r = 0; r < kTogether; ++r) {
      const int64_t e = b + r * 256 + threadIdx.x;
      if (e < L) sw[e] = make_int2(x[r], y[r]);
      c += (x[r] != -2);
    }
  }
  for (int d = 32; d >= 1; d >>= 1) c += __shfl_xor(c, d, 64);
  if (__lane_id() == 0) part[threadIdx.x >> 6] = c;
  __syncthreads();
  if (threadIdx.x == 0) atomicAdd(count, part[0] + part[1] + part[2] + part[3]);
}

int walk_grid(int32_t total, int32_t per_wave) {
  const int64_t waves = (total + (int64_t)per_wave - 1) / per_wave;
  return (int)((waves * 64 + kWalkThreads - 1) / kWalkThreads);
}

}  // namespace

// Every buffer of a ranking is taken from the scratch before the first
// launch (the level sizes follow from the list length, the number of heads
// and the launch shape alone), so a fixed-size arena can be checked, or a
// pool request fail, before anything is enqueued.
struct LrLevel {
  int4* rec;        // this level's records (level 1: the sublist records)
  int32_t T, hb;    // records and the index of the first head record
  int4* el;         // per record: {sublist, exclusive local len, down} of the level above
  int2* off;        // per record: exclusive prefix {len, down} from its head
  int ks;           // splitter spacing of the level above (2^ks)
  int32_t S_up;     // chunk splitters of the level above
  int32_t per_wave; // sublists per wavefront of the level above's walk
};

struct LrPlan {
  int ks1 = 0;
  int32_t S1 = 0, cont_max = 0, T1 = 0, per_wave1 = 0;
  uint64_t* packed = nullptr;
  int4* rec1 = nullptr;
  int32_t* ctr = nullptr;
  bool direct = false;  // the whole list goes to k_rank_lds
  std::vector<LrLevel> lv;
};

constexpr int32_t kLongList = 1 << 25;
constexpr int kLongSpacing = 5;
constexpr int32_t kShortLevel = 1 << 21;

static void list_rank_plan(Ctx* c, Scratch& sc, int32_t L, int32_t H, int weighted, bool local, LrPlan* pl) {
  const int32_t lds_max = H <= kLdsHeads ? kLdsMax : kLdsMaxHeads;
  // One workgroup ranks a short list by itself, one launch in place of three.
  // By this / by level 1 and a final level, us: plain lists (whose ranks it
  // writes itself) 16 / 29 at 2000 elements, 29 / 38 at 8000, 39 / 39 at 12000;
  // weighted lists 29 / 41 and 43 / 47, in id order 26 / 31 and 35 / 32.
  pl->direct = L <= kLdsDirect && H <= kLdsHeads;
  if (pl->direct) {
    pl->T1 = L;
    pl->packed = sc.get<uint64_t>((size_t)L * (weighted == 2 ? 2 : 1));
    pl->lv.assign(1, {nullptr, L, 0, nullptr, sc.get<int2>((size_t)L), 0, 0, 0});
    return;
  }
  // Level-1 splitter spacing K = 2^ks1 (a sublist averages K elements).
  // Shorter lists keep more, shorter sublists: below about 2^25 elements the
  // walk is bound by its dependent steps rather than by line fetches, so the
  // spacing drops by half per factor 4 of length (2^24 -> 16, 2^22 -> 8,
  // 2^20 -> 4), down to 4; the context's value is the largest spacing used.
  // From 2^25 elements on a spacing below 32 is doubled: the sublists' offsets,
  // which every element gathers, are then half as many. Spacing 16 / 32, us:
  // random lists of 24.5M elements 1220 / 1242, of 2^25 1719 / 1687, of 2^26 4878 /
  // 4635; random trees of 12.5M nodes 2348 / 2368, of 2^24 3131 / 3075, a path
  // 2172 / 2222 and 3056 / 2964, 30M 6377 / 6183; a batch of 2^25 local elements
  // 3899 / 4070.
  pl->ks1 = std::min(c->lr.k1_log2, std::max(2, (floor_log2(L) - 15) / 2));
  if (!local && L >= kLongList && pl->ks1 < kLongSpacing) ++pl->ks1;
  pl->S1 = (int32_t)(((int64_t)L + (1 << pl->ks1) - 1) >> pl->ks1);
  pl->cont_max = L / kCap + H + 64;
  pl->T1 = pl->S1 + H + pl->cont_max;
  pl->packed = sc.get<uint64_t>((size_t)L * (weighted == 2 ? 2 : 1));
  pl->rec1 = sc.get<int4>((size_t)pl->T1);
  pl->ctr = sc.get<int32_t>(4);
  // sublists per wavefront: the context's value, fewer when that would leave
  // under 4096 wavefronts (at least 64, one per lane)
  pl->per_wave1 = std::min(c->lr.per_wave1, std::max(64, (pl->S1 + H) >> 12));
  pl->lv.clear();
  pl->lv.push_back({pl->rec1, pl->T1, pl->S1, nullptr, nullptr, 0, 0, 0});
  for (;;) {
    LrLevel& cur = pl->lv.back();
    if (cur.T <= lds_max) break;
    // The walk of a short level lasts as long as its longest sublist, about 2^ks
    // ln(sublists) dependent steps of 0.5 us (that of a long one as long as its
    // total work), so there three levels of spacing 4 are quicker than two of 8,
    // unless there are so many heads that the lists are short and a level shrinks
    // little. Calls with spacing 8 / by this rule, us: 10^6 nodes with tables 335
    // / 328, 10^6 weighted elements 149 / 142, 2^21 nodes 510 / 496, 3 * 10^5
    // elements 112 / 97, 2^23 482 / 462 (and 2^22 292 / 296: how long the longest
    // sublist is varies by some us from list to list); with 1747 heads in 2^20
    // elements spacing 4 would cost 127 / 136.
    const int kn = c->lr.kn_log2;
    const int widest = cur.T <= kShortLevel && H <= kLdsHeads ? std::min(2, kn) : kn;
    int ks = std::min(2, c->lr.kn_log2);
    while (ks < widest && (((int64_t)cur.T + (1 << ks) - 1) >> ks) + H > lds_max) ++ks;
    const int32_t S = (int32_t)(((int64_t)cur.T + (1 << ks) - 1) >> ks);
    const int32_t Tn = S + H;
    if ((int64_t)Tn * 2 > cur.T) break;  // many heads: shrinking stalls
    cur.el = sc.get<int4>((size_t)cur.T);
    int4* rec = sc.get<int4>((size_t)Tn);
    cur.ks = ks;
    cur.S_up = S;
    cur.per_wave = std::min(c->lr.per_waven, std::max(64, Tn >> 12));
    pl->lv.push_back({rec, Tn, S, nullptr, nullptr, 0, 0, 0});
  }
  for (auto& l : pl->lv) l.off = sc.get<int2>((size_t)l.T);
}

constexpr int32_t kLocalXcd = 1 << 20;  // elements of a list up to which an XCD keeps its own stretch

static int list_rank_launch(Ctx* c, const LrPlan& pl, const int32_t* succ, int32_t L, const int32_t* heads,
                            int32_t H, bool tree_weights, const int32_t* expected_reach, hipStream_t s,
                            bool empty_head_ok, int weighted, int32_t local_len) {
  const int32_t S1 = pl.S1, T1 = pl.T1, cont_max = pl.cont_max;
  if (pl.direct) {
    const int ks = rank_lds_ks(L);
    if (tree_weights) return ET_EINVAL;  // (never: small.hip builds trees of so few half-edges)
    static_assert(2 * (kSmallTreeMax + 1) > kLdsDirect, "a tour that comes here is longer");
    const auto kern = weighted == 2 ? k_rank_lds<IN_PAIR2> : weighted ? k_rank_lds<IN_PAIR> : k_rank_lds<IN_SUCC>;
    ET_PROF(c, s, "k_rank_lds");
    hipLaunchKernelGGL(kern, dim3(1), dim3(kFinalThreads), rank_lds_bytes(L, H), s, succ, L, heads, 0, H,
                       empty_head_ok, ks, kSalt,
                       pl.packed, pl.lv[0].off, nullptr, nullptr, expected_reach, c->d_status);
    return hipGetLastError() == hipSuccess ? ET_OK : ET_EHIP;
  }
  hipLaunchKernelGGL(k_lr_init, dim3(ceil_div(cont_max, 256)), dim3(256), 0, s, pl.ctr, pl.rec1, S1 + H, T1);
  // Where the lists are local (a batch of trees: a tree's half-edges lie
  // together) a wavefront takes one round of sublists only, so that the
  // workgroups in flight cover a short stretch of the array, whose lines stay
  // in the cache until all their elements are passed; and where two such trees
  // fit an XCD's L2, each XCD takes its own stretch. Level 1 in us, as for one
  // list / one round / one round and a stretch per XCD: 4096 trees of 2^12
  // nodes 880 / 693 / 595, 300 of 2^16 1110 / 949 / 753, 64 of 2^18 1016 / 831 /
  // 735, 16 of 2^20 976 / 858 / 902, 4 of 2^22 1015 / 923 / 1096; one tree of
  // 2^24 866 / 901 / 900.
  const bool local = local_len > 0;
  // With the doubled spacing a wavefront covers twice as much of the array, and
  // with 256 sublists there are only half as many of them. Where ids follow the
  // order of the list its lines then leave the cache half used; fewer sublists
  // keep them and cost a random list nothing, a random tour little. 256 / 128 / 64
  // a wavefront (spacing 16 and 256), us: list of 2^25 elements in order 1159 /
  // 1067 / 996 (992), random 1688 / 1656 / 1687, 2^26 in order 2231 / 2079 / 1907
  // (1927), random 4543 / 4595 / 4635; tree of 2^24 nodes on 64 legs 2282 / 2266 /
  // 2111 (2160), random 3055 / 3075 / 3142, 30M on 64 legs 4428 / 3752 / 3472 (3594),
  // random 6236 / 6183 / 6081.
  const int32_t long_wave = tree_weights ? 128 : 64;
  const int32_t per_wave1 = local                ? 64
                            : L >= kLongList ? std::min(pl.per_wave1, long_wave)
                                             : pl.per_wave1;
  const dim3 g1(walk_grid(S1 + H, per_wave1));
  if (tree_weights) {
    ET_PROF(c, s, "k_walk1<true>");
    hipLaunchKernelGGL(k_walk1<true>, g1, dim3(kWalkThreads), 0, s, succ, L, heads, H, pl.ks1, kSalt, S1,
                       per_wave1, pl.packed, pl.rec1, pl.ctr, S1 + H, cont_max, empty_head_ok, c->d_status,
                       local && local_len <= kLocalXcd);
  } else if (weighted) {
    ET_PROF(c, s, weighted == 2 ? "k_walk1w<true>" : "k_walk1w<false>");
    const auto kern = weighted == 2 ? k_walk1w<true> : k_walk1w<false>;
    hipLaunchKernelGGL(kern, g1, dim3(kWalkThreads), 0, s, succ, L, heads, H, pl.ks1, kSalt, S1, per_wave1,
                       pl.packed, pl.rec1, pl.ctr, S1 + H, cont_max, empty_head_ok, c->d_status);
  } else {
    ET_PROF(c, s, "k_walk1<false>");
    hipLaunchKernelGGL(k_walk1<false>, g1, dim3(kWalkThreads), 0, s, succ, L, heads, H, pl.ks1, kSalt, S1,
                       per_wave1, pl.packed, pl.rec1, pl.ctr, S1 + H, cont_max, empty_head_ok, c->d_status,
                       local && local_len <= kLocalXcd);
  }
  // upper levels: level k's records are walked into level k+1's
  const auto& lv = pl.lv;
  for (size_t k = 0; k + 1 < lv.size(); ++k) {
    const LrLevel& cur = lv[k];
    const int32_t Tn = lv[k + 1].T;
    ET_PROF(c, s, "k_walkN");
    hipLaunchKernelGGL(k_walkN, dim3(walk_grid(Tn, cur.per_wave)), dim3(kWalkThreads), 0, s, cur.rec, cur.T,
                       cur.hb, H, cur.ks, kSalt ^ (uint32_t)(k + 1), cur.S_up, cur.per_wave, cur.el, lv[k + 1].rec,
                       c->d_status);
  }
  const LrLevel& top = lv.back();
  if (H <= kLdsHeads && top.T <= kLdsMax) {
    const int ks = rank_lds_ks(top.T);
    ET_PROF(c, s, "k_rank_lds");
    hipLaunchKernelGGL(k_rank_lds<IN_REC>, dim3(1), dim3(kFinalThreads), rank_lds_bytes(top.T, H), s,
                       reinterpret_cast<const int32_t*>(top.rec), top.T, nullptr, top.hb, H, false, ks,
                       kSalt ^ (uint32_t)lv.size(), nullptr, top.off, nullptr, pl.ctr + 1, expected_reach, c->d_status);
  } else if (top.T <= kLdsMaxHeads) {
    ET_PROF(c, s, "k_final_lds");
    hipLaunchKernelGGL(k_final_lds, dim3(1), dim3(kFinalThreads), 0, s, top.rec, top.T, top.hb, H, top.off,
                       pl.ctr + 1, expected_reach, c->d_status);
  } else {
    {
      ET_PROF(c, s, "k_final_walk");
      hipLaunchKernelGGL(k_final_walk, dim3(ceil_div(H, 256)), dim3(256), 0, s, top.rec, top.T, top.hb, H,
                         top.off, pl.ctr + 1, c->d_status);
    }
    hipLaunchKernelGGL(k_check_reached, dim3(1), dim3(1), 0, s, pl.ctr + 1, expected_reach, c->d_status);
  }
  for (int k = (int)lv.size() - 2; k >= 0; --k) {
    ET_PROF(c, s, "k_push_down");
    // the level-1 offsets compact where one word is enough
    const auto kern = k > 0 || tree_weights || weighted == 2 ? k_push_down<0>
                      : weighted                               ? k_push_down<2>
                                                               : k_push_down<1>;
    hipLaunchKernelGGL(kern, dim3(ceil_div(lv[k].T, 256)), dim3(256), 0, s, lv[k].rec, lv[k].el, lv[k].T,
                       lv[k + 1].off, lv[k + 1].T, lv[k].off, c->d_status);
  }
  return hipGetLastError() == hipSuccess ? ET_OK : ET_EHIP;
}

int list_rank_prepare() {
  for (const void* kern :
       {reinterpret_cast<const void*>(k_rank_lds<IN_REC>), reinterpret_cast<const void*>(k_rank_lds<IN_SUCC>),
        reinterpret_cast<const void*>(k_rank_lds<IN_PAIR>), reinterpret_cast<const void*>(k_rank_lds<IN_PAIR2>)})
    if (hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize,
                            (int)rank_lds_bytes(kLdsMax, kLdsHeads)) != hipSuccess)
      return ET_EHIP;
  return ET_OK;
}

// the level-1 offsets of a plain ranking (lengths) or of sums alone, as the
// launches above leave them: compact if they come from a push-down
static OffWord off_word(const LrPlan& pl, int weighted) {
  const int32_t* p = reinterpret_cast<const int32_t*>(pl.lv[0].off);
  return pl.lv.size() > 1 ? OffWord{p, 0} : OffWord{p + (weighted ? 1 : 0), 1};
}

int list_rank_core(Ctx* c, Scratch& sc, const int32_t* succ, int32_t len, const int32_t* heads,
                   int32_t nheads, bool tree_weights, const int32_t* expected_reach, LRResult* out,
                   hipStream_t s, bool empty_head_ok, int weighted, int32_t local_len) {
  LrPlan pl;
  list_rank_plan(c, sc, len, nheads, weighted, local_len > 0, &pl);
  if (sc.failed) return ET_ENOMEM;
  const int rc = list_rank_launch(c, pl, succ, len, heads, nheads, tree_weights, expected_reach, s, empty_head_ok,
                                  weighted, local_len);
  out->packed = pl.packed;
  out->off = pl.lv[0].off;
  out->word = off_word(pl, weighted);
  out->nsub = pl.T1;
  return rc;
}

// Plain ranking with the scratch taken from `sc` (the pool, or an arena):
// every buffer is reserved before the first launch.
static int list_rank_with(Ctx* c, Scratch& sc, const int32_t* succ, int32_t len, const int32_t* heads,
                          int32_t nheads, int32_t* rank, hipStream_t s) {
  LrPlan pl;
  list_rank_plan(c, sc, len, nheads, 0, false, &pl);
  if (sc.failed || sc.counting) return sc.failed ? ET_ENOMEM : ET_OK;
  if (pl.direct) {  // sees every element itself: nothing to count, no records to add up
    const int ks = rank_lds_ks(len);
    ET_PROF(c, s, "k_rank_lds");
    hipLaunchKernelGGL(k_rank_lds<IN_SUCC>, dim3(1), dim3(kFinalThreads), rank_lds_bytes(len, nheads), s, succ, len,
                       heads, 0, nheads, false, ks, kSalt, nullptr, nullptr, rank, nullptr, nullptr, c->d_status);
    return hipGetLastError() == hipSuccess ? ET_OK : ET_EHIP;
  }
  int rc = list_rank_launch(c, pl, succ, len, heads, nheads, false, nullptr, s, false, 0, 0);
  if (rc) return rc;
  {
    ET_PROF(c, s, "k_rank_fix");
    // elements per lane: few on a list whose blocks would not fill the GPU
    const int per = kFixTogether * (len < (1 << 22) ? 1 : 4);
    hipLaunchKernelGGL(k_rank_fix, dim3(ceil_div(len, 256 * per)), dim3(256), 0, s, succ, pl.packed, len, per,
                       off_word(pl, 0), pl.T1, rank, pl.ctr + 2, c->d_status);
  }
  hipLaunchKernelGGL(k_check_reached, dim3(1), dim3(1), 0, s, pl.ctr + 1, pl.ctr + 2, c->d_status);
  return hipGetLastError() == hipSuccess ? ET_OK : ET_EHIP;
}

int list_rank_generic(Ctx* c, const int32_t* succ, int32_t len, const int32_t* heads, int32_t nheads,
                      int32_t* rank, hipStream_t s) {
  if (len == 0) return ET_OK;
  Scratch sc(c, s);
  return list_rank_with(c, sc, succ, len, heads, nheads, rank, s);
}

size_t list_rank_plan_bytes(const Ctx* c, int32_t len, int32_t nheads, int weighted, bool local) {
  if (len == 0) return 0;
  Ctx shape;  // the plan reads only the launch shape
  shape.lr = c ? c->lr : LrShape{};
  Scratch count(&shape, nullptr, nullptr, 0);
  LrPlan pl;
  list_rank_plan(&shape, count, len, nheads, weighted, local, &pl);
  // as pool blocks: every block, the last one too, takes whole 256-byte units
  return (count.used + 255) & ~(size_t)255;
}

size_t list_rank_scratch_bytes(Ctx* c, int32_t len, int32_t nheads) {
  if (len == 0) return 0;
  Scratch count(c, nullptr, nullptr, 0);
  (void)list_rank_with(c, count, nullptr, len, nullptr, nheads, nullptr, nullptr);
  return count.used;
}

int list_rank_arena(Ctx* c, void* arena, size_t bytes, const int32_t* succ, int32_t len, const int32_t* heads,
                    int32_t nheads, int32_t* rank, hipStream_t s) {
  if (len == 0) return ET_OK;
  Scratch sc(c, s, arena, bytes);
  return list_rank_with(c, sc, succ, len, heads, nheads, rank, s);
}

int list_scan_generic(Ctx* c, const int32_t* succ, const int32_t* weights, int32_t len, const int32_t* heads,
                      int32_t nheads, int32_t* rank, int32_t* sum, hipStream_t s) {
  if (len == 0) return ET_OK;
  Scratch sc(c, s);
  int32_t* expected = sc.get<int32_t>(1);
  int2* sw = sc.get<int2>((size_t)len);
  if (sc.failed) return ET_ENOMEM;
  hipLaunchKernelGGL(k_set_scalar, dim3(1), dim3(1), 0, s, expected, 0);
  {
    ET_PROF(c, s, "k_pair_count");
    hipLaunchKernelGGL(k_pair_count, dim3(pair_blocks(len)), dim3(256), 0, s, succ, weights, len, sw,
                       expected);
  }
  LRResult r;
  int rc = list_rank_core(c, sc, reinterpret_cast<const int32_t*>(sw), len, heads, nheads, false, expected, &r, s,
                          false, rank ? 2 : 1);
  if (rc) return rc;
  {
    ET_PROF(c, s, rank ? "k_scan_fix<true>" : "k_scan_fix<false>");
    const auto kern = rank ? k_scan_fix<true> : k_scan_fix<false>;
    hipLaunchKernelGGL(kern, dim3(ceil_div(len, 256)), dim3(256), 0, s, sw, r.packed, len, r.off, r.word, r.nsub, rank, sum,
                       c->d_status);
  }
  return hipGetLastError() == hipSuccess ? ET_OK : ET_EHIP;
}

}  // namespace et
