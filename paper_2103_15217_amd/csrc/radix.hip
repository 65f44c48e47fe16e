// Stable grouping of the children of every node by parent id.
//
// The paper builds the DCEL by lexicographically sorting half-edges
// (Section 2.1) and remarks that this sort dominates construction. With a
// parent array as input the half-edges of node x are its children, and a
// stable sort of the child ids by parent id puts every node's children next
// to each other in ascending id order, which is all the successor step
// needs. This is an LSD radix sort over the ceil(log2 n) key bits, in as few
// passes as the digits of plan_passes() allow (2 of 9 and 8 bits at n = 2^17, 2
// of 11 and 10 at 2^21, 3 of 8 at 2^24, 3 of 9 at 2^27):
//
//   upsweep    per 4096-element tile, a digit histogram (one LDS histogram
//              per wavefront), stored digit-major so that one exclusive scan
//              gives every (digit, tile) its output offset;
//   scan       the array scan of scan.hip;
//   downsweep  512 lanes per tile; each wavefront ranks its 8 rounds of 64
//              keys stably: a ballot a bit finds the lanes that share a digit, the
//              lowest such lane bumps the wavefront's LDS counter for that
//              digit, and the eight wavefront counters are chained per
//              digit. The tile is then sorted by digit in LDS and written
//              out run by run, so consecutive lanes store to consecutive
//              addresses.
//
// Both kernels take their tile from xcd_block(): workgroups are handed to the
// eight XCDs in turn, and each XCD is given a contiguous range of tiles, so
// the runs of one digit that adjacent tiles write (neighbours in the output)
// and the histogram entries they write meet in the same L2, which merges
// their partial lines before they go to memory. With the 512-lane shape
// this takes a downsweep pass over 2^24 uniform keys from 126 to 83 us, and
// one of a 2^24-node tree build from 116 to 91 us.
//
// The first pass reads the parent array directly (the root's -1 becomes the
// all-ones key and sorts last), validates it, finds the root, and writes
// the successor of every down half-edge of a leaf (2c -> 2c+1).
#include "et_internal.hpp"

namespace et {
namespace {

constexpr int kThreads = 256;  // histogram pass
constexpr int kWaves = kThreads / 64;
constexpr int kRounds = 16;
constexpr int kTile = kThreads * kRounds;  // 4096 keys per tile
constexpr int kDownThreads = 512;          // downsweep: 8 wavefronts of 8 rounds per tile
constexpr int kDownWaves = kDownThreads / 64;
constexpr int kDownRounds = kTile / kDownThreads;
constexpr int kMaxBits = 11;               // widest digit; kernels are built for 256 to 2048 digits

__device__ __forceinline__ uint32_t parent_key(int32_t p, int32_t n) {
  return (p >= 0 && p < n) ? (uint32_t)p : 0xffffffffu;
}

// What a first pass reads: a parent array (values: the node ids) or the targets
// of the half-edges of an edge list (values: the half-edge ids); later passes
// read the keys and values of the pass before.
enum SortIn { IN_KEYS, IN_PARENT, IN_TARGET };

// scalars[0] = root id, scalars[1] = number of roots
template <SortIn IN, int DIG>
__global__ __launch_bounds__(kThreads) void k_upsweep(const void* __restrict__ keys_in, HalfEdges he, int32_t n,
                                                      int shift, int nbits, int32_t ntiles,
                                                      uint32_t* __restrict__ hist,
                                                      int32_t* __restrict__ succ, int32_t* __restrict__ scalars,
                                                      uint32_t* __restrict__ status) {
  __shared__ uint32_t h[kWaves][DIG];
  const int wave = threadIdx.x >> 6;
  const uint32_t mask = (1u << nbits) - 1u;
  for (int i = threadIdx.x; i < kWaves * DIG; i += kThreads) (&h[0][0])[i] = 0;
  __syncthreads();
  const int32_t tile = xcd_block(ntiles);
  const int64_t base = (int64_t)tile * kTile;
  bool bad = false;
  // all of a lane's loads first (guarded, not cut short), then the counts
  uint32_t raw[kRounds];
#pragma unroll
  for (int r = 0; r < kRounds; ++r) {
    const int64_t idx = base + r * kThreads + threadIdx.x;
    if (IN == IN_TARGET) raw[r] = idx < n ? (uint32_t)he.target(idx) : 0u;
    else raw[r] = idx < n ? static_cast<const uint32_t*>(keys_in)[idx] : 0u;
  }
#pragma unroll
  for (int r = 0; r < kRounds; ++r) {
    const int64_t idx = base + r * kThreads + threadIdx.x;
    if (idx >= n) break;
    uint32_t key;
    if (IN == IN_TARGET) {
      // the other half-edge of the edge is the neighbouring lane's
      const uint32_t x = raw[r], y = (uint32_t)__shfl_xor((int32_t)x, 1, 64);
      if (x >= (uint32_t)he.n || x == y) bad = true;
      key = he.clamp((int32_t)x);
    } else if (IN == IN_PARENT) {
      const int32_t p = (int32_t)raw[r];
      key = parent_key(p, n);
      if (p == -1) {
        atomicAdd(&scalars[1], 1);
        scalars[0] = (int32_t)idx;
        succ[2 * idx] = -2;
        succ[2 * idx + 1] = -2;
      } else {
        if (p < 0 || p >= n || p == idx) bad = true;
        // succ(2c) = 2c+1 (a leaf unless the successor step writes the first
        // child); succ(2c+1) is always written by that step, so the pair is
        // stored whole: one full 8-byte store instead of a strided 4-byte one
        reinterpret_cast<int2*>(succ)[idx] = make_int2((int32_t)(2 * idx + 1), -2);
      }
    } else {
      key = raw[r];
    }
    atomicAdd(&h[wave][(key >> shift) & mask], 1u);
  }
  if (bad) flag(status, ST_BAD_PARENT);
  __syncthreads();
  for (int d = threadIdx.x; d <= (int)mask; d += kThreads)
    hist[(int64_t)d * ntiles + tile] = h[0][d] + h[1][d] + h[2][d] + h[3][d];
}

// BY_SOURCE: the last pass by target gives out every half-edge with its source
// for a key. The gather (6M half-edges: 95 us in a kernel of its own, 24 MB out
// and in again) is made from the sorted tile, all of a lane's loads together.
template <SortIn IN, bool BY_SOURCE, int DIG>
__global__ __launch_bounds__(kDownThreads, 2) void k_downsweep(const void* __restrict__ keys_in,
                                                        const int32_t* __restrict__ vals_in, HalfEdges he, int32_t n,
                                                        int shift, int nbits, int32_t ntiles,
                                                        const uint32_t* __restrict__ offsets,
                                                        uint32_t* __restrict__ keys_out,
                                                        int32_t* __restrict__ vals_out) {
  constexpr int kPer = (DIG + kDownThreads - 1) / kDownThreads;  // digits owned by one thread in the tile scan
  __shared__ __align__(16) uint16_t cnt[kDownWaves][DIG];  // (a wavefront has 512 keys, a tile 4096)
  __shared__ uint32_t lstart[DIG];   // tile-local start of each digit's run
  __shared__ uint32_t gstart[DIG];   // global start of this tile's run of each digit
  __shared__ uint32_t skey[kTile];
  __shared__ int32_t sval[kTile];
  const int wave = threadIdx.x >> 6;
  const uint32_t mask = (1u << nbits) - 1u;
  for (int i = threadIdx.x; i < kDownWaves * DIG / 2; i += kDownThreads) reinterpret_cast<uint32_t*>(&cnt[0][0])[i] = 0;
  __syncthreads();
  const int32_t tile = xcd_block(ntiles);
  const int64_t tbase = (int64_t)tile * kTile;
  const int64_t wbase = tbase + (int64_t)wave * (64 * kDownRounds) + __lane_id();
  const uint64_t below = lanemask_lt();
  uint32_t key[kDownRounds];
  int32_t val[kDownRounds];
  uint32_t rnk[kDownRounds];
#pragma unroll
  for (int r = 0; r < kDownRounds; ++r) {
    const int64_t idx = wbase + r * 64;
    const bool valid = idx < n;
    if (IN == IN_TARGET) {
      key[r] = valid ? he.clamp(he.target(idx)) : 0u;
      val[r] = (int32_t)idx;
    } else if (IN == IN_PARENT) {
      key[r] = valid ? parent_key(static_cast<const int32_t*>(keys_in)[idx], n) : 0u;
      val[r] = (int32_t)idx;
    } else {
      key[r] = valid ? static_cast<const uint32_t*>(keys_in)[idx] : 0u;
      val[r] = valid ? vals_in[idx] : 0;
    }
    const uint32_t dg = (key[r] >> shift) & mask;
    uint64_t peers = __ballot(valid);
#pragma unroll
    for (int b = 0; b < (DIG > 1024 ? 11 : DIG > 512 ? 10 : DIG > 256 ? 9 : 8); ++b) {
      if (b >= nbits) break;
      const bool bit = (dg >> b) & 1u;
      const uint64_t bal = __ballot(bit);
      peers &= bit ? bal : ~bal;
    }
    const uint32_t lower = (uint32_t)__popcll(peers & below);
    const uint32_t c0 = cnt[wave][dg];
    rnk[r] = c0 + lower;
    if (valid && lower == 0) cnt[wave][dg] = (uint16_t)(c0 + (uint32_t)__popcll(peers));
  }
  __syncthreads();
  // per digit: chain the wave counters, then an exclusive scan over digits
  // gives each digit's run inside the tile; thread t owns digits kPer*t ..
  // kPer*t + kPer - 1
  {
    uint32_t tots[kPer];
    uint32_t tot = 0;
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
      const int d = kPer * threadIdx.x + q;
      uint32_t td = 0;
      if (d < DIG && d <= (int)mask) {
#pragma unroll
        for (int w = 0; w < kDownWaves; ++w) {
          const uint32_t c = cnt[w][d];
          cnt[w][d] = (uint16_t)td;  // exclusive prefix over the waves
          td += c;
        }
        gstart[d] = offsets[(int64_t)d * ntiles + tile];
      }
      tots[q] = td;
      tot += td;
    }
    // block exclusive scan of the per-thread totals over the 512 threads (8 waves)
    uint32_t inc = tot;
    const int lane = __lane_id();
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const uint32_t u = __shfl_up(inc, o, 64);
      if (lane >= o) inc += u;
    }
    __shared__ uint32_t wsum[kDownWaves];
    if (lane == 63) wsum[wave] = inc;
    __syncthreads();
    uint32_t run = inc - tot;
    for (int w = 0; w < wave; ++w) run += wsum[w];
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
      const int d = kPer * threadIdx.x + q;
      if (d < DIG) lstart[d] = run;
      run += tots[q];
    }
  }
  __syncthreads();
  // place every key at its tile-local sorted position
#pragma unroll
  for (int r = 0; r < kDownRounds; ++r) {
    const int64_t idx = wbase + r * 64;
    if (idx < n) {
      const uint32_t dg = (key[r] >> shift) & mask;
      const uint32_t lp = lstart[dg] + cnt[wave][dg] + rnk[r];
      skey[lp] = key[r];
      sval[lp] = val[r];
    }
  }
  __syncthreads();
  // write the tile out digit run by digit run: consecutive lanes, consecutive addresses
  const int valid_in_tile = (int)min<int64_t>((int64_t)kTile, n - tbase);
  if (BY_SOURCE) {
#pragma unroll
    for (int r = 0; r < kDownRounds; ++r) {
      const int i = r * kDownThreads + threadIdx.x;
      key[r] = i < valid_in_tile ? (uint32_t)he.source(sval[i]) : 0u;
    }
  }
#pragma unroll
  for (int r = 0; r < kDownRounds; ++r) {
    const int i = r * kDownThreads + threadIdx.x;
    if (i < valid_in_tile) {
      const uint32_t k = skey[i];
      const uint32_t dg = (k >> shift) & mask;
      const uint32_t pos = gstart[dg] + (uint32_t)i - lstart[dg];
      keys_out[pos] = BY_SOURCE ? he.clamp((int32_t)key[r]) : k;
      vals_out[pos] = sval[i];
    }
  }
}

__global__ void k_reset_root(int32_t* __restrict__ scalars) {
  scalars[0] = -1;
  scalars[1] = 0;
}

// Digit widths of the passes over `bits` key bits of n keys, balanced: as few
// passes as digits of 9 bits allow, or of 11 bits up to 2^21 keys. Longer
// digits make shorter runs in a tile and more histogram entries, and where the
// tiles are no more than two a compute unit a saved pass (four launches) is
// worth more than both: widest digit 8 / 9 / 10 / 11 bits, time of the Euler
// tour in us, 245 / 214 (66000 nodes, 2 passes of 9), 310 / 309 / 296 (300000),
// 430 / 428 / 392 (2^20), 552 / 552 / 554 / 519 (2^21). At 2.5M nodes 11 bits
// cost 604 / 616, at 4M 775 / 819. For the longest arrays the traffic counts,
// three passes of 9 bits before four of 7 (2^25 nodes 5299 / 5219, 2^26 11305 /
// 11267) but not of 10 (2^27: 24175 with 9, 24449 with 10).
int plan_passes(int bits, int64_t n, int* width) {
  const int widest = n <= (1 << 21) ? kMaxBits : 9;
  const int passes = (bits + widest - 1) / widest;
  for (int p = 0; p < passes; ++p) width[p] = bits / passes + (p < bits % passes ? 1 : 0);
  return passes;
}

int key_bits(int64_t n) {
  int bits = 1;
  while (bits < 31 && (1ll << bits) < n) ++bits;
  return bits;
}

// entries of the widest pass's histogram (the first digit is the widest)
int64_t hist_entries(int bits, int32_t n) {
  int width[8];
  plan_passes(bits, n, width);
  return ((int64_t)1 << width[0]) * ceil_div(n, kTile);
}

// the kernels for a digit width
template <SortIn IN>
auto upsweep_for(int nbits) {
  return nbits > 10  ? k_upsweep<IN, 2048>
         : nbits > 9 ? k_upsweep<IN, 1024>
         : nbits > 8 ? k_upsweep<IN, 512>
                     : k_upsweep<IN, 256>;
}
template <SortIn IN, bool BY_SOURCE>
auto downsweep_for(int nbits) {
  return nbits > 10  ? k_downsweep<IN, BY_SOURCE, 2048>
         : nbits > 9 ? k_downsweep<IN, BY_SOURCE, 1024>
         : nbits > 8 ? k_downsweep<IN, BY_SOURCE, 512>
                     : k_downsweep<IN, BY_SOURCE, 256>;
}

// one pass: histograms, their scan, the scatter
template <SortIn IN, bool BY_SOURCE>
int sort_pass(Ctx* c, const void* kin, const int32_t* vin, HalfEdges he, int32_t n, int shift, int nbits,
              uint32_t* hist, uint32_t* kout, int32_t* vout, int32_t* succ, int32_t* scalars, hipStream_t s) {
  const int32_t ntiles = ceil_div(n, kTile);
  {
    ET_PROF(c, s, IN == IN_KEYS ? "k_upsweep<false>" : "k_upsweep<true>");
    hipLaunchKernelGGL(upsweep_for<IN>(nbits), dim3(ntiles), dim3(kThreads), 0, s, kin, he, n, shift, nbits, ntiles,
                       hist, succ, scalars, c->d_status);
  }
  const int rc = scan_u32(c, hist, hist, ((int64_t)1 << nbits) * ntiles, ScanOp::Add, true, s);
  if (rc) return rc;
  {
    ET_PROF(c, s, IN == IN_KEYS ? "k_downsweep<false>" : "k_downsweep<true>");
    hipLaunchKernelGGL((downsweep_for<IN, BY_SOURCE>(nbits)), dim3(ntiles), dim3(kDownThreads), 0, s, kin, vin, he, n,
                       shift, nbits, ntiles, hist, kout, vout);
  }
  return ET_OK;
}

}  // namespace

// histograms of every tile and the ping-pong keys and values, plus the
// largest histogram scan's partials
size_t group_by_parent_scratch_bytes(int32_t n) {
  int width[8];
  const int passes = plan_passes(key_bits(n), n, width);
  size_t scan = 0;
  for (int p = 0; p < passes; ++p)
    scan = std::max(scan, scan_scratch_bytes(((int64_t)1 << width[p]) * ceil_div(n, kTile)));
  return scratch_block<uint32_t>((size_t)hist_entries(key_bits(n), n)) + scratch_block<uint32_t>((size_t)n) +
         scratch_block<int32_t>((size_t)n) + scan;
}

// keys_out / vals_out receive the stable order; scalars[0] = root, scalars[1]
// = number of roots; succ[2c] of every non-root c is set to 2c+1 and
// succ[2c+1] to -2 (the successor step writes it), both root ids to -2.
int group_by_parent_impl(Ctx* c, const int32_t* parent, int32_t n, uint32_t* keys_out, int32_t* vals_out,
                         int32_t* succ, int32_t* scalars, hipStream_t s) {
  const int bits = key_bits(n);
  int width[8];
  const int passes = plan_passes(bits, n, width);
  Scratch sc(c, s);
  uint32_t* hist = sc.get<uint32_t>((size_t)hist_entries(bits, n));
  uint32_t* tk = sc.get<uint32_t>((size_t)n);
  int32_t* tv = sc.get<int32_t>((size_t)n);
  if (sc.failed) return ET_ENOMEM;
  hipLaunchKernelGGL(k_reset_root, dim3(1), dim3(1), 0, s, scalars);
  const void* kin = parent;
  const int32_t* vin = nullptr;
  for (int p = 0, shift = 0; p < passes; shift += width[p], ++p) {
    const bool to_out = ((passes - 1 - p) % 2) == 0;
    uint32_t* kout = to_out ? keys_out : tk;
    int32_t* vout = to_out ? vals_out : tv;
    const auto pass = p == 0 ? sort_pass<IN_PARENT, false> : sort_pass<IN_KEYS, false>;
    const int rc = pass(c, kin, vin, HalfEdges{}, n, shift, width[p], hist, kout, vout, succ, scalars, s);
    if (rc) return rc;
    kin = kout;
    vin = vout;
  }
  return hipGetLastError() == hipSuccess ? ET_OK : ET_EHIP;
}

// The half-edges of an edge list in lexicographic order of {source, target}:
// stably by target, then stably by source, in passes over the half-edge ids
// between {key0, val0} and {key1, val1}; key1 / val1 receive the sources and
// the ids. Ends out of range are flagged (as are self-loops) and count as 0.
int sort_half_edges(Ctx* c, HalfEdges he, int32_t L, uint32_t* key0, int32_t* val0, uint32_t* key1, int32_t* val1,
                    hipStream_t s) {
  const int bits = key_bits(he.n);
  int width[8];
  const int passes = plan_passes(bits, L, width);
  Scratch sc(c, s);
  uint32_t* hist = sc.get<uint32_t>((size_t)hist_entries(bits, L));
  if (sc.failed) return ET_ENOMEM;
  const void* kin = nullptr;
  const int32_t* vin = nullptr;
  for (int q = 0, shift = 0; q < 2 * passes; ++q) {
    const int p = q % passes;
    if (p == 0) shift = 0;
    const bool last_by_target = q == passes - 1;
    const auto pass = q == 0 ? (last_by_target ? sort_pass<IN_TARGET, true> : sort_pass<IN_TARGET, false>)
                             : (last_by_target ? sort_pass<IN_KEYS, true> : sort_pass<IN_KEYS, false>);
    uint32_t* kout = (q & 1) ? key1 : key0;  // an even number of passes: the last one is odd
    int32_t* vout = (q & 1) ? val1 : val0;
    const int rc = pass(c, kin, vin, he, L, shift, width[p], hist, kout, vout, nullptr, nullptr, s);
    if (rc) return rc;
    shift += width[p];
    kin = kout;
    vin = vout;
  }
  return hipGetLastError() == hipSuccess ? ET_OK : ET_EHIP;
}

}  // namespace et
