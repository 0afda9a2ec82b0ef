// Initialization stage (Sec. 2.1, stage 1): leaf assignment and a stable sort
// of the points by leaf Morton key, plus gather/scatter of per-point rows.
//
// The sort is a least-significant-digit radix sort of the 2*depth-bit keys in
// as few passes as digits of at most 9 bits allow (one up to depth 4, two up
// to depth 9, three above; a 10-bit digit's runs in a tile are too short:
// 460 us in two passes against 410 in three at 2^24 points, depth 10), or of
// at most 8 bits below kWideFrom points (two passes up to depth 8).  A
// pass is three launches: digit counts of each workgroup's contiguous range
// of items, an exclusive scan of every digit's row of counts, and a scatter.
// The scatter ranks a tile of items stably
// (wave ballots over the digit's bits, counts per wave, a scan over the
// digits), reorders the tile in LDS and writes runs of equal digits to
// consecutive addresses.  Every rank follows from the input order, so the
// result is stable and deterministic.  Up to kSmall points one workgroup
// sorts in LDS in one launch, by digits of at most 8 bits.
//
// Keys are formed from the points again in the first pass instead of being
// stored by the counting launch: 8 bytes read for 4 written and 4 read.
//
// Bound by the scatters: at 2^24 points, depth 10, 85 us a pass for 256 MB
// read and written (53 us at the rate of a large copy), 40 + 2 x 14 us of
// counting, 3 x 6 of scans, 26 of leaf starts.  Whole build, against 4-bit
// digits with five launches a pass: 382 us against 762 at 2^24 points, 47
// against 125 at 2^20 (depth 8), 11 against 48 at 4096 (depth 4).
#include <algorithm>

#include "fmm2d_internal.h"

namespace fmm2d {

using tree_ws::align256;

constexpr int kThreads = 512;             // of a counting or scattering workgroup
constexpr int kWaves = kThreads / 64;
constexpr int kMaxBits = 9, kMaxBins = 1 << kMaxBits;
constexpr int kMaxBlocks = 512;           // ranges: two workgroups a compute unit (1024: 16% slower at 4M points)
constexpr int64_t kSmall = 8192;          // points one workgroup sorts by itself
constexpr int64_t kWideFrom = 65536;      // points from which digits of 9 bits are used

// The passes of one build: digit width, passes, items a thread (tile), ranges.
struct SortPlan {
  int bits, passes, items, blocks;
  int64_t range;  // items of a workgroup, a multiple of the tile
};

static SortPlan plan_of(int64_t n, int depth) {
  SortPlan p;
  // 8-bit digits below kWideFrom points keep the counts within the workspace
  const int most = n < kWideFrom ? 8 : kMaxBits;
  p.passes = (2 * depth + most - 1) / most;
  p.bits = (2 * depth + p.passes - 1) / p.passes;
  // tiles of 4096 items once they give a workgroup to every compute unit
  // (48 against 53 us at 2^20 points; 38 against 34 at 250000), of 2048
  // below; tiles of 8192 leave too few waves a unit (530 against 410 us at
  // 2^24 points)
  p.items = n >= int64_t(256) * kThreads * 8 ? 8 : 4;
  const int64_t tile = int64_t(kThreads) * p.items, tiles = (n + tile - 1) / tile;
  p.blocks = int(tiles < kMaxBlocks ? tiles : kMaxBlocks);
  p.range = (tiles + p.blocks - 1) / p.blocks * tile;
  p.blocks = int((n + p.range - 1) / p.range);
  return p;
}

struct TreeWs {
  uint32_t *keys[2];
  int32_t *vals;
  uint32_t *count;  // [bins][blocks], a row's exclusive scan after scan_rows_kernel
  uint32_t *total;  // [bins]
  uint32_t *bad;    // [blocks]: a point of the range lies outside the domain
  size_t bytes;
};

static TreeWs carve(void *ws, int64_t n, int bins, int blocks) {
  char *p = static_cast<char *>(ws);
  TreeWs w;
  const size_t kb = align256(size_t(n) * 4);
  w.keys[0] = reinterpret_cast<uint32_t *>(p); p += kb;
  w.keys[1] = reinterpret_cast<uint32_t *>(p); p += kb;
  w.vals = reinterpret_cast<int32_t *>(p); p += kb;
  w.count = reinterpret_cast<uint32_t *>(p); p += align256(size_t(bins) * blocks * 4);
  w.total = reinterpret_cast<uint32_t *>(p); p += align256(size_t(bins) * 4);
  w.bad = reinterpret_cast<uint32_t *>(p); p += align256(size_t(blocks) * 4);
  w.bytes = size_t(p - static_cast<char *>(ws));
  return w;
}

size_t build_tree_ws_bytes(int64_t n, int depth) {
  (void)depth;
  return tree_ws::bytes(n);
}

// Leaf key of a point; `bad` is set for one outside [0,1]^2 (NaN included).
__device__ inline uint32_t leaf_key(float2 p, int depth, bool &bad) {
  const bool inside = (p.x >= 0.f && p.x <= 1.f && p.y >= 0.f && p.y <= 1.f);
  bad = bad || !inside;
  const float side = float(1 << depth);  // x * 2^depth is exact in FP32
  const int lim = (1 << depth) - 1;
  const int ix = inside ? min(int(floorf(p.x * side)), lim) : 0;
  const int iy = inside ? min(int(floorf(p.y * side)), lim) : 0;
  return morton2(uint32_t(ix), uint32_t(iy));
}

// Inclusive scan over the wave.
__device__ inline uint32_t wave_scan(uint32_t v, int lane) {
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const uint32_t u = __shfl_up(v, d);
    if (lane >= d) v += u;
  }
  return v;
}

// In place: exclusive scan of v[0..bins) in LDS by the whole workgroup;
// `part` holds one value a wave.  Starts and ends with a barrier.
template <int THREADS>
__device__ inline void block_scan(uint32_t *v, int bins, uint32_t *part) {
  const int t = threadIdx.x, wave = t >> 6, lane = t & 63;
  const int per = (bins + THREADS - 1) / THREADS;  // consecutive values of a thread
  __syncthreads();
  uint32_t s = 0;
  for (int i = 0; i < per; ++i) s += t * per + i < bins ? v[t * per + i] : 0u;
  const uint32_t inc = wave_scan(s, lane);
  if (lane == 63) part[wave] = inc;
  __syncthreads();
  uint32_t off = inc - s;
  for (int w = 0; w < wave; ++w) off += part[w];
  for (int i = 0; i < per; ++i) {
    if (t * per + i >= bins) break;
    const uint32_t x = v[t * per + i];
    v[t * per + i] = off;
    off += x;
  }
  __syncthreads();
}

// Stable ranks of a tile.  Wave w holds items (w ITEMS + r) 64 + lane in
// round r, so (wave, round, lane) is the tile's order.  rank[r] becomes the
// number of earlier items of the same digit in the wave; hist[w][d] the
// number of items with digit d in wave w.
template <int ITEMS, int BITS>
__device__ inline void wave_ranks(const int (&dig)[ITEMS], uint16_t (&rank)[ITEMS], volatile uint16_t *hist,
                                  int lane) {
  const uint64_t lt_mask = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
#pragma unroll
  for (int r = 0; r < ITEMS; ++r) {
    const bool live = dig[r] >= 0;
    uint64_t same = __ballot(live);
#pragma unroll
    for (int b = 0; b < BITS; ++b) {
      const int bit = (dig[r] << (31 - b)) >> 31;  // 0 or -1
      const uint64_t m = __ballot(bit != 0);
      same &= ~(m ^ uint64_t(int64_t(bit)));
    }
    if (live) {
      const uint32_t before = hist[dig[r]];
      rank[r] = uint16_t(before + __popcll(same & lt_mask));
      // the wave's LDS accesses complete in order: all lanes have read
      if ((same & lt_mask) == 0) hist[dig[r]] = uint16_t(before + __popcll(same));
    }
    __builtin_amdgcn_wave_barrier();
  }
}

// Digit counts of each range, from the points (FIRST) or the keys.
template <bool FIRST>
__global__ __launch_bounds__(kThreads) void digit_count_kernel(const float2 *__restrict__ xy,
                                                               const uint32_t *__restrict__ keys, int64_t n, int depth,
                                                               int shift, int bits, int64_t range,
                                                               uint32_t *__restrict__ count,
                                                               uint32_t *__restrict__ bad) {
  __shared__ uint32_t hist[kMaxBins];
  const int bins = 1 << bits;
  for (int d = threadIdx.x; d < bins; d += kThreads) hist[d] = 0;
  __syncthreads();
  const int64_t b0 = blockIdx.x * range, b1 = min(b0 + range, n);
  bool out = false;
  int64_t i = b0 + threadIdx.x;
  constexpr int kAhead = 8;  // loads in flight a thread
  for (; i + (kAhead - 1) * kThreads < b1; i += kAhead * kThreads) {
    float2 z[kAhead];
    uint32_t key[kAhead];
#pragma unroll
    for (int r = 0; r < kAhead; ++r) {
      if (FIRST) z[r] = xy[i + r * kThreads];
      else key[r] = keys[i + r * kThreads];
    }
#pragma unroll
    for (int r = 0; r < kAhead; ++r) {
      if (FIRST) key[r] = leaf_key(z[r], depth, out);
      atomicAdd(&hist[(key[r] >> shift) & uint32_t(bins - 1)], 1u);
    }
  }
  for (; i < b1; i += kThreads) {
    const uint32_t key = FIRST ? leaf_key(xy[i], depth, out) : keys[i];
    atomicAdd(&hist[(key >> shift) & uint32_t(bins - 1)], 1u);
  }
  const int any = __syncthreads_or(out);
  for (int d = threadIdx.x; d < bins; d += kThreads) count[int64_t(d) * gridDim.x + blockIdx.x] = hist[d];
  if (FIRST && threadIdx.x == 0) bad[blockIdx.x] = any ? 1u : 0u;
}

// Exclusive scan of each digit's row of counts (one wave a row, at most
// kMaxBlocks values) and the row's total; the first pass also collects the
// domain flag.
__global__ __launch_bounds__(256) void scan_rows_kernel(uint32_t *__restrict__ count, int bins, int blocks,
                                                        uint32_t *__restrict__ total,
                                                        const uint32_t *__restrict__ bad,
                                                        uint32_t *__restrict__ domain_flag) {
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  if (domain_flag && blockIdx.x == 0 && wave == 0) {
    bool any = false;
    for (int b = lane; b < blocks; b += 64) any = any || bad[b] != 0u;
    if (__ballot(any) == 0ull) {
      if (lane == 0) *domain_flag = 0u;
    } else if (lane == 0) {
      *domain_flag = 1u;
    }
  }
  const int d = blockIdx.x * 4 + wave;
  if (d >= bins) return;
  uint32_t *row = count + int64_t(d) * blocks;
  uint32_t run = 0;
  for (int b0 = 0; b0 < blocks; b0 += 64) {
    const int b = b0 + lane;
    const uint32_t v = b < blocks ? row[b] : 0u;
    const uint32_t inc = wave_scan(v, lane);
    if (b < blocks) row[b] = run + inc - v;
    run += __shfl(inc, 63);
  }
  if (lane == 0) total[d] = run;
}

struct ScatterArgs {
  const float2 *xy;     // the points: the caller's, or with xout those of the pass before
  const uint32_t *kin;  // keys and values of the pass before
  const int32_t *vin;
  uint32_t *kout;
  int32_t *vout;
  int64_t n;
  int depth, shift;
  int32_t *leaf_start;
  const float *qin;   // with xout, the caller's charges (or null)
  const uint2 *qvin;  // with xout, (charge, value) of the pass before, values without charges
  float2 *xout;       // the points in this pass's order, if they are wanted
  uint2 *qvout;       // with xout: (charge, value), or null in the last pass, which
  float *qout;        // writes vout (or null: not wanted) and qout
};

// One pass's scatter.  FIRST: keys from the points, values are the indices.
// kout may be null (a single pass needs no sorted keys); leaf_start is then
// the digits' starts, written by workgroup 0.
//
// POINTS: the points move along, so that the last pass leaves them sorted, in
// runs instead of by random reads afterwards (4e6 points, depth 9: gathers of
// 140 us).  Their keys are formed anew in each pass, and between passes a
// point's value and charge are one 8-byte item (qv; without CHARGES the value
// alone), so a digit's run in a
// tile is two pieces of 8 bytes an item and not four of 8 and 4: each piece's
// ends are lines that several tiles write (first scatter of 4e6 points, depth
// 9: 57 us against 78, with keys moved too; of 6.5e6, depth 8: 74 against 92;
// counting reads the points again for it, 12 and 16 us against 7;
// the second one 82 us, 72 without the permutation and 66 without charges).
template <int ITEMS, int BITS, bool FIRST, bool POINTS, bool CHARGES>
__global__ __launch_bounds__(kThreads) void digit_scatter_kernel(ScatterArgs a, int64_t range,
                                                                 const uint32_t *__restrict__ count,
                                                                 const uint32_t *__restrict__ total) {
  constexpr int kTile = kThreads * ITEMS, bins = 1 << BITS;
  __shared__ uint2 buf[kTile];                  // what moves, in digit order
  __shared__ uint16_t hist[kWaves][bins];       // per wave counts, then offsets
  __shared__ uint32_t start[bins], goff[bins];  // of each digit: in the tile, in the output
  __shared__ uint32_t part[kWaves];
  const float2 *__restrict__ xy = a.xy;
  const uint32_t *__restrict__ kin = a.kin;
  const int32_t *__restrict__ vin = a.vin;
  const uint2 *__restrict__ qvin = a.qvin;
  const uint32_t *__restrict__ idin = reinterpret_cast<const uint32_t *>(a.qvin);
  uint32_t *const buf32 = reinterpret_cast<uint32_t *>(buf);
  const float *__restrict__ qin = a.qin;
  const int64_t n = a.n;
  const uint32_t mask = uint32_t(bins - 1);
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, shift = a.shift, depth = a.depth;
  for (int d = threadIdx.x; d < bins; d += kThreads) goff[d] = total[d];
  block_scan<kThreads>(goff, bins, part);
  if (a.leaf_start && blockIdx.x == 0) {
    for (int d = threadIdx.x; d < bins; d += kThreads) a.leaf_start[d] = int32_t(goff[d]);
    if (threadIdx.x == 0) a.leaf_start[bins] = int32_t(n);
    __syncthreads();
  }
  for (int d = threadIdx.x; d < bins; d += kThreads) goff[d] += count[int64_t(d) * gridDim.x + blockIdx.x];

  const int64_t b0 = blockIdx.x * range, b1 = min(b0 + range, n);
  for (int64_t t0 = b0; t0 < b1; t0 += kTile) {
    const int live = int(min(int64_t(kTile), b1 - t0));
    uint32_t key[ITEMS];
    uint2 kv[ITEMS];  // (key, value); POINTS: (charge, value)
    int dig[ITEMS];
    uint16_t rank[ITEMS];
    float2 z[ITEMS];
    const int at = wave * ITEMS * 64 + lane;
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
      const int e = at + r * 64;
      const int64_t i = t0 + (e < live ? e : 0);
      bool out = false;
      if (FIRST || POINTS) z[r] = xy[i];
      key[r] = FIRST || POINTS ? leaf_key(z[r], depth, out) : kin[i];
      if (POINTS && !FIRST) kv[r] = CHARGES ? qvin[i] : make_uint2(0u, idin[i]);
      else if (POINTS) kv[r] = make_uint2(CHARGES ? __float_as_uint(qin[i]) : 0u, uint32_t(i));
      else kv[r] = make_uint2(key[r], FIRST ? uint32_t(i) : uint32_t(vin[i]));
      dig[r] = e < live ? int((key[r] >> shift) & mask) : -1;
    }
    for (int d = lane; d < bins; d += 64) hist[wave][d] = 0;
    __builtin_amdgcn_wave_barrier();
    wave_ranks<ITEMS, BITS>(dig, rank, hist[wave], lane);
    __syncthreads();
    for (int d = threadIdx.x; d < bins; d += kThreads) {
      uint32_t run = 0;
#pragma unroll
      for (int w = 0; w < kWaves; ++w) {
        const uint32_t c = hist[w][d];
        hist[w][d] = uint16_t(run);
        run += c;
      }
      start[d] = run;
    }
    block_scan<kThreads>(start, bins, part);
    int pos[ITEMS];
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
      pos[r] = dig[r] >= 0 ? int(start[dig[r]]) + hist[wave][dig[r]] + rank[r] : -1;
      if (pos[r] >= 0) buf[pos[r]] = POINTS ? make_uint2(__float_as_uint(z[r].x), __float_as_uint(z[r].y)) : kv[r];
    }
    __syncthreads();
    uint32_t dst[ITEMS];
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
      const int e = r * kThreads + threadIdx.x;
      if (e < live) {
        const uint2 v = buf[e];
        const float2 p = make_float2(__uint_as_float(v.x), __uint_as_float(v.y));
        bool out = false;
        const uint32_t d = ((POINTS ? leaf_key(p, depth, out) : v.x) >> shift) & mask;
        dst[r] = goff[d] + uint32_t(e) - start[d];
        if (POINTS) {
          a.xout[dst[r]] = p;
        } else {
          if (a.kout) a.kout[dst[r]] = v.x;
          a.vout[dst[r]] = int32_t(v.y);
        }
      }
    }
    __syncthreads();
    // the digits' next output addresses
    for (int d = threadIdx.x; d < bins; d += kThreads)
      goff[d] += (d + 1 < bins ? start[d + 1] : uint32_t(live)) - start[d];
    if (POINTS) {
#pragma unroll
      for (int r = 0; r < ITEMS; ++r) {
        if (pos[r] < 0) continue;
        if (CHARGES) buf[pos[r]] = kv[r];
        else buf32[pos[r]] = kv[r].y;
      }
      __syncthreads();
#pragma unroll
      for (int r = 0; r < ITEMS; ++r) {
        const int e = r * kThreads + threadIdx.x;
        if (e >= live) continue;
        const uint2 v = CHARGES ? buf[e] : make_uint2(0u, buf32[e]);
        if (a.qvout) {
          if (CHARGES) a.qvout[dst[r]] = v;
          else reinterpret_cast<uint32_t *>(a.qvout)[dst[r]] = v.y;
        } else {
          if (a.vout) a.vout[dst[r]] = int32_t(v.y);
          if (CHARGES) a.qout[dst[r]] = __uint_as_float(v.x);
        }
      }
      __syncthreads();
    }
  }
}

// leaf_start[m] = first sorted position whose key is >= m: a binary search
// within the range of m's top digit (the last pass's totals, scanned here;
// without totals one range of all keys).
// The keys are those of the sorted points where keys is null.
__global__ __launch_bounds__(256) void leaf_start_kernel(const uint32_t *__restrict__ keys,
                                                         const float2 *__restrict__ points, int depth, int64_t n,
                                                         int64_t nleaf, int shift, int bins,
                                                         const uint32_t *__restrict__ total,
                                                         int32_t *__restrict__ leaf_start) {
  __shared__ uint32_t base[kMaxBins], part[4];
  for (int d = threadIdx.x; d < bins; d += 256) base[d] = total ? total[d] : 0u;
  block_scan<256>(base, bins, part);
  const int64_t step = int64_t(gridDim.x) * 256;
  for (int64_t m = blockIdx.x * int64_t(256) + threadIdx.x; m <= nleaf; m += step) {
    const int d = int(m >> shift);
    int64_t lo = d < bins ? int64_t(base[d]) : n, hi = d + 1 < bins ? int64_t(base[d + 1]) : n;
    while (lo < hi) {
      const int64_t mid = (lo + hi) >> 1;
      bool out = false;
      if (int64_t(keys ? keys[mid] : leaf_key(points[mid], depth, out)) < m) lo = mid + 1;
      else hi = mid;
    }
    leaf_start[m] = int32_t(lo);
  }
}

// The whole build of at most kSmall points by one workgroup of 1024 threads:
// the same passes on 8-bit digits, with the items in registers and reordered
// through LDS.  Bound by its chain of barriers and waits, 11 us for 4096
// points at depth 4 (13 with keys and indices exchanged one after the other
// and the sorted points gathered from memory), 14.5 at depth 8 (15.6); of that
// about 2 us are any launch's.  Leaf starts come from the sorted keys in LDS; a tree of more
// than kSmallLeaves leaves leaves them to leaf_start_kernel and the keys in
// keys_out.
constexpr int kSmallThreads = 1024, kSmallWaves = kSmallThreads / 64;
constexpr int64_t kSmallLeaves = 4096;  // four searches a thread

template <int ITEMS>
__global__ __launch_bounds__(kSmallThreads) void small_tree_kernel(const float2 *__restrict__ xy, int n, int depth,
                                                                   int32_t *__restrict__ perm,
                                                                   int32_t *__restrict__ leaf_start,
                                                                   uint32_t *__restrict__ keys_out,
                                                                   uint32_t *__restrict__ domain_flag,
                                                                   const float *__restrict__ q,
                                                                   float2 *__restrict__ xs, float *__restrict__ qs) {
  constexpr int kBins = 256;
  __shared__ uint32_t buf[kSmallThreads * ITEMS];
  __shared__ uint16_t hist[kSmallWaves][kBins];
  __shared__ uint32_t start[kBins], part[kSmallWaves];
  // the points and charges in the caller's order, for the gather at the end
  __shared__ float2 points[kSmallThreads * ITEMS];
  __shared__ float charges[kSmallThreads * ITEMS];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  uint32_t key[ITEMS];
  int32_t val[ITEMS];
  bool out = false;
  const int at = wave * ITEMS * 64 + lane;
#pragma unroll
  for (int r = 0; r < ITEMS; ++r) {
    const int e = at + r * 64;
    const float2 z = e < n ? xy[e] : make_float2(0.f, 0.f);
    key[r] = leaf_key(z, depth, out);
    val[r] = e;
    points[e] = z;
    if (xs && q) charges[e] = e < n ? q[e] : 0.f;
  }
  const int any = __syncthreads_or(out);
  if (threadIdx.x == 0) *domain_flag = any ? 1u : 0u;
  const int passes = (2 * depth + 7) / 8, bits = (2 * depth + passes - 1) / passes, bins = 1 << bits;
  constexpr int kIndexBits = 13;
  static_assert((1 << kIndexBits) >= kSmallThreads * ITEMS, "an index fits");
  const bool packed = 2 * depth + kIndexBits <= 32;  // key and index change places as one word
  for (int shift = 0; shift < 2 * depth; shift += bits) {
    int dig[ITEMS], pos[ITEMS];
    uint16_t rank[ITEMS];
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) dig[r] = at + r * 64 < n ? int((key[r] >> shift) & uint32_t(bins - 1)) : -1;
    for (int d = lane; d < bins; d += 64) hist[wave][d] = 0;
    __builtin_amdgcn_wave_barrier();
    wave_ranks<ITEMS, 8>(dig, rank, hist[wave], lane);
    __syncthreads();
    if (int(threadIdx.x) < bins) {
      uint32_t run = 0;
#pragma unroll
      for (int w = 0; w < kSmallWaves; ++w) {
        const uint32_t c = hist[w][threadIdx.x];
        hist[w][threadIdx.x] = uint16_t(run);
        run += c;
      }
      start[threadIdx.x] = run;
    }
    block_scan<kSmallThreads>(start, bins, part);
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
      pos[r] = dig[r] >= 0 ? int(start[dig[r]]) + hist[wave][dig[r]] + rank[r] : -1;
      if (pos[r] >= 0) buf[pos[r]] = packed ? key[r] << kIndexBits | uint32_t(val[r]) : uint32_t(val[r]);
    }
    __syncthreads();
    if (packed) {
#pragma unroll
      for (int r = 0; r < ITEMS; ++r) {
        if (dig[r] < 0) continue;
        const uint32_t w = buf[at + r * 64];
        key[r] = w >> kIndexBits;
        val[r] = int32_t(w & ((1u << kIndexBits) - 1u));
      }
      continue;
    }
#pragma unroll
    for (int r = 0; r < ITEMS; ++r)
      if (dig[r] >= 0) val[r] = int32_t(buf[at + r * 64]);
    __syncthreads();
#pragma unroll
    for (int r = 0; r < ITEMS; ++r)
      if (pos[r] >= 0) buf[pos[r]] = key[r];
    __syncthreads();
#pragma unroll
    for (int r = 0; r < ITEMS; ++r)
      if (dig[r] >= 0) key[r] = buf[at + r * 64];
  }
  // buf holds the sorted keys, packed with the indices or not
#pragma unroll
  for (int r = 0; r < ITEMS; ++r)
    if (at + r * 64 < n) {
      if (perm) perm[at + r * 64] = val[r];
      if (xs) xs[at + r * 64] = points[val[r]];
      if (xs && q) qs[at + r * 64] = charges[val[r]];
      if (keys_out) keys_out[at + r * 64] = key[r];
    }
  if (keys_out) return;
  const int nleaf = 1 << (2 * depth);
  if (passes == 1) {  // the digits are the leaves
    for (int m = threadIdx.x; m <= nleaf; m += kSmallThreads) leaf_start[m] = m < nleaf ? int32_t(start[m]) : n;
    return;
  }
  for (int m = threadIdx.x; m <= nleaf; m += kSmallThreads) {
    int lo = 0, hi = n;
    while (lo < hi) {
      const int mid = (lo + hi) >> 1;
      if (int(packed ? buf[mid] >> kIndexBits : buf[mid]) < m) lo = mid + 1;
      else hi = mid;
    }
    leaf_start[m] = lo;
  }
}

__global__ void empty_tree_kernel(int64_t nleaf, int32_t *__restrict__ leaf_start, uint32_t *__restrict__ flag) {
  const int64_t m = blockIdx.x * int64_t(blockDim.x) + threadIdx.x;
  if (m <= nleaf) leaf_start[m] = 0;
  if (m == 0) *flag = 0u;
}

template <int ITEMS, int BITS>
static void launch_scatter(bool first, const SortPlan &pl, const TreeWs &w, const ScatterArgs &a, hipStream_t s) {
  const dim3 g(unsigned(pl.blocks)), b(kThreads);
#define LAUNCH(FIRST, POINTS, CHARGES)                                                                          \
  hipLaunchKernelGGL((digit_scatter_kernel<ITEMS, BITS, FIRST, POINTS, CHARGES>), g, b, 0, s, a, pl.range, w.count, \
                     w.total)
  if (!a.xout) {
    if (first) LAUNCH(true, false, false);
    else LAUNCH(false, false, false);
  } else if (a.qin) {
    if (first) LAUNCH(true, true, true);
    else LAUNCH(false, true, true);
  } else {
    if (first) LAUNCH(true, true, false);
    else LAUNCH(false, true, false);
  }
#undef LAUNCH
}

size_t sort_points_ws_bytes(int64_t n) {
  return align256(tree_ws::bytes(n)) + 2 * align256(size_t(n) * 8);
}

int launch_build_tree(const float *xy, int64_t n, int depth, int32_t *perm, int32_t *leaf_start,
                      uint32_t *domain_flag, void *ws, hipStream_t s) {
  return launch_sort_points(xy, nullptr, n, depth, perm, leaf_start, domain_flag, nullptr, nullptr, ws, s);
}

int launch_sort_points(const float *xy, const float *q, int64_t n, int depth, int32_t *perm, int32_t *leaf_start,
                       uint32_t *domain_flag, float *xs, float *qs, void *ws, hipStream_t s) {
  float2 *xsorted = reinterpret_cast<float2 *>(xs);
  const int64_t nleaf = int64_t(1) << (2 * depth);
  const float2 *z = reinterpret_cast<const float2 *>(xy);
  if (n == 0) {
    hipLaunchKernelGGL(empty_tree_kernel, dim3(unsigned((nleaf + 1 + 255) / 256)), dim3(256), 0, s, nleaf, leaf_start,
                       domain_flag);
    return check_launch("build_tree");
  }
  const unsigned lblocks = unsigned(std::min<int64_t>((nleaf + 1 + 255) / 256, 2048));
  if (n <= kSmall) {
    const dim3 g(1), b(kSmallThreads);
    uint32_t *ko = nleaf > kSmallLeaves ? static_cast<uint32_t *>(ws) : nullptr;
    if (n <= kSmallThreads)
      hipLaunchKernelGGL(small_tree_kernel<1>, g, b, 0, s, z, int(n), depth, perm, leaf_start, ko, domain_flag,
                         q, xsorted, qs);
    else if (n <= 4 * kSmallThreads)
      hipLaunchKernelGGL(small_tree_kernel<4>, g, b, 0, s, z, int(n), depth, perm, leaf_start, ko, domain_flag,
                         q, xsorted, qs);
    else
      hipLaunchKernelGGL(small_tree_kernel<8>, g, b, 0, s, z, int(n), depth, perm, leaf_start, ko, domain_flag,
                         q, xsorted, qs);
    if (ko)
      hipLaunchKernelGGL(leaf_start_kernel, dim3(lblocks), dim3(256), 0, s, ko, static_cast<const float2 *>(nullptr), depth,
                         n, nleaf, 2 * depth + 1, 1, static_cast<const uint32_t *>(nullptr), leaf_start);
    return check_launch("build_tree");
  }
  const SortPlan pl = plan_of(n, depth);
  const TreeWs w = carve(ws, n, 1 << pl.bits, pl.blocks);
  if (w.bytes > build_tree_ws_bytes(n, depth))
    return set_error(FMM2D_EWORKSPACE, "build_tree: the sort needs %zu bytes", w.bytes);
  const dim3 g(unsigned(pl.blocks)), b(kThreads);
  uint32_t *kin = nullptr, *kout = w.keys[0];
  int32_t *vin = nullptr;
  // with points: their second buffer and one of (charge, value) lie behind the
  // tree build's workspace; the other takes the place of the keys, which are
  // formed from the points
  char *extra = static_cast<char *>(ws) + align256(tree_ws::bytes(n));
  float2 *xtmp = reinterpret_cast<float2 *>(extra);
  uint2 *qv[2] = {reinterpret_cast<uint2 *>(w.keys[0]), reinterpret_cast<uint2 *>(extra + align256(size_t(n) * 8))};
  const float2 *xin = z;
  for (int pass = 0; pass < pl.passes; ++pass) {
    const bool first = pass == 0, last = pass == pl.passes - 1, only = pl.passes == 1;
    const int shift = pass * pl.bits, bits = last ? 2 * depth - shift : pl.bits, bins = 1 << bits;
    // values (and points) alternate between the outputs and the workspace so
    // that the last pass writes the outputs
    const bool own = (pl.passes - 1 - pass) % 2 == 0;
    int32_t *vout = own ? perm : w.vals;
    float2 *xout = !xs ? nullptr : own ? xsorted : xtmp;
    if (first || xs)
      hipLaunchKernelGGL(digit_count_kernel<true>, g, b, 0, s, xin, kin, n, depth, shift, bits, pl.range, w.count, w.bad);
    else
      hipLaunchKernelGGL(digit_count_kernel<false>, g, b, 0, s, z, kin, n, depth, shift, bits, pl.range, w.count,
                         w.bad);
    hipLaunchKernelGGL(scan_rows_kernel, dim3(unsigned((bins + 3) / 4)), dim3(256), 0, s, w.count, bins, pl.blocks,
                       w.total, w.bad, first ? domain_flag : nullptr);
    ScatterArgs sa{xin, kin, vin, only ? nullptr : kout, vout, n, depth, shift, only ? leaf_start : nullptr,
                   nullptr, nullptr, nullptr, nullptr, nullptr};
    if (xs) {
      sa.qin = q;
      sa.qvin = qv[(pass + 1) % 2];
      sa.xout = xout;
      sa.qvout = last ? nullptr : qv[pass % 2];
      sa.qout = q ? qs : nullptr;
    }
    switch (bits) {
#define X(N_)                                                       \
  case N_:                                                          \
    if (pl.items == 8) launch_scatter<8, N_>(first, pl, w, sa, s);  \
    else launch_scatter<4, N_>(first, pl, w, sa, s);                \
    break;
      X(2) X(3) X(4) X(5) X(6) X(7) X(8) X(9)
#undef X
    }
    if (last && !only)
      hipLaunchKernelGGL(leaf_start_kernel, dim3(lblocks), dim3(256), 0, s, xs ? static_cast<const uint32_t *>(nullptr) : kout,
                         xsorted, depth, n, nleaf,
                         shift, bins, w.total, leaf_start);
    kin = kout;
    kout = kout == w.keys[0] ? w.keys[1] : w.keys[0];
    vin = vout;
    if (xs) xin = xout;
  }
  return check_launch("build_tree");
}

__global__ void gather_kernel(const float *__restrict__ src, const int32_t *__restrict__ perm, int64_t n, int width,
                              float *__restrict__ dst, bool scatter) {
  const int64_t e = blockIdx.x * int64_t(blockDim.x) + threadIdx.x;
  if (e >= n * width) return;
  const int64_t i = e / width;
  const int c = int(e - i * width);
  if (scatter) dst[int64_t(perm[i]) * width + c] = src[e];
  else dst[e] = src[int64_t(perm[i]) * width + c];
}

// Rows of 1, 2 or 4 floats (charges, positions, complex values; pairs of
// complex values) move as one vector access per row: no index division, and
// one load of perm per row.
template <typename V>
__global__ void gather_rows_kernel(const V *__restrict__ src, const int32_t *__restrict__ perm, int64_t n,
                                   V *__restrict__ dst, bool scatter) {
  const int64_t i = blockIdx.x * int64_t(blockDim.x) + threadIdx.x;
  if (i >= n) return;
  const int64_t j = perm[i];
  if (scatter) dst[j] = src[i];
  else dst[i] = src[j];
}

template <typename V>
void launch_rows(const float *src, const int32_t *perm, int64_t n, float *dst, bool scatter, hipStream_t s) {
  hipLaunchKernelGGL(gather_rows_kernel<V>, dim3(unsigned((n + 255) / 256)), dim3(256), 0, s,
                     reinterpret_cast<const V *>(src), perm, n, reinterpret_cast<V *>(dst), scatter);
}

int launch_gather(const float *src, const int32_t *perm, int64_t n, int width, float *dst, bool scatter,
                  hipStream_t s) {
  if (n == 0) return FMM2D_OK;
  const uintptr_t align = reinterpret_cast<uintptr_t>(src) | reinterpret_cast<uintptr_t>(dst);
  if (width == 1) launch_rows<float>(src, perm, n, dst, scatter, s);
  else if (width == 2 && align % 8 == 0) launch_rows<float2>(src, perm, n, dst, scatter, s);
  else if (width == 4 && align % 16 == 0) launch_rows<float4>(src, perm, n, dst, scatter, s);
  else {
    const int64_t tot = n * width;
    hipLaunchKernelGGL(gather_kernel, dim3(unsigned((tot + 255) / 256)), dim3(256), 0, s, src, perm, n, width, dst,
                       scatter);
  }
  return check_launch(scatter ? "scatter" : "gather");
}

}  // namespace fmm2d
