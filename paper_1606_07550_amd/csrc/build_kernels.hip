// CSR builder for gfx950: validate + symmetrise + drop self loops (degree
// count, prefix sum, scatter), a segmented row sort binned by row length
// with in-place dedup, and the degree-order orientation into a DAG.
//
// The paper keeps, per node, a vector of adjacent nodes held in sorted order
// (Section 5.1); an undirected edge is stored in both endpoints' vectors.
// Here all vectors live in one array: row v occupies adj[off[v], off[v+1])
// of which the first deg[v] entries are the sorted, duplicate-free
// neighbours once the build is done.
#include <algorithm>

#include "device_common.h"
#include "kernels.h"

namespace tricc {

// ---------------------------------------------------------------------------
// a1: validation and raw degree count (both directions, loops dropped)
__global__ __launch_bounds__(256) void k_degree_raw(const int32_t* __restrict__ src,
                                                    const int32_t* __restrict__ dst, int64_t m_raw,
                                                    int32_t n, int32_t* __restrict__ cnt,
                                                    int32_t* __restrict__ err) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  bool bad = false;
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < m_raw; e += stride) {
    const int32_t u = src[e], v = dst[e];
    if ((uint32_t)u >= (uint32_t)n || (uint32_t)v >= (uint32_t)n) { bad = true; continue; }
    if (u == v) continue;
    atomicAdd(&cnt[u], 1);
    atomicAdd(&cnt[v], 1);
  }
  if (__ballot(bad) && lane_id() == 0) atomicOr(err, 1);
}

hipError_t launch_degree_raw(const int32_t* src, const int32_t* dst, int64_t m_raw, int32_t n,
                             int32_t* cnt, int32_t* err, hipStream_t s) {
  if (m_raw == 0) return hipSuccess;
  k_degree_raw<<<grid_for(m_raw, 256 * 8, 1u << 16), 256, 0, s>>>(src, dst, m_raw, n, cnt, err);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Exclusive prefix sum (reduce, scan of block sums, apply).
constexpr int kScanThreads = 256;
constexpr int kScanItems = 16;
constexpr int64_t kScanTile = kScanThreads * kScanItems;

int64_t scan_tmp_elems(int64_t n) { return (n + kScanTile - 1) / kScanTile + 2; }

template <typename Tin>
__global__ __launch_bounds__(kScanThreads) void k_scan_reduce(const Tin* __restrict__ in, int64_t n,
                                                              int64_t* __restrict__ bsum) {
  __shared__ int64_t lds[kScanThreads / kWave + 1];
  const int64_t base = (int64_t)blockIdx.x * kScanTile;
  int64_t acc = 0;
#pragma unroll
  for (int k = 0; k < kScanItems; ++k) {
    const int64_t i = base + (int64_t)k * kScanThreads + threadIdx.x;
    if (i < n) acc += (int64_t)in[i];
  }
  const int64_t t = block_sum<int64_t, kScanThreads>(acc, lds);
  if (threadIdx.x == 0) bsum[blockIdx.x] = t;
}

// Single block: exclusive scan of nb block sums in place; bsum[nb] = total.
__global__ __launch_bounds__(1024) void k_scan_blocks(int64_t* __restrict__ bsum, int64_t nb) {
  __shared__ int64_t lds[1024 / kWave + 1];
  int64_t carry = 0;
  for (int64_t base = 0; base < nb; base += 1024) {
    const int64_t i = base + threadIdx.x;
    const int64_t x = i < nb ? bsum[i] : 0;
    int64_t tot;
    const int64_t ex = block_excl_scan<int64_t, 1024>(x, lds, &tot);
    if (i < nb) bsum[i] = carry + ex;
    carry += tot;
  }
  if (threadIdx.x == 0) bsum[nb] = carry;
}

template <typename Tin>
__global__ __launch_bounds__(kScanThreads) void k_scan_apply(const Tin* __restrict__ in, int64_t n,
                                                             const int64_t* __restrict__ bsum,
                                                             int64_t* __restrict__ out, int64_t nb) {
  __shared__ int64_t lds[kScanThreads / kWave + 1];
  const int64_t base = (int64_t)blockIdx.x * kScanTile;
  // blocked arrangement: thread t owns kScanItems consecutive elements
  int64_t v[kScanItems];
  int64_t acc = 0;
  const int64_t tb = base + (int64_t)threadIdx.x * kScanItems;
#pragma unroll
  for (int k = 0; k < kScanItems; ++k) {
    const int64_t i = tb + k;
    v[k] = i < n ? (int64_t)in[i] : 0;
    acc += v[k];
  }
  int64_t tot;
  int64_t run = bsum[blockIdx.x] + block_excl_scan<int64_t, kScanThreads>(acc, lds, &tot);
#pragma unroll
  for (int k = 0; k < kScanItems; ++k) {
    const int64_t i = tb + k;
    if (i < n) out[i] = run;
    run += v[k];
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) out[n] = bsum[nb];
}

template <typename Tin>
static hipError_t scan_impl(const Tin* in, int64_t n, int64_t* out, int64_t* tmp, hipStream_t s) {
  const int64_t nb = (n + kScanTile - 1) / kScanTile;
  if (nb == 0) {
    return hipMemsetAsync(out, 0, sizeof(int64_t), s);
  }
  k_scan_reduce<Tin><<<(unsigned)nb, kScanThreads, 0, s>>>(in, n, tmp);
  k_scan_blocks<<<1, 1024, 0, s>>>(tmp, nb);
  k_scan_apply<Tin><<<(unsigned)nb, kScanThreads, 0, s>>>(in, n, tmp, out, nb);
  return hipGetLastError();
}

hipError_t launch_scan_i32(const int32_t* in, int64_t n, int64_t* out, int64_t* tmp, hipStream_t s) {
  return scan_impl<int32_t>(in, n, out, tmp, s);
}

// ---------------------------------------------------------------------------
// a1/a3: scatter both directions into the row segments (unsorted).
__global__ __launch_bounds__(256) void k_scatter(const int32_t* __restrict__ src,
                                                 const int32_t* __restrict__ dst, int64_t m_raw,
                                                 const int64_t* __restrict__ off,
                                                 int32_t* __restrict__ cur, int32_t* __restrict__ adj) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < m_raw; e += stride) {
    const int32_t u = src[e], v = dst[e];
    if (u == v) continue;
    adj[off[u] + atomicAdd(&cur[u], 1)] = v;
    adj[off[v] + atomicAdd(&cur[v], 1)] = u;
  }
}

hipError_t launch_scatter(const int32_t* src, const int32_t* dst, int64_t m_raw, const int64_t* off,
                          int32_t* cur, int32_t* adj, hipStream_t s) {
  if (m_raw == 0) return hipSuccess;
  k_scatter<<<grid_for(m_raw, 256 * 8, 1u << 16), 256, 0, s>>>(src, dst, m_raw, off, cur, adj);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// a1-a3, partitioned: the same raw rows without a global atomic per entry.
// Node v lies in partition v >> pbits (2^pbits consecutive ids, at most
// kPartMax partitions). Pass A counts each partition's entries with LDS
// histograms (and checks the ids); pass B moves every entry, i.e. each pair
// seen from each of its endpoints, into its partition's slice of a staging
// array (other endpoint in pv, the row as a 16-bit local index in pu),
// reserving one range per (tile, partition); passes C and D take one chunk
// of one partition per block with one LDS counter per node of the
// partition: C adds up the raw row lengths, D reserves each row's range and
// places the entries. Self loops are dropped in A and B.
constexpr int kPartMax = kPartMaxParts;
constexpr int kPartMinBits = 10, kPartMaxBits = 14;
constexpr int kPartNT = 1024;
constexpr int kPartPairs = 16;  // pairs per thread per tile in pass B
constexpr int64_t kPartTile = (int64_t)kPartNT * kPartPairs;
constexpr int kRowsNT = 1024;
constexpr int kRowsUnroll = 2;  // groups of 8 entries per thread per step
constexpr int64_t kRowsChunk = int64_t(1) << 18;  // entries per block in C and D

int part_bits(int64_t n) {
  if (n <= 0) return -1;
  int b = kPartMinBits;
  while (b < kPartMaxBits && ((n + (int64_t(1) << b) - 1) >> b) > 1024) ++b;
  return ((n + (int64_t(1) << b) - 1) >> b) <= kPartMax ? b : -1;
}

// Adds one to cnt[p] in LDS for every active lane and returns the lane's place
// among the counts so far. Lanes that all have the same p (a graph of one
// partition, a batch of small graphs, pairs grouped by node) take one atomic
// together: 64 on one address follow each other (200 graphs of 64 to 65,536
// nodes, build to results: 2.18 -> 2.13 ms).
__device__ __forceinline__ uint32_t take_place(uint32_t* cnt, int32_t p) {
  const int32_t p0 = __builtin_amdgcn_readfirstlane(p);
  if (__ballot(p != p0)) return atomicAdd(&cnt[p], 1u);
  const uint64_t m = __ballot(true);
  const int below = mask_below(m);
  uint32_t first = 0;
  if (below == 0) first = atomicAdd(&cnt[p0], (uint32_t)__popcll(m));
  return (uint32_t)__builtin_amdgcn_readfirstlane((int)first) + (uint32_t)below;
}

__global__ __launch_bounds__(kPartNT) void k_part_count(const int32_t* __restrict__ src,
                                                       const int32_t* __restrict__ dst, int64_t m_raw, int32_t n,
                                                       int pbits, int32_t P, uint32_t* __restrict__ ptotal,
                                                       int32_t* __restrict__ err) {
  __shared__ uint32_t hist[kPartMax];
  for (int b = threadIdx.x; b < P; b += kPartNT) hist[b] = 0;
  __syncthreads();
  const int64_t stride = (int64_t)gridDim.x * kPartNT;
  bool bad = false;
  for (int64_t e = (int64_t)blockIdx.x * kPartNT + threadIdx.x; e < m_raw; e += stride) {
    const int32_t u = src[e], v = dst[e];
    if ((uint32_t)u >= (uint32_t)n || (uint32_t)v >= (uint32_t)n) { bad = true; continue; }
    if (u == v) continue;  // dropped, as a pair with an id out of range is (the build is refused later)
    take_place(hist, u >> pbits);
    take_place(hist, v >> pbits);
  }
  if (__ballot(bad) && lane_id() == 0) atomicOr(err, 1);
  __syncthreads();
  for (int b = threadIdx.x; b < P; b += kPartNT)
    if (hist[b]) atomicAdd(&ptotal[b], hist[b]);
}

// Chunks of a partition of t entries (an empty one has one too: its block
// writes the empty rows' offsets).
__device__ __forceinline__ int64_t part_chunks(int64_t t) { return t > 0 ? (t + kRowsChunk - 1) / kRowsChunk : 1; }

// Single block: pstart = exclusive scan of the partition sizes, cstart =
// exclusive scan of their chunk counts.
__global__ __launch_bounds__(1024) void k_part_scan(const uint32_t* __restrict__ ptotal, int32_t P,
                                                    int64_t* __restrict__ pstart, int64_t* __restrict__ cstart) {
  __shared__ int64_t lds[1024 / kWave + 1];
  int64_t c0 = 0, c1 = 0;
  for (int32_t base = 0; base < P; base += 1024) {
    const int32_t i = base + threadIdx.x;
    const int64_t t = i < P ? (int64_t)ptotal[i] : 0;
    const int64_t ch = i < P ? part_chunks(t) : 0;
    int64_t tot0, tot1;
    const int64_t e0 = block_excl_scan<int64_t, 1024>(t, lds, &tot0);
    const int64_t e1 = block_excl_scan<int64_t, 1024>(ch, lds, &tot1);
    if (i < P) {
      pstart[i] = c0 + e0;
      cstart[i] = c1 + e1;
    }
    c0 += tot0;
    c1 += tot1;
  }
  if (threadIdx.x == 0) {
    pstart[P] = c0;
    cstart[P] = c1;
  }
}

// A pair that pass B places: both ids in range (pass A flags the others, and
// counts as pass B does) and not a self loop.
__device__ __forceinline__ bool pair_ok(int32_t u, int32_t v, int32_t n) {
  return (uint32_t)u < (uint32_t)n && (uint32_t)v < (uint32_t)n && u != v;
}

// Pass B.
__global__ __launch_bounds__(kPartNT) void k_part_place(const int32_t* __restrict__ src,
                                                       const int32_t* __restrict__ dst, int64_t m_raw, int32_t n,
                                                       int pbits,
                                                       int32_t P, const int64_t* __restrict__ pstart,
                                                       uint32_t* __restrict__ pcur, int32_t* __restrict__ pv,
                                                       uint16_t* __restrict__ pu) {
  __shared__ uint32_t hist[kPartMax];
  __shared__ int64_t hoff[kPartMax];
  const int64_t ntiles = (m_raw + kPartTile - 1) / kPartTile;
  const int32_t lmask = (1 << pbits) - 1;
  for (int64_t tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
    for (int b = threadIdx.x; b < P; b += kPartNT) hist[b] = 0;
    __syncthreads();
    const int64_t base = tile * kPartTile + threadIdx.x;
    int32_t a[kPartPairs], c[kPartPairs];
#pragma unroll
    for (int k = 0; k < kPartPairs; ++k) {
      const int64_t e = base + (int64_t)k * kPartNT;
      a[k] = -1;
      c[k] = -1;
      if (e < m_raw) {
        a[k] = src[e];
        c[k] = dst[e];
      }
    }
    uint32_t ra[kPartPairs], rc[kPartPairs];
#pragma unroll
    for (int k = 0; k < kPartPairs; ++k) {
      if (!pair_ok(a[k], c[k], n)) a[k] = -1;  // also past the end
      if (a[k] >= 0) {
        ra[k] = atomicAdd(&hist[a[k] >> pbits], 1u);
        rc[k] = atomicAdd(&hist[c[k] >> pbits], 1u);
      }
    }
    __syncthreads();
    for (int b = threadIdx.x; b < P; b += kPartNT) {
      const uint32_t h = hist[b];
      if (h) hoff[b] = pstart[b] + atomicAdd(&pcur[b], h);
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kPartPairs; ++k) {
      if (a[k] < 0) continue;
      const int64_t p = hoff[a[k] >> pbits] + ra[k];
      pv[p] = c[k];
      pu[p] = (uint16_t)(a[k] & lmask);
      const int64_t q = hoff[c[k] >> pbits] + rc[k];
      pv[q] = a[k];
      pu[q] = (uint16_t)(c[k] & lmask);
    }
    __syncthreads();  // hist and hoff are reused by the next tile
  }
}

// Pass B with coalesced stores, for at most kStagedParts partitions: a tile
// of kStagedPairs pairs is ranked per partition (LDS atomics), scanned, and
// staged in LDS in partition order; each partition's run then goes to its
// reserved range with consecutive lanes on consecutive addresses, instead
// of one cache line per lane.
// ONE: all pairs are one tile, so its counts are the partitions' sizes and pass
// A, whose other work is to flag ids out of range, is left out (5,003 pairs on
// 1,000 nodes, whole count: 163 -> 147 us, part of it by take_place).
constexpr int kStagedParts = 1024;
constexpr int kStagedNT = 1024;
constexpr int kStagedPairs = 8192;
constexpr int kStagedPer = kStagedPairs / kStagedNT;

template <bool ONE>
__global__ __launch_bounds__(kStagedNT) void k_part_place_staged(const int32_t* __restrict__ src,
                                                                 const int32_t* __restrict__ dst, int64_t m_raw,
                                                                 int32_t n, int pbits, int32_t P,
                                                                 const uint32_t* __restrict__ ptotal,
                                                                 int64_t* __restrict__ pstart,
                                                                 int64_t* __restrict__ cstart,
                                                                 uint32_t* __restrict__ pcur, int32_t* __restrict__ pv,
                                                                 uint16_t* __restrict__ pu,
                                                                 int32_t* __restrict__ err) {
  __shared__ uint32_t cnt[kStagedParts];   // entries of each partition in the tile
  __shared__ uint32_t lst[kStagedParts];   // their exclusive prefix (run start in the stage)
  __shared__ int64_t hoff[kStagedParts];   // global start of the run
  __shared__ int32_t sv[2 * kStagedPairs];  // staged other endpoint
  __shared__ int32_t ss[2 * kStagedPairs];  // staged row endpoint
  __shared__ uint32_t red[kStagedNT / kWave + 1];
  const int64_t ntiles = (m_raw + kStagedPairs - 1) / kStagedPairs;
  const int32_t lmask = (1 << pbits) - 1;
  static_assert(kStagedParts == kStagedNT, "one partition per thread in the scans");
  // every block scans the partition sizes itself (one launch less); thread b
  // keeps partition b's start, block 0 writes the starts for the later passes
  __shared__ int64_t red64[kStagedNT / kWave + 1];
  int64_t mystart = 0;
  auto starts = [&](int64_t psize) {
    int64_t all;
    mystart = block_excl_scan<int64_t, kStagedNT>(psize, red64, &all);
    if (blockIdx.x == 0) {
      int64_t chunks;
      const int64_t mychunk =
          block_excl_scan<int64_t, kStagedNT>(threadIdx.x < P ? part_chunks(psize) : 0, red64, &chunks);
      if (threadIdx.x < P) {
        pstart[threadIdx.x] = mystart;
        cstart[threadIdx.x] = mychunk;
      }
      if (threadIdx.x == 0) {
        pstart[P] = all;
        cstart[P] = chunks;
      }
    }
  };
  if (!ONE) starts(threadIdx.x < P ? (int64_t)ptotal[threadIdx.x] : 0);
  for (int64_t tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
    for (int b = threadIdx.x; b < P; b += kStagedNT) cnt[b] = 0;
    __syncthreads();
    int32_t a[kStagedPer], c[kStagedPer];
    uint32_t ra[kStagedPer], rc[kStagedPer];
    const int64_t base = tile * kStagedPairs + threadIdx.x;
#pragma unroll
    for (int k = 0; k < kStagedPer; ++k) {
      const int64_t e = base + (int64_t)k * kStagedNT;
      a[k] = -1;
      c[k] = -1;
      if (e < m_raw) {
        a[k] = src[e];
        c[k] = dst[e];
      }
    }
    bool bad = false;
#pragma unroll
    for (int k = 0; k < kStagedPer; ++k) {
      if (ONE && base + (int64_t)k * kStagedNT < m_raw)
        bad |= (uint32_t)a[k] >= (uint32_t)n || (uint32_t)c[k] >= (uint32_t)n;
      if (!pair_ok(a[k], c[k], n)) a[k] = -1;  // also past the end
      if (a[k] >= 0) {
        ra[k] = take_place(cnt, a[k] >> pbits);
        rc[k] = take_place(cnt, c[k] >> pbits);
      }
    }
    if (ONE && __ballot(bad) && lane_id() == 0) atomicOr(err, 1);
    __syncthreads();
    if (ONE) starts(threadIdx.x < P ? (int64_t)cnt[threadIdx.x] : 0);
    const uint32_t mine = threadIdx.x < P ? cnt[threadIdx.x] : 0u;
    uint32_t tot;
    const uint32_t run = block_excl_scan<uint32_t, kStagedNT>(mine, red, &tot);
    if (threadIdx.x < P) {
      lst[threadIdx.x] = run;
      if (mine) hoff[threadIdx.x] = mystart + (ONE ? 0u : atomicAdd(&pcur[threadIdx.x], mine));
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kStagedPer; ++k) {
      if (a[k] < 0) continue;
      const uint32_t i = lst[a[k] >> pbits] + ra[k];
      sv[i] = c[k];
      ss[i] = a[k];
      const uint32_t j = lst[c[k] >> pbits] + rc[k];
      sv[j] = a[k];
      ss[j] = c[k];
    }
    __syncthreads();
    for (uint32_t t = threadIdx.x; t < tot; t += kStagedNT) {
      const int32_t r = ss[t];
      const int32_t p = r >> pbits;
      const int64_t pos = hoff[p] + (t - lst[p]);
      pv[pos] = sv[t];
      pu[pos] = (uint16_t)(r & lmask);
    }
    __syncthreads();  // the stage and the tables are reused by the next tile
  }
}

// Passes C and D. A partition held by one chunk is finished by one block of
// mode 0: row lengths, their prefix inside the partition (whose slice starts
// at pstart[p], so no scan over all nodes is needed) and the entries. One
// spread over several chunks takes three launches: mode 0 adds up its row
// lengths (global atomics on the zeroed len), mode 1 (one block per
// partition) turns them into row offsets and clears the cursors cur, mode 2
// reserves each row's range and places the entries. The launcher leaves
// modes 1 and 2 out when no partition can have two chunks.
__device__ __forceinline__ void part_offsets(int32_t v0, int32_t W, int64_t pb, int64_t total, int32_t n,
                                             uint32_t* cnt, const int32_t* __restrict__ len,
                                             int64_t* __restrict__ raw_off, int32_t* __restrict__ cur,
                                             uint32_t* red) {
  // cnt (LDS) = row lengths (loaded from len when it is given) -> offsets
  // inside the partition; one run of W / kRowsNT rows per thread
  if (len) {
    for (int j = threadIdx.x; j < W; j += kRowsNT) {
      cnt[j] = (uint32_t)len[v0 + j];
      cur[v0 + j] = 0;
    }
    __syncthreads();
  }
  const int per = (W + kRowsNT - 1) / kRowsNT;
  const int j0 = threadIdx.x * per, j1 = min(W, j0 + per);
  uint32_t sum = 0;
  for (int j = j0; j < j1; ++j) sum += cnt[j];
  uint32_t tot;
  uint32_t run = block_excl_scan<uint32_t, kRowsNT>(sum, red, &tot);
  for (int j = j0; j < j1; ++j) {
    const uint32_t k = cnt[j];
    cnt[j] = run;
    run += k;
  }
  __syncthreads();
  for (int j = threadIdx.x; j < W; j += kRowsNT) raw_off[v0 + j] = pb + (int64_t)cnt[j];
  if (threadIdx.x == 0 && v0 + W == n) raw_off[n] = total;
}

__global__ __launch_bounds__(kRowsNT) void k_part_rows(int mode, int pbits, int32_t P, int32_t n,
                                                      const int64_t* __restrict__ pstart,
                                                      const int64_t* __restrict__ cstart,
                                                      const uint16_t* __restrict__ pu,
                                                      const int32_t* __restrict__ pv, int32_t* __restrict__ len,
                                                      int64_t* __restrict__ raw_off,
                                                      int32_t* __restrict__ cur, int32_t* __restrict__ adj) {
  __shared__ uint32_t cnt[1 << kPartMaxBits];
  __shared__ uint32_t red[kRowsNT / kWave + 1];
  int32_t p;
  int64_t c = 0;
  if (mode == 1) {
    p = (int32_t)blockIdx.x;
  } else {
    c = blockIdx.x;
    if (c >= cstart[P]) return;
    int32_t lo = 0, hi = P - 1;  // partition of chunk c: the last p with cstart[p] <= c
    while (lo < hi) {
      const int32_t mid = (lo + hi + 1) >> 1;
      if (cstart[mid] <= c) lo = mid; else hi = mid - 1;
    }
    p = lo;
  }
  const bool single = cstart[p + 1] - cstart[p] == 1;
  if (mode != 0 && single) return;  // finished by mode 0
  const int64_t pb = pstart[p];
  const int32_t v0 = p << pbits;
  const int32_t W = min(1 << pbits, n - v0);
  if (mode == 1) {
    part_offsets(v0, W, pb, pstart[P], n, cnt, len, raw_off, cur, red);
    return;
  }
  const int64_t i0 = pb + (c - cstart[p]) * kRowsChunk;
  const int64_t i1 = min(pstart[p + 1], i0 + kRowsChunk);
  for (int j = threadIdx.x; j < W; j += kRowsNT) cnt[j] = 0;
  __syncthreads();
  // aligned groups of 8 entries, one 16-byte load of local rows each (the
  // group start rounds down inside the array; the last group may read up
  // to 7 entries past the end, inside the staging area's padding); entries
  // outside [i0, i1) are masked
  const int64_t g0 = i0 & ~int64_t(7);
  for (int64_t gs = g0 + 8 * (int64_t)threadIdx.x; gs < i1; gs += 8 * kRowsNT * kRowsUnroll) {
    uint4 w[kRowsUnroll];
#pragma unroll
    for (int k = 0; k < kRowsUnroll; ++k) {
      const int64_t at = gs + (int64_t)k * 8 * kRowsNT;
      w[k] = at < i1 ? *reinterpret_cast<const uint4*>(pu + at) : make_uint4(0, 0, 0, 0);
    }
#pragma unroll
    for (int k = 0; k < kRowsUnroll; ++k) {
      const int64_t at = gs + (int64_t)k * 8 * kRowsNT;
      const uint32_t ws[4] = {w[k].x, w[k].y, w[k].z, w[k].w};
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        const int64_t i = at + q;
        if (i >= i0 && i < i1) atomicAdd(&cnt[(ws[q >> 1] >> (16 * (q & 1))) & 0xffffu], 1u);
      }
    }
  }
  __syncthreads();
  if (single) {
    for (int j = threadIdx.x; j < W; j += kRowsNT) len[v0 + j] = (int32_t)cnt[j];
    __syncthreads();
    part_offsets(v0, W, pb, pstart[P], n, cnt, nullptr, raw_off, nullptr, red);
  } else if (mode == 0) {
    for (int j = threadIdx.x; j < W; j += kRowsNT) {
      const uint32_t k = cnt[j];
      if (k) atomicAdd(&len[v0 + j], (int32_t)k);
    }
    return;
  } else {
    for (int j = threadIdx.x; j < W; j += kRowsNT) {
      const uint32_t k = cnt[j];
      if (k) cnt[j] = (uint32_t)(raw_off[v0 + j] - pb) + (uint32_t)atomicAdd(&cur[v0 + j], (int32_t)k);
    }
  }
  __syncthreads();
  for (int64_t gs = g0 + 8 * (int64_t)threadIdx.x; gs < i1; gs += 8 * kRowsNT * kRowsUnroll) {
    uint4 w[kRowsUnroll];
    int4 xa[kRowsUnroll], xb[kRowsUnroll];
#pragma unroll
    for (int k = 0; k < kRowsUnroll; ++k) {
      const int64_t at = gs + (int64_t)k * 8 * kRowsNT;
      const bool ok = at < i1;
      w[k] = ok ? *reinterpret_cast<const uint4*>(pu + at) : make_uint4(0, 0, 0, 0);
      xa[k] = ok ? *reinterpret_cast<const int4*>(pv + at) : make_int4(0, 0, 0, 0);
      xb[k] = ok ? *reinterpret_cast<const int4*>(pv + at + 4) : make_int4(0, 0, 0, 0);
    }
#pragma unroll
    for (int k = 0; k < kRowsUnroll; ++k) {
      const int64_t at = gs + (int64_t)k * 8 * kRowsNT;
      const uint32_t ws[4] = {w[k].x, w[k].y, w[k].z, w[k].w};
      const int32_t xs[8] = {xa[k].x, xa[k].y, xa[k].z, xa[k].w, xb[k].x, xb[k].y, xb[k].z, xb[k].w};
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        const int64_t i = at + q;
        if (i >= i0 && i < i1) adj[pb + atomicAdd(&cnt[(ws[q >> 1] >> (16 * (q & 1))) & 0xffffu], 1u)] = xs[q];
      }
    }
  }
}

// Clears what the build accumulates into: the header, the partition counters
// and (len given) the row lengths.
__global__ __launch_bounds__(256) void k_build_clear(int32_t* __restrict__ hdr, int32_t words,
                                                     uint32_t* __restrict__ part, int32_t nparts,
                                                     int32_t* __restrict__ len, int32_t n) {
  const int64_t stride = (int64_t)gridDim.x * 256;
  const int64_t i0 = (int64_t)blockIdx.x * 256 + threadIdx.x;
  for (int64_t i = i0; i < words; i += stride) hdr[i] = 0;
  for (int64_t i = i0; i < nparts; i += stride) part[i] = 0;
  if (len)
    for (int64_t i = i0; i < n; i += stride) len[i] = 0;
}

hipError_t launch_build_clear(int32_t* hdr, int32_t words, uint32_t* part, int32_t nparts, int32_t* len, int32_t n,
                              hipStream_t s) {
  const int64_t most = std::max<int64_t>(std::max(words, nparts), len ? n : 0);
  k_build_clear<<<grid_for(most, 256 * 4, 2048), 256, 0, s>>>(hdr, words, part, nparts, len, n);
  return hipGetLastError();
}

// One tile of the staged placing holds all pairs.
static bool part_one_tile(int64_t m_raw, int32_t P) { return m_raw <= kStagedPairs && P <= kStagedParts; }

hipError_t launch_part_count(const int32_t* src, const int32_t* dst, int64_t m_raw, int32_t n, int pbits, int32_t P,
                             uint32_t* ptotal, int32_t* err, hipStream_t s) {
  if (m_raw == 0 || part_one_tile(m_raw, P)) return hipSuccess;
  k_part_count<<<grid_for(m_raw, kPartNT * 16, 2048), kPartNT, 0, s>>>(src, dst, m_raw, n, pbits, P, ptotal, err);
  return hipGetLastError();
}

// Partition starts and chunk starts, then pass B.
hipError_t launch_part_place(const int32_t* src, const int32_t* dst, int64_t m_raw, int32_t n, int pbits, int32_t P,
                             const uint32_t* ptotal, int64_t* pstart, int64_t* cstart, uint32_t* pcur, int32_t* pv,
                             uint16_t* pu, int32_t* err, hipStream_t s) {
  if (m_raw == 0) return hipSuccess;
  if (part_one_tile(m_raw, P)) {
    k_part_place_staged<true><<<1, kStagedNT, 0, s>>>(src, dst, m_raw, n, pbits, P, nullptr, pstart, cstart, nullptr,
                                                      pv, pu, err);
    return hipGetLastError();
  }
  if (P <= kStagedParts) {
    k_part_place_staged<false><<<grid_for(m_raw, kStagedPairs, 4096), kStagedNT, 0, s>>>(
        src, dst, m_raw, n, pbits, P, ptotal, pstart, cstart, pcur, pv, pu, nullptr);
    return hipGetLastError();
  }
  k_part_scan<<<1, 1024, 0, s>>>(ptotal, P, pstart, cstart);
  k_part_place<<<grid_for(m_raw, (int)kPartTile, 4096), kPartNT, 0, s>>>(src, dst, m_raw, n, pbits, P, pstart, pcur,
                                                                         pv, pu);
  return hipGetLastError();
}

bool part_may_split(int64_t entries) { return entries > kRowsChunk; }

hipError_t launch_part_rows(int pbits, int32_t P, int32_t n, int64_t max_entries, const int64_t* pstart,
                            const int64_t* cstart, const uint16_t* pu, const int32_t* pv, int32_t* len,
                            int64_t* raw_off, int32_t* cur, int32_t* adj, hipStream_t s) {
  // every partition has at most ceil(size / chunk) <= size / chunk + 1 chunks
  const unsigned blocks = (unsigned)(max_entries / kRowsChunk + P);
  k_part_rows<<<blocks, kRowsNT, 0, s>>>(0, pbits, P, n, pstart, cstart, pu, pv, len, raw_off, cur, adj);
  if (part_may_split(max_entries)) {
    k_part_rows<<<(unsigned)P, kRowsNT, 0, s>>>(1, pbits, P, n, pstart, cstart, pu, pv, len, raw_off, cur, adj);
    k_part_rows<<<blocks, kRowsNT, 0, s>>>(2, pbits, P, n, pstart, cstart, pu, pv, len, raw_off, cur, adj);
  }
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Tiles of nodes of the two-pass layouts (row classes, DAG layout): at most
// kLayoutMaxTiles, so that every block of the second pass can add up the sums
// of the tiles before its own. sums holds one column per tile.
constexpr int kLayoutNT = 1024;
constexpr int64_t kLayoutMaxTiles = 1024;
enum : int { kLqOut = 0, kLqIn = 1, kLqBin = 2, kLqInBin = 8, kLqItems = 14, kLqDeg2 = 20, kLqMaxD = 21, kLqMaxP = 22,
             kLayoutQ = 23 };

int64_t layout_tile(int64_t n) {
  const int64_t per = (n + kLayoutNT * kLayoutMaxTiles - 1) / (kLayoutNT * kLayoutMaxTiles);
  return kLayoutNT * (per > 0 ? per : 1);
}

// ---------------------------------------------------------------------------
// Row classes by raw length.
__device__ __forceinline__ int row_class(int32_t len, int32_t bitmap_min) {
  if (len <= 1) return kRowTrivial;
  if (len <= 8) return kRow8;
  if (len <= 16) return kRow16;
  if (len <= 32) return kRow32;
  if (len <= 64) return kRow64;
  if (len <= 128) return kRow128;
  if (len <= 256) return kRow256;
  if (len <= 512) return kRow512;
  if (len <= 1024) return kRow1024;
  if (len <= 4096) return kRow4k;
  if (len <= 8192) return kRow8k;
  if (len <= 16384) return kRow16k;
  if (len <= 32768) return kRow32k;
  return len < bitmap_min ? kRowMerge : kRowLarge;
}

// Rows by class, listed class-major: pass 1 leaves each tile's class counts,
// pass 2 adds up the counts of the classes and tiles before its own and
// places its rows with wave ballots and one LDS cursor per class. Rows of
// length <= 1 are not listed; their degree is set here. Tiles as for the DAG
// layout (at most 1,024 of them), so no scan stands between the passes: as a
// histogram, a three-launch scan, an offset gather and a placement it took
// six launches.
__global__ __launch_bounds__(kLayoutNT) void k_rows_count(int32_t n, int64_t tile, int32_t bitmap_min,
                                                          const int32_t* __restrict__ len,
                                                          int32_t* __restrict__ deg, int32_t* __restrict__ sums) {
  __shared__ int32_t acc[kNumRowClasses];
  if (threadIdx.x < kNumRowClasses) acc[threadIdx.x] = 0;
  __syncthreads();
  const int64_t t0 = (int64_t)blockIdx.x * tile, t1 = min((int64_t)n, t0 + tile);
  int32_t nc[kNumRowClasses] = {};  // wave-uniform
  for (int64_t b = t0; b < t1; b += kLayoutNT) {
    const int64_t v = b + threadIdx.x;
    int c = kRowTrivial;
    if (v < t1) {
      const int32_t L = len[v];
      c = row_class(L, bitmap_min);
      if (c == kRowTrivial) deg[v] = L;
    }
#pragma unroll
    for (int q = kRowTrivial + 1; q < kNumRowClasses; ++q) nc[q] += (int32_t)__popcll(__ballot(c == q));
  }
  if (lane_id() == 0)
#pragma unroll
    for (int q = kRowTrivial + 1; q < kNumRowClasses; ++q)
      if (nc[q]) atomicAdd(&acc[q], nc[q]);
  __syncthreads();
  if (threadIdx.x < kNumRowClasses) sums[(int64_t)threadIdx.x * gridDim.x + blockIdx.x] = acc[threadIdx.x];
}

__global__ __launch_bounds__(kLayoutNT) void k_rows_place(int32_t n, int64_t tile, int32_t bitmap_min,
                                                          const int32_t* __restrict__ len,
                                                          const int32_t* __restrict__ sums,
                                                          int32_t* __restrict__ list, int64_t* __restrict__ cls_off) {
  __shared__ int32_t prev[kNumRowClasses], all[kNumRowClasses], cur[kNumRowClasses];
  const int lane = lane_id(), wv = threadIdx.x / kWave;
  const int nt = (int)gridDim.x, me = (int)blockIdx.x;
  if (wv < kNumRowClasses) {
    int32_t p = 0, a = 0;
    for (int b = lane; b < nt; b += kWave) {
      const int32_t x = sums[(int64_t)wv * nt + b];
      a += x;
      if (b < me) p += x;
    }
    p = group_sum<int32_t, kWave>(p);
    a = group_sum<int32_t, kWave>(a);
    if (lane == 0) {
      prev[wv] = p;
      all[wv] = a;
    }
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    int32_t o = 0;
    for (int q = 0; q < kNumRowClasses; ++q) {
      if (me == 0) cls_off[q] = o;
      cur[q] = o + prev[q];
      o += all[q];
    }
    if (me == 0) cls_off[kNumRowClasses] = o;
  }
  __syncthreads();
  const int64_t t0 = (int64_t)me * tile, t1 = min((int64_t)n, t0 + tile);
  for (int64_t b = t0; b < t1; b += kLayoutNT) {
    const int64_t v = b + threadIdx.x;
    const int c = v < t1 ? row_class(len[v], bitmap_min) : kRowTrivial;
#pragma unroll
    for (int q = kRowTrivial + 1; q < kNumRowClasses; ++q) {
      const uint64_t m = __ballot(c == q);
      if (!m) continue;
      int32_t at = 0;
      if (lane == 0) at = atomicAdd(&cur[q], (int32_t)__popcll(m));
      at = __builtin_amdgcn_readfirstlane(at);
      if (c == q) list[at + mask_below(m)] = (int32_t)v;
    }
  }
}

hipError_t launch_row_classes(int32_t n, const int32_t* len, int32_t* deg, int32_t* sums, int32_t* list,
                              int64_t* cls_off, hipStream_t s) {
  static_assert(kNumRowClasses <= kLayoutNT / kWave && kNumRowClasses <= kLayoutQ, "one wavefront per class");
  if (n <= 0) return hipSuccess;
  const int64_t tile = layout_tile(n);
  const unsigned nt = (unsigned)((n + tile - 1) / tile);
  const int32_t least = row_bitmap_min(n);
  k_rows_count<<<nt, kLayoutNT, 0, s>>>(n, tile, least, len, deg, sums);
  k_rows_place<<<nt, kLayoutNT, 0, s>>>(n, tile, least, len, sums, list, cls_off);
  return hipGetLastError();
}

__global__ void k_gather_offsets(const int64_t* __restrict__ prefix, const int64_t* __restrict__ at, int k,
                                 int64_t* __restrict__ out) {
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < k; i += gridDim.x * blockDim.x) out[i] = prefix[at[i]];
}

hipError_t launch_gather_offsets(const int64_t* prefix, const int64_t* at, int k, int64_t* out, hipStream_t s) {
  if (k <= 0) return hipSuccess;
  k_gather_offsets<<<(unsigned)std::min(1024, (k + 255) / 256), 256, 0, s>>>(prefix, at, k, out);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
template <int G>
__device__ __forceinline__ constexpr uint64_t group_bits() {
  return G >= 64 ? ~0ull : ((1ull << (G & 63)) - 1);
}

// Rows of up to G entries: a group of G lanes sorts one row in registers with
// a bitonic network over __shfl_xor, then compacts the unique values. blk:
// the block's place among the class's blocks of 256 / G rows.
template <int G>
__device__ __forceinline__ void sort_small(int64_t blk, const int32_t* __restrict__ rows, int32_t nrows,
                                           const int64_t* __restrict__ off, const int32_t* __restrict__ len,
                                           int32_t* __restrict__ adj, int32_t* __restrict__ deg) {
  const int64_t gi = blk * (256 / G) + threadIdx.x / G;
  const int g = threadIdx.x % G;
  const bool active = gi < nrows;
  int32_t v = 0, L = 0;
  int64_t beg = 0;
  int32_t x = kPad;
  if (active) {
    v = rows[gi];
    beg = off[v];
    L = len[v];
    if (g < L) x = adj[beg + g];
  }
#pragma unroll
  for (int k = 2; k <= G; k <<= 1) {
#pragma unroll
    for (int j = k >> 1; j > 0; j >>= 1) {
      const int32_t y = __shfl_xor(x, j, G);
      const bool up = (g & k) == 0;
      const bool low = (g & j) == 0;
      x = (low == up) ? min(x, y) : max(x, y);
    }
  }
  const int32_t prev = __shfl_up(x, 1, G);
  const bool uniq = active && x != kPad && (g == 0 || x != prev);
  const uint64_t mask = __ballot(uniq);
  const int shift = lane_id() & ~(G - 1);
  const uint64_t gm = (mask >> shift) & group_bits<G>();
  if (uniq) adj[beg + __popcll(gm & ((1ull << g) - 1))] = x;
  if (active && g == 0) deg[v] = (int32_t)__popcll(gm);
}

// Rows of up to 64 * E raw entries: one wavefront per row, the
// row in registers (id i in lane i % 64, register i / 64), a bitonic network
// whose strides >= 64 swap registers inside a lane and whose smaller strides
// exchange with the lane i ^ j by a shuffle, so no LDS and no barrier.
// Then an in-order dedup and a compacted, coalesced write to the row start.
template <int E>
__device__ __forceinline__ void sort_wave(int64_t blk, const int32_t* __restrict__ rows, int32_t nrows,
                                          const int64_t* __restrict__ off, const int32_t* __restrict__ len,
                                          int32_t* __restrict__ adj, int32_t* __restrict__ deg) {
  constexpr int P = kWave * E;
  const int lane = lane_id();
  const int64_t r = blk * (256 / kWave) + threadIdx.x / kWave;
  if (r >= nrows) return;
  const int32_t v = rows[r];
  const int64_t beg = off[v];
  const int32_t L = len[v];
  int32_t x[E];
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const int32_t i = e * kWave + lane;
    x[e] = i < L ? adj[beg + i] : kPad;
  }
#pragma unroll
  for (int k = 2; k <= P; k <<= 1) {
#pragma unroll
    for (int j = k >> 1; j > 0; j >>= 1) {
      if (j >= kWave) {
#pragma unroll
        for (int e = 0; e < E; ++e) {
          const int pe = e ^ (j / kWave);
          if (pe > e) {
            const bool up = ((e * kWave) & k) == 0;  // k > 64: the lane bits do not matter
            const int32_t a = x[e], b = x[pe];
            x[e] = up ? min(a, b) : max(a, b);
            x[pe] = up ? max(a, b) : min(a, b);
          }
        }
      } else {
#pragma unroll
        for (int e = 0; e < E; ++e) {
          const int32_t y = __shfl_xor(x[e], j, kWave);
          const bool up = ((e * kWave + lane) & k) == 0;
          const bool lo = (lane & j) == 0;
          x[e] = (lo == up) ? min(x[e], y) : max(x[e], y);
        }
      }
    }
  }
  int32_t base = 0;
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const int32_t i = e * kWave + lane;
    int32_t prev = __shfl_up(x[e], 1, kWave);
    if (e > 0) {
      const int32_t last = __builtin_amdgcn_readlane(x[e > 0 ? e - 1 : 0], kWave - 1);
      if (lane == 0) prev = last;
    }
    const bool u = i < L && (i == 0 || x[e] != prev);
    const uint64_t m = __ballot(u);
    if (u) adj[beg + base + mask_below(m)] = x[e];
    base += (int32_t)__popcll(m);
  }
  if (lane == 0) deg[v] = base;
}

// Rows of up to 64 * E * W ids: one block of W wavefronts holds
// the row in registers (id i in wavefront i / (64 E), register (i / 64) % E,
// lane i % 64) and runs a bitonic network on it: strides below 64 exchange
// by shuffles, strides below 64 E swap registers inside a lane, and only the
// strides of 64 E and up go through LDS (write, barrier, read of the partner,
// barrier). The stages run in a loop over k with the strides unrolled, which
// keeps the code small. The network spans only the next power of two Q >= L
// (the first Q ids, ascending; the pads beyond are left as they are), and
// wavefronts wholly past Q skip the register and shuffle stages. Then the
// unique ids, compacted to the row start, and deg[v].
template <int E, int W>
struct SortBlockLds {
  int32_t s[kWave * E * W];
  int32_t wsum[W + 1];
  int32_t wlast[W];
};

template <int E, int W>
__device__ __forceinline__ void sort_block(SortBlockLds<E, W>& lds, int32_t v, const int64_t* __restrict__ off,
                                           const int32_t* __restrict__ len, int32_t* __restrict__ adj,
                                           int32_t* __restrict__ deg) {
  constexpr int PW = kWave * E;  // ids per wavefront
  constexpr int P = PW * W;
  int32_t* s = lds.s;
  int32_t* wsum = lds.wsum;
  int32_t* wlast = lds.wlast;
  const int lane = lane_id();
  const int wv = threadIdx.x / kWave;
  const int32_t i0 = wv * PW + lane;  // index of x[0]; x[e] is i0 + 64 e
  const int64_t beg = off[v];
  const int32_t L = len[v];
  int32_t Q = 2;
  while (Q < L) Q <<= 1;
  const bool idle = wv * PW >= Q;  // wavefront-uniform
  int32_t x[E];
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const int32_t i = i0 + e * kWave;
    x[e] = i < L ? adj[beg + i] : kPad;
  }
  for (int k = 2; k <= Q; k <<= 1) {
#pragma unroll
    for (int j = P / 2; j > 0; j >>= 1) {
      if (j >= k) continue;  // block-uniform: the strides of stage k are k / 2 .. 1
      if (j >= PW) {
#pragma unroll
        for (int e = 0; e < E; ++e) s[i0 + e * kWave] = x[e];
        __syncthreads();
#pragma unroll
        for (int e = 0; e < E; ++e) {
          const int32_t i = i0 + e * kWave;
          const int32_t y = s[i ^ j];
          const bool up = (i & k) == 0;
          const bool lo = (i & j) == 0;
          x[e] = (lo == up) ? min(x[e], y) : max(x[e], y);
        }
        __syncthreads();
      } else if (idle) {
        continue;
      } else if (j >= kWave) {
#pragma unroll
        for (int e = 0; e < E; ++e) {
          const int pe = e ^ (j / kWave);
          if (pe > e) {
            const bool up = ((wv * PW + e * kWave) & k) == 0;  // k > 64: the lane bits do not matter
            const int32_t a = x[e], b = x[pe];
            x[e] = up ? min(a, b) : max(a, b);
            x[pe] = up ? max(a, b) : min(a, b);
          }
        }
      } else {
#pragma unroll
        for (int e = 0; e < E; ++e) {
          const int32_t y = __shfl_xor(x[e], j, kWave);
          const bool up = ((i0 + e * kWave) & k) == 0;
          const bool lo = (lane & j) == 0;
          x[e] = (lo == up) ? min(x[e], y) : max(x[e], y);
        }
      }
    }
  }
  // in-order dedup: the id before x[0] of lane 0 is the previous wavefront's
  // last; the unique flags are formed twice (count, then write) rather than
  // kept in registers
  if (lane == kWave - 1) wlast[wv] = x[E - 1];
  __syncthreads();
  const int32_t before = wv > 0 ? wlast[wv > 0 ? wv - 1 : 0] : 0;
  auto unique = [&](int e) -> uint64_t {
    const int32_t i = i0 + e * kWave;
    int32_t prev = __shfl_up(x[e], 1, kWave);
    if (lane == 0) prev = e > 0 ? __builtin_amdgcn_readlane(x[e > 0 ? e - 1 : 0], kWave - 1) : before;
    return __ballot(i < L && (i == 0 || x[e] != prev));
  };
  int32_t cnt = 0;
#pragma unroll
  for (int e = 0; e < E; ++e) cnt += (int32_t)__popcll(unique(e));
  if (lane == 0) wsum[wv] = cnt;
  __syncthreads();
  int32_t base = 0;
  for (int q = 0; q < wv; ++q) base += wsum[q];
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const uint64_t um = unique(e);
    if ((um >> lane) & 1) adj[beg + base + mask_below(um)] = x[e];
    base += (int32_t)__popcll(um);
  }
  if (wv == W - 1 && lane == 0) deg[v] = base;
}

template <int E, int W>
__global__ __launch_bounds__(kWave * W) void k_sort_block(const int32_t* __restrict__ rows,
                                                          const int64_t* __restrict__ off,
                                                          const int32_t* __restrict__ len,
                                                          int32_t* __restrict__ adj, int32_t* __restrict__ deg) {
  __shared__ SortBlockLds<E, W> lds;
  sort_block<E, W>(lds, rows[blockIdx.x], off, len, adj, deg);
}

// Rows of up to 4,096 entries in two launches (above 256 entries, and the
// rest, whose kernel needs a third of the registers), the blocks of the
// longest rows first: the last of them run beside the shorter classes instead
// of alone before the next launch, and a small graph pays one launch, not one
// per class.
struct SortPlan {
  int32_t row0[kSortClasses];   // first row in the list, from kRow4k down to kRow8
  int32_t nrows[kSortClasses];
  uint32_t blk0[kSortClasses];  // first block in the class's launch
};

// Class of block b of a launch of the classes [k0, k1).
__device__ __forceinline__ int sort_plan_class(const SortPlan& plan, int k0, int k1, uint32_t b) {
  int k = k0;
  for (int q = k0 + 1; q < k1; ++q)
    if (b >= plan.blk0[q]) k = q;
  return k;
}

__global__ __launch_bounds__(256) void k_sort_rows_long(SortPlan plan, const int32_t* __restrict__ list,
                                                        const int64_t* __restrict__ off,
                                                        const int32_t* __restrict__ len, int32_t* __restrict__ adj,
                                                        int32_t* __restrict__ deg) {
  __shared__ SortBlockLds<16, 4> lds;
  const int k = sort_plan_class(plan, 0, kSortLongClasses, blockIdx.x);
  const int64_t blk = blockIdx.x - plan.blk0[k];
  const int32_t* rows = list + plan.row0[k];
  switch (kRow4k - k) {
    case kRow4k: sort_block<16, 4>(lds, rows[blk], off, len, adj, deg); break;
    case kRow1024: sort_wave<16>(blk, rows, plan.nrows[k], off, len, adj, deg); break;
    default: sort_wave<8>(blk, rows, plan.nrows[k], off, len, adj, deg); break;
  }
}

// Blocks b0 .. of the launch's classes (the launcher cuts long launches up: a
// loop over blocks in the kernel took 4% more of a build of rows of 10 entries).
__global__ __launch_bounds__(256) void k_sort_rows_short(SortPlan plan, uint32_t b0,
                                                         const int32_t* __restrict__ list,
                                                         const int64_t* __restrict__ off,
                                                         const int32_t* __restrict__ len, int32_t* __restrict__ adj,
                                                         int32_t* __restrict__ deg) {
  const uint32_t b = b0 + blockIdx.x;
  const int k = sort_plan_class(plan, kSortLongClasses, kSortClasses, b);
  const int64_t blk = b - plan.blk0[k];
  const int32_t* rows = list + plan.row0[k];
  const int32_t n = plan.nrows[k];
  switch (kRow4k - k) {
    case kRow256: sort_wave<4>(blk, rows, n, off, len, adj, deg); break;
    case kRow128: sort_wave<2>(blk, rows, n, off, len, adj, deg); break;
    case kRow64: sort_small<64>(blk, rows, n, off, len, adj, deg); break;
    case kRow32: sort_small<32>(blk, rows, n, off, len, adj, deg); break;
    case kRow16: sort_small<16>(blk, rows, n, off, len, adj, deg); break;
    default: sort_small<8>(blk, rows, n, off, len, adj, deg); break;
  }
}

// Bitonic compare-exchanges of one stride j of stage k on kSortRun ids held
// by one thread in registers (x[r] is id base + r); run-local strides only.
constexpr int kSortRun = 32;
__device__ __forceinline__ void run_stage(int32_t (&x)[kSortRun], int base, int j, int k) {
#pragma unroll
  for (int r = 0; r < kSortRun; ++r) {
    const int pr = r ^ j;
    if (pr > r) {
      const bool up = ((base + r) & k) == 0;
      const int32_t a = x[r], b = x[pr];
      x[r] = up ? min(a, b) : max(a, b);
      x[pr] = up ? max(a, b) : min(a, b);
    }
  }
}

// Rows of up to CAP entries: one block sorts one row (or one chunk) in LDS
// with a bitonic network. Each thread owns a run of 32 consecutive ids: the
// strides below 32 run in its registers (one LDS read and write for all of
// them, the first five stages in one pass), the larger strides in LDS, one
// barrier each. The LDS holds id i at i + i / 32, so a run's ids sit in
// distinct banks for the 32 lanes that read them together. DEDUP: compact
// the unique values in place and write deg; otherwise write the sorted chunk
// back as is.
template <int CAP, int NT, bool DEDUP>
__global__ __launch_bounds__(NT) void k_sort_lds(const int32_t* __restrict__ rows,
                                                 const int64_t* __restrict__ seg_beg,
                                                 const int32_t* __restrict__ seg_len,
                                                 const int64_t* __restrict__ off,
                                                 const int32_t* __restrict__ len,
                                                 int32_t* __restrict__ adj, int32_t* __restrict__ deg) {
  constexpr int R = kSortRun;
  static_assert(CAP % R == 0 && CAP / R <= NT, "one run per thread");
  __shared__ int32_t s[CAP + CAP / R];
  __shared__ int32_t lds_scan[NT / kWave + 1];
  auto at = [](int i) { return i + (i >> 5); };
  int32_t v = -1;
  int64_t beg;
  int32_t L;
  if (DEDUP) {
    v = rows[blockIdx.x];
    beg = off[v];
    L = len[v];
  } else {
    beg = seg_beg[blockIdx.x];
    L = seg_len[blockIdx.x];
  }
  int P = R;
  while (P < L) P <<= 1;
  for (int i = threadIdx.x; i < P; i += NT) s[at(i)] = i < L ? adj[beg + i] : kPad;
  __syncthreads();
  const int g = threadIdx.x;
  const bool owner = g < P / R;  // thread g owns ids g R .. g R + R - 1, at g (R + 1) + r
  int32_t x[R];
  if (owner) {
#pragma unroll
    for (int r = 0; r < R; ++r) x[r] = s[g * (R + 1) + r];
#pragma unroll
    for (int k = 2; k <= R; k <<= 1) {
#pragma unroll
      for (int j = k >> 1; j > 0; j >>= 1) run_stage(x, g * R, j, k);
    }
#pragma unroll
    for (int r = 0; r < R; ++r) s[g * (R + 1) + r] = x[r];
  }
  __syncthreads();
  for (int k = 2 * R; k <= P; k <<= 1) {
    for (int j = k >> 1; j >= R; j >>= 1) {
      for (int i = threadIdx.x; i < (P >> 1); i += NT) {
        const int lo = ((i & ~(j - 1)) << 1) | (i & (j - 1));
        const int hi = lo + j;
        const bool up = (lo & k) == 0;
        const int32_t a = s[at(lo)], b = s[at(hi)];
        if ((a > b) == up) { s[at(lo)] = b; s[at(hi)] = a; }
      }
      __syncthreads();
    }
    if (owner) {
#pragma unroll
      for (int r = 0; r < R; ++r) x[r] = s[g * (R + 1) + r];
#pragma unroll
      for (int j = R >> 1; j > 0; j >>= 1) run_stage(x, g * R, j, k);
#pragma unroll
      for (int r = 0; r < R; ++r) s[g * (R + 1) + r] = x[r];
    }
    __syncthreads();
  }
  if (!DEDUP) {
    for (int i = threadIdx.x; i < L; i += NT) adj[beg + i] = s[at(i)];
    return;
  }
  int32_t carry = 0;
  for (int base = 0; base < L; base += NT) {
    const int i = base + threadIdx.x;
    const int32_t x0 = i < L ? s[at(i)] : kPad;
    const bool u = i < L && (i == 0 || x0 != s[at(i - 1)]);
    int32_t tot;
    const int32_t ex = block_excl_scan<int32_t, NT>(u ? 1 : 0, lds_scan, &tot);
    if (u) adj[beg + carry + ex] = x0;
    carry += tot;
  }
  if (threadIdx.x == 0) deg[v] = carry;
}

// Long rows: the ids of a row that fall into one range of 32 * WORDS ids are
// set in an LDS bitmap (which drops the repeats) and written out in order,
// each wavefront its share of the words. One block per row and range. With
// one range (n <= 32 * WORDS) the row is rewritten in place; with more, each
// block also counts the row's entries below its range, writes its ids to the
// span of `out` that starts there, and k_row_compact closes the gaps.
// Against sorting networks in LDS (above 32,768 entries chunk sorts and merge
// passes), whose one block per row left the chip idle: build + count of an R-MAT
// graph of 240k nodes 1,890 -> 1,331 us, R-MAT 24 94.9 -> 91.5 ms. Bound by the
// LDS passes over the words where rows are short for their range (about 8 us a
// range), by reading the row once per range where they are long: rows with few
// entries per range stay with the networks and merges (see row_bitmap_min).
constexpr int kBitmapNT = 1024;
constexpr int kBitmapUnroll = 8;
constexpr int kBitmapWords = kBitmapIds / 32;  // 128 KB of LDS
constexpr int kBitmapWordsSmall = 8192;        // 2^18 ids, four blocks per CU

template <int WORDS>
__global__ __launch_bounds__(kBitmapNT) void k_sort_bitmap(const int32_t* __restrict__ rows, int32_t nrows,
                                                           int32_t ranges, int32_t n,
                                                           const int64_t* __restrict__ off,
                                                           const int32_t* __restrict__ len, int32_t* adj,
                                                           int32_t* __restrict__ out, int32_t* __restrict__ deg,
                                                           int2* __restrict__ part) {
  constexpr int NW = kBitmapNT / kWave;
  __shared__ uint4 map[WORDS / 4];
  __shared__ int32_t wtot[NW], wlow[NW];
  // the ranges of one row run on one XCD (blocks go to the 8 XCDs in turn):
  // its entries come from that L2 after the first read
  const int32_t per = 8 * ranges;
  const int32_t row = (int32_t)(blockIdx.x / per) * 8 + (int32_t)(blockIdx.x % per) % 8;
  const int32_t r = (int32_t)(blockIdx.x % per) / 8;
  if (row >= nrows) return;
  const int lane = lane_id(), wv = threadIdx.x / kWave;
  const int32_t v = rows[row];
  const int64_t beg = off[v];
  const int32_t L = len[v];
  const int32_t base = r * (32 * WORDS);
  const uint32_t lim = (uint32_t)min((int64_t)32 * WORDS, (int64_t)n - base);
  const int quads = ((int)((lim + 31) / 32) + 3) / 4;
  for (int i = threadIdx.x; i < quads; i += kBitmapNT) map[i] = make_uint4(0, 0, 0, 0);
  __syncthreads();
  uint32_t* word = reinterpret_cast<uint32_t*>(map);
  int32_t low = 0;
  for (int32_t i0 = threadIdx.x; i0 < L; i0 += kBitmapNT * kBitmapUnroll) {
    int32_t x[kBitmapUnroll];
#pragma unroll
    for (int q = 0; q < kBitmapUnroll; ++q) {
      const int32_t i = i0 + q * kBitmapNT;
      x[q] = i < L ? adj[beg + i] : kPad;  // kPad is above every range (ids are below it)
    }
#pragma unroll
    for (int q = 0; q < kBitmapUnroll; ++q) {
      const uint32_t d = (uint32_t)(x[q] - base);
      // equal ids of neighbouring lanes (in rows of 16) set the bit once: atomics
      // on one word follow each other (4M pairs all alike, build 4.2 -> 1.2 ms)
      const uint32_t y = (uint32_t)x[q] + 1u;  // not 0, which the first lane of a row gets
      const bool again = dpp<0x111>(y) == y;
      if (d < lim && !again) atomicOr(&word[d >> 5], 1u << (d & 31));
      low += x[q] < base;
    }
  }
  low = group_sum<int32_t, kWave>(low);
  __syncthreads();
  // wavefront w owns quads [w seg, (w + 1) seg)
  const int seg = (quads + NW * kWave - 1) / (NW * kWave) * kWave;
  const int q0 = wv * seg, q1 = min(quads, q0 + seg);
  int32_t cnt = 0;
  for (int i = q0 + lane; i < q1; i += kWave) {
    const uint4 w = map[i];
    cnt += __popc(w.x) + __popc(w.y) + __popc(w.z) + __popc(w.w);
  }
  cnt = group_sum<int32_t, kWave>(cnt);
  if (lane == 0) {
    wtot[wv] = cnt;
    wlow[wv] = low;
  }
  __syncthreads();
  int32_t at = 0, tot = 0, lower = 0;
#pragma unroll
  for (int k = 0; k < NW; ++k) {
    if (k < wv) at += wtot[k];
    tot += wtot[k];
    lower += wlow[k];
  }
  int32_t* O = ranges == 1 ? adj + beg : out + beg + lower;
  for (int i = q0; i < q1; i += kWave) {
    const uint4 w = i + lane < q1 ? map[i + lane] : make_uint4(0, 0, 0, 0);
    const int32_t c = __popc(w.x) + __popc(w.y) + __popc(w.z) + __popc(w.w);
    if (!__ballot(c != 0)) continue;
    const int32_t incl = wave_incl_scan(c);
    int32_t o = at + incl - c;
    const uint32_t ws[4] = {w.x, w.y, w.z, w.w};
    const int32_t id0 = base + (i + lane) * 128;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      uint32_t bits = ws[k];
      while (bits) {
        O[o++] = id0 + 32 * k + __builtin_ctz(bits);
        bits &= bits - 1;
      }
    }
    at += __builtin_amdgcn_readlane(incl, kWave - 1);
  }
  if (threadIdx.x == 0) {
    if (ranges == 1) deg[v] = tot;
    else part[(int64_t)row * ranges + r] = make_int2(lower, tot);
  }
}

// Joins the ranges of each row: range r's ids move from out[off + lower_r ..]
// to adj behind those of the ranges before it. One block per row and range.
__global__ __launch_bounds__(256) void k_row_compact(const int32_t* __restrict__ rows, int32_t ranges,
                                                     const int64_t* __restrict__ off, const int2* __restrict__ part,
                                                     const int32_t* __restrict__ out, int32_t* __restrict__ adj,
                                                     int32_t* __restrict__ deg) {
  __shared__ int32_t red[256 / kWave + 1];
  const int32_t row = (int32_t)(blockIdx.x / ranges), r = (int32_t)(blockIdx.x % ranges);
  const int2* mine = part + (int64_t)row * ranges;
  int32_t before = 0;
  for (int32_t k = threadIdx.x; k < r; k += 256) before += mine[k].y;
  int32_t at;
  (void)block_excl_scan<int32_t, 256>(before, red, &at);
  const int32_t v = rows[row];
  const int64_t beg = off[v];
  const int2 m = mine[r];
  const int32_t* I = out + beg + m.x;
  int32_t* O = adj + beg + at;
  for (int32_t i = threadIdx.x; i < m.y; i += 256) O[i] = I[i];
  if (r == ranges - 1 && threadIdx.x == 0) deg[v] = at + m.y;
}

// Sorts and dedups the rows of every class but kRowMerge in place and writes
// deg; which go by bitmap: row_first_bitmap_class.
hipError_t launch_sort_rows(const int32_t* rowlist, const int64_t* cls_off, int32_t n, const int64_t* off,
                            const int32_t* len, int32_t* adj, int32_t* deg, int32_t* tmp, int32_t* scratch,
                            hipStream_t s) {
  const int32_t ranges = row_ranges(n);
  SortPlan plan;
  uint32_t blocks[2] = {};  // long, short
  for (int k = 0; k < kSortClasses; ++k) {
    const int cls = kRow4k - k, x = k >= kSortLongClasses;
    plan.row0[k] = (int32_t)cls_off[cls];
    plan.nrows[k] = (int32_t)(cls_off[cls + 1] - cls_off[cls]);
    plan.blk0[k] = blocks[x];
    blocks[x] += row_sort_blocks(plan.nrows[k], k);
  }
  const int first = row_first_bitmap_class(n);
  for (int cls = kRow8k; cls < std::min<int>(first, kRowMerge); ++cls) {
    const int32_t nrows = (int32_t)(cls_off[cls + 1] - cls_off[cls]);
    const int32_t* rows = rowlist + cls_off[cls];
    if (nrows == 0) continue;
    if (cls == kRow8k) k_sort_block<16, 8><<<nrows, 512, 0, s>>>(rows, off, len, adj, deg);
    else if (cls == kRow16k) k_sort_block<16, 16><<<nrows, 1024, 0, s>>>(rows, off, len, adj, deg);
    else k_sort_lds<32768, 1024, true><<<nrows, 1024, 0, s>>>(rows, nullptr, nullptr, off, len, adj, deg);
  }
  if (blocks[0] > 0) k_sort_rows_long<<<blocks[0], 256, 0, s>>>(plan, rowlist, off, len, adj, deg);
  for (uint32_t b0 = 0; b0 < blocks[1]; b0 += kRowShortGrid)
    k_sort_rows_short<<<row_short_grid(blocks[1] - b0), 256, 0, s>>>(plan, b0, rowlist, off, len, adj, deg);
  const int32_t nbig = (int32_t)(cls_off[kNumRowClasses] - cls_off[first]);
  if (nbig > 0) {
    const int32_t* rows = rowlist + cls_off[first];
    int2* part = reinterpret_cast<int2*>(scratch);
    const unsigned grid = (unsigned)row_bitmap_blocks(nbig, ranges);
    if (n <= 32 * kBitmapWordsSmall)
      k_sort_bitmap<kBitmapWordsSmall><<<grid, kBitmapNT, 0, s>>>(rows, nbig, 1, n, off, len, adj, tmp, deg, part);
    else
      k_sort_bitmap<kBitmapWords><<<grid, kBitmapNT, 0, s>>>(rows, nbig, ranges, n, off, len, adj, tmp, deg, part);
    const hipError_t e = hipGetLastError();  // the next kernel follows what this one writes
    if (e != hipSuccess) return e;
    if (ranges > 1)
      k_row_compact<<<(unsigned)(nbig * ranges), 256, 0, s>>>(rows, ranges, off, part, tmp, adj, deg);
  }
  return hipGetLastError();
}

hipError_t launch_sort_chunks(const int64_t* chunk_beg, const int32_t* chunk_len, int32_t nchunks,
                              int32_t* buf, hipStream_t s) {
  if (nchunks == 0) return hipSuccess;
  k_sort_lds<kMergeChunk, 1024, false><<<nchunks, 1024, 0, s>>>(nullptr, chunk_beg, chunk_len, nullptr, nullptr, buf,
                                                                 nullptr);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Merge pass for the rows of kRowMerge (merge path partition, A first on ties).
constexpr int kMergeItems = 8;
static_assert(kMergeTile == 256 * kMergeItems, "tile");

__global__ __launch_bounds__(256) void k_merge(const int64_t* __restrict__ a_beg, const int32_t* __restrict__ la_,
                                               const int32_t* __restrict__ lb_, const int64_t* __restrict__ out_beg,
                                               const int64_t* __restrict__ tile_off, int32_t njobs,
                                               const int32_t* __restrict__ in, int32_t* __restrict__ out) {
  const int64_t tile = blockIdx.x;
  int lo = 0, hi = njobs - 1;  // job = last k with tile_off[k] <= tile
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (tile_off[mid] <= tile) lo = mid; else hi = mid - 1;
  }
  const int job = lo;
  const int32_t la = la_[job], lb = lb_[job];
  const int32_t* A = in + a_beg[job];
  const int32_t* B = A + la;
  int32_t* O = out + out_beg[job];
  const int64_t k0l = (tile - tile_off[job]) * (int64_t)kMergeTile + (int64_t)threadIdx.x * kMergeItems;
  if (k0l >= (int64_t)la + lb) return;
  const int32_t k0 = (int32_t)k0l;
  int32_t b0 = max(0, k0 - lb), e0 = min(k0, la);
  while (b0 < e0) {
    const int32_t mid = (b0 + e0) >> 1;
    if (A[mid] <= B[k0 - 1 - mid]) b0 = mid + 1; else e0 = mid;
  }
  int32_t i = b0, j = k0 - b0;
#pragma unroll
  for (int t = 0; t < kMergeItems; ++t) {
    if (k0 + t >= la + lb) break;
    const bool takeA = j >= lb || (i < la && A[i] <= B[j]);
    O[k0 + t] = takeA ? A[i] : B[j];
    if (takeA) ++i; else ++j;
  }
}

hipError_t launch_merge_pass(const int64_t* a_beg, const int32_t* la, const int32_t* lb,
                             const int64_t* out_beg, const int64_t* tile_off, int32_t njobs,
                             int64_t ntiles, const int32_t* buf_in, int32_t* buf_out, hipStream_t s) {
  if (njobs == 0 || ntiles == 0) return hipSuccess;
  k_merge<<<(unsigned)ntiles, 256, 0, s>>>(a_beg, la, lb, out_beg, tile_off, njobs, buf_in, buf_out);
  return hipGetLastError();
}

constexpr int kDedupNT = 1024;
constexpr int kDedupPer = 4;  // consecutive entries per thread per step

__global__ __launch_bounds__(kDedupNT) void k_dedup_rows(const int32_t* __restrict__ rows,
                                                         const int64_t* __restrict__ seg_beg,
                                                         const int32_t* __restrict__ len,
                                                         const int32_t* __restrict__ sorted,
                                                         const int64_t* __restrict__ off,
                                                         int32_t* __restrict__ adj, int32_t* __restrict__ deg) {
  __shared__ int32_t lds_scan[kDedupNT / kWave + 1];
  const int32_t v = rows[blockIdx.x];
  const int32_t L = len[v];
  const int32_t* S = sorted + seg_beg[blockIdx.x];
  int32_t* D = adj + off[v];
  int32_t carry = 0;
  for (int base = 0; base < L; base += kDedupNT * kDedupPer) {
    const int i0 = base + threadIdx.x * kDedupPer;
    int32_t x[kDedupPer];
    bool u[kDedupPer];
    int32_t c = 0;
    int32_t prev = i0 > 0 && i0 - 1 < L ? S[i0 - 1] : kPad;
#pragma unroll
    for (int q = 0; q < kDedupPer; ++q) {
      const int i = i0 + q;
      x[q] = i < L ? S[i] : kPad;
      u[q] = i < L && (i == 0 || x[q] != prev);
      prev = x[q];
      c += u[q];
    }
    __syncthreads();  // every read of this step precedes the writes (S may alias D)
    int32_t tot;
    int32_t at = carry + block_excl_scan<int32_t, kDedupNT>(c, lds_scan, &tot);
#pragma unroll
    for (int q = 0; q < kDedupPer; ++q)
      if (u[q]) D[at++] = x[q];
    carry += tot;
    __syncthreads();
  }
  if (threadIdx.x == 0) deg[v] = carry;
}

hipError_t launch_dedup_rows(const int32_t* rows, const int64_t* seg_beg, int32_t nrows,
                             const int32_t* len, const int32_t* sorted, const int64_t* off,
                             int32_t* adj, int32_t* deg, hipStream_t s) {
  if (nrows == 0) return hipSuccess;
  k_dedup_rows<<<nrows, kDedupNT, 0, s>>>(rows, seg_beg, len, sorted, off, adj, deg);
  return hipGetLastError();
}

__global__ void k_gather_rows(const int32_t* __restrict__ rows, int32_t nr, const int64_t* __restrict__ off,
                              const int32_t* __restrict__ len, int64_t* __restrict__ out_off,
                              int32_t* __restrict__ out_len) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < nr) { out_off[i] = off[rows[i]]; out_len[i] = len[rows[i]]; }
}

hipError_t launch_gather_rows(const int32_t* rows, int32_t nr, const int64_t* off, const int32_t* len,
                              int64_t* out_off, int32_t* out_len, hipStream_t s) {
  if (nr == 0) return hipSuccess;
  k_gather_rows<<<(nr + 255) / 256, 256, 0, s>>>(rows, nr, off, len, out_off, out_len);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// a4: orientation in one pass over every row plus a copy. The pass counts
// d+(v) and partitions row v into the same span of `part`: N+(v) (ascending)
// from the front, N-(v) from the back in reverse order. After d+ and d- are
// scanned, the copy streams both parts to dcol[doff[v]..] and
// dincol[dinoff[v]..], each ascending. Rows of raw length <= kOrientShort:
// a group of kOrientG lanes per row, grid-stride; medium rows: a wavefront
// each; long rows: a block each (both listed contiguously by the row
// classes).
// Degree classes for the rank test: class(d) = 0 below 64, 1 below 512, 2
// below 4096, else 3, two bits per node (16 nodes per word, 4 MB for 2^24
// nodes, small enough to stay in L2). A class order agrees with the degree
// order, so w ranks above v whenever class(w) > class(v), and below it
// whenever class(w) < class(v); only nodes of one class need d(w) itself.
// At R-MAT 24 about 3 in 4 edges join nodes of different classes, which
// saves that many random gathers of d(w).
__device__ __forceinline__ uint32_t deg_class(int32_t d) {
  return (uint32_t)(d >= 64) + (uint32_t)(d >= 512) + (uint32_t)(d >= 4096);
}

// True when w ranks above v (rank = (key, id), key = d by default); kv, cv =
// key(v), class(key(v)). The classes agree with any key order, so the same
// test serves the degree order and a caller's order (e.g. degeneracy).
__device__ __forceinline__ bool ranks_above(int32_t kv, uint32_t cv, int32_t v, int32_t w,
                                            const int32_t* __restrict__ key, const uint32_t* __restrict__ cls) {
  if (cls) {  // uniform
    const uint32_t cw = (cls[w >> 4] >> (2 * (w & 15))) & 3u;
    if (cw != cv) return cw > cv;
  }
  return rank_below(kv, v, key[w], w);
}

__global__ __launch_bounds__(256) void k_deg_class(int32_t n, const int32_t* __restrict__ key,
                                                   uint32_t* __restrict__ cls) {
  const int64_t words = ((int64_t)n + 15) / 16;
  for (int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; k < words; k += (int64_t)gridDim.x * blockDim.x) {
    uint32_t word = 0;
    for (int j = 0; j < 16; ++j) {
      const int64_t v = k * 16 + j;
      if (v < n) word |= deg_class(key[v]) << (2 * j);
    }
    cls[k] = word;
  }
}

constexpr int kOrientG = 8;
constexpr int32_t kOrientShort = 64;
constexpr int kOrientShortUnroll = 4;  // steps of G entries issued together (short rows)
constexpr int kOrientMedUnroll = 4;    // chunks of 64 entries issued together (medium rows)

// Short rows, a group of 8 lanes each (grid-stride over all nodes, the listed
// rows left out). blk of nblk: this block's place among them.
__device__ __forceinline__ void orient_short(int64_t blk, int64_t nblk, int32_t n, const int32_t* __restrict__ len,
                                             const int64_t* __restrict__ off,
                                             const int32_t* __restrict__ deg, const int32_t* __restrict__ key,
                                             const uint32_t* __restrict__ cls, const int32_t* __restrict__ adj,
                                             int32_t* __restrict__ dplus, int32_t* __restrict__ part) {
  constexpr int G = kOrientG;
  const int64_t ngroups = nblk * (256 / G);
  const int g = threadIdx.x % G;
  const int shift = lane_id() & ~(G - 1);
  for (int64_t v = blk * (256 / G) + threadIdx.x / G; v < n; v += ngroups) {
    if (len[v] > kOrientShort) continue;
    const int32_t dv = deg[v], kv = key[v];
    const uint32_t cv = deg_class(kv);
    const int64_t rb = off[v];
    const int32_t* row = adj + rb;
    int32_t* prow = part + rb;
    int32_t c = 0;
    for (int32_t b = 0; b < dv; b += G * kOrientShortUnroll) {
      int32_t w[kOrientShortUnroll];
      bool f[kOrientShortUnroll];
#pragma unroll
      for (int q = 0; q < kOrientShortUnroll; ++q) {
        const int32_t i = b + q * G + g;
        w[q] = i < dv ? row[i] : 0;
      }
#pragma unroll
      for (int q = 0; q < kOrientShortUnroll; ++q) {
        const int32_t i = b + q * G + g;
        f[q] = i < dv && ranks_above(kv, cv, (int32_t)v, w[q], key, cls);
      }
#pragma unroll
      for (int q = 0; q < kOrientShortUnroll; ++q) {
        const int32_t i = b + q * G + g;
        const uint32_t mask = (uint32_t)(__ballot(f[q]) >> shift) & ((1u << G) - 1);
        const int32_t below = __popc(mask & ((1u << g) - 1));
        if (f[q]) prow[c + below] = w[q];
        else if (i < dv) prow[dv - 1 - (i - (c + below))] = w[q];
        c += __popc(mask);
      }
    }
    if (g == 0) dplus[v] = c;
  }
}

// Rows of medium length: one wavefront per row (grid-stride), ballot-ordered
// compaction, no block barriers.
__device__ __forceinline__ void orient_medium(int64_t blk, int64_t nblk, const int32_t* __restrict__ rows,
                                              int32_t nrows, const int64_t* __restrict__ off,
                                              const int32_t* __restrict__ deg, const int32_t* __restrict__ key,
                                              const uint32_t* __restrict__ cls, const int32_t* __restrict__ adj,
                                              int32_t* __restrict__ dplus, int32_t* __restrict__ part) {
  const int64_t nwaves = nblk * (256 / kWave);
  const int l = lane_id();
  for (int64_t r = blk * (256 / kWave) + threadIdx.x / kWave; r < nrows; r += nwaves) {
    const int32_t v = rows[r];
    const int32_t dv = deg[v], kv = key[v];
    const uint32_t cv = deg_class(kv);
    const int64_t rb = off[v];
    const int32_t* row = adj + rb;
    int32_t* prow = part + rb;
    int32_t c = 0;
    // kOrientMedUnroll chunks of 64 entries per step: their row loads, then
    // their degree gathers, are issued together
    for (int32_t b = 0; b < dv; b += kWave * kOrientMedUnroll) {
      int32_t w[kOrientMedUnroll];
      bool f[kOrientMedUnroll];
#pragma unroll
      for (int q = 0; q < kOrientMedUnroll; ++q) {
        const int32_t i = b + q * kWave + l;
        w[q] = i < dv ? row[i] : 0;
      }
#pragma unroll
      for (int q = 0; q < kOrientMedUnroll; ++q) {
        const int32_t i = b + q * kWave + l;
        f[q] = i < dv && ranks_above(kv, cv, v, w[q], key, cls);
      }
#pragma unroll
      for (int q = 0; q < kOrientMedUnroll; ++q) {
        const int32_t i = b + q * kWave + l;
        const uint64_t m = __ballot(f[q]);
        const int32_t below = mask_below(m);
        if (f[q]) prow[c + below] = w[q];
        else if (i < dv) prow[dv - 1 - (i - (c + below))] = w[q];
        c += (int32_t)__popcll(m);
      }
    }
    if (l == 0) dplus[v] = c;
  }
}

// Both in one launch, the medium rows' blocks first: their last ones run
// beside the short rows.
__global__ __launch_bounds__(256) void k_orient(unsigned nmed_blocks, const int32_t* __restrict__ med_rows,
                                                int32_t nmed, int32_t n, const int32_t* __restrict__ len,
                                                const int64_t* __restrict__ off, const int32_t* __restrict__ deg,
                                                const int32_t* __restrict__ key, const uint32_t* __restrict__ cls,
                                                const int32_t* __restrict__ adj, int32_t* __restrict__ dplus,
                                                int32_t* __restrict__ part) {
  if (blockIdx.x < nmed_blocks)
    orient_medium(blockIdx.x, nmed_blocks, med_rows, nmed, off, deg, key, cls, adj, dplus, part);
  else
    orient_short(blockIdx.x - nmed_blocks, gridDim.x - nmed_blocks, n, len, off, deg, key, cls, adj, dplus, part);
}

constexpr int kOrientLongNT = 1024;
constexpr int kOrientLongPer = 4;  // consecutive entries per thread per step

__global__ __launch_bounds__(kOrientLongNT) void k_orient_long(const int32_t* __restrict__ rows,
                                                               const int64_t* __restrict__ off,
                                                               const int32_t* __restrict__ deg,
                                                               const int32_t* __restrict__ key,
                                                               const uint32_t* __restrict__ cls,
                                                               const int32_t* __restrict__ adj,
                                                               int32_t* __restrict__ dplus,
                                                               int32_t* __restrict__ part) {
  __shared__ int32_t lds[kOrientLongNT / kWave + 1];
  const int32_t v = rows[blockIdx.x];
  const int32_t dv = deg[v], kv = key[v];
  const uint32_t cv = deg_class(kv);
  const int64_t rb = off[v];
  const int32_t* row = adj + rb;
  int32_t* prow = part + rb;
  int32_t c = 0;
  for (int32_t b = 0; b < dv; b += kOrientLongNT * kOrientLongPer) {
    const int32_t i0 = b + threadIdx.x * kOrientLongPer;
    int32_t w[kOrientLongPer];
    bool f[kOrientLongPer];
    int32_t k = 0;
#pragma unroll
    for (int q = 0; q < kOrientLongPer; ++q) w[q] = i0 + q < dv ? row[i0 + q] : 0;
#pragma unroll
    for (int q = 0; q < kOrientLongPer; ++q) {
      f[q] = i0 + q < dv && ranks_above(kv, cv, v, w[q], key, cls);
      k += f[q];
    }
    int32_t tot;
    int32_t o = c + block_excl_scan<int32_t, kOrientLongNT>(k, lds, &tot);  // out-entries before i0
#pragma unroll
    for (int q = 0; q < kOrientLongPer; ++q) {
      const int32_t i = i0 + q;
      if (i >= dv) break;
      if (f[q]) prow[o++] = w[q];
      else prow[dv - 1 - (i - o)] = w[q];
    }
    c += tot;
  }
  if (threadIdx.x == 0) dplus[v] = c;
}

// Copy of the partitioned rows: N+(v) = part[off[v] .. off[v] + d+(v)) to
// dcol[doff[v] ..]; N-(v) = part[off[v] + d(v) - 1 - k], k < d-(v), to
// dincol[dinoff[v] + k] (ascending again). G lanes per row (G = 8, 64 or
// 256), rows short (all rows of raw length <= kOrientShort, grid-stride),
// or listed.
template <int G>
__device__ __forceinline__ void orient_copy_row(int32_t v, int g, const int64_t* __restrict__ off,
                                                const int32_t* __restrict__ deg,
                                                const int32_t* __restrict__ dplus,
                                                const int32_t* __restrict__ part, const int64_t* __restrict__ doff,
                                                int32_t* __restrict__ dcol, const int64_t* __restrict__ dinoff,
                                                int32_t* __restrict__ dincol) {
  constexpr int U = 4;  // loads of each list issued together per step
  const int32_t dv = deg[v], dp = dplus[v];
  const int32_t di = dincol ? dv - dp : 0;
  const int32_t* prow = part + off[v];
  const int32_t* pend = prow + dv - 1;
  int32_t* out = dcol + doff[v];
  int32_t* in = dincol ? dincol + dinoff[v] : nullptr;
  const int32_t dm = max(dp, di);
  for (int32_t k0 = g; k0 < dm; k0 += G * U) {
    int32_t a[U], b[U];
#pragma unroll
    for (int q = 0; q < U; ++q) {
      const int32_t k = k0 + q * G;
      a[q] = k < dp ? prow[k] : 0;
      b[q] = k < di ? pend[-k] : 0;
    }
#pragma unroll
    for (int q = 0; q < U; ++q) {
      const int32_t k = k0 + q * G;
      if (k < dp) out[k] = a[q];
      if (k < di) in[k] = b[q];
    }
  }
}

// The copies of all rows in one launch: blocks for the long rows (a block per
// row), then the medium ones (a wavefront per row), then all short ones.
struct CopyGrid {
  unsigned long_blocks, medium_blocks;
};

__global__ __launch_bounds__(256) void k_orient_copy(CopyGrid grid, const int32_t* __restrict__ long_rows,
                                                     int32_t nlong, const int32_t* __restrict__ medium_rows,
                                                     int32_t nmedium, int32_t n, const int64_t* __restrict__ off,
                                                     const int32_t* __restrict__ len,
                                                     const int32_t* __restrict__ deg,
                                                     const int32_t* __restrict__ dplus,
                                                     const int32_t* __restrict__ part,
                                                     const int64_t* __restrict__ doff, int32_t* __restrict__ dcol,
                                                     const int64_t* __restrict__ dinoff,
                                                     int32_t* __restrict__ dincol) {
  int64_t blk = blockIdx.x;
  if (blk < grid.long_blocks) {
    for (int64_t r = blk; r < nlong; r += grid.long_blocks)
      orient_copy_row<256>(long_rows[r], threadIdx.x, off, deg, dplus, part, doff, dcol, dinoff, dincol);
    return;
  }
  blk -= grid.long_blocks;
  if (blk < grid.medium_blocks) {
    const int64_t step = (int64_t)grid.medium_blocks * (256 / kWave);
    for (int64_t r = blk * (256 / kWave) + threadIdx.x / kWave; r < nmedium; r += step)
      orient_copy_row<kWave>(medium_rows[r], threadIdx.x % kWave, off, deg, dplus, part, doff, dcol, dinoff, dincol);
    return;
  }
  blk -= grid.medium_blocks;
  constexpr int G = kOrientG;
  const int64_t step = ((int64_t)gridDim.x - grid.long_blocks - grid.medium_blocks) * (256 / G);
  for (int64_t v = blk * (256 / G) + threadIdx.x / G; v < n; v += step) {
    if (len[v] > kOrientShort) continue;
    orient_copy_row<G>((int32_t)v, threadIdx.x % G, off, deg, dplus, part, doff, dcol, dinoff, dincol);
  }
}

// Up to this many ids the keys themselves stay in L2 (4 MB per XCD): no class
// words, which cost a launch to form.
constexpr int32_t kOrientClassMin = 1 << 20;

hipError_t launch_orient(int32_t n, const int64_t* off, const int32_t* len, const int32_t* deg, const int32_t* key,
                         const int32_t* adj, const int32_t* medium_rows, int32_t nmedium, const int32_t* long_rows,
                         int32_t nlong, uint32_t* cls, int32_t* dplus, int32_t* part, hipStream_t s) {
  if (n == 0) return hipSuccess;
  if (!key) key = deg;
  if (n <= kOrientClassMin) cls = nullptr;
  if (cls) k_deg_class<<<grid_for(((int64_t)n + 15) / 16, 256, 4096), 256, 0, s>>>(n, key, cls);
  if (nlong > 0)
    k_orient_long<<<nlong, kOrientLongNT, 0, s>>>(long_rows, off, deg, key, cls, adj, dplus, part);
  const unsigned mb = nmedium > 0 ? grid_for((int64_t)nmedium * kWave, 256, 1u << 14) : 0;
  const unsigned sb = grid_for((int64_t)n * kOrientG, 256, 1u << 16);
  k_orient<<<mb + sb, 256, 0, s>>>(mb, medium_rows, nmedium, n, len, off, deg, key, cls, adj, dplus, part);
  return hipGetLastError();
}

hipError_t launch_orient_copy(int32_t n, const int64_t* off, const int32_t* len, const int32_t* deg,
                              const int32_t* dplus, const int32_t* part, const int32_t* medium_rows, int32_t nmedium,
                              const int32_t* long_rows, int32_t nlong, const int64_t* doff, int32_t* dcol,
                              const int64_t* dinoff, int32_t* dincol, hipStream_t s) {
  if (n == 0) return hipSuccess;
  CopyGrid g;
  g.long_blocks = (unsigned)std::min(nlong, 1 << 14);
  g.medium_blocks = nmedium > 0 ? grid_for((int64_t)nmedium * kWave, 256, 1u << 14) : 0;
  const unsigned sb = grid_for((int64_t)n * kOrientG, 256, 1u << 16);
  k_orient_copy<<<g.long_blocks + g.medium_blocks + sb, 256, 0, s>>>(g, long_rows, nlong, medium_rows, nmedium, n, off,
                                                                 len, deg, dplus, part, doff, dcol, dinoff, dincol);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Graphs handed over as a CSR (rows d_col[rowptr[v] .. rowptr[v+1])).
// Row v's bounds: rowptr[0] == 0, non-decreasing, rowptr[n] == nnz.
__device__ __forceinline__ bool csr_row_ok(int64_t v, int32_t n, int64_t nnz, int64_t b, int64_t e) {
  return !(b > e || b < 0 || e > nnz || (v == 0 && b != 0) || (v == n - 1 && e != nnz));
}

__global__ __launch_bounds__(256) void k_csr_bounds(int32_t n, int64_t nnz, const int64_t* __restrict__ rowptr,
                                                    int32_t* __restrict__ err) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  bool bad = false;
  for (int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; v < n; v += stride)
    bad |= !csr_row_ok(v, n, nnz, rowptr[v], rowptr[v + 1]);
  if (n == 0 && blockIdx.x == 0 && threadIdx.x == 0 && (rowptr[0] != 0 || nnz != 0)) bad = true;
  if (__ballot(bad) && lane_id() == 0) atomicOr(err, 4);
}

// Rows taken as they are: off = rowptr, len = deg = row lengths (0 for a row
// whose bounds are bad: bit 4 of err[0]), adj = col, and the rows checked: ids in
// [0, n) (else bit 1), without the row's own id (else bit 2) and strictly
// ascending (else err[1] is not 0). Entries are shared out evenly, whatever the
// rows' lengths: one wavefront per row took 446 us at R-MAT 20, most of them on
// its few rows of 10^4 to 6 10^4 entries. A step that does not rise from
// col[i - 1] to col[i] is right only where a row starts: err[1] is the number of
// such steps less those at row starts. (A search of the row offsets at each such
// step, one a row, missed the L2 where the offsets outgrow it: a CSR of 4M nodes
// and 200M entries, whole count, 15.1 ms, now 11.8; 13.4 with a wavefront per row.)
// A row's own id is searched in its sorted row, inside the array whatever it holds.
__global__ __launch_bounds__(256) void k_csr_take(int32_t n, int64_t nnz, const int64_t* __restrict__ rowptr,
                                                  const int32_t* __restrict__ col, int64_t* __restrict__ off,
                                                  int32_t* __restrict__ len, int32_t* __restrict__ deg,
                                                  int32_t* __restrict__ adj, int32_t* __restrict__ err) {
  __shared__ int32_t red[256 / kWave];
  const int64_t stride = (int64_t)gridDim.x * 256;
  const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x;
  int32_t bad = 0, falls = 0;
  for (int64_t v = t; v < n; v += stride) {
    const int64_t b = rowptr[v], e = rowptr[v + 1];
    const bool ok = csr_row_ok(v, n, nnz, b, e);
    if (!ok) bad |= 4;
    const int32_t l = ok ? (int32_t)(e - b) : 0;
    off[v] = b;
    len[v] = l;
    deg[v] = l;
    if (l > 0) {
      if (b > 0 && col[b - 1] >= col[b]) --falls;
      int64_t lo = b, hi = e;
      while (lo < hi) {
        const int64_t mid = (lo + hi) >> 1;
        if (col[mid] < (int32_t)v) lo = mid + 1; else hi = mid;
      }
      if (lo < e && col[lo] == (int32_t)v) bad |= 2;
    }
  }
  if (t == 0) {
    off[n] = rowptr[n];
    if (n == 0 && (rowptr[0] != 0 || nnz != 0)) bad |= 4;
  }
  constexpr int U = 4;
  for (int64_t i0 = t; i0 < nnz; i0 += stride * U) {
    int32_t x[U], y[U];
#pragma unroll
    for (int q = 0; q < U; ++q) {
      const int64_t i = i0 + q * stride;
      x[q] = i < nnz ? col[i] : 0;
      y[q] = i < nnz && i > 0 ? col[i - 1] : INT32_MIN;
    }
#pragma unroll
    for (int q = 0; q < U; ++q) {
      const int64_t i = i0 + q * stride;
      if (i >= nnz) break;
      adj[i] = x[q];
      if ((uint32_t)x[q] >= (uint32_t)n) bad |= 1;
      falls += i > 0 && y[q] >= x[q];
    }
  }
#pragma unroll
  for (int bit = 1; bit <= 4; bit <<= 1)
    if (__ballot(bad & bit) && lane_id() == 0) atomicOr(&err[0], bit);
  falls = block_sum<int32_t, 256>(falls, red);
  if (threadIdx.x == 0 && falls) atomicAdd(&err[1], falls);
}

// src[i] = v for every entry i of row v: the CSR as a list of (v, w) pairs.
__global__ __launch_bounds__(256) void k_csr_expand(int32_t n, const int64_t* __restrict__ rowptr,
                                                    int32_t* __restrict__ src) {
  const int lane = lane_id();
  const int64_t nw = (int64_t)gridDim.x * (blockDim.x / kWave);
  for (int64_t v = (int64_t)blockIdx.x * (blockDim.x / kWave) + threadIdx.x / kWave; v < n; v += nw) {
    const int64_t b = rowptr[v], e = rowptr[v + 1];
    for (int64_t i = b + lane; i < e; i += kWave) src[i] = (int32_t)v;
  }
}

hipError_t launch_csr_bounds(int32_t n, int64_t nnz, const int64_t* rowptr, int32_t* err, hipStream_t s) {
  k_csr_bounds<<<grid_for(n > 0 ? n : 1, 256, 1u << 16), 256, 0, s>>>(n, nnz, rowptr, err);
  return hipGetLastError();
}

hipError_t launch_csr_take(int32_t n, int64_t nnz, const int64_t* rowptr, const int32_t* col, int64_t* off,
                           int32_t* len, int32_t* deg, int32_t* adj, int32_t* err, hipStream_t s) {
  // eight blocks a CU fill it, and each adds to err[1] once
  k_csr_take<<<grid_for(std::max<int64_t>(n, nnz / 4), 256, 2048), 256, 0, s>>>(n, nnz, rowptr, col, off, len,
                                                                                  deg, adj, err);
  return hipGetLastError();
}

hipError_t launch_csr_expand(int32_t n, const int64_t* rowptr, int32_t* src, hipStream_t s) {
  if (n == 0) return hipSuccess;
  k_csr_expand<<<grid_for(n, 4, 1u << 16), 256, 0, s>>>(n, rowptr, src);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// a2 of the DAG and a5 together: offsets of the out- and in-lists, the
// edge-existence records, the node bins, the in-list owners by bin and their
// chunk prefix, in two passes over (d, d+). Pass 1 leaves one column of sums
// per tile of nodes; pass 2 adds up the columns before its own, so that no
// separate scan of the sums is needed (at most 1,024 tiles), and places its
// nodes with wave ballots and one LDS cursor per bin. Bound by launches and
// host round trips on small graphs, by about 60 bytes of traffic a node on
// large ones. Measured against two classifications, three scans and four
// single-purpose kernels (31 launches, five round trips; now two launches,
// one round trip): build + count of G(10^4, 10^5) 497 -> 301 us, an R-MAT
// graph of 240k nodes 2,339 -> 2,019 us.
// Node u with d+(u) >= 2: the first bin whose limit holds d+; else -1.
__device__ __forceinline__ int node_bin(int32_t p, const BinParams& bp) {
  if (p < 2) return -1;
  int b = kNumBins - 1;
#pragma unroll
  for (int q = kNumBins - 2; q >= 0; --q)
    if (p <= bp.limit[q]) b = q;
  return b;
}

// In-list pass owners: 3 <= d+(w) <= limit[4], at least one in-neighbour.
__device__ __forceinline__ int in_bin(int32_t d, int32_t p, const BinParams& bp) {
  if (!bp.min_side || p < 3 || d - p < 1 || p > bp.limit[kNumBins - 2]) return -1;
  int b = kNumBins - 2;
#pragma unroll
  for (int q = kNumBins - 3; q >= 0; --q)
    if (p <= bp.limit[q]) b = q;
  return b;
}

// In-list chunks of an owner of bin b (chunk = what the bin's table holds).
__device__ __forceinline__ int32_t in_chunks(int32_t din, int b, const BinParams& bp) {
  int32_t c = 1;
#pragma unroll
  for (int q = 0; q < kNumBins; ++q)
    if (q == b) c = bp.cap[q];
  return (int32_t)(((int64_t)din + c - 1) / c);
}

__device__ __forceinline__ int32_t wave_max_i32(int32_t x) {
#pragma unroll
  for (int o = kWave / 2; o > 0; o >>= 1) x = max(x, __shfl_xor(x, o, kWave));
  return x;
}

__global__ __launch_bounds__(kLayoutNT) void k_layout_count(int32_t n, int64_t tile,
                                                            const int32_t* __restrict__ deg,
                                                            const int32_t* __restrict__ dplus, BinParams bp,
                                                            int32_t* __restrict__ sums) {
  __shared__ int32_t acc[kLayoutQ];
  if (threadIdx.x < kLayoutQ) acc[threadIdx.x] = 0;
  __syncthreads();
  const int64_t t0 = (int64_t)blockIdx.x * tile, t1 = min((int64_t)n, t0 + tile);
  int32_t sp = 0, si = 0, c2 = 0, mxd = 0, mxp = 0;  // c2 and the bin counts are wave-uniform
  int32_t nb[kNumBins] = {}, ib[kNumBins] = {}, it[kNumBins] = {};
  for (int64_t b = t0; b < t1; b += kLayoutNT) {
    const int64_t v = b + threadIdx.x;
    const int32_t d = v < t1 ? deg[v] : 0, p = v < t1 ? dplus[v] : 0;
    sp += p;
    si += d - p;
    mxd = max(mxd, d);
    mxp = max(mxp, p);
    c2 += (int32_t)__popcll(__ballot(d >= 2));
    const int x = node_bin(p, bp), y = in_bin(d, p, bp);
#pragma unroll
    for (int q = 0; q < kNumBins; ++q) nb[q] += (int32_t)__popcll(__ballot(x == q));
    if (__ballot(y >= 0)) {
      const int32_t k = y >= 0 ? in_chunks(d - p, y, bp) : 0;
#pragma unroll
      for (int q = 0; q < kNumBins; ++q) {
        ib[q] += (int32_t)__popcll(__ballot(y == q));
        it[q] += y == q ? k : 0;
      }
    }
  }
  sp = group_sum<int32_t, kWave>(sp);
  si = group_sum<int32_t, kWave>(si);
  mxd = wave_max_i32(mxd);
  mxp = wave_max_i32(mxp);
#pragma unroll
  for (int q = 0; q < kNumBins; ++q) it[q] = group_sum<int32_t, kWave>(it[q]);
  if (lane_id() == 0) {
    atomicAdd(&acc[kLqOut], sp);
    atomicAdd(&acc[kLqIn], si);
    atomicAdd(&acc[kLqDeg2], c2);
    atomicMax(&acc[kLqMaxD], mxd);
    atomicMax(&acc[kLqMaxP], mxp);
#pragma unroll
    for (int q = 0; q < kNumBins; ++q) {
      if (nb[q]) atomicAdd(&acc[kLqBin + q], nb[q]);
      if (ib[q]) atomicAdd(&acc[kLqInBin + q], ib[q]);
      if (it[q]) atomicAdd(&acc[kLqItems + q], it[q]);
    }
  }
  __syncthreads();
  if (threadIdx.x < kLayoutQ) sums[(int64_t)threadIdx.x * gridDim.x + blockIdx.x] = acc[threadIdx.x];
}

// OFFSETS: the offsets and records too (of a new DAG), else the bins alone.
template <bool OFFSETS>
__global__ __launch_bounds__(kLayoutNT) void k_layout_place(int32_t n, int64_t tile, BinParams bp,
                                                            const int32_t* __restrict__ sums, LayoutOut o) {
  __shared__ int32_t prev[kLayoutQ], all[kLayoutQ];
  __shared__ int32_t ncur[kNumBins];
  __shared__ unsigned long long icur[kNumBins];  // list position << 32 | chunk
  __shared__ unsigned long long red[kLayoutNT / kWave + 1];
  const int lane = lane_id(), wv = threadIdx.x / kWave;
  const int nt = (int)gridDim.x, me = (int)blockIdx.x;
  for (int q = wv; q < kLayoutQ; q += kLayoutNT / kWave) {
    int32_t p = 0, a = 0;
    for (int b = lane; b < nt; b += kWave) {
      const int32_t x = sums[(int64_t)q * nt + b];
      if (q >= kLqMaxD) a = max(a, x);
      else a += x;
      if (b < me) p += x;
    }
    p = group_sum<int32_t, kWave>(p);
    a = q >= kLqMaxD ? wave_max_i32(a) : group_sum<int32_t, kWave>(a);
    if (lane == 0) {
      prev[q] = p;
      all[q] = a;
    }
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    int64_t nb = 0, ib = 0, it = 0;
    for (int q = 0; q <= kNumBins; ++q) {
      if (me == 0) {
        o.bin_off[q] = nb;
        o.in_off[q] = ib;
        o.in_items[q] = it;
      }
      if (q == kNumBins) break;
      ncur[q] = (int32_t)nb + prev[kLqBin + q];
      icur[q] = ((unsigned long long)(ib + prev[kLqInBin + q]) << 32) | (unsigned long long)(it + prev[kLqItems + q]);
      nb += all[kLqBin + q];
      ib += all[kLqInBin + q];
      it += all[kLqItems + q];
    }
    if (me == 0) {
      if (OFFSETS) {
        o.doff[n] = all[kLqOut];
        o.dinoff[n] = all[kLqIn];
        o.stats[0] = all[kLqMaxD];
        o.stats[1] = all[kLqMaxP];
        o.stats[2] = all[kLqDeg2];
        *o.m = all[kLqOut];
      }
      if (bp.min_side) o.incoff[ib] = it;
      for (int q = 0; q < kNumBins - 1; ++q) o.limit[q] = bp.limit[q];
      for (int q = 0; q < kNumBins; ++q) o.cap[q] = bp.cap[q];
    }
  }
  __syncthreads();
  int64_t runp = prev[kLqOut], runi = prev[kLqIn];
  const int64_t t0 = (int64_t)me * tile, t1 = min((int64_t)n, t0 + tile);
  for (int64_t b = t0; b < t1; b += kLayoutNT) {
    const int64_t v = b + threadIdx.x;
    const bool in = v < t1;
    const int32_t d = in ? o.deg[v] : 0, p = in ? o.dplus[v] : 0;
    if (OFFSETS) {
      unsigned long long tot;
      // both sums stay below 2^31: one scan of the two packed
      const unsigned long long ex = block_excl_scan<unsigned long long, kLayoutNT>(
          ((unsigned long long)(uint32_t)p << 32) | (unsigned long long)(uint32_t)(d - p), red, &tot);
      if (in) {
        o.doff[v] = runp + (int64_t)(ex >> 32);
        o.dinoff[v] = runi + (int64_t)(ex & 0xffffffffull);
        o.din[v] = d - p;
        o.rec[v] = make_int2((int32_t)(uint32_t)o.raw_off[v], d);
      }
      runp += (int64_t)(tot >> 32);
      runi += (int64_t)(tot & 0xffffffffull);
    } else {
      __syncthreads();  // the lists ascend by 1,024 ids here too
    }
    const int x = node_bin(p, bp), y = in_bin(d, p, bp);
#pragma unroll
    for (int q = 0; q < kNumBins; ++q) {
      const uint64_t m = __ballot(x == q);
      if (!m) continue;
      int32_t at = 0;
      if (lane == 0) at = atomicAdd(&ncur[q], (int32_t)__popcll(m));
      at = __builtin_amdgcn_readfirstlane(at);
      if (x == q) o.binlist[at + mask_below(m)] = (int32_t)v;
    }
    if (!__ballot(y >= 0)) continue;
    const int32_t k = y >= 0 ? in_chunks(d - p, y, bp) : 0;
#pragma unroll
    for (int q = 0; q < kNumBins; ++q) {
      const uint64_t m = __ballot(y == q);
      if (!m) continue;
      const int32_t kq = y == q ? k : 0;
      const int32_t incl = wave_incl_scan(kq);
      const int32_t sum = __builtin_amdgcn_readlane(incl, kWave - 1);
      unsigned long long at = 0;
      if (lane == 0)
        at = atomicAdd(&icur[q], ((unsigned long long)__popcll(m) << 32) | (unsigned long long)(uint32_t)sum);
      const int32_t ap = __builtin_amdgcn_readfirstlane((int32_t)(at >> 32));
      const int32_t ac = __builtin_amdgcn_readfirstlane((int32_t)(at & 0xffffffffull));
      if (y == q) {
        const int32_t i = ap + mask_below(m);
        o.inlist[i] = (int32_t)v;
        o.incoff[i] = (int64_t)ac + incl - kq;
      }
    }
  }
}

hipError_t launch_layout(int32_t n, const BinParams& bp, bool offsets, int32_t* sums, const LayoutOut& o,
                         hipStream_t s) {
  if (n <= 0) return hipSuccess;
  const int64_t tile = layout_tile(n);
  const unsigned nt = (unsigned)((n + tile - 1) / tile);
  k_layout_count<<<nt, kLayoutNT, 0, s>>>(n, tile, o.deg, o.dplus, bp, sums);
  if (offsets) k_layout_place<true><<<nt, kLayoutNT, 0, s>>>(n, tile, bp, sums, o);
  else k_layout_place<false><<<nt, kLayoutNT, 0, s>>>(n, tile, bp, sums, o);
  return hipGetLastError();
}

// Chunk -> owner map of the in-list items, so that a work item finds its
// owner with one load instead of a search over the chunk prefix. The list's
// length is read on the device. An owner's run of chunks is written by its
// lane, runs above kOwnerRun (hubs with a small table) by the wavefront: one
// lane alone took 6,300 stores for the largest hub of R-MAT 24.
constexpr int32_t kOwnerRun = 16;

__global__ __launch_bounds__(256) void k_in_owners(const int64_t* __restrict__ nlist_at,
                                                   const int64_t* __restrict__ coff, int32_t* __restrict__ owner) {
  const int64_t nlist = *nlist_at;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  const int lane = lane_id();
  for (int64_t b = (int64_t)blockIdx.x * blockDim.x; b < nlist; b += stride) {  // uniform trip count
    const int64_t i = b + threadIdx.x;
    int64_t c0 = 0;
    int32_t k = 0;
    if (i < nlist) {
      c0 = coff[i];
      k = (int32_t)(coff[i + 1] - c0);
    }
    for (int32_t c = 0; c < k && k <= kOwnerRun; ++c) owner[c0 + c] = (int32_t)i;
    uint64_t big = __ballot(k > kOwnerRun);
    while (big) {
      const int src = __builtin_ctzll(big);
      big &= big - 1;
      const int32_t kk = __shfl(k, src, kWave), ii = __shfl((int32_t)i, src, kWave);
      const int64_t cc = __shfl((int32_t)c0, src, kWave);  // chunks stay below 2^31
      for (int32_t c = lane; c < kk; c += kWave) owner[cc + c] = ii;
    }
  }
}

hipError_t launch_in_owners(int32_t n, const int64_t* nlist, const int64_t* coff, int32_t* owner, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  k_in_owners<<<grid_for(n, 256 * 4, 4096), 256, 0, s>>>(nlist, coff, owner);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// sum over DAG edges u->w of d+(u) + d+(w): the list elements a merge-based
// intersection reads (the algorithmic-bytes measure of the hot loop).
__global__ __launch_bounds__(256) void k_list_elems(int32_t n, const int64_t* __restrict__ doff,
                                                    const int32_t* __restrict__ dcol,
                                                    unsigned long long* __restrict__ out) {
  const int64_t nwaves = (int64_t)gridDim.x * (blockDim.x / kWave);
  const int64_t w0 = (int64_t)blockIdx.x * (blockDim.x / kWave) + threadIdx.x / kWave;
  const int l = lane_id();
  unsigned long long acc = 0;
  for (int64_t u = w0; u < n; u += nwaves) {
    const int64_t b = doff[u], e = doff[u + 1];
    const unsigned long long du = (unsigned long long)(e - b);
    for (int64_t p = b + l; p < e; p += kWave) {
      const int32_t w = dcol[p];
      acc += du + (unsigned long long)(doff[w + 1] - doff[w]);
    }
  }
  acc = group_sum<unsigned long long, kWave>(acc);
  if (l == 0 && acc) atomicAdd(out, acc);
}

hipError_t launch_list_elems(int32_t n, const int64_t* doff, const int32_t* dcol, unsigned long long* out,
                             hipStream_t s) {
  if (n == 0) return hipSuccess;
  k_list_elems<<<grid_for((int64_t)n * kWave, 256, 1u << 14), 256, 0, s>>>(n, doff, dcol, out);
  return hipGetLastError();
}

// Per-bin algorithmic sizes: every DAG edge u->w with d+(u) >= 2 is charged
// to the bin whose kernel counts it: w's bin (by d+(w)) when the min-side
// rule hands it to w's in-list (d+(u) < d+(w) <= w_max), else u's bin.
// elems[b] += d+(u) + d+(w), edges[b] += 1. Wave per node, grid-stride.
__device__ __forceinline__ int bin_of(int32_t d, const int32_t* lim) {
  int b = kNumBins - 1;
#pragma unroll
  for (int q = kNumBins - 2; q >= 0; --q)
    if (d <= lim[q]) b = q;
  return b;
}

// Per bin b, over the DAG edges u->w that bin b's kernel counts (min-side
// ownership with w_max; w_max = 0 counts every edge from its tail):
//   elems[b]  sum of d+(u) + d+(w) (what a merge of both lists reads)
//   edges[b]  number of such edges
//   kbytes[b] bytes the min-side kernel moves for the bin when nothing is
//             reused between its work items: per out-list item u, its row
//             bounds (16), N+(u) for the table (4 d+(u)), the row bounds of
//             every w (16 d+(u)) and the T credits (8 (d+(u) + 1)); per
//             streamed list its ids (4 per id); per in-list chunk of w (din
//             in-neighbours, chunks of cap[b]), its bounds (32), N+(w) for
//             the table and the credits (12 d+(w) + 8); per in-neighbour its
//             entry and row bounds (20) and, if its list is streamed, its
//             credit (8).
__global__ __launch_bounds__(256) void k_bin_elems(int32_t n, const int64_t* __restrict__ doff,
                                                   const int32_t* __restrict__ dcol,
                                                   const int32_t* __restrict__ din,
                                                   const int32_t* __restrict__ limit,
                                                   const int32_t* __restrict__ cap, int32_t w_max,
                                                   unsigned long long* __restrict__ elems,
                                                   unsigned long long* __restrict__ edges,
                                                   unsigned long long* __restrict__ kbytes) {
  int32_t lim[kNumBins - 1];
#pragma unroll
  for (int q = 0; q < kNumBins - 1; ++q) lim[q] = limit[q];
  const int64_t nwaves = (int64_t)gridDim.x * (blockDim.x / kWave);
  const int l = lane_id();
  unsigned long long acc[kNumBins] = {}, eacc[kNumBins] = {}, kacc[kNumBins] = {};
  for (int64_t u = (int64_t)blockIdx.x * (blockDim.x / kWave) + threadIdx.x / kWave; u < n; u += nwaves) {
    const int64_t beg = doff[u], end = doff[u + 1];
    const int32_t du = (int32_t)(end - beg);
    const int bu = bin_of(du, lim);
    if (l == 0) {
      unsigned long long kb = 0;
      if (du >= 2) kb += 16ull + 28ull * (unsigned long long)du + 8ull;
      const int32_t di = din ? din[u] : 0;
      if (w_max > 0 && du >= 3 && du <= w_max && di >= 1) {
        const int32_t c = max(1, cap[bu]);
        const unsigned long long chunks = (unsigned long long)((di + c - 1) / c);
        kb += chunks * (40ull + 12ull * (unsigned long long)du) + 20ull * (unsigned long long)di;
      }
#pragma unroll
      for (int q = 0; q < kNumBins; ++q)
        if (q == bu) kacc[q] += kb;
    }
    if (du < 2) continue;
    for (int64_t p = beg + l; p < end; p += kWave) {
      const int32_t w = dcol[p];
      const int32_t dw = (int32_t)(doff[w + 1] - doff[w]);
      const bool in_side = du < dw && dw <= w_max;
      const int b = in_side ? bin_of(dw, lim) : bu;
      const unsigned long long kb = in_side ? 4ull * (unsigned long long)du + 8ull : 4ull * (unsigned long long)dw;
#pragma unroll
      for (int q = 0; q < kNumBins; ++q)
        if (q == b) { acc[q] += (unsigned long long)(du + dw); eacc[q] += 1; kacc[q] += kb; }
    }
  }
#pragma unroll
  for (int q = 0; q < kNumBins; ++q) {
    const unsigned long long a = group_sum<unsigned long long, kWave>(acc[q]);
    const unsigned long long e = group_sum<unsigned long long, kWave>(eacc[q]);
    const unsigned long long k = group_sum<unsigned long long, kWave>(kacc[q]);
    if (l == 0 && a) atomicAdd(&elems[q], a);
    if (l == 0 && e) atomicAdd(&edges[q], e);
    if (l == 0 && k) atomicAdd(&kbytes[q], k);
  }
}

hipError_t launch_bin_elems(int32_t n, const int64_t* doff, const int32_t* dcol, const int32_t* din,
                            const int32_t* limit, const int32_t* cap, int32_t w_max, unsigned long long* elems,
                            unsigned long long* edges, unsigned long long* kbytes, hipStream_t s) {
  if (n == 0) return hipSuccess;
  k_bin_elems<<<grid_for((int64_t)n * kWave, 256, 1u << 14), 256, 0, s>>>(n, doff, dcol, din, limit, cap, w_max,
                                                                         elems, edges, kbytes);
  return hipGetLastError();
}

// Streaming copy, 16 bytes per lane per iteration (the bandwidth probe).
__global__ __launch_bounds__(256) void k_probe_copy(uint4* __restrict__ dst, const uint4* __restrict__ src,
                                                    int64_t n16) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n16; i += stride) dst[i] = src[i];
}

hipError_t launch_probe_copy(void* dst, const void* src, size_t bytes, hipStream_t s) {
  const int64_t n16 = (int64_t)(bytes / 16);
  if (n16 == 0) return hipSuccess;
  k_probe_copy<<<grid_for(n16, 256 * 4, 8192), 256, 0, s>>>(static_cast<uint4*>(dst),
                                                            static_cast<const uint4*>(src), n16);
  return hipGetLastError();
}

// Packed batch -> disjoint union: the graph of edge e is found by binary
// search over edge_off (G + 1 entries). With src null only dst is mapped (the
// column array of a packed CSR, whose rows already sit at global positions).
__global__ __launch_bounds__(256) void k_batch_relabel(int32_t G, const int64_t* __restrict__ node_off,
                                                       const int64_t* __restrict__ edge_off,
                                                       const int32_t* __restrict__ src,
                                                       const int32_t* __restrict__ dst, int64_t m_raw,
                                                       int32_t* __restrict__ gsrc, int32_t* __restrict__ gdst,
                                                       int32_t* __restrict__ err) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  bool bad = false;
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < m_raw; e += stride) {
    int32_t lo = 0, hi = G - 1;  // last g with edge_off[g] <= e
    while (lo < hi) {
      const int32_t mid = (lo + hi + 1) >> 1;
      if (edge_off[mid] <= e) lo = mid; else hi = mid - 1;
    }
    const int64_t base = node_off[lo];
    const int64_t ng = node_off[lo + 1] - base;
    const int32_t u = src ? src[e] : 0, v = dst[e];
    if (u < 0 || v < 0 || u >= ng || v >= ng) {
      bad = true;
      if (src) gsrc[e] = -1;  // out of range in the union too: its build refuses the batch
      gdst[e] = src ? -1 : (int32_t)base;  // keeps the CSR well formed; refused by err
      continue;
    }
    if (src) gsrc[e] = (int32_t)(base + u);
    gdst[e] = (int32_t)(base + v);
  }
  if (err && __ballot(bad) && lane_id() == 0) atomicOr(err, 1);
}

hipError_t launch_batch_relabel(int32_t num_graphs, const int64_t* node_off, const int64_t* edge_off,
                                const int32_t* src, const int32_t* dst, int64_t m_raw, int32_t* gsrc,
                                int32_t* gdst, int32_t* err, hipStream_t s) {
  if (m_raw == 0) return hipSuccess;
  k_batch_relabel<<<grid_for(m_raw, 256 * 8, 1u << 16), 256, 0, s>>>(num_graphs, node_off, edge_off, src, dst,
                                                                     m_raw, gsrc, gdst, err);
  return hipGetLastError();
}

}  // namespace tricc
