// Edge-existence tests over the simple graph's sorted rows (IsEdge, among
// the graph methods of Section 4). Section 5.1 tests an edge by a search in
// a node's sorted neighbour vector, O(log deg_max) in its complexity table;
// here each lane takes one query and searches the shorter of the two rows,
// so the cost is O(log min(d(u), d(v))) dependent loads.
#include "device_common.h"
#include "kernels.h"

namespace tricc {

namespace {

// True when key is in adj[lo, hi) (ascending, unique): halving, id by id.
__device__ __forceinline__ bool row_has_short(const int32_t* __restrict__ adj, uint32_t lo, uint32_t hi, int32_t key) {
  while (lo < hi) {
    const uint32_t mid = lo + ((hi - lo) >> 1);
    const int32_t x = adj[mid];
    if (x == key) return true;
    if (x < key) lo = mid + 1;
    else hi = mid;
  }
  return false;
}

// The same (lo < hi) by aligned blocks of W ids, each read by W / 4 independent loads and
// settled whole: key is in it, between its ids, or to one side. The first block is
// the one where key would be if the row's ids were spread as the graph's degrees
// are: share, the part of all rows' entries that lie before key's own row, which
// the key's record holds. (Spread evenly over the ids, the guess failed where low
// ids have high degrees: 3M tests on an R-MAT graph of 65k nodes with its ids as
// made 82 us, so 63, by halving 66; 4M nodes 184, so 125, by halving 190.) From
// there the steps to the key's side double until it is passed, then the bracket
// is halved, so a row of clustered ids costs at most about twice the blocks of a
// halving from the start. Blocks at the row's ends hold ids of other rows (the
// array is padded to whole blocks); only [lo, hi) counts. Bound by misses of the
// random reads (halving id by id: 4.3 per test on 4M nodes and 67M pairs, two of
// them the records).
template <int W>
__device__ __forceinline__ bool row_has(const int32_t* __restrict__ adj, uint32_t lo, uint32_t hi, int32_t key,
                                        float share) {
  constexpr uint32_t LG = W == 16 ? 4 : 3, ALL = (1u << W) - 1u;
  static_assert(W == 8 || W == 16, "whole 32- or 64-byte blocks");
  const int4* blocks = reinterpret_cast<const int4*>(adj);
  uint32_t blo = lo >> LG, bhi = (hi - 1) >> LG;
  uint32_t g = min(bhi, blo + (uint32_t)(share * (float)(bhi - blo + 1)));
  uint32_t step = 1;
  int side = 0;  // of the last step; 2 once the key's side has changed
  while (true) {
    int4 x[W / 4];
#pragma unroll
    for (int k = 0; k < W / 4; ++k) x[k] = blocks[(size_t)g * (W / 4) + k];
    uint32_t hit = 0;
#pragma unroll
    for (int k = 0; k < W / 4; ++k) {
      const int32_t v[4] = {x[k].x, x[k].y, x[k].z, x[k].w};
#pragma unroll
      for (int j = 0; j < 4; ++j) hit |= v[j] == key ? 1u << (4 * k + j) : 0u;
    }
    if (hit) {
      const uint32_t base = g << LG;
      uint32_t in = ALL;  // this row's ids of the block
      if (base < lo) in &= ALL << (lo - base);
      if (hi - base < (uint32_t)W) in &= ALL >> (W - (hi - base));
      if (hit & in) return true;
    }
    int d;
    if (g > blo && x[0].x > key) {  // a block that is not the row's first begins with its ids
      bhi = g - 1;
      d = -1;
    } else if (g < bhi && x[W / 4 - 1].w < key) {  // one that is not its last ends with them
      blo = g + 1;
      d = 1;
    } else {
      return false;
    }
    if (side == 0) side = d;
    else if (side != d) side = 2;
    if (side == 2) {
      g = blo + ((bhi - blo) >> 1);
    } else {
      g = d < 0 ? (bhi - blo + 1 > step ? bhi + 1 - step : blo) : (bhi - blo + 1 > step ? blo + step - 1 : bhi);
      step <<= 1;
    }
  }
}

constexpr int kQueryNT = 256;

// rec[v] = (row start of v as uint32, d(v)): one 8-byte load gives both,
// so a query fetches its two records in one round trip.
// One query per thread (grid-stride): out[i] = 1 if {u[i], v[i]} is an edge,
// 0 if not (u == v included), kEdgeQueryBadId if an id is outside [0, n).
// W: ids per block of the row search, 0 for the halving. A wavefront whose rows are
// all short goes by halving in any case: whole blocks of them are mostly other rows'
// ids. 3M tests, half edges, us by blocks / with this: 2M nodes joined to one hub 156 /
// 124, by preferential attachment 4M nodes with one edge each 206 / 165 and 1M
// with 16 158 / 142, uniform 8M nodes and 40M pairs 235 / 187, R-MAT of 4M nodes and
// 64M pairs 160 / 152 (rows up to 16 and 32 halved: 168, 142, 233, 152 and 169, 142,
// 242, 152; all by halving 123, 169, 234, 241, 263).
constexpr int32_t kShortRow = 8;
template <int W>
__global__ __launch_bounds__(kQueryNT) void k_has_edges(int64_t q, const int32_t* __restrict__ qu,
                                                        const int32_t* __restrict__ qv, int32_t n,
                                                        const int2* __restrict__ rec,
                                                        const int64_t* __restrict__ entries,
                                                        const int32_t* __restrict__ adj,
                                                        uint8_t* __restrict__ out) {
  const int64_t stride = (int64_t)gridDim.x * kQueryNT;
  const float inv = 1.0f / (float)max(*entries, (int64_t)1);
  for (int64_t i = (int64_t)blockIdx.x * kQueryNT + threadIdx.x; i < q; i += stride) {
    const int32_t u = qu[i], v = qv[i];
    uint8_t r = 0;
    if ((uint32_t)u >= (uint32_t)n || (uint32_t)v >= (uint32_t)n) {
      r = kEdgeQueryBadId;
    } else if (u != v) {
      const int2 ru = rec[u], rv = rec[v];
      const bool su = ru.y <= rv.y;  // search the shorter row
      const int2 ra = su ? ru : rv;
      const uint32_t lo = (uint32_t)ra.x;
      const uint32_t hi = lo + (uint32_t)ra.y;
      const int32_t key = su ? v : u;
      if constexpr (W == 0) {
        r = row_has_short(adj, lo, hi, key) ? 1 : 0;
      } else {
        const float share = (float)(uint32_t)(su ? rv.x : ru.x) * inv;  // of all rows' entries, before key's row
        if (!__ballot(ra.y > kShortRow)) r = row_has_short(adj, lo, hi, key) ? 1 : 0;
        else r = ra.y > 0 && row_has<W>(adj, lo, hi, key, share) ? 1 : 0;
      }
    }
    out[i] = r;
  }
}

}  // namespace

// m edges in rows of 8m bytes: blocks of 16 ids (what a miss fetches) once the
// rows are well past the L2s of 4 MB, blocks of 8 below. 3M tests of which half
// are edges, us with halving / 8 / 16: R-MAT of 4M nodes and 32M pairs 232 / 149
// / 147 (ids as made 220 / 137 / 134), of 262k nodes and 2M pairs 113 / 70 / 72
// (100 / 71 / 73); uniform 1M nodes and 15M pairs 266 / 149 / 147, 200k and 2.4M
// 155 / 83 / 85, 50k and 150k 68 / 57 / 59, 400k and 800k 98 / 97 / 97, 4M and 8M
// 191 / 189 / 188; a grid of 2,048 x 2,048 nodes 186 with each. Random pairs
// alone, R-MAT of 65k nodes and 524k pairs 52 / 49 / 50.
// Up to kQueryFew tests go by halving: a call ends with its slowest lane, whose
// steps from a guess that failed and back are more, and each longer, than a
// halving's through ids that its first loads brought. us with halving / blocks,
// of a call alone, R-MAT of 65k nodes and 1M pairs: 1,000 tests 18.7 / 20.2,
// 65,000 19.9 / 22.3, 262,144 24.7 / 24.9, 400,000 29.8 / 27.8; 500k nodes joined
// to 20 hubs: 65,000 tests 20.6 / 28.6, 262,144 32 / 36, 400,000 45 / 42; uniform
// 1M nodes and 16M pairs: 65,000 tests 20 / 20, 180,000 28.3 / 26.8, 262,144 35.5
// / 30.1. Not where an eighth of all ordered pairs of ids are edges: nearly every
// guess is right then (2,500 nodes all joined: 65,000 tests 22.5 / 19.1).
constexpr int64_t kQueryFew = 3 << 16;

hipError_t launch_has_edges(int64_t q, const int32_t* qu, const int32_t* qv, int32_t n, int64_t m, const int32_t* rec,
                            const int64_t* entries, const int32_t* adj, uint8_t* out, hipStream_t s) {
  if (q <= 0) return hipSuccess;
  int64_t blocks = (q + kQueryNT - 1) / kQueryNT;
  if (blocks > (int64_t(1) << 20)) blocks = int64_t(1) << 20;
  const int2* r = reinterpret_cast<const int2*>(rec);
  const bool dense = 8 * m >= (int64_t)n * n;
  if (q <= kQueryFew && !dense)
    k_has_edges<0><<<(unsigned)blocks, kQueryNT, 0, s>>>(q, qu, qv, n, r, entries, adj, out);
  else if (8 * m <= (int64_t(20) << 20))
    k_has_edges<8><<<(unsigned)blocks, kQueryNT, 0, s>>>(q, qu, qv, n, r, entries, adj, out);
  else
    k_has_edges<16><<<(unsigned)blocks, kQueryNT, 0, s>>>(q, qu, qv, n, r, entries, adj, out);
  return hipGetLastError();
}

}  // namespace tricc
