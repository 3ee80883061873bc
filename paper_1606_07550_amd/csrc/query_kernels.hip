// Edge-existence tests over the simple graph's sorted rows (IsEdge, among
// the graph methods of Section 4). Section 5.1 tests an edge by a search in
// a node's sorted neighbour vector, O(log deg_max) in its complexity table;
// here each lane takes one query and searches the shorter of the two rows,
// so the cost is O(log min(d(u), d(v))) dependent loads.
#include "device_common.h"
#include "kernels.h"

namespace tricc {

namespace {

// True when key is in adj[lo, hi) (ascending, unique, lo < hi): halving, id by
// id. Few instructions: for graphs of short rows that the L2 holds.
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

// The same (ids in [0, n), inv_n = 1 / n) by aligned blocks of W ids, each read
// by W / 4 independent loads and settled whole: key is in it, between its ids, or
// to one side. The first block is the one that would hold key if the row's ids
// were spread evenly; from there the steps to the key's side double until it is
// passed, then the bracket is halved, so a row of clustered ids costs at most
// about twice the blocks of a halving from the start. Blocks at the row's ends
// hold ids of other rows (the array is padded to whole blocks); only [lo, hi)
// counts. Bound by misses of the random reads (halving id by id: 4.3 per test on
// 4M nodes and 67M pairs, two of them the records).
template <int W>
__device__ __forceinline__ bool row_has(const int32_t* __restrict__ adj, uint32_t lo, uint32_t hi, int32_t key,
                                        float inv_n) {
  constexpr uint32_t LG = W == 16 ? 4 : 3, ALL = (1u << W) - 1u;
  static_assert(W == 8 || W == 16, "whole 32- or 64-byte blocks");
  const int4* blocks = reinterpret_cast<const int4*>(adj);
  uint32_t blo = lo >> LG, bhi = (hi - 1) >> LG;
  uint32_t g = min(bhi, blo + (uint32_t)((float)key * inv_n * (float)(bhi - blo + 1)));
  uint32_t step = 1;
  int side = 0;  // of the last step; 2 once the key's side has changed
  while (true) {
    const uint32_t base = g << LG;
    uint32_t in = ALL;  // this row's ids of the block
    if (base < lo) in &= ALL << (lo - base);
    if (hi - base < (uint32_t)W) in &= ALL >> (W - (hi - base));
    int4 x[W / 4];
#pragma unroll
    for (int k = 0; k < W / 4; ++k) x[k] = blocks[(size_t)g * (W / 4) + k];
    // lane bits of the ids that pass a test
    auto ids = [&](auto test) {
      uint32_t m = 0;
#pragma unroll
      for (int k = 0; k < W / 4; ++k) {
        const int32_t v[4] = {x[k].x, x[k].y, x[k].z, x[k].w};
#pragma unroll
        for (int j = 0; j < 4; ++j) m |= test(v[j]) ? 1u << (4 * k + j) : 0u;
      }
      return m & in;
    };
    if (ids([&](int32_t v) { return v == key; })) return true;
    if (blo == bhi) return false;
    const uint32_t lt = ids([&](int32_t v) { return v < key; });
    int d;
    if (lt == 0u) {
      if (g == blo) return false;
      bhi = g - 1;
      d = -1;
    } else if (lt == in) {
      if (g == bhi) return false;
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
// W: ids per block of the row search, 0 for the halving.
template <int W>
__global__ __launch_bounds__(kQueryNT) void k_has_edges(int64_t q, const int32_t* __restrict__ qu,
                                                        const int32_t* __restrict__ qv, int32_t n,
                                                        const int2* __restrict__ rec,
                                                        const int32_t* __restrict__ adj,
                                                        uint8_t* __restrict__ out) {
  const int64_t stride = (int64_t)gridDim.x * kQueryNT;
  const float inv_n = 1.0f / (float)n;
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
      if constexpr (W == 0) r = row_has_short(adj, lo, hi, key) ? 1 : 0;
      else r = ra.y > 0 && row_has<W>(adj, lo, hi, key, inv_n) ? 1 : 0;
    }
    out[i] = r;
  }
}

}  // namespace

// m edges in rows of 8m bytes. Blocks of 16 ids (what a miss fetches) once the
// rows are well past the L2s of 4 MB, blocks of 8 below, and the halving for
// short rows (mean degree under 10) that an L2 holds a good part of. Tests of
// which half are edges, ids relabelled, us with halving / 8 / 16: 4M tests on 4M
// nodes, 67M pairs 325 / 207 / 202; 20M on 1M nodes, 15M pairs 1190 / 697 / 697
// (uniform 1667 / 1062 / 1005); 3M on 200k nodes, 2.4M pairs 108 / 104 / 112 (uniform
// 139 / 84 / 88) and 1M pairs 80 / 88 / 94 (82 / 79 / 83); on 50k nodes, 150k
// pairs 55 / 61 / 63. Ids left as R-MAT makes them, all tests edges: 4M nodes
// 454 / 447 / 397, 262k nodes and 2M pairs 165 / 175 / 182.
hipError_t launch_has_edges(int64_t q, const int32_t* qu, const int32_t* qv, int32_t n, int64_t m, const int32_t* rec,
                            const int32_t* adj, uint8_t* out, hipStream_t s) {
  if (q <= 0) return hipSuccess;
  int64_t blocks = (q + kQueryNT - 1) / kQueryNT;
  if (blocks > (int64_t(1) << 20)) blocks = int64_t(1) << 20;
  const int2* r = reinterpret_cast<const int2*>(rec);
  if (m < 5 * (int64_t)n && 8 * m <= (int64_t(12) << 20))
    k_has_edges<0><<<(unsigned)blocks, kQueryNT, 0, s>>>(q, qu, qv, n, r, adj, out);
  else if (8 * m <= (int64_t(20) << 20))
    k_has_edges<8><<<(unsigned)blocks, kQueryNT, 0, s>>>(q, qu, qv, n, r, adj, out);
  else
    k_has_edges<16><<<(unsigned)blocks, kQueryNT, 0, s>>>(q, qu, qv, n, r, adj, out);
  return hipGetLastError();
}

}  // namespace tricc
