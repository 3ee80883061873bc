// Edge-existence tests over the simple graph's sorted rows (IsEdge, among
// the graph methods of Section 4). Section 5.1 tests an edge by a search in
// a node's sorted neighbour vector, O(log deg_max) in its complexity table;
// here each lane takes one query and searches the shorter of the two rows,
// so the cost is O(log min(d(u), d(v))) dependent loads.
#include "device_common.h"
#include "kernels.h"

namespace tricc {

namespace {

// True when key is in adj[lo, hi) (ascending, unique, lo < hi; ids in [0, n),
// inv_n = 1 / n). The row is searched by aligned blocks of 16 ids (64 bytes, what
// a miss fetches), each read by four independent loads and settled whole: key is
// in it, between its ids, or to one side. The first block is the one that would
// hold key if the row's ids were spread evenly; from there the steps to the
// key's side double until it is passed, then the bracket is halved, so a row of
// clustered ids costs at most about twice the blocks of a halving from the
// start. Blocks at the row's ends hold ids of other rows (the array is padded to
// whole blocks); only [lo, hi) counts.
// Bound by misses of the random reads (a halving id by id: 4.3 per test on 4M
// nodes and 67M pairs, two of them the records). 4M tests, half of them edges:
// 325 -> 202 us there with relabelled ids, 178 -> 116 us on 262k nodes and 4M
// pairs; ids left as R-MAT makes them, all edges: 454 -> 397 us on 4M nodes; on
// 262k nodes, whose rows stay in the L2, 165 -> 182 us. Blocks of 8 ids: 207 us
// in the first case, 447 us in the third.
__device__ __forceinline__ bool row_has(const int32_t* __restrict__ adj, uint32_t lo, uint32_t hi, int32_t key,
                                        float inv_n) {
  constexpr uint32_t W = 16, LG = 4, ALL = (1u << W) - 1u;  // ids per block
  const int4* blocks = reinterpret_cast<const int4*>(adj);
  uint32_t blo = lo >> LG, bhi = (hi - 1) >> LG;
  uint32_t g = min(bhi, blo + (uint32_t)((float)key * inv_n * (float)(bhi - blo + 1)));
  uint32_t step = 1;
  int side = 0;  // of the last step; 2 once the key's side has changed
  while (true) {
    const uint32_t base = g << LG;
    uint32_t in = ALL;  // this row's ids of the block
    if (base < lo) in &= ALL << (lo - base);
    if (hi - base < W) in &= ALL >> (W - (hi - base));
    int4 x[W / 4];
#pragma unroll
    for (int k = 0; k < (int)W / 4; ++k) x[k] = blocks[(size_t)g * (W / 4) + k];
    // lane bits of the ids that pass a test
    auto ids = [&](auto test) {
      uint32_t m = 0;
#pragma unroll
      for (int k = 0; k < (int)W / 4; ++k) {
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
      r = ra.y > 0 && row_has(adj, lo, lo + (uint32_t)ra.y, su ? v : u, inv_n) ? 1 : 0;
    }
    out[i] = r;
  }
}

}  // namespace

hipError_t launch_has_edges(int64_t q, const int32_t* qu, const int32_t* qv, int32_t n, const int32_t* rec,
                            const int32_t* adj, uint8_t* out, hipStream_t s) {
  if (q <= 0) return hipSuccess;
  int64_t blocks = (q + kQueryNT - 1) / kQueryNT;
  if (blocks > (int64_t(1) << 20)) blocks = int64_t(1) << 20;
  k_has_edges<<<(unsigned)blocks, kQueryNT, 0, s>>>(q, qu, qv, n, reinterpret_cast<const int2*>(rec), adj, out);
  return hipGetLastError();
}

}  // namespace tricc
