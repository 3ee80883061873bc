// Induced-subgraph extraction for query batches (subgraph extraction is one
// of the graph manipulation methods in the paper's table of methods,
// Section 4; node ids keep their identity, Section 3.1).
//
// A batch holds Q queries; query q is the node set S_q = nodes[qoff[q] ..
// qoff[q+1]) of the resident graph (distinct ids), and its induced subgraph
// G[S_q] gets local ids = positions in S_q. Every undirected edge {v,w} of
// the resident graph with v, w in S_q and v < w (by id) is emitted once as
// the pair (pos(v), pos(w)).
//
// Membership is a per-query open-addressing table in global memory (2^k >=
// max(4, 2|S_q|) slots): buckets of four node ids, filled in order, so that one
// 16-byte read settles most look-ups, and the slots' positions in an array
// apart, read for hits only. Rows of the resident CSR are scanned in chunks of
// kServeChunk neighbours, one wavefront per few (item, chunk), so hub rows
// spread over many waves. Exact counts per chunk, a prefix sum, then an ordered
// fill give a deterministic pair list.
#include <algorithm>

#include "device_common.h"
#include "kernels.h"

namespace tricc {

constexpr int32_t kServeChunk = 2048;

namespace {

// query of flat item i: last q with qoff[q] <= i
__device__ __forceinline__ int32_t find_query(const int64_t* qoff, int32_t Q, int64_t i) {
  int32_t lo = 0, hi = Q - 1;
  while (lo < hi) {
    const int32_t mid = (lo + hi + 1) >> 1;
    if (qoff[mid] <= i) lo = mid; else hi = mid - 1;
  }
  return lo;
}

// Home bucket of x among nb buckets.
__device__ __forceinline__ uint32_t qbucket(int32_t x, uint32_t nb) {
  return __umulhi((uint32_t)x * 0x9E3779B1u, nb);
}

// Slot of x in a bucket read as q (0 .. 3), or -1.
__device__ __forceinline__ int bucket_slot(int4 q, int32_t x) {
  return q.x == x ? 0 : q.y == x ? 1 : q.z == x ? 2 : q.w == x ? 3 : -1;
}

}  // namespace

// Clears the ids of every query table (total slots, a multiple of 4).
__global__ __launch_bounds__(256) void k_serve_clear(int4* __restrict__ keys, int64_t total4) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < total4; i += stride)
    keys[i] = make_int4(-1, -1, -1, -1);
}

// Inserts every (node, position) and writes the number of row chunks and
// the query of each item; flags node ids outside [0, n) or repeated inside
// one query.
__global__ __launch_bounds__(256) void k_serve_insert(int32_t Q, const int64_t* __restrict__ qoff,
                                                      const int32_t* __restrict__ nodes,
                                                      const int64_t* __restrict__ toff, int32_t* __restrict__ keys,
                                                      int32_t* __restrict__ places, int32_t n,
                                                      const int32_t* __restrict__ deg,
                                                      int32_t* __restrict__ nchunks, int32_t* __restrict__ qidx,
                                                      int32_t* __restrict__ err) {
  const int64_t N = qoff[Q];
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < N; i += stride) {
    const int32_t q = find_query(qoff, Q, i);
    qidx[i] = q;
    const int32_t v = nodes[i];
    if ((uint32_t)v >= (uint32_t)n) {
      atomicOr(err, 1);
      nchunks[i] = 0;
      continue;
    }
    const int64_t t = toff[q];
    const uint32_t nb = (uint32_t)(toff[q + 1] - t) / 4;
    uint32_t b = qbucket(v, nb);
    int k = 0;
    while (true) {
      const int64_t at = t + 4 * (int64_t)b + k;
      const int prev = atomicCAS(&keys[at], -1, v);
      if (prev == -1) { places[at] = (int32_t)(i - qoff[q]); break; }
      if (prev == v) { atomicOr(err, 2); break; }
      if (++k == 4) {
        k = 0;
        b = b + 1 == nb ? 0 : b + 1;
      }
    }
    nchunks[i] = (deg[v] + kServeChunk - 1) / kServeChunk;
  }
}

// Item of every row chunk (the chunk prefix coff inverted), so that a
// chunk finds its item with one load instead of a search.
__global__ __launch_bounds__(256) void k_serve_items(int64_t N, const int64_t* __restrict__ coff,
                                                     int32_t* __restrict__ item) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < N; i += stride)
    for (int64_t c = coff[i]; c < coff[i + 1]; ++c) item[c] = (int32_t)i;
}

// `per` (item, chunk)s per wavefront: pass 0 counts the emitted pairs of each
// into cnt[c]; pass 1 writes them, in row order, at pos[c]. A lane holds what one
// chunk needs (its row, query, table: four dependent loads), and four loads of 64
// row ids, then their home buckets, are in flight together: the kernel waits for
// memory, and with a chunk at a time, 64 ids a step and a table probed slot by
// slot the steps of a row followed each other. 100 queries of 16 to 100,000 nodes
// of an R-MAT graph of 2^20 (363M row ids, 53M pairs): 22.7 -> 21.3 ms, both
// passes together 5.2 ms of it.
constexpr int kServeUnroll = 4;

template <int PASS>
__global__ __launch_bounds__(256) void k_serve_pairs(int32_t per, int32_t Q, const int64_t* __restrict__ qoff,
                                                     const int32_t* __restrict__ nodes,
                                                     const int64_t* __restrict__ coff,  // chunk prefix per item
                                                     const int32_t* __restrict__ item,  // item of each chunk
                                                     const int32_t* __restrict__ qidx,  // query of each item
                                                     const int64_t* __restrict__ toff,
                                                     const int32_t* __restrict__ keys,
                                                     const int32_t* __restrict__ places,
                                                     const int64_t* __restrict__ off,
                                                     const int32_t* __restrict__ deg,
                                                     const int32_t* __restrict__ adj,
                                                     int32_t* __restrict__ cnt, const int64_t* __restrict__ pos,
                                                     int32_t* __restrict__ psrc, int32_t* __restrict__ pdst) {
  constexpr int U = kServeUnroll;
  const int64_t C = coff[qoff[Q]];
  const int64_t step = (int64_t)gridDim.x * (blockDim.x / kWave) * per;
  const int l = lane_id();
  for (int64_t c0 = ((int64_t)blockIdx.x * (blockDim.x / kWave) + threadIdx.x / kWave) * per; c0 < C; c0 += step) {
    const int32_t here = (int32_t)min((int64_t)per, C - c0);
    int32_t lv = 0, lp = 0, ln = 0;
    uint32_t lnb = 0;
    int64_t lt = 0, lb = 0, lat = 0;
    if (l < here) {
      const int64_t c = c0 + l;
      const int64_t i = item[c];
      const int32_t q = qidx[i];
      lv = nodes[i];
      lp = (int32_t)(i - qoff[q]);
      lt = toff[q];
      lnb = (uint32_t)(toff[q + 1] - lt) / 4;
      const int32_t b0 = (int32_t)(c - coff[i]) * kServeChunk;
      ln = min(deg[lv] - b0, kServeChunk);
      lb = off[lv] + b0;
      if (PASS == 1) lat = pos[c];
    }
    int32_t mine = 0;  // pairs of this lane's chunk
    for (int32_t k = 0; k < here; ++k) {
      const int32_t v = __builtin_amdgcn_readlane(lv, k);
      const int32_t pv = __builtin_amdgcn_readlane(lp, k);
      const int32_t n = __builtin_amdgcn_readlane(ln, k);
      const uint32_t nb = (uint32_t)__builtin_amdgcn_readlane((int)lnb, k);
      const int32_t* row = adj + __shfl(lb, k, kWave);
      const int64_t t = __shfl(lt, k, kWave);
      const int64_t base = PASS == 1 ? __shfl(lat, k, kWave) : 0;
      const int4* buckets = reinterpret_cast<const int4*>(keys + t);
      int32_t found = 0;
      for (int32_t p = 0; p < n; p += U * kWave) {
        int32_t x[U];
        uint32_t b[U];
        int4 e[U];
#pragma unroll
        for (int r = 0; r < U; ++r) x[r] = p + r * kWave + l < n ? row[p + r * kWave + l] : -1;
#pragma unroll
        for (int r = 0; r < U; ++r) {
          b[r] = qbucket(x[r], nb);
          e[r] = make_int4(-1, -1, -1, -1);
          if (x[r] > v) e[r] = buckets[b[r]];
        }
#pragma unroll
        for (int r = 0; r < U; ++r) {
          if (p + r * kWave >= n) break;
          const bool want = x[r] > v;
          int s = want ? bucket_slot(e[r], x[r]) : -1;
          while (want && s < 0 && e[r].w >= 0) {  // a full bucket: the next one
            b[r] = b[r] + 1 == nb ? 0 : b[r] + 1;
            e[r] = buckets[b[r]];
            s = bucket_slot(e[r], x[r]);
          }
          const uint64_t m = __ballot(s >= 0);
          if (PASS == 1 && s >= 0) {
            const int64_t at = base + found + mask_below(m);
            psrc[at] = pv;
            pdst[at] = places[t + 4 * (int64_t)b[r] + s];
          }
          found += (int32_t)__popcll(m);
        }
      }
      if (l == k) mine = found;
    }
    if (PASS == 0 && l < here) cnt[c0 + l] = mine;
  }
}

// pair offsets of each query: pairs of query q start at pos[coff[qoff[q]]]
__global__ void k_serve_query_pairs(int32_t Q, const int64_t* __restrict__ qoff, const int64_t* __restrict__ coff,
                                    const int64_t* __restrict__ pos, int64_t* __restrict__ qpairs) {
  const int32_t q = blockIdx.x * blockDim.x + threadIdx.x;
  if (q <= Q) qpairs[q] = pos[coff[qoff[q]]];
}

// The tables: `total` slots (a multiple of 4), their ids first, then their places.
hipError_t launch_serve_clear(int32_t* tab, int64_t total, hipStream_t s) {
  if (total == 0) return hipSuccess;
  k_serve_clear<<<grid_for(total / 4, 256, 1u << 14), 256, 0, s>>>(reinterpret_cast<int4*>(tab), total / 4);
  return hipGetLastError();
}

hipError_t launch_serve_insert(int32_t Q, const int64_t* qoff, const int32_t* nodes, int64_t N, const int64_t* toff,
                               int32_t* tab, int64_t total, int32_t n, const int32_t* deg, int32_t* nchunks,
                               int32_t* qidx, int32_t* err, hipStream_t s) {
  if (N == 0) return hipSuccess;
  k_serve_insert<<<grid_for(N, 256, 1u << 14), 256, 0, s>>>(Q, qoff, nodes, toff, tab, tab + total, n, deg, nchunks,
                                                            qidx, err);
  return hipGetLastError();
}

hipError_t launch_serve_items(int64_t N, const int64_t* coff, int32_t* item, hipStream_t s) {
  if (N == 0) return hipSuccess;
  k_serve_items<<<grid_for(N, 256, 1u << 14), 256, 0, s>>>(N, coff, item);
  return hipGetLastError();
}

// A wavefront takes up to 16 chunks, fewer where the chip's 8,192 would not get
// two turns each.
hipError_t launch_serve_pairs(int pass, int32_t Q, const int64_t* qoff, const int32_t* nodes, const int64_t* coff,
                              int64_t C, const int32_t* item, const int32_t* qidx, const int64_t* toff,
                              const int32_t* tab, int64_t total, const int64_t* off, const int32_t* deg,
                              const int32_t* adj, int32_t* cnt, const int64_t* pos, int32_t* psrc, int32_t* pdst,
                              hipStream_t s) {
  if (C == 0) return hipSuccess;
  const int32_t per = (int32_t)std::clamp<int64_t>(C / 16384, 1, 16);
  const unsigned grid = grid_for((C + per - 1) / per, 256 / kWave, 1u << 14);
  if (pass == 0)
    k_serve_pairs<0><<<grid, 256, 0, s>>>(per, Q, qoff, nodes, coff, item, qidx, toff, tab, tab + total, off, deg, adj,
                                          cnt, pos, psrc, pdst);
  else
    k_serve_pairs<1><<<grid, 256, 0, s>>>(per, Q, qoff, nodes, coff, item, qidx, toff, tab, tab + total, off, deg, adj,
                                          cnt, pos, psrc, pdst);
  return hipGetLastError();
}

hipError_t launch_serve_query_pairs(int32_t Q, const int64_t* qoff, const int64_t* coff, const int64_t* pos,
                                    int64_t* qpairs, hipStream_t s) {
  k_serve_query_pairs<<<(Q + 1 + 255) / 256, 256, 0, s>>>(Q, qoff, coff, pos, qpairs);
  return hipGetLastError();
}

}  // namespace tricc
