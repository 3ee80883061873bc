// Core numbers by parallel level-synchronous peeling (k-core analysis,
// among the analytics methods of Section 4; Section 5 names the
// Batagelj-Zaversnik decomposition, which removes nodes in order of their
// current degree). Here every node whose current degree is at most k is
// removed together (core number k), and the removals lower their
// neighbours' current degrees with atomics; a neighbour that falls to k
// joins the next frontier of the same level. Levels with no node are
// skipped: a scan that finds no frontier reports the smallest current
// degree left.
//
// Scans of every node left are made once per window of levels [k, U]: the
// scan at k also lists the nodes left with current degree <= U (the near
// list), and the peels append every node whose current degree falls from
// U + 1 to U. Every node left with current degree <= U is thus on the near
// list, so the levels up to U scan that list alone.
//
// The whole peeling is a state machine on the device: one kernel per step (a
// scan or one round of a level), every block of which works out the step from
// the state and the counters that the step before left, so the host only
// launches steps ahead and reads the state now and then. The steps are short
// (a frontier of tens to thousands of nodes), so the decomposition is bound by
// their number and latency: R-MAT 20 takes 888 steps of about 5 us and the gap
// to the next, 7.7 ms in all, against 32.4 ms with a read-back after each scan
// and every fourth round and rows walked by one wavefront each.
//
// With `order` given, each node also records the round in which it was
// removed (rounds count every frontier, across levels). A node removed in
// round r had current degree <= k then, counting exactly its neighbours
// removed in round r or later, so orienting every edge towards the later
// (round, id) gives out-degrees at most the core number: the degeneracy
// ordering.
#include <algorithm>
#include <cstring>

#include "device_common.h"
#include "kernels.h"

namespace tricc {

namespace {

constexpr int kCoreNT = 256;
constexpr int kPeelG = 8;  // lanes per node in the peel of large frontiers
// Levels per window of the peeling: a scan of every node left opens a window
// [k, k + kCoreWindow], whose levels then scan the near list only.
constexpr int32_t kCoreWindow = 32;
// A level's rounds start at multiples of this many in the order values: part of
// the results, which stay what they are however the rounds are launched.
constexpr int32_t kOrderRounds = 4;
constexpr int32_t kNoDegree = 0x7fffffff;

enum : int32_t { kCoreScan = 0, kCorePeel = 1, kCoreDone = 2 };

// The step that a launch is to do. Buffers: the frontier is F[fb] (nf nodes),
// the near list near[xb] (nx nodes), the candidates of a full scan all ids or
// the list A[ab] (ncand either way).
struct CoreState {
  int32_t phase, k, U, nf, fb, nx, xb, listed, ab, ncand, left, round, rounds, maxc, full, listing;
};
// Counters of a step: frontier found (scan) or next frontier (peel),
// survivors listed, near nodes added, smallest degree above k seen.
struct CoreCount {
  int32_t f, survivors, near, least;
};

// What follows the levels done so far: a scan for level k, or the end.
__host__ __device__ __forceinline__ void core_plan(CoreState& s, int32_t n, int32_t k_stop) {
  if (!(s.left > 0 && (k_stop < 0 || s.k < k_stop))) {
    s.phase = kCoreDone;
    return;
  }
  s.phase = kCoreScan;
  s.full = s.k > s.U || s.nx == 0;
  s.listing = 0;
  if (s.full) {
    s.U = s.k + kCoreWindow;
    if (k_stop >= 0 && s.U > k_stop - 1) s.U = k_stop - 1;  // no level at or above k_stop is peeled
    // full scans list the survivors for the next one once at most a quarter
    // of the nodes are left
    s.listing = s.listed || s.left <= n / 4;
  }
}

// The state after step s, whose counters were c.
__host__ __device__ __forceinline__ void core_next(CoreState& s, const CoreCount& c, int32_t n, int32_t k_stop) {
  if (s.phase == kCoreScan) {
    s.xb ^= 1;
    s.nx = c.near;
    if (s.listing) {
      s.ab ^= 1;
      s.listed = 1;
      s.ncand = c.survivors;
    }
    if (c.f > 0) {
      s.phase = kCorePeel;
      s.nf = c.f;
      s.fb = 0;
      s.rounds = 0;
      return;
    }
    // no node at this level: the smallest current degree seen comes next
    if (c.least != kNoDegree) s.k = c.least;
    else if (s.full) s.left = 0;  // no node left at all
    else s.k = s.U + 1;           // none left in the window: every node left is above U
    core_plan(s, n, k_stop);
  } else if (s.phase == kCorePeel) {
    s.left -= s.nf;
    s.rounds += 1;
    s.nx += c.near;
    s.nf = c.f;
    s.fb ^= 1;
    if (s.nf > 0) return;
    s.round += (s.rounds + kOrderRounds - 1) / kOrderRounds * kOrderRounds;
    s.maxc = s.k;
    s.k += 1;
    core_plan(s, n, k_stop);
  }
}

// Layout of the counter area (64 int32): two states, three counter sets.
__device__ __forceinline__ CoreState* core_state(int32_t* cnt, int i) {
  return reinterpret_cast<CoreState*>(cnt) + (i & 1);
}
__device__ __forceinline__ CoreCount* core_count(int32_t* cnt, int i) {
  return reinterpret_cast<CoreCount*>(cnt + 2 * sizeof(CoreState) / 4) + i % 3;
}
static_assert(2 * sizeof(CoreState) + 3 * sizeof(CoreCount) <= 256, "counter area");

__global__ __launch_bounds__(kCoreNT) void k_core_init(int32_t n, int32_t k_stop, const int32_t* __restrict__ deg,
                                                       int32_t* __restrict__ cur, int32_t* __restrict__ core,
                                                       int32_t* __restrict__ cnt) {
  const int64_t stride = (int64_t)gridDim.x * kCoreNT;
  for (int64_t v = (int64_t)blockIdx.x * kCoreNT + threadIdx.x; v < n; v += stride) {
    cur[v] = deg[v];
    core[v] = -1;
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    CoreState s{};
    s.U = -1;
    s.ncand = n;
    s.left = n;
    core_plan(s, n, k_stop);
    *core_state(cnt, 0) = s;
    *core_count(cnt, 0) = CoreCount{0, 0, 0, kNoDegree};
    *core_count(cnt, 1) = CoreCount{0, 0, 0, kNoDegree};
  }
}

struct CoreArrays {
  const int64_t* off;
  const int32_t* deg;
  const int32_t* adj;
  int32_t* cur;
  int32_t* core;
  int32_t* order;  // may be null
  int32_t* F[2];
  int32_t* A[2];
  int32_t* near[2];
  int32_t* cnt;
};

// Scan for level k: among the candidates, the nodes left whose current degree
// is <= k become the frontier; the others still left are listed (listing) and
// go on the near list up to degree U. A block takes tiles of kScanTile
// candidates and adds each tile's items to the three lists with one atomic per
// list: one counter takes about 100 atomics per microsecond, which held up the
// first levels, whose near lists hold most nodes, when every wavefront issued
// its own (first scan of R-MAT 20: 422 us for 10^6 nodes, the next 32 near
// lists 180 to 10 us each).
constexpr int kScanPer = 8;
constexpr int kScanTile = kCoreNT * kScanPer;

struct ScanLds {
  int32_t count[3], base[3];
};

__device__ __forceinline__ void core_scan(const CoreState& s, const CoreArrays& g, CoreCount* c, ScanLds& lds) {
  const int32_t na = s.full ? s.ncand : s.nx;
  const int32_t* list = s.full ? (s.listed ? g.A[s.ab] : nullptr) : g.near[s.xb];
  int32_t* const q[3] = {g.F[0], g.near[s.xb ^ 1], g.A[s.ab ^ 1]};
  int32_t* const cnt[3] = {&c->f, &c->near, &c->survivors};
  const int lists = s.listing ? 3 : 2;
  const int64_t stride = (int64_t)gridDim.x * kScanTile;
  int32_t mn = kNoDegree;
  for (int64_t b = (int64_t)blockIdx.x * kScanTile; b < na; b += stride) {  // uniform trip count
    if (threadIdx.x < 3) lds.count[threadIdx.x] = 0;
    __syncthreads();
    int32_t v[kScanPer];
    uint32_t on[3] = {0, 0, 0};  // bit r: item r goes on the list
#pragma unroll
    for (int r = 0; r < kScanPer; ++r) {
      const int64_t i = b + r * kCoreNT + threadIdx.x;
      v[r] = i < na ? (list ? list[i] : (int32_t)i) : -1;
    }
#pragma unroll
    for (int r = 0; r < kScanPer; ++r) {
      if (v[r] < 0 || g.core[v[r]] >= 0) continue;
      const int32_t d = g.cur[v[r]];
      if (d <= s.k) {
        g.core[v[r]] = s.k;
        if (g.order) g.order[v[r]] = s.round;
        on[0] |= 1u << r;
      } else {
        mn = min(mn, d);
        if (d <= s.U) on[1] |= 1u << r;
        on[2] |= 1u << r;
      }
    }
    // the wavefront's place in the tile, then the tile's in the list
    int32_t at[3];
    for (int l = 0; l < lists; ++l) {
      int32_t k = 0;
#pragma unroll
      for (int r = 0; r < kScanPer; ++r) k += (int32_t)__popcll(__ballot((on[l] >> r) & 1u));
      int32_t w = 0;
      if (lane_id() == 0 && k) w = atomicAdd(&lds.count[l], k);
      at[l] = __builtin_amdgcn_readfirstlane(w);
    }
    __syncthreads();
    if (threadIdx.x < lists) {
      const int32_t k = lds.count[threadIdx.x];
      if (k) lds.base[threadIdx.x] = atomicAdd(cnt[threadIdx.x], k);
    }
    __syncthreads();
    for (int l = 0; l < lists; ++l) {
      int32_t p = lds.base[l] + at[l];
#pragma unroll
      for (int r = 0; r < kScanPer; ++r) {
        const bool take = (on[l] >> r) & 1u;
        const uint64_t m = __ballot(take);
        if (take) q[l][p + mask_below(m)] = v[r];
        p += (int32_t)__popcll(m);
      }
    }
  }
#pragma unroll
  for (int o = kWave / 2; o > 0; o >>= 1) mn = min(mn, __shfl_xor(mn, o, kWave));
  if (lane_id() == 0 && mn != kNoDegree &&
      mn < __hip_atomic_load(&c->least, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
    atomicMin(&c->least, mn);
}

// Rows up to this length are walked by an 8-lane group of a wavefront that holds
// eight of them; longer ones, and all rows of frontiers of at most kPeelFew
// nodes, by a wavefront each. Full decomposition, ms, short rows up to 16 / 32 /
// 64: a lattice of 128^3 nodes and 26 neighbours 18.8 / 8.2 / 8.1, 10^6 nodes of
// 16 edges by preferential attachment 9.4 / 5.8 / 4.8, R-MAT 24 (64M pairs) 15.6 /
// 15.3 / 15.1; kPeelFew 64 / 128 / 256 / 512: R-MAT 18 4.96 / 4.79 / 4.64 / 4.55.
constexpr int32_t kPeelShort = 64;
constexpr int32_t kPeelFew = 512;
// Steps of a walk issued together: their loads and atomic subtractions are
// in flight at once, since each waits on a round trip to memory.
constexpr int kPeelU = 8;

// kPeelU steps of a walk over row[0, d): the entries j0 + q * W + t, q <
// kPeelU (t = the lane's place among the W walkers): every neighbour left
// loses one from its current degree; the one decrement from k + 1 to k gives
// it core number k and puts it on the next frontier, the one from U + 1 to U
// on the near list. Every lane of the wavefront calls it: all its items of a list
// take one atomic, both lists' in flight together (a step waits for it).
__device__ __forceinline__ void peel_steps(const int32_t* __restrict__ row, int32_t d, int32_t j0, int32_t W,
                                           int32_t t, const CoreState& s, const CoreArrays& g, CoreCount* c) {
  int32_t w[kPeelU];
  bool live[kPeelU];
#pragma unroll
  for (int q = 0; q < kPeelU; ++q) {
    const int32_t j = j0 + q * W + t;
    live[q] = j < d;
    w[q] = live[q] ? row[j] : 0;
  }
#pragma unroll
  for (int q = 0; q < kPeelU; ++q) live[q] = live[q] && g.core[w[q]] < 0;
  int32_t old[kPeelU];
#pragma unroll
  for (int q = 0; q < kPeelU; ++q) old[q] = live[q] ? atomicSub(&g.cur[w[q]], 1) : 0;
  // bit q of take: entry q falls to k; of enter: it falls to U (at the window's
  // last level the frontier is all that enters)
  uint32_t take = 0, enter = 0;
  int32_t nt = 0, ne = 0;
#pragma unroll
  for (int q = 0; q < kPeelU; ++q) {
    take |= live[q] && old[q] == s.k + 1 ? 1u << q : 0u;
    enter |= live[q] && old[q] == s.U + 1 && s.U > s.k ? 1u << q : 0u;
    nt += (int32_t)__popcll(__ballot((take >> q) & 1u));
    ne += (int32_t)__popcll(__ballot((enter >> q) & 1u));
  }
  if (nt + ne == 0) return;
  int32_t at = 0, et = 0;
  if (lane_id() == 0 && nt) at = atomicAdd(&c->f, nt);
  if (lane_id() == 0 && ne) et = atomicAdd(&c->near, ne);
  at = __builtin_amdgcn_readfirstlane(at);
  et = __builtin_amdgcn_readfirstlane(et) + s.nx;
#pragma unroll
  for (int q = 0; q < kPeelU; ++q) {
    const bool t = (take >> q) & 1u, e = (enter >> q) & 1u;
    const uint64_t tm = __ballot(t), em = __ballot(e);
    if (t) {
      g.core[w[q]] = s.k;
      if (g.order) g.order[w[q]] = s.round + s.rounds + 1;
      g.F[s.fb ^ 1][at + mask_below(tm)] = w[q];
    }
    if (e) g.near[s.xb][et + mask_below(em)] = w[q];
    at += (int32_t)__popcll(tm);
    et += (int32_t)__popcll(em);
  }
}

// A frontier node as its walkers need it: row length and start (0 past the end).
struct PeelRow {
  int32_t d;
  int64_t at;
};
__device__ __forceinline__ PeelRow peel_row(int64_t i, int32_t nf, const int32_t* F, const CoreArrays& g) {
  PeelRow r{0, 0};
  if (i < nf) {
    const int32_t v = F[i];
    r.d = g.deg[v];
    r.at = g.off[v];
  }
  return r;
}

// The short rows among 8 frontier nodes (lane l holds that of group l / 8 in r),
// one per 8-lane group of a wavefront.
__device__ __forceinline__ void peel_short(const PeelRow& r, const CoreState& s, const CoreArrays& g, CoreCount* c) {
  const int32_t ds = r.d <= kPeelShort ? r.d : 0;
  int32_t dmax = ds;
#pragma unroll
  for (int o = kWave / 2; o > 0; o >>= 1) dmax = max(dmax, __shfl_xor(dmax, o, kWave));
  for (int32_t j0 = 0; j0 < dmax; j0 += kPeelG * kPeelU)
    peel_steps(g.adj + r.at, ds, j0, kPeelG, threadIdx.x % kPeelG, s, g, c);
}

// One round. Short rows go eight nodes to a wavefront, whose pushes take one
// atomic together: one counter takes about 100 atomics per microsecond, so with
// a wavefront per node rounds of 4,096 nodes of degree 4 took 22 us, and 40 where
// both lists grew (a grid of 2,048 x 2,048 nodes 45 and 79 ms, now 19 and 19).
// Long rows: with many nodes (more than 8 per wavefront) one after the other by
// the wavefront that holds them, else by a wavefront each, or by several blocks
// each when the frontier is smaller than the grid (late levels: tens of nodes
// with rows of thousands of entries, which one wavefront walks 512 at a time).
__device__ __forceinline__ void core_peel(const CoreState& s, const CoreArrays& g, CoreCount* c) {
  constexpr int WPB = kCoreNT / kWave, GPW = kWave / kPeelG;  // wavefronts a block, groups a wavefront
  const int32_t* F = g.F[s.fb];
  const int32_t nf = s.nf;
  const int lane = lane_id(), wv = threadIdx.x / kWave;
  const int32_t blocks = (int32_t)gridDim.x, waves = blocks * WPB;
  if (nf <= GPW * waves) {
    // groups of eight nodes go to the first wavefront of each block first
    const int32_t me = wv * blocks + (int32_t)blockIdx.x;
    const PeelRow mine = peel_row((int64_t)me * GPW + lane / kPeelG, nf, F, g);
    const int32_t shortest = nf <= kPeelFew ? 0 : kPeelShort;  // rows above it are walked one by one
    if (nf <= blocks) {
      const int32_t per = blocks / nf;  // blocks per node
      const int32_t i = (int32_t)blockIdx.x % nf, part = (int32_t)blockIdx.x / nf;
      if (part < per) {
        const PeelRow r = peel_row(i, nf, F, g);
        if (r.d > shortest)
          for (int32_t j0 = part * kCoreNT * kPeelU; j0 < r.d; j0 += per * kCoreNT * kPeelU)
            peel_steps(g.adj + r.at, r.d, j0, kCoreNT, threadIdx.x, s, g, c);
      }
    } else {
      for (int32_t i = me; i < nf; i += waves) {
        const PeelRow r = peel_row(i, nf, F, g);
        if (r.d <= shortest) continue;
        for (int32_t j0 = 0; j0 < r.d; j0 += kWave * kPeelU) peel_steps(g.adj + r.at, r.d, j0, kWave, lane, s, g, c);
      }
    }
    if (nf > kPeelFew) peel_short(mine, s, g, c);
    return;
  }
  const int64_t step = (int64_t)waves * GPW;
  for (int64_t b = ((int64_t)blockIdx.x * WPB + wv) * GPW; b < nf; b += step) {  // wave-uniform
    const PeelRow r = peel_row(b + lane / kPeelG, nf, F, g);
    peel_short(r, s, g, c);
    // long rows: the whole wavefront on each in turn (group leaders' bits)
    uint64_t longs = __ballot(lane % kPeelG == 0 && r.d > kPeelShort);
    while (longs) {
      const int src = __builtin_ctzll(longs);
      longs &= longs - 1;
      const int32_t d = __shfl(r.d, src, kWave);
      const int64_t at = ((int64_t)__shfl((int32_t)(r.at >> 32), src, kWave) << 32) |
                         (uint32_t)__shfl((int32_t)r.at, src, kWave);
      for (int32_t j0 = 0; j0 < d; j0 += kWave * kPeelU) peel_steps(g.adj + at, d, j0, kWave, lane, s, g, c);
    }
  }
}

// Step i (1, 2, ..): forms its state from state and counters of step i - 1,
// does it into counters i, and prepares what step i + 1 reads: state i and
// zeroed counters i + 1 (those of step i - 2, which nothing reads any more).
__global__ __launch_bounds__(kCoreNT) void k_core_step(int step, int32_t n, int32_t k_stop, CoreArrays g) {
  CoreState s = *core_state(g.cnt, step - 1);
  if (step > 1) core_next(s, *core_count(g.cnt, step - 1), n, k_stop);
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    *core_state(g.cnt, step) = s;
    *core_count(g.cnt, step + 1) = CoreCount{0, 0, 0, kNoDegree};
  }
  CoreCount* c = core_count(g.cnt, step);
  __shared__ ScanLds lds;
  if (s.phase == kCoreScan) core_scan(s, g, c, lds);
  else if (s.phase == kCorePeel) core_peel(s, g, c);
}

// After step `step`, if the peeling has ended with it: the nodes left get k_stop.
__global__ __launch_bounds__(kCoreNT) void k_core_fill(int step, int32_t n, int32_t k_stop, CoreArrays g) {
  CoreState s = *core_state(g.cnt, step);
  core_next(s, *core_count(g.cnt, step), n, k_stop);
  if (s.phase != kCoreDone || s.left == 0) return;
  const int64_t stride = (int64_t)gridDim.x * kCoreNT;
  for (int64_t v = (int64_t)blockIdx.x * kCoreNT + threadIdx.x; v < n; v += stride)
    if (g.core[v] < 0) g.core[v] = k_stop;
}

unsigned core_grid(int64_t work) {
  int64_t b = (work + kCoreNT - 1) / kCoreNT;
  return (unsigned)(b < 1 ? 1 : b > 8192 ? 8192 : b);
}

CoreArrays core_arrays(const CoreBuffers& b) {
  return CoreArrays{b.off, b.deg, b.adj, b.cur, b.core, b.order, {b.F[0], b.F[1]}, {b.A[0], b.A[1]},
                    {b.near[0], b.near[1]}, b.cnt};
}

}  // namespace

hipError_t launch_core_init(int32_t n, int32_t k_stop, const CoreBuffers& b, hipStream_t s) {
  k_core_init<<<core_grid(n), kCoreNT, 0, s>>>(n, k_stop, b.deg, b.cur, b.core, b.cnt);
  return hipGetLastError();
}

hipError_t launch_core_steps(int first, int count, int32_t n, int32_t k_stop, const CoreBuffers& b, hipStream_t s) {
  // four blocks a CU: with 512 blocks the first levels took longer (8.0 ms at
  // R-MAT 20), with more the short steps
  const unsigned grid = std::min(core_grid((int64_t)n * kPeelG), 1024u);
  const CoreArrays g = core_arrays(b);
  for (int i = first; i < first + count; ++i) k_core_step<<<grid, kCoreNT, 0, s>>>(i, n, k_stop, g);
  return hipGetLastError();
}

CoreProgress core_progress(const int32_t* cnt, int step, int32_t n, int32_t k_stop) {
  CoreState s;
  CoreCount c;
  std::memcpy(&s, cnt + (step & 1) * (sizeof(CoreState) / 4), sizeof(s));
  std::memcpy(&c, cnt + 2 * (sizeof(CoreState) / 4) + step % 3 * (sizeof(CoreCount) / 4), sizeof(c));
  core_next(s, c, n, k_stop);
  return CoreProgress{s.phase == kCoreDone, s.left, s.maxc};
}

hipError_t launch_core_fill(int step, int32_t n, int32_t k_stop, const CoreBuffers& b, hipStream_t s) {
  k_core_fill<<<core_grid(n), kCoreNT, 0, s>>>(step, n, k_stop, core_arrays(b));
  return hipGetLastError();
}

}  // namespace tricc
