// 4- and 5-clique counts (clique detection, among the graph-motif methods of
// Section 4): the triangle method one and two sizes up on the same
// degree-ordered DAG. A 4-clique u < w < x < z (by rank) is met once, at u:
// w in N+(u), x in C = N+(u) ∩ N+(w), z in N+(x) ∩ C; a 5-clique adds one
// more level of the same intersection.
#include "device_common.h"
#include "kernels.h"
#include "tables.h"

namespace tricc {

namespace {

constexpr int kK4NT = 256;
// Loads of 64 ids per step while rows are built, two steps in flight (four
// steps of 1 to 3 loads measured no faster).
constexpr int kK4U = 4;
// Out-degrees up to 64 take the kernel with a wavefront per node; up to
// kK4BitsLow and kK4BitsMid the bit-row kernel with 256 and 512 threads (14 and
// 48 KB of LDS); up to kK4BitsMax the one with 1,024 threads and 144 KB (one
// block per CU); up to 2,048 the pass kernel over quarters of the positions
// (1,024 threads, 142 KB); up to 4,096 the pass kernel over sixteenths
// (150 KB); up to kK4Cap = 8,192 the pass kernel over blocks of 64
// positions (2 words per row, 102 KB).
constexpr int kK4BitsSmall = 64;
// A wavefront's node has its lists streamed packed where their mean length is
// below this, else one by one, 64 ids a step either way (500k nodes of out-degree
// 20 in a ring, 4-cliques: one by one 3.3 ms, packed 1.8, with NEAR tables 0.50;
// 60-cliques 1.46 -> 0.81 -> 0.22; R-MAT of 1M nodes and 4M pairs 0.89 -> 0.94;
// bounds of 16, 32 and 100 took 3.4, 1.8 and 1.8 ms of the ring).
constexpr int32_t kK4PackMean = 64;
constexpr int kK4BitsLow = 256;
constexpr int kK4BitsMid = 512;
constexpr int kK4BitsMax = 1024;

// Position of the first element >= x in L[0, P), P a power of two and L
// ascending (padded past its length with kPad, above every id): fixed
// halving steps, no data-dependent exit. Every element before the result is
// below x, so x is in L iff L[result] == x.
__device__ __forceinline__ int32_t pow2_lower_pos(const int32_t* L, int32_t P, int32_t x) {
  int32_t p = 0;
  for (int32_t s = P >> 1; s > 0; s >>= 1)
    if (L[p + s - 1] < x) p += s;
  return p;
}

// Places of the ids of N+(u) in it, by a table in LDS (cuckoo, or buckets where
// a build gives up): two reads that do not depend on each other find an id,
// against a chain of log2 d in a search of the sorted list. The tables of small
// nodes have few slots, so their keys take NEAR slots: without, every build gave
// up on lists of neighbouring ids and a bucket chain held most of them (4-cliques
// of 200k nodes joined to the 50 on each side 3.8 ms, now 0.79; R-MAT of 240k
// nodes 1.66 ms either way).
constexpr bool kPlaceNear = true;
template <int SLOTS>
struct PlaceTable {
  int4 K[SLOTS / 4];
  uint16_t place[SLOTS];
  int32_t fail;
};

// Table of src[0, d) (d <= SLOTS / 2) for a group of G lanes, g = lane in group;
// true for the cuckoo layout. Callers separate it from the table's last use.
template <int G, int SLOTS>
__device__ __forceinline__ bool build_places(PlaceTable<SLOTS>& S, const int32_t* __restrict__ src, int32_t d, int g) {
  int32_t* K = reinterpret_cast<int32_t*>(S.K);
  for (int s = g; s < SLOTS; s += G) K[s] = -1;
  if (g == 0) S.fail = 0;
  group_sync<G>();
  for (int i = g; i < d; i += G)
    if (!cuckoo_insert<SLOTS, kPlaceNear>(K, src[i])) S.fail = 1;
  group_sync<G>();
  const bool ck = __builtin_amdgcn_readfirstlane(S.fail) == 0;
  if (!ck) {
    for (int s = g; s < SLOTS; s += G) K[s] = -1;
    group_sync<G>();
    for (int i = g; i < d; i += G) bucket_insert<SLOTS / 4>(K, src[i]);
    group_sync<G>();
  }
  for (int i = g; i < d; i += G) {
    const int32_t x = src[i];
    S.place[ck ? cuckoo_find<SLOTS, kPlaceNear>(K, x) : table_find<SLOTS>(K, x)] = (uint16_t)i;
  }
  group_sync<G>();
  return ck;
}

// Bit rows of the subgraph induced on N+(u) = dcol[ub, ub + d): for the lists
// i = wv, wv + NW, .. every id of N+(w_i) that is in N+(u) calls set(i, place).
// Begin and length of 64 lists at a time sit in the lanes; of each list, U
// loads of 64 ids are in flight while the ones before are looked up.
template <int NW, int U, typename Probe, typename Set>
__device__ __forceinline__ void stream_rows(int32_t wv0, int32_t d, int64_t ub, const int64_t* __restrict__ doff,
                                            const int32_t* __restrict__ dcol, const uint16_t* place, Probe probe,
                                            Set set) {
  const int32_t wv = __builtin_amdgcn_readfirstlane(wv0);
  const int lane = lane_id();
  for (int32_t i0 = wv; i0 < d; i0 += NW * kWave) {
    const int32_t left = (d - i0 + NW - 1) / NW;
    const int32_t cnt = left < kWave ? left : kWave;
    int32_t vb = 0, vn = 0;
    if (lane < cnt) {
      const int32_t w = dcol[ub + i0 + lane * NW];
      const int64_t b = doff[w];
      vb = (int32_t)b;
      vn = (int32_t)(doff[w + 1] - b);
    }
    int32_t k = 0, p = 0;
    int32_t b = __builtin_amdgcn_readlane(vb, 0), n = __builtin_amdgcn_readlane(vn, 0);
    auto advance = [&](int32_t (&cur)[U], int32_t (&nxt)[U]) -> bool {
      int32_t nk = k, nb = b, nn = n, np = p + U * kWave;
      if (np >= n) {
        nk = k + 1;
        np = 0;
        nn = 0;
        if (nk < cnt) {
          nb = __builtin_amdgcn_readlane(vb, nk);
          nn = __builtin_amdgcn_readlane(vn, nk);
        }
      }
      load_chunk<U>(nxt, dcol + nb, np, nn, lane);
      const int32_t rem = n - p;
#pragma unroll
      for (int q = 0; q < U; ++q) {
        if (q * kWave >= rem) break;
        int off;
        if (probe(cur[q], lane + q * kWave < rem, &off)) set(i0 + k * NW, (int32_t)place[off >> 2]);
      }
      if (np == 0 && nk >= cnt) return false;
      k = nk;
      b = nb;
      n = nn;
      p = np;
      return true;
    };
    int32_t x[U], y[U];
    load_chunk<U>(x, dcol + b, 0, n, lane);
    while (advance(x, y) && advance(y, x)) {
    }
  }
}

// Both layouts of the table.
template <int NW, int U, int SLOTS, typename Set>
__device__ __forceinline__ void stream_rows_of(bool ck, int32_t wv, int32_t d, int64_t ub,
                                               const int64_t* __restrict__ doff, const int32_t* __restrict__ dcol,
                                               const PlaceTable<SLOTS>& S, Set set) {
  if (ck)
    stream_rows<NW, U>(wv, d, ub, doff, dcol, S.place, CuckooProbe<SLOTS, kPlaceNear>{reinterpret_cast<const int32_t*>(S.K)}, set);
  else
    stream_rows<NW, U>(wv, d, ub, doff, dcol, S.place, BucketProbe<SLOTS / 4>{S.K}, set);
}

// Block-wide total of the per-lane counts, one 64-bit atomic per block.
// `red` holds NW values (the block's wavefronts); contains __syncthreads().
template <int NW>
__device__ __forceinline__ void k4_block_total(unsigned long long acc, unsigned long long* red,
                                               unsigned long long* total) {
  const int wv = threadIdx.x / kWave;
#pragma unroll
  for (int o = kWave / 2; o > 0; o >>= 1) acc += __shfl_xor(acc, o, kWave);
  __syncthreads();
  if (lane_id() == 0) red[wv] = acc;
  __syncthreads();
  if (threadIdx.x == 0) {
    unsigned long long t = 0;
    for (int q = 0; q < NW; ++q) t += red[q];
    if (t) atomicAdd(total, t);
  }
}

// Nodes with DMIN < d+(u) <= DMAX (and d+(u) >= 3): one block of NT threads
// per node. The block scans `chunk` (<= NT) consecutive ids at a time
// (grid-stride over such chunks), queues the ones in range in LDS, then
// takes them in turn. The block builds the subgraph induced on N+(u) as bit rows in
// LDS (row i: the places in N+(u) of N+(w_i) ∩ N+(u), each wavefront
// building the rows of its w's by looking N+(w) up in a table of N+(u)); then every pair
// (w, x) with x in row w adds popcount(row w & row x): the z that close the
// 4-clique {u, w, x, z}. Rows take RS = 2^rs words (RS >= d / 32), and the
// lanes of a wavefront cover 64 / RS rows x at once, one word each. LISTED:
// the x of row w are first listed in LDS by ballot; otherwise (rows of 32
// words, DMIN >= 512) they are taken two at a time straight from row w's
// bits, which leaves the LDS for 1,024 threads. The row's words lie in the lanes
// and those without a bit are passed over: read from LDS one after the other,
// they were nearly all the time of sparse rows (10,000 nodes with no edge among
// their 1,000 neighbours: 7.2 ms, 7.6 beside the table look-ups, now 1.36).
template <int DMIN, int DMAX, int NT, bool LISTED>
__global__ __launch_bounds__(NT) void k_count_k4_bits(int32_t n, int32_t chunk, const int64_t* __restrict__ doff,
                                                      const int32_t* __restrict__ dcol,
                                                      unsigned long long* __restrict__ total) {
  constexpr int NW = NT / kWave;
  static_assert(DMAX % 32 == 0 && DMAX <= 65536, "positions are stored in 16 bits");
  static_assert(LISTED || (DMIN >= 512 && DMAX <= 1024), "unlisted rows must be 32 words");
  __shared__ PlaceTable<2 * DMAX> S;
  __shared__ uint32_t B[DMAX * (DMAX / 32)];
  __shared__ uint16_t Pl[LISTED ? NW : 1][LISTED ? DMAX : 1];
  __shared__ unsigned long long red[NW];
  __shared__ int32_t Q[NT];
  __shared__ int32_t Qn;
  const int wv = threadIdx.x / kWave;
  const int lane = lane_id();
  unsigned long long acc = 0;
  for (int64_t base = (int64_t)blockIdx.x * chunk; base < n; base += (int64_t)gridDim.x * chunk) {
    __syncthreads();  // the previous chunk's queue has been taken
    if (threadIdx.x == 0) Qn = 0;
    __syncthreads();
    const int64_t v = base + threadIdx.x;
    if ((int)threadIdx.x < chunk && v < n) {
      const int32_t dv = (int32_t)(doff[v + 1] - doff[v]);
      if (dv >= 3 && dv > DMIN && dv <= DMAX) Q[atomicAdd(&Qn, 1)] = (int32_t)v;
    }
    __syncthreads();
    const int32_t nq = Qn;
    for (int32_t qi = 0; qi < nq; ++qi) {  // block-uniform
      const int32_t u = Q[qi];
      const int64_t ub = doff[u];
      const int32_t d = (int32_t)(doff[u + 1] - ub);
      const int rs = d <= 32 ? 0 : 32 - __builtin_clz((uint32_t)((d + 31) / 32 - 1));
      const int RS = 1 << rs;
      __syncthreads();  // the table and B of the previous node are no longer read
      for (int32_t q = threadIdx.x; q < d * RS; q += NT) B[q] = 0u;
      const bool ck = build_places<NT>(S, dcol + ub, d, threadIdx.x);
      stream_rows_of<NW, kK4U>(ck, wv, d, ub, doff, dcol, S,
                               [&](int32_t i, int32_t p) { atomicOr(&B[i * RS + (p >> 5)], 1u << (p & 31)); });
      __syncthreads();
      for (int32_t i = wv; i < d && !LISTED; i += NW) {
        // RS == 32: half-wave h takes the h-th of each next two bits of row i, whose
        // words lie in the lanes
        const int32_t k = lane & 31;
        const bool second = lane >= 32;
        const uint32_t bik = B[i * 32 + k];
        uint32_t some = (uint32_t)__ballot(bik != 0u);  // words with bits left
        uint32_t word = 0u;
        int32_t kw = 0;
        auto next = [&]() -> int32_t {  // -1 after the last
          if (word == 0u) {
            if (some == 0u) return -1;
            kw = __builtin_ctz(some);
            some &= some - 1u;
            word = (uint32_t)__builtin_amdgcn_readlane((int32_t)bik, kw);
          }
          const int32_t x = kw * 32 + __builtin_ctz(word);
          word &= word - 1u;
          return x;
        };
        while (true) {
          const int32_t xa = next();
          if (xa < 0) break;
          const int32_t xb = next();
          const int32_t x = second ? xb : xa;
          if (x >= 0) acc += (unsigned long long)__popc(bik & B[x * 32 + k]);
          if (xb < 0) break;
        }
      }
      for (int32_t i = wv; i < d && LISTED; i += NW) {
        const uint32_t* Bi = B + i * RS;
        int32_t np = 0;  // wave-uniform: the x of row i, listed
        for (int32_t b0 = 0; b0 < d; b0 += kWave) {
          const int32_t b = b0 + lane;
          const bool bit = b < d && ((Bi[b >> 5] >> (b & 31)) & 1u);
          const uint64_t m = __ballot(bit);
          if (bit) Pl[wv][np + mask_below(m)] = (uint16_t)b;
          np += (int32_t)__popcll(m);
        }
        wave_sync();
        if (np >= 2) {  // a clique needs x and z in row i
          const int32_t k = lane & (RS - 1);
          const int32_t js = lane >> rs;
          const uint32_t bik = Bi[k];
          for (int32_t j0 = 0; j0 < np; j0 += (kWave >> rs)) {
            const int32_t jj = j0 + js;
            if (jj < np) acc += (unsigned long long)__popc(bik & B[(int32_t)Pl[wv][jj] * RS + k]);
          }
        }
        wave_sync();  // the next row reuses Pl
      }
    }
  }
  k4_block_total<NW>(acc, red, total);
}

// Nodes with 3 <= d+(u) <= 64: a wavefront per node and no block barrier. The
// subgraph's adjacency is a 64-bit word per place p, of the places i whose list
// has p: built in LDS (the ids of a list set bits of different words), then held
// by lane p. For each place x the lanes whose word has x add popcount(word & word
// x), every 4-clique once, as by rows. The nodes of a block's chunk of ids go to
// its wavefronts in turn. Eight wavefronts a SIMD are asked for: left to itself the
// allocation took 87 scalar registers, of 80 that eight may have (1M R-MAT nodes
// with 4M pairs 0.96 -> 0.92 ms, the ring of out-degree 50 0.80 -> 0.75). Three quarters of the nodes of an
// R-MAT graph are this small; a block of 256 threads for each spent their time
// in barriers.
__global__ __launch_bounds__(kK4NT, 8) void k_count_k4_small(int32_t n, int32_t chunk, const int64_t* __restrict__ doff,
                                                          const int32_t* __restrict__ dcol,
                                                          unsigned long long* __restrict__ total) {
  constexpr int NW = kK4NT / kWave;
  __shared__ PlaceTable<2 * kK4BitsSmall> S[NW];
  __shared__ unsigned long long R[NW][kWave];
  __shared__ int2 lists[NW][kWave];  // offset and row of the lists that are not empty
  __shared__ PackStarts starts[NW];
  __shared__ unsigned long long red[NW];
  const int wv = threadIdx.x / kWave;
  const int lane = lane_id();
  uint32_t* B = reinterpret_cast<uint32_t*>(R[wv]);
  unsigned long long acc = 0;
  const int64_t step = (int64_t)gridDim.x * chunk;
  for (int64_t base = (int64_t)blockIdx.x * chunk; base < n; base += step) {
    const int32_t ids = (int32_t)min((int64_t)chunk, (int64_t)n - base);
    for (int32_t v0 = 0; v0 < ids; v0 += NW * kWave) {
      const int32_t vi = v0 + wv + lane * NW;  // ids in turn
      int32_t d0 = 0;
      int64_t b0 = 0;
      if (vi < ids) {
        b0 = doff[base + vi];
        d0 = (int32_t)(doff[base + vi + 1] - b0);
      }
      uint64_t todo = __ballot(d0 >= 3 && d0 <= kK4BitsSmall);
      while (todo) {
        const int src = __builtin_ctzll(todo);
        todo &= todo - 1;
        const int32_t d = __builtin_amdgcn_readlane(d0, src);
        const int64_t ub = __builtin_amdgcn_readlane((int32_t)b0, src);  // DAG offsets stay below 2^30
        int32_t vb = 0, vn = 0;
        if (lane < d) {
          const int32_t w = dcol[ub + lane];
          const int64_t b = doff[w];
          vb = (int32_t)b;
          vn = (int32_t)(doff[w + 1] - b);
        }
        const int32_t incl = wave_incl_scan(vn);
        const int32_t total = __builtin_amdgcn_readlane(incl, kWave - 1);
        wave_sync();  // the table and rows of the previous node are no longer read
        R[wv][lane] = 0ull;
        const uint64_t some = __ballot(vn > 0);
        if (vn > 0) lists[wv][mask_below(some)] = make_int2(vb - (incl - vn), lane);
        const bool ck = build_places<kWave>(S[wv], dcol + ub, d, lane);
        auto set = [&](int32_t i, int32_t p) { atomicOr(&B[2 * p + (i >> 5)], 1u << (i & 31)); };
        if (total < kK4PackMean * d) {
          auto packed = [&](auto probe) {
            stream_lists(
                vn, incl - vn, total, starts[wv], dcol, [&](int32_t k) { return lists[wv][k]; },
                [&](int32_t x, int32_t i, bool valid) {
                  int off;
                  if (probe(x, valid, &off)) set(i, (int32_t)S[wv].place[off >> 2]);
                });
          };
          if (ck) packed(CuckooProbe<2 * kK4BitsSmall, kPlaceNear>{reinterpret_cast<const int32_t*>(S[wv].K)});
          else packed(BucketProbe<2 * kK4BitsSmall / 4>{S[wv].K});
        } else {
          stream_rows_of<1, kK4U>(ck, 0, d, ub, doff, dcol, S[wv], set);
        }
        wave_sync();
        const unsigned long long row = R[wv][lane];
        const int32_t lo = (int32_t)(uint32_t)row, hi = (int32_t)(uint32_t)(row >> 32);
        uint32_t c = 0;
        for (int32_t x = 0; x < d; ++x) {
          const unsigned long long rx = ((unsigned long long)(uint32_t)__builtin_amdgcn_readlane(hi, x) << 32) |
                                        (uint32_t)__builtin_amdgcn_readlane(lo, x);
          if ((row >> x) & 1ull) c += (uint32_t)__popcll(row & rx);
        }
        acc += c;
      }
    }
  }
  k4_block_total<NW>(acc, red, total);
}

// Nodes with DMIN < d+(u) <= CAP: bit rows over blocks of PCOLS positions.
// Full rows (up to CAP / 32 words for CAP rows) do not fit in LDS, so the
// block of 1,024 threads makes one pass per PCOLS positions: it builds that
// block of every row (PCOLS / 32 words per row, 128 KB for CAP rows); then
// each wavefront streams N+(w) again, places its ids in N+(u), and for every
// x found (the hits of 64 ids, 64 / (PCOLS / 32) x at a time) adds
// popcount(row w & row x) over the block. Summed over the passes this is the
// count the full rows give. Nodes are queued from chunks of ids as in the
// bit-row kernel.
constexpr int kK4QNT = 1024;
constexpr int kK4QWaves = kK4QNT / kWave;

template <int DMIN, int CAP, int PCOLS>
__global__ __launch_bounds__(kK4QNT) void k_count_k4_passes(int32_t n, int32_t chunk,
                                                            const int64_t* __restrict__ doff,
                                                            const int32_t* __restrict__ dcol,
                                                            unsigned long long* __restrict__ total) {
  constexpr int kK4QCols = PCOLS;
  constexpr int kK4QWords = PCOLS / 32;
  static_assert(PCOLS % 32 == 0 && kK4QWords <= kWave && CAP <= 65536, "pass layout");
  __shared__ int32_t L[CAP];
  __shared__ uint32_t B[CAP * kK4QWords];
  __shared__ uint16_t H[kK4QWaves][kWave];
  __shared__ unsigned long long red[kK4QWaves];
  __shared__ int32_t Q[kK4QNT];
  __shared__ int32_t Qn;
  const int wv = threadIdx.x / kWave;
  const int lane = lane_id();
  unsigned long long acc = 0;
  for (int64_t base = (int64_t)blockIdx.x * chunk; base < n; base += (int64_t)gridDim.x * chunk) {
    __syncthreads();  // the previous chunk's queue has been taken
    if (threadIdx.x == 0) Qn = 0;
    __syncthreads();
    const int64_t v = base + threadIdx.x;
    if ((int)threadIdx.x < chunk && v < n) {
      const int64_t dv = doff[v + 1] - doff[v];
      if (dv > DMIN && dv <= CAP) Q[atomicAdd(&Qn, 1)] = (int32_t)v;
    }
    __syncthreads();
    const int32_t nq = Qn;
    for (int32_t qi = 0; qi < nq; ++qi) {  // block-uniform
      const int32_t u = Q[qi];
      const int64_t ub = doff[u];
      const int32_t d = (int32_t)(doff[u + 1] - ub);
      const int32_t P = 1 << (32 - __builtin_clz((uint32_t)(d - 1)));  // power of two >= d, <= CAP
      __syncthreads();  // L and B of the previous node are no longer read
      for (int32_t i = threadIdx.x; i < P; i += kK4QNT) L[i] = i < d ? dcol[ub + i] : kPad;
      for (int32_t q = 0; q * kK4QCols < d; ++q) {
        __syncthreads();  // L written; the previous quarter's rows no longer read
        for (int32_t e = threadIdx.x; e < d * kK4QWords; e += kK4QNT) B[e] = 0u;
        __syncthreads();
        for (int32_t i = wv; i < d; i += kK4QWaves) {  // quarter q of row i
          const int32_t w = L[i];
          const int64_t wb = doff[w];
          const int32_t dw = (int32_t)(doff[w + 1] - wb);
          for (int32_t t = lane; t < dw; t += kWave) {
            const int32_t y = dcol[wb + t];
            const int32_t p = pow2_lower_pos(L, P, y);
            if (L[p] == y && p / kK4QCols == q)
              atomicOr(&B[i * kK4QWords + (p % kK4QCols) / 32], 1u << (p & 31));
          }
        }
        __syncthreads();
        const int32_t k = lane & (kK4QWords - 1);
        const int32_t j = lane / kK4QWords;
        for (int32_t i = wv; i < d; i += kK4QWaves) {  // the x of row i, quarter q of the AND
          const int32_t w = L[i];
          const int64_t wb = doff[w];
          const int32_t dw = (int32_t)(doff[w + 1] - wb);
          const uint32_t bw = B[i * kK4QWords + k];
          for (int32_t t0 = 0; t0 < dw; t0 += kWave) {
            const int32_t t = t0 + lane;
            bool hit = false;
            int32_t p = 0;
            if (t < dw) {
              const int32_t y = dcol[wb + t];
              p = pow2_lower_pos(L, P, y);
              hit = L[p] == y;
            }
            const uint64_t m = __ballot(hit);
            const int32_t nh = (int32_t)__popcll(m);
            if (hit) H[wv][mask_below(m)] = (uint16_t)p;
            wave_sync();
            for (int32_t g = 0; g < nh; g += kWave / kK4QWords) {
              const int32_t jj = g + j;
              if (jj < nh) acc += (unsigned long long)__popc(bw & B[(int32_t)H[wv][jj] * kK4QWords + k]);
            }
            wave_sync();  // H is rewritten by the next 64 ids
          }
        }
      }
    }
  }
  k4_block_total<kK4QWaves>(acc, red, total);
}

// 5-cliques, nodes with DMIN < d+(u) <= DMAX (and d+(u) >= 4): the bit rows
// of the subgraph induced on N+(u) are built as for the 4-clique kernel; a
// 5-clique u < w < x < y < z is then w's row bit x, y a bit of the AND of
// rows w and x, and z a bit of that AND with row y. Each wavefront takes rows
// w in turn and walks the x of row w one at a time: every lane forms one
// word of the AND of rows w and x (lane & (RS - 1)), the y in it are listed
// in LDS (per lane, in bit order, after a scan of the lanes' popcounts), and
// groups of 64 / RS lanes add popcount(AND & row y), one word each. The y are
// listed where the table was: apart they took 44,088 bytes of LDS for out-degrees
// up to 512, three blocks a CU instead of four (50k nodes in a ring joined to the
// 200 on each side 555 -> 603 ms, now 474; R-MAT of 262k nodes and 4M pairs 56.3 -> 51.6, now 44.5).
template <int DMIN, int DMAX, int NT>
__global__ __launch_bounds__(NT) void k_count_k5_bits(int32_t n, int32_t chunk, const int64_t* __restrict__ doff,
                                                      const int32_t* __restrict__ dcol,
                                                      unsigned long long* __restrict__ total) {
  constexpr int NW = NT / kWave;
  static_assert(DMAX % 32 == 0 && DMAX <= 1024, "rows of at most 32 words");
  __shared__ union {
    PlaceTable<2 * DMAX> S;  // while the rows are built
    uint16_t Y[NW][DMAX];    // after that
  } lds;
  __shared__ uint32_t B[DMAX * (DMAX / 32)];
  PlaceTable<2 * DMAX>& S = lds.S;
  uint16_t(&Y)[NW][DMAX] = lds.Y;
  __shared__ unsigned long long red[NW];
  __shared__ int32_t Q[NT];
  __shared__ int32_t Qn;
  static_assert(DMAX > kK4BitsMid ||
                    sizeof(lds) + sizeof(B) + sizeof(red) + sizeof(Q) + sizeof(Qn) <= 160 * 1024 / 4,
                "four blocks a CU");
  const int wv = threadIdx.x / kWave;
  const int lane = lane_id();
  unsigned long long acc = 0;
  for (int64_t base = (int64_t)blockIdx.x * chunk; base < n; base += (int64_t)gridDim.x * chunk) {
    __syncthreads();  // the previous chunk's queue has been taken
    if (threadIdx.x == 0) Qn = 0;
    __syncthreads();
    const int64_t v = base + threadIdx.x;
    if ((int)threadIdx.x < chunk && v < n) {
      const int32_t dv = (int32_t)(doff[v + 1] - doff[v]);
      if (dv >= 4 && dv > DMIN && dv <= DMAX) Q[atomicAdd(&Qn, 1)] = (int32_t)v;
    }
    __syncthreads();
    const int32_t nq = Qn;
    for (int32_t qi = 0; qi < nq; ++qi) {  // block-uniform
      const int32_t u = Q[qi];
      const int64_t ub = doff[u];
      const int32_t d = (int32_t)(doff[u + 1] - ub);
      const int rs = d <= 32 ? 0 : 32 - __builtin_clz((uint32_t)((d + 31) / 32 - 1));
      const int RS = 1 << rs;
      __syncthreads();  // Y and B of the previous node are no longer read
      for (int32_t q = threadIdx.x; q < d * RS; q += NT) B[q] = 0u;
      const bool ck = build_places<NT>(S, dcol + ub, d, threadIdx.x);
      stream_rows_of<NW, kK4U>(ck, wv, d, ub, doff, dcol, S,
                               [&](int32_t i, int32_t p) { atomicOr(&B[i * RS + (p >> 5)], 1u << (p & 31)); });
      __syncthreads();
      const int32_t k = lane & (RS - 1);
      const int32_t js = lane >> rs;
      for (int32_t i = wv; i < d; i += NW) {
        const uint32_t* Bi = B + i * RS;
        const uint32_t bik = Bi[k];
        for (int32_t kw = 0; kw < RS; ++kw) {
          uint32_t word = Bi[kw];  // wave-uniform
          while (word) {
            const int32_t x = kw * 32 + __builtin_ctz(word);
            word &= word - 1u;
            const uint32_t wx = bik & B[x * RS + k];
            // list the y of wx: lanes 0 .. RS-1 own one word each
            const int32_t c = lane < RS ? __popc(wx) : 0;
            const int32_t incl = wave_incl_scan(c);
            const int32_t ny = __builtin_amdgcn_readlane(incl, kWave - 1);
            if (ny < 2) continue;  // y and z both lie in wx (wave-uniform)
            if (lane < RS) {
              uint32_t bits = wx;
              int32_t o = incl - c;
              while (bits) {
                Y[wv][o++] = (uint16_t)(lane * 32 + __builtin_ctz(bits));
                bits &= bits - 1u;
              }
            }
            wave_sync();
            for (int32_t g = 0; g < ny; g += (kWave >> rs)) {
              const int32_t jj = g + js;
              if (jj < ny) acc += (unsigned long long)__popc(wx & B[(int32_t)Y[wv][jj] * RS + k]);
            }
            wave_sync();  // Y is rewritten for the next x
          }
        }
      }
    }
  }
  k4_block_total<NW>(acc, red, total);
}

__global__ void k_zero_one(unsigned long long* p) {
  if (threadIdx.x == 0) *p = 0ull;
}

}  // namespace

// Chunk of ids per scan step: enough chunks to fill `target` blocks, at
// most `nt` ids (one per thread).
static int32_t k4_chunk(int32_t n, int64_t target, int32_t nt) {
  const int64_t c = ((int64_t)n + target - 1) / target;
  return (int32_t)(c < 1 ? 1 : c > nt ? nt : c);
}

static unsigned k4_grid(int32_t n, int32_t chunk, int64_t cap) {
  const int64_t g = ((int64_t)n + chunk - 1) / chunk;
  return (unsigned)(g < cap ? g : cap);
}

// The bit-row kernels get a block per few ids (the dispatcher balances them; a
// grid of a few blocks a CU took 30% longer on an R-MAT graph of 240k nodes).
// Kernels of out-degrees that the graph does not reach are left out. Measured
// on that graph, largest out-degree 396: 3.35 -> 1.60 ms against one bit-row
// kernel for all out-degrees up to 512 whose rows were built by searches of
// N+(u) (of the 1.60 ms, 0.40 up to out-degree 64, 0.71 up to 256).
hipError_t launch_count_k4(int32_t n, int64_t max_outdeg, const int64_t* doff, const int32_t* dcol,
                           unsigned long long* total, hipStream_t s) {
  k_zero_one<<<1, 64, 0, s>>>(total);
  if (n > 0 && max_outdeg >= 3) {
    const int32_t cs = k4_chunk(n, 16384, 1024);
    k_count_k4_small<<<k4_grid(n, cs, 16384), kK4NT, 0, s>>>(n, cs, doff, dcol, total);
    const int32_t cm = k4_chunk(n, 65536, kK4NT);
    if (max_outdeg > kK4BitsSmall)
      k_count_k4_bits<kK4BitsSmall, kK4BitsLow, kK4NT, true><<<k4_grid(n, cm, 65536), kK4NT, 0, s>>>(n, cm, doff, dcol,
                                                                                                  total);
    if (max_outdeg > kK4BitsLow)
      k_count_k4_bits<kK4BitsLow, kK4BitsMid, 512, true><<<k4_grid(n, cm, 65536), 512, 0, s>>>(n, cm, doff, dcol, total);
    const int32_t cb = k4_chunk(n, 1024, 1024);
    if (max_outdeg > kK4BitsMid)
      k_count_k4_bits<kK4BitsMid, kK4BitsMax, 1024, false><<<k4_grid(n, cb, 1024), 1024, 0, s>>>(n, cb, doff, dcol,
                                                                                                total);
    if (max_outdeg > kK4BitsMax)
      k_count_k4_passes<kK4BitsMax, 2048, 512><<<k4_grid(n, cb, 1024), kK4QNT, 0, s>>>(n, cb, doff, dcol, total);
    if (max_outdeg > 2048)
      k_count_k4_passes<2048, 4096, 256><<<k4_grid(n, cb, 1024), kK4QNT, 0, s>>>(n, cb, doff, dcol, total);
    if (max_outdeg > 4096)
      k_count_k4_passes<4096, kK4Cap, 64><<<k4_grid(n, cb, 1024), kK4QNT, 0, s>>>(n, cb, doff, dcol, total);
  }
  return hipGetLastError();
}

// One kernel takes all nodes up to out-degree 512: a node above 256 takes a block
// up to a millisecond, and in a launch of their own the few such nodes left the
// chip idle (R-MAT of 100k nodes, largest out-degree 259: 11.8 ms in two
// launches, 9.4 in one; 10.9 before the table look-ups). Without such nodes the
// kernel for up to 256 lets more blocks share a CU.
hipError_t launch_count_k5(int32_t n, int64_t max_outdeg, const int64_t* doff, const int32_t* dcol,
                           unsigned long long* total, hipStream_t s) {
  k_zero_one<<<1, 64, 0, s>>>(total);
  if (n > 0 && max_outdeg >= 4) {
    const int32_t cm = k4_chunk(n, 65536, kK4NT);
    if (max_outdeg <= kK4BitsLow)
      k_count_k5_bits<0, kK4BitsLow, kK4NT><<<k4_grid(n, cm, 65536), kK4NT, 0, s>>>(n, cm, doff, dcol, total);
    else
      k_count_k5_bits<0, kK4BitsMid, kK4NT><<<k4_grid(n, cm, 65536), kK4NT, 0, s>>>(n, cm, doff, dcol, total);
    const int32_t cb = k4_chunk(n, 2048, 512);
    if (max_outdeg > kK4BitsMid)
      k_count_k5_bits<kK4BitsMid, kK5Cap, 512><<<k4_grid(n, cb, 2048), 512, 0, s>>>(n, cb, doff, dcol, total);
  }
  return hipGetLastError();
}

}  // namespace tricc
