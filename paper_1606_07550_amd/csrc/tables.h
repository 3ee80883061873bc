// Id tables in LDS (bucket and cuckoo layouts) and streams of lists, shared by
// the intersection and clique kernels.
#pragma once
#include "device_common.h"

namespace tricc {

template <int G>
__device__ __forceinline__ void group_sync() {
  if constexpr (G > kWave) __syncthreads();
  else wave_sync();
}

// Open-addressing table of NB buckets of 4 int32 keys (-1 = empty), probed
// bucket by bucket: a lookup is normally one 16-byte LDS read.
template <int NB>
__device__ __forceinline__ int bucket_insert(int32_t* K, int32_t x) {
  uint32_t b = hash_slot(x, __builtin_ctz(NB));
  while (true) {
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if (atomicCAS(&K[4 * b + j], -1, x) == -1) return (int)(4 * b + j);
    b = (b + 1) & (NB - 1);
  }
}

// Slot of x, or -1. `first` is the already-loaded bucket hash_slot(x).
template <int NB>
__device__ __forceinline__ int bucket_match(const int4* Kb, int32_t x, uint32_t b, int4 q) {
  while (true) {
    if (q.x == x) return (int)(4 * b);
    if (q.y == x) return (int)(4 * b + 1);
    if (q.z == x) return (int)(4 * b + 2);
    if (q.w == x) return (int)(4 * b + 3);
    if (q.w < 0) return -1;  // keys fill a bucket in order: an empty last slot ends the chain
    b = (b + 1) & (NB - 1);
    q = Kb[b];
  }
}

template <int SLOTS>
__device__ __forceinline__ int table_find(const int32_t* K, int32_t x) {
  constexpr int NB = SLOTS / 4;
  const int4* Kb = reinterpret_cast<const int4*>(K);
  const uint32_t b = hash_slot(x, __builtin_ctz(NB));
  return bucket_match<NB>(Kb, x, b, Kb[b]);
}

// Looks x up in the bucket table: true when the lane is valid and x is in
// the table, with *off the byte offset inside the counter array C of x's
// slot (slot j of bucket b is counter 4b + j, at byte 16b + 4j). One 16-byte
// read unless x's home bucket is full and does not hold x (rare in a sparse
// table). The matching slot comes from four compares whose lane masks are
// combined on the scalar unit.
template <int NB>
__device__ __forceinline__ bool bucket_credit(const int4* Kb, int32_t x, bool valid, int* off) {
  uint32_t b = hash_slot(x, __builtin_ctz(NB));
  int4 q = Kb[b];
  bool e1 = q.y == x, e2 = q.z == x, e3 = q.w == x;
  bool hit = (q.x == x) | e1 | e2 | e3;
  int o = (int)(b << 4) + ((e1 | e3) ? 4 : 0) + ((e2 | e3) ? 8 : 0);
  bool more = valid & !hit & (q.w >= 0);
  while (more) {
    b = (b + 1) & (NB - 1);
    q = Kb[b];
    e1 = q.y == x;
    e2 = q.z == x;
    e3 = q.w == x;
    hit = (q.x == x) | e1 | e2 | e3;
    o = (int)(b << 4) + ((e1 | e3) ? 4 : 0) + ((e2 | e3) ? 8 : 0);
    more = !hit & (q.w >= 0);
  }
  *off = o;
  return valid & hit;
}

// Two-choice cuckoo table of SLOTS int32 keys (-1 = empty), one key per
// slot (Pagh and Rodler 2001; built in parallel with atomic exchanges as in
// Alcantara et al. 2009): key x sits in slot a(x) or b(x), so a lookup is two
// 4-byte LDS reads and two compares, with no probe loop. Ids share a slot
// pair when their low 24 bits agree.
// Both slots by the top bits of products (hash_slot): ids that lie close
// together fall into close slots, which keeps the bank conflicts of a stream of
// them low, but a table of few slots has no room for many such ids. NEAR: the
// second slot by lower bits of the first's product, where the constant is the
// golden section and neighbours fall far apart.
template <int SLOTS, bool NEAR = false>
__device__ __forceinline__ void cuckoo_pos(int32_t x, uint32_t* a, uint32_t* b) {
  constexpr int bits = __builtin_ctz(SLOTS);
  const uint32_t lo = (uint32_t)x & 0xFFFFFFu;
  *a = (lo * 0x9E3779u) >> (32 - bits);
  *b = NEAR ? ((lo * 0x9E3779u) >> (24 - bits)) & (SLOTS - 1) : (lo * 0x3C6EF3u) >> (32 - bits);
}

// The same two slots as byte offsets (4 x slot).
template <int SLOTS, bool NEAR = false>
__device__ __forceinline__ void cuckoo_off(int32_t x, uint32_t* a, uint32_t* b) {
  cuckoo_pos<SLOTS, NEAR>(x, a, b);
  *a <<= 2;
  *b <<= 2;
}

// Eviction chains longer than this give up: the caller then rebuilds the
// node's table in the bucket layout.
constexpr int kCuckooMaxChain = 48;

// Inserts x (absent from the table; keys are distinct). Each thread holds
// exactly one key outside the table at any time, so concurrent inserts lose
// nothing while they succeed. False: the chain gave up and the key it held
// is not in the table.
template <int SLOTS, bool NEAR = false>
__device__ __forceinline__ bool cuckoo_insert(int32_t* K, int32_t x) {
  uint32_t a, b;
  cuckoo_pos<SLOTS, NEAR>(x, &a, &b);
  if (atomicCAS(&K[a], -1, x) == -1 || atomicCAS(&K[b], -1, x) == -1) return true;
  uint32_t pos = a;
#pragma unroll 1
  for (int it = 0; it < kCuckooMaxChain; ++it) {
    x = atomicExch(&K[pos], x);
    if (x == -1) return true;
    cuckoo_pos<SLOTS, NEAR>(x, &a, &b);  // the evicted key moves to its other slot
    pos = pos == a ? b : a;
  }
  return false;
}

// Slot of x in a complete cuckoo table, or -1.
template <int SLOTS, bool NEAR = false>
__device__ __forceinline__ int cuckoo_find(const int32_t* K, int32_t x) {
  uint32_t a, b;
  cuckoo_pos<SLOTS, NEAR>(x, &a, &b);
  return K[a] == x ? (int)a : K[b] == x ? (int)b : -1;
}

// Probes of the streaming loops: true when the lane is valid and x is in the
// table, with *off the byte offset of x's counter in C (4 x slot). The
// callers count the hits (per lane in a register on the long-list path, so
// that no scalar instruction is spent per 64 ids).
template <int NB>
struct BucketProbe {
  const int4* Kb;
  __device__ __forceinline__ bool operator()(int32_t x, bool valid, int* off) const {
    return bucket_credit<NB>(Kb, x, valid, off);
  }
};

template <int SLOTS, bool NEAR = false>
struct CuckooProbe {
  const int32_t* K;
  __device__ __forceinline__ bool operator()(int32_t x, bool valid, int* off) const {
    x = valid ? x : -2;  // in no table
    uint32_t a, b;
    cuckoo_off<SLOTS, NEAR>(x, &a, &b);
    const char* Kc = reinterpret_cast<const char*>(K);
    const bool ea = *reinterpret_cast<const int32_t*>(Kc + a) == x;
    const bool eb = *reinterpret_cast<const int32_t*>(Kc + b) == x;
    *off = (int)(ea ? a : b);
    return ea | eb;
  }
};

// U chunks of 64 ids of L[p..n) into x, through a raw buffer view of
// L[p..n): the offsets are lane * 4 + k * 256, which its range check covers
// exactly, so lanes past n read 0 without a memory access. All U loads are
// issued, which keeps the wait counts of the caller's pipeline exact.
template <int U>
__device__ __forceinline__ void load_chunk(int32_t (&x)[U], const int32_t* L, int32_t p, int32_t n, int lane) {
  static_assert(U * kWave * 4 <= 4096, "per-load offsets must fit the 12-bit immediate field");
  const int32_t left = n > p ? n - p : 0;
  const __amdgpu_buffer_rsrc_t rs =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<int32_t*>(L + p), (short)0, left * 4, kRawBufferWord3);
#pragma unroll
  for (int k = 0; k < U; ++k) x[k] = __builtin_amdgcn_raw_buffer_load_b32(rs, lane * 4 + k * kWave * 4, 0, 0);
}

// Steps of 64 ids whose gathers are issued together in the packed streams.
constexpr int kPackUnroll = 3;

// Positions of a concatenation of lists whose starts are marked at a time: five
// steps of the packed streams, one bit a position.
constexpr int32_t kPackWindow = 5 * kPackUnroll * kWave;
struct PackStarts {
  uint64_t bits[(kPackWindow / kWave + 1) & ~1];
};

// The concatenation of 64 lists, one per lane (begin b, length n, 0 for none),
// 64 ids per step: body(x, k, valid) gets the lane's id and the number of its
// list among the lists that are not empty. The list of position t is the number
// of list starts in (0, t]: the starts are marked as bits in LDS, so a step
// takes one read of 64 bits, a lane-mask count and, through where(k), the offset
// of list k against its place in the concatenation. (A search of the lanes'
// prefixes by shuffles is six dependent LDS round trips and 30 instructions a
// step.) kPackUnroll independent gathers are in flight before their bodies.
template <typename Where, typename Body>
__device__ __forceinline__ void stream_lists(int32_t n, int32_t ex, int32_t total, PackStarts& P,
                                             const int32_t* __restrict__ dcol, Where where, Body body) {
  const int lane = lane_id();
  uint32_t* bits = reinterpret_cast<uint32_t*>(P.bits);
  int32_t before = 0;  // starts in (0, t0]
  for (int32_t w0 = 0; w0 < total; w0 += kPackWindow) {
    wave_sync();  // the previous window's bits are no longer read
    if (lane < (int)(sizeof(PackStarts) / 4)) bits[lane] = 0u;
    wave_sync();
    const int32_t at = ex - 1 - w0;
    if (n > 0 && (uint32_t)at < (uint32_t)kPackWindow) atomicOr(&bits[at >> 5], 1u << (at & 31));
    wave_sync();
    const int32_t end = min(total, w0 + kPackWindow);
    for (int32_t t0 = w0; t0 < end; t0 += kPackUnroll * kWave) {
      int32_t x[kPackUnroll], kk[kPackUnroll];
#pragma unroll
      for (int r = 0; r < kPackUnroll; ++r) {
        const int32_t t = t0 + r * kWave + lane;
        const uint64_t mv = P.bits[(t0 - w0) / kWave + r];
        const uint64_t m = ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(mv >> 32)) << 32) |
                           (uint32_t)__builtin_amdgcn_readfirstlane((int)mv);
        const int2 l = where(before + mask_below(m));
        before += (int32_t)__popcll(m);
        x[r] = t < total ? dcol[l.x + t] : -1;
        kk[r] = l.y;
      }
#pragma unroll
      for (int r = 0; r < kPackUnroll; ++r) {
        if (t0 + r * kWave >= total) break;
        body(x[r], kk[r], t0 + r * kWave + lane < total);
      }
    }
  }
}

}  // namespace tricc
