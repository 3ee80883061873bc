// Which rows of the graph build are sorted how, and the launch sizes that
// follow. Host arithmetic only.
#pragma once
#include <stdint.h>

#include <algorithm>

namespace tricc {

// Row classes by raw length.
enum RowClass : int {
  kRowTrivial = 0,  // len <= 1
  kRow8, kRow16, kRow32, kRow64,  // register bitonic sort by a lane group
  kRow128, kRow256, kRow512, kRow1024,  // register bitonic sort by a wavefront
  kRow4k,      // <= 4096, register bitonic sort by a block of 4 wavefronts
  kRow8k,      // <= 8192, by 8 wavefronts, or by bitmap (see row_first_bitmap_class)
  kRow16k,     // <= 16384, by 16 wavefronts, or by bitmap
  kRow32k,     // <= 32768, by a bitonic network in LDS, or by bitmap
  kRowMerge,   // > 32768 but short for the graph's ids: chunk sorts and merges
  kRowLarge,   // > 32768, by bitmap
  kNumRowClasses
};

// Ids per bitmap (128 KB of LDS): a graph of n nodes has row_ranges(n) ranges
// of them, and a row sorted by bitmap costs a block per range, whatever it holds.
constexpr int32_t kBitmapIds = 1 << 20;
inline int32_t row_ranges(int64_t n) { return (int32_t)((n + kBitmapIds - 1) / kBitmapIds); }

// Rows go by bitmap from these lengths on. One range: above 4,096 entries,
// where the register networks need a block of 8 wavefronts and more. More
// ranges: above 16,384 entries, and with at least 1,024 entries per range. Build
// of 3,000 rows of 17,000 entries, networks / bitmaps, ms: 2^25 ids (32 ranges)
// 8.7 / 10.3, 2^26 11.7 / 16.2, 2^27 39.3 / 49.3, and at 2^24 (16 ranges) 6.3 by
// bitmaps; of 300 rows of 200,000 entries, merges (an older build around them) /
// bitmaps: 2^25 ids 13.2 / 9.0, 2^26 17.1 / 13.1.
constexpr int32_t kBitmapMinPerRange = 1024;
inline int32_t row_bitmap_min(int64_t n) {
  const int32_t r = row_ranges(n);
  return r <= 1 ? 4097 : std::max(16385, kBitmapMinPerRange * r);
}
inline int row_first_bitmap_class(int64_t n) {
  const int32_t least = row_bitmap_min(n);
  return least <= 4097 ? kRow8k : least <= 16385 ? kRow32k : kRowLarge;
}

// Blocks of 1,024 threads for nrows rows sorted by bitmap (groups of 8 rows).
// A launch takes less than 2^32 threads in a dimension, 2^22 such blocks: rows
// sorted by bitmap hold 1,024 entries a range and more, of at most 2^31.
inline int64_t row_bitmap_blocks(int64_t nrows, int32_t ranges) { return (nrows + 7) / 8 * 8 * ranges; }

// Rows per block of 256 threads in the joint launches of the classes kRow4k,
// kRow1024, .., kRow8; the first kSortLongClasses of them form one launch, the
// others the other, cut up into launches of kRowShortGrid blocks (2^28 threads):
// 2^31 entries in rows of 2 make 2^25 blocks, twice what a launch takes, and rows
// of two classes can pass that where neither would alone.
constexpr int kSortClasses = kRow4k - kRow8 + 1;
constexpr int kSortLongClasses = kRow4k - kRow256;
constexpr int kSortRowsPerBlock[kSortClasses] = {1, 4, 4, 4, 4, 4, 8, 16, 32};
constexpr uint32_t kRowShortGrid = 1u << 20;
inline uint32_t row_sort_blocks(int64_t nrows, int k) {
  return (uint32_t)((nrows + kSortRowsPerBlock[k] - 1) / kSortRowsPerBlock[k]);
}
inline uint32_t row_short_grid(uint32_t blocks) { return std::min(blocks, kRowShortGrid); }

}  // namespace tricc
