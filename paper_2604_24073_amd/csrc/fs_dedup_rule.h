// Which form the index half of a batch takes: one workgroup (fs_small.hip), or a chain of launches whose dedup goes by ranges
// of keys (fs_bucket.hip) or by radix passes (fs_unique.hip).  Host code only, no HIP, so that the rules can be compiled and
// looked at by themselves.
#pragma once

#include <stdint.h>

namespace fs {

#ifndef FS_RADIX_BITS
#define FS_RADIX_BITS 9
#endif
constexpr int kRadixBits = FS_RADIX_BITS;                 // most bits one pass may sort (11 would sort 22-bit row IDs in
                                                          // two passes, but every scatter workgroup then scans a
                                                          // [tile][2048] table and lives four times as long beside the
                                                          // class passes: measured slower, 105.2 against 103.0 us per step)

// bits of a row ID of a table of num_rows rows (of unknown size: 63)
inline int key_bits_of(int64_t num_rows) {
    if (num_rows <= 0) return 63;
    int kb = 1;
    while (kb < 63 && (1ll << kb) < num_rows) ++kb;
    return kb;
}
inline int radix_passes(int key_bits) { return (key_bits + kRadixBits - 1) / kRadixBits; }

// IDs of a batch whose index half fits the LDS of one workgroup, and the most it takes.  On the caller's stream: up to where
// the chain of launches over many workgroups is the faster one (a whole step, one workgroup against the chain: 1024 IDs
// 25.4 / 40.7 us, 4096 40.1 / 53.4, 6144 53.8 / 62.2, 8192 59.9 / 62.6).  Ahead of time a launch costs whatever runs beside
// it and the workgroup has the iterations ahead to finish, but it must keep up with them, and it sorts by 8 bits a pass.
// Ten steps, one workgroup / the chain, tables of 64 columns, median of three processes: two passes, 11000 IDs, one table of
// 500 rows 263 / 315 us, of 65536 283 / 310, three 439 / 591 and 500 / 568; 12200 IDs 263 / 303, 290 / 315, 445 / 591, 521 /
// 524.  Three passes, of 1 M rows, one and three tables: 9000 IDs 309 / 318, 565 / 572; 10200 320 / 315, 573 / 540; 11000
// 322 / 318, 590 / 527; 12200 336 / 319, 620 / 540.
constexpr int64_t kSmallIds = 16384;
constexpr int kSmallBits = 8;                             // most bits of a radix pass
constexpr int64_t kSmallIdsInline = 8192;
constexpr int64_t kSmallIdsAhead = 10240, kSmallIdsAheadTwoPasses = 12288;
inline int64_t small_index_ids(bool callers_stream, int key_bits) {
    return callers_stream ? kSmallIdsInline : key_bits <= 2 * kSmallBits ? kSmallIdsAheadTwoPasses : kSmallIdsAhead;
}
static_assert(kSmallIdsAheadTwoPasses <= kSmallIds && kSmallIdsInline <= kSmallIds, "what the LDS holds");

// Dedup by ranges of keys: most IDs of a batch (a place and a rank share 32 bits), IDs of a tile, most ranges, and the IDs
// a range is meant to hold (up to that many; a power of two of ranges).
constexpr int64_t kBucketIdsMax = 1 << 20;
constexpr int kBucketTile = 2048;
constexpr int kMaxBuckets = 1024;
constexpr int kBucketMean = 768;
inline int ranges_log2(int64_t n) {
    int k = 0;
    while ((1 << k) < kMaxBuckets && ((int64_t)kBucketMean << k) < n) ++k;
    return k;
}
// IDs of a batch from which the ranges are 1024: two to a compute unit (58 KB of LDS each), 512 of them run at once.
constexpr int64_t kBucketOneWave = (int64_t)kBucketMean << 9;

// By ranges or by radix passes?  Four launches by ranges, whatever the keys (up to 49152 IDs three; three or two where the
// order alone is wanted); two per radix pass of up to 9 key bits and two more.  Radix / ranges, us (tables of 64 fp32 columns,
// Zipf IDs), all of them of the form with four launches:
//   one pass (512 rows): radix at every size.  The dedup alone, 9 k IDs 22 / 25, 131 k 23 / 29, 393 k 26 / 34, 786 k 32 / 55;
//     ten steps of 60 k 281 / 313, of 500 k 776 / 814; self-contained step of 500 k 98 / 117; 65 k samples up to 500 long
//     balanced 73.9 / 78.2.  (Below five rows and 34 k IDs the ranges lead, 28 / 23; no table is as small.)
//   two passes (2^18 rows): ranges while they run all at once, 20 k IDs 36 / 28, 393216 43 / 41; beyond it depends on what is
//     beside them.  Alone 393217 43 / 47, 550 k 47 / 54, 786 k 52 / 60.  Of an index half, where the smaller workgroups find
//     a place beside the row work sooner, ten steps 500 k 866 / 865, 700 k 1129 / 1093, 1 M 1585 / 1487 (200 k rows 1790 /
//     1632), self-contained step of 400 k 121 / 124, of 700 k 160 / 156.
//   three and more: ranges at every size they can take.  4 M rows alone 300 k 62 / 44, 786 k 77 / 73, 1 M 86 / 82 (mean of 16
//     batches, those with a range beyond LDS among them); ten steps of 1 M 2200 / 2038; 2^30 rows alone, 1 M 118 / 88.  Only
//     batches of next to nothing but one row are the slower for it (400 k times one row 54 / 60), and those with a range beyond
//     LDS (1 M in runs of fifty 71 / 83).
// most_ids, key_bits: the largest batch and the widest key of the dedups that share the launches; alone: an operation of its
// own, not part of an index half.
inline bool dedup_by_ranges(int64_t most_ids, int key_bits, bool alone) {
    if (key_bits > 31 || most_ids > kBucketIdsMax) return false;
    const int passes = radix_passes(key_bits);
    return passes >= 3 || (passes == 2 && (!alone || most_ids <= kBucketOneWave));
}

}  // namespace fs
