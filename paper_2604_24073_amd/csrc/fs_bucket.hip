// Dedup of one iteration's row IDs by ranges: the batch is cut into ranges of keys of about equal weight, every range is
// sorted, stably, by one workgroup in LDS.  Same outputs as the radix sort of fs_unique.hip, bit for bit, in four
// launches (up to 49152 IDs three) instead of eight (two per radix pass, two for the compaction):
//
//   sample     a stratified sample of the batch is sorted by one workgroup, every fourth entry becomes a boundary (up to 64
//              ranges, 49152 IDs, the partition finds the boundaries by itself)
//   partition  every tile of 2048 IDs is put in the order of its ranges, on the spot: a workgroup's output goes where its
//              input lay, with a table of where each range starts in each tile
//   sort       one workgroup per range collects its pieces from the tiles (tile order = batch order), sorts them and
//              lists its distinct rows; the table gives its place in the sorted batch, so nothing is scattered
//              across the chip and no launch has to count digits first
//   compact    the distinct rows of the ranges, closed up
//
// What bounds it: launches and dependent rounds, not bytes (a few MB).  Sample, partition, sort, compact of one batch alone,
// against the passes and the compaction of the radix sort: 34 k IDs 5 + 7 + 14 + 4 us against 54 (without the sample 10.6 + 12
// + 4.8), 297 k 10 + 9 + 19 + 4 against 62.  Beside the class passes the smaller workgroups count as well: the passes of
// tables of one row width leave a SIMD 64 registers (those of tables of several widths next to none, fs_fused.hip), so
// that 512 threads of 64 registers start as soon as one workgroup of theirs ends, where the 1024 threads of a radix pass
// wait for most of a compute unit.  Ten steps of a 4M x 128 table 1040 -> 972 us, of eight tables 5630 -> 5490.
// Ranges of 384 IDs (256 threads) or of 768 (512 threads): the same within 1 %; 1024 threads: 1012 and 5500.
//
// Row popularity is Zipf, so a row can have any share of the batch.  A row that the sample meets often enough to fill
// whole ranges gets a range of its own: boundaries are whole numbers, and a run of equal boundaries v, v, v, v becomes
// v, v + 1, v + 1, v + 1.  The range [v, v + 1) needs no sorting, and the empty ranges behind it help to write it.
// Four samples a range keep the others near the mean: the weight of a range is a sum of four waiting times.  Its workgroup
// holds 4096 IDs, 5.3 times the mean at 768 a range, the most up to 786432 IDs; beyond, the ranges grow to 1024 IDs at 2^20.
// Of 300 batches of a size (Zipf 1.05, 1.1 and 1.2, nearly distinct, 100 rows with 55 % of the occurrences) this many had a
// larger range: none up to 786432 IDs (largest 4032), 3 or 4 of 850 k to 950 k, 12 of 1 M, 29 of 2^20 (largest 5896).  Such a
// range is sorted in memory by its one workgroup: the dedup of 2^20 IDs took 88 to 98 us then, 79 to 82 otherwise, the radix
// sort 82 to 83.  The sample's places are spread by a hash inside their strata, so that a pattern in the batch (sequences of
// one length, say) does not line up with them; a batch made so that the sample misses where its IDs are takes 1.0 ms of 100 k
// IDs, 3.8 ms of 300 k.
//
// A range takes 58 KB of LDS whatever its size (32 KB for keys and places, 24 KB of masks and counters): two workgroups to a
// compute unit alone, one beside the class passes.
#include "fs_common.h"
#include "fs_device.h"

namespace fs {

constexpr int kBucketThreads = 512;                      // sample, sort
constexpr int kBucketWaves = kBucketThreads / kWave;
constexpr int kBucketKpt = 8;                            // most elements of a range a thread sorts
constexpr int kBucketCap = kBucketThreads * kBucketKpt;  // elements of a range that fit the LDS of its workgroup
constexpr int kSamplesLog2 = 2;                          // samples per range
constexpr int kSamplesMost = kMaxBuckets << kSamplesLog2;
constexpr int kSampleThreads = 256;
constexpr int kOwnCutsLog2 = 6;                          // most ranges (log2) whose cuts the partition finds by itself
constexpr int kPartThreads = 256;
constexpr int kPartWaves = kPartThreads / kWave;
constexpr int kPartKpt = kBucketTile / kPartThreads;
constexpr int kRangesPer = kMaxBuckets / kPartThreads;
constexpr int kBucketBits = 8;                           // most bits of a radix pass inside a range
constexpr int kBucketRadix = 1 << kBucketBits;
constexpr int kBucketTiles = (int)(kBucketIdsMax / kBucketTile);
static_assert(kRangesPer * kPartThreads == kMaxBuckets, "whole rounds");
static_assert(kBucketTiles <= kBucketThreads && kBucketRadix <= kBucketThreads, "a thread per tile, a thread per digit");
static_assert(kBucketTile <= 65536, "places inside a tile take 16 bits");

struct bucket_dev_job {
    const int64_t *ids;
    int n, tiles, log2;                                  // IDs, tiles, log2 of the ranges
    int64_t num_rows;
    uint32_t *part_keys;                                 // [n] keys of every tile in the order of its ranges
    uint16_t *part_place;                                // [n] place in its tile of every one of them
    uint16_t *table;                                     // [tiles][ranges] where a range starts in a tile
    uint32_t *cut;                                       // [ranges - 1] every fourth of the sample in order
    int32_t *first, *size, *heads;                       // [ranges] first sorted position, positions, distinct rows
    uint32_t *row_key;                                   // [n] distinct rows of a range, from its first position on
    int32_t *row_seg;                                    // [n] their first positions
    int32_t *rank;                                       // [n] distinct rows of the range up to a position (for the inverse)
    uint32_t *big_key[2];                                // [n] each: a range that does not fit LDS
    int32_t *big_idx[2];
    int64_t *unique;
    int32_t *seg_offsets, *perm, *inverse;
    int64_t *n_unique_dev, *sorted_ids;
    fs_zigzag deal;                                          // order alone: n > 0: dealt to n ranks, whose shares begin at
    int64_t *rank_offsets;                                   // [n + 1]
};
struct bucket_dev_batch {
    bucket_dev_job j[kMaxBatch];
};

template <int WAVES>
struct sort_shared {
    uint64_t mask[WAVES][kBucketRadix];
    uint32_t cnt[WAVES][kBucketRadix];
    uint32_t base[kBucketRadix];
    uint32_t part[kBucketRadix / kWave];
};
typedef sort_shared<kBucketWaves> bucket_sort_shared;

// lanes of my wavefront with my digit (a lane that is not valid has no peers of its own).  All MOST bits, whatever the
// digits use: a bit that is 0 in every lane changes nothing, and a branch around it costs more.
template <int MOST>
__device__ __forceinline__ uint64_t digit_peers(uint32_t digit, bool valid) {
    const uint64_t all = __ballot(valid);
    uint32_t lo = (uint32_t)all, hi = (uint32_t)(all >> 32);
#pragma unroll
    for (int b = 0; b < MOST; ++b) {
        const uint32_t m = (uint32_t)((int)(digit << (31 - b)) >> 31);      // my bit in every position
        const uint64_t bal = __ballot(m != 0);
        lo &= ~((uint32_t)bal ^ m);
        hi &= ~((uint32_t)(bal >> 32) ^ m);
    }
    return (uint64_t)lo | ((uint64_t)hi << 32);
}
__device__ __forceinline__ uint32_t peers_before(uint64_t peers) {
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(peers >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)peers, 0));
}

// Stable sort of the n elements in skey (with their values in sval) by the low `bits` bits of their keys, LSD radix
// passes.  Round r of wavefront w has the 64 elements from (w * KPT + r) * 64 on.  The ranks wait beside the values in
// LDS, so that a pass has keys, values and places of its elements in registers only while they change places.
constexpr int kPlaceBits = 20;
constexpr uint32_t kPlaceMask = (1u << kPlaceBits) - 1u;
static_assert(kBucketIdsMax <= 1ll << kPlaceBits, "a place and a rank share a word");
template <int WAVES>
__device__ __forceinline__ void clear_counters(sort_shared<WAVES> &sh) {
    for (int i = threadIdx.x; i < WAVES * kBucketRadix; i += WAVES * kWave) (&sh.cnt[0][0])[i] = 0u;
}
// The elements of a wavefront with the same digit, in order: every lane sets its bit in the digit's mask, reads the mask
// and clears it again, reads the digit's count and adds itself to it.  A wavefront's LDS accesses are carried out in
// their order, so none of the five waits for another and the rounds follow each other; ballots over the bits of the
// digit cost ten times the instructions.  The mask comes back whole, the count as it stood before the round.
template <int WAVES>
__device__ __forceinline__ void rank_round(sort_shared<WAVES> &sh, int w, uint32_t digit, bool valid, uint64_t &peers,
                                           uint32_t &old) {
    peers = 0;
    old = 0;
    if (valid) {
        uint64_t *m = &sh.mask[w][digit];
        uint32_t *c = &sh.cnt[w][digit];
        (void)__hip_atomic_fetch_or(m, 1ull << (threadIdx.x & (kWave - 1)), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
        wave_lds_order();
        peers = __hip_atomic_load(m, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
        old = __hip_atomic_load(c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
        wave_lds_order();
        __hip_atomic_store(m, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
        (void)__hip_atomic_fetch_add(c, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
    }
    wave_lds_order();
}
template <int KPT, int WAVES>
__device__ __forceinline__ void sort_in_lds(int n, int bits, uint32_t *skey, uint32_t *sval, sort_shared<WAVES> &sh) {
    static_assert(kBucketRadix <= WAVES * kWave, "a thread per digit");
    static_assert(KPT * WAVES * kWave <= 1 << (32 - kPlaceBits), "a place and a rank share a word");
    const int lane = threadIdx.x & (kWave - 1);
    const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave);
    const int e0 = w * (kWave * KPT) + lane;
    const int passes = (bits + kBucketBits - 1) / kBucketBits;
    const int per = (bits + passes - 1) / passes;
    const uint32_t mask = (1u << per) - 1u;
    clear_counters(sh);
    for (int i = threadIdx.x; i < WAVES * kBucketRadix; i += WAVES * kWave) (&sh.mask[0][0])[i] = 0ull;
    for (int pass = 0; pass < passes; ++pass) {
        const int shift = pass * per;
        __syncthreads();
        // G rounds side by side: their loads, then their accesses to the counters, then their ranks
        constexpr int G = KPT < 4 ? KPT : 4;
#pragma unroll 1
        for (int r0 = 0; r0 < KPT; r0 += G) {
            uint32_t digit[G], v[G], old[G];
            uint64_t peers[G];
#pragma unroll
            for (int g = 0; g < G; ++g) {
                const int e = e0 + (r0 + g) * kWave;          // past n: whatever the LDS holds, never used
                digit[g] = (skey[e] >> shift) & mask;
                v[g] = sval[e] & kPlaceMask;
            }
#pragma unroll
            for (int g = 0; g < G; ++g) rank_round(sh, w, digit[g], e0 + (r0 + g) * kWave < n, peers[g], old[g]);
#pragma unroll
            for (int g = 0; g < G; ++g)
                sval[e0 + (r0 + g) * kWave] = v[g] | ((old[g] + peers_before(peers[g])) << kPlaceBits);
        }
        __syncthreads();
        if (threadIdx.x < kBucketRadix) {                     // a digit a thread: prefix over the waves, then over the digits
            uint32_t run = 0;
#pragma unroll
            for (int i = 0; i < WAVES; ++i) {
                const uint32_t v = sh.cnt[i][threadIdx.x];
                sh.cnt[i][threadIdx.x] = run;
                run += v;
            }
            const uint32_t incl = wave_inclusive_scan<uint32_t>(run);
            sh.base[threadIdx.x] = incl - run;
            if (lane == kWave - 1) sh.part[w] = incl;
        }
        __syncthreads();
        uint32_t part[kBucketRadix / kWave];
        part[0] = 0;
#pragma unroll
        for (int i = 1; i < kBucketRadix / kWave; ++i) part[i] = part[i - 1] + sh.part[i - 1];
        uint32_t key[KPT], val[KPT];                          // val: place in the batch, then place to go to
#pragma unroll
        for (int r = 0; r < KPT; ++r) {
            const int e = e0 + r * kWave;
            key[r] = skey[e];
            const uint32_t v = sval[e], digit = (key[r] >> shift) & mask, q = digit / kWave;
            const uint32_t pos = (q == 0 ? part[0] : q == 1 ? part[1] : q == 2 ? part[2] : part[3]) + sh.base[digit] +
                                 sh.cnt[w][digit] + (v >> kPlaceBits);
            val[r] = (v & kPlaceMask) | (pos << kPlaceBits);
        }
        __syncthreads();
        clear_counters(sh);
#pragma unroll
        for (int r = 0; r < KPT; ++r)
            if (e0 + r * kWave < n) {
                skey[val[r] >> kPlaceBits] = key[r];
                sval[val[r] >> kPlaceBits] = val[r];
            }
    }
    __syncthreads();
}

__device__ __forceinline__ void sort_any(int n, int bits, uint32_t *skey, uint32_t *sval, bucket_sort_shared &sh) {
    if (n <= kBucketThreads) sort_in_lds<1>(n, bits, skey, sval, sh);
    else if (n <= 2 * kBucketThreads) sort_in_lds<2>(n, bits, skey, sval, sh);
    else if (n <= 4 * kBucketThreads) sort_in_lds<4>(n, bits, skey, sval, sh);
    else sort_in_lds<kBucketKpt>(n, bits, skey, sval, sh);
}

__device__ __forceinline__ int bits_of(uint32_t x) { return x ? 32 - __builtin_clz(x) : 0; }

// ---- sample ------------------------------------------------------------------------------------------------------
// Place of the i-th of m samples: somewhere in the i-th m-th of the batch.
__device__ __forceinline__ int sample_place(int i, int m_log2, int n) {
    const int a = (int)(((int64_t)i * n) >> m_log2), b = (int)(((int64_t)(i + 1) * n) >> m_log2);
    uint32_t h = (uint32_t)i * 0x9E3779B1u;
    h ^= h >> 15;
    h *= 0x85EBCA77u;
    h ^= h >> 13;
    const int len = b > a ? b - a : 1;
    const int p = a + (int)(((uint64_t)h * (uint32_t)len) >> 32);
    return p < n ? p : n - 1;
}

// One workgroup of 256 threads: beside four workgroups of the batch update a compute unit has registers for one wavefront a
// SIMD, and up to 512 ranges (393216 IDs) this one takes 60.  With 512 threads it waited for one of them to end, and the whole
// index half of a self-contained step behind it (297 k IDs 140.0 -> 138.1 us).  Beyond, with 101 registers and 46 KB of LDS, it
// waits all the same, and is 1.5 us longer alone than with 512 threads (400 k IDs 59.3 -> 60.9).  The sort with 256 threads, in turn with this one: the same step 137.1 / 135.1, but plain operations
// of 34 k IDs 66.6 / 69.9, balancing 65 k samples 86.3 / 88.8, ten pipelined steps of a 64 M row table 1042 / 1051.
template <int MOST>
__global__ __launch_bounds__(kSampleThreads) void bucket_sample_kernel(const bucket_dev_batch batch) {
    FS_WG_TRACE(13);
    const bucket_dev_job &job = batch.j[blockIdx.x];
    if (job.n == 0) return;
    __shared__ uint32_t key[MOST], val[MOST];
    __shared__ sort_shared<kSampleThreads / kWave> sh;
    const int ranges = 1 << job.log2, m_log2 = job.log2 + kSamplesLog2, m = 1 << m_log2;
    const uint32_t last_key = (uint32_t)(job.num_rows - 1);
#pragma unroll 4
    for (int i = threadIdx.x; i < m; i += kSampleThreads) {
        const uint32_t k = (uint32_t)job.ids[sample_place(i, m_log2, job.n)];
        key[i] = k < last_key ? k : last_key;                 // IDs out of range go to the last range, where nobody looks
    }
    __syncthreads();
    const int bits = bits_of(last_key | 1u);
    if (m <= 2 * kSampleThreads) sort_in_lds<2>(m, bits, key, val, sh);
    else if (m <= 4 * kSampleThreads) sort_in_lds<4>(m, bits, key, val, sh);
    else if (m <= 8 * kSampleThreads) sort_in_lds<8>(m, bits, key, val, sh);
    else sort_in_lds<MOST / kSampleThreads>(m, bits, key, val, sh);
    for (int e = threadIdx.x; e < ranges - 1; e += kSampleThreads) job.cut[e] = key[(e + 1) << kSamplesLog2];
}
static_assert(kSamplesMost <= kBucketCap, "sorted like a range");

// First key of the range behind range i: of a run of cuts v, v, v the first is v, the others v + 1.
__device__ __forceinline__ uint32_t bound_at(const uint32_t *__restrict__ cut, int i) {
    const uint32_t v = cut[i];
    return v + ((i > 0 && cut[i - 1] == v) ? 1u : 0u);
}

// number of boundaries i in [0, n) with bound_at(i) < x; one whole wavefront, 64-ary
__device__ __forceinline__ int bounds_below(const uint32_t *__restrict__ cut, int n, uint32_t x) {
    const int lane = threadIdx.x & (kWave - 1);
    int lo = 0, hi = n;
    while (lo < hi) {
        const int step = (hi - lo + kWave - 1) / kWave;
        const int probe = lo + (lane + 1) * step - 1;
        const int cnt = __popcll(__ballot(probe < hi && bound_at(cut, probe) < x));
        lo += cnt * step;
        const int nhi = lo + step - 1;
        hi = nhi < hi ? nhi : hi;
    }
    return lo;
}

// The cuts of a few ranges without a launch of their own: every tile takes the same sample, an entry a thread, and ranks its
// entries by counting (equal ones in their order).  The first tile writes the cuts down for the sort.  With 64 ranges 256
// comparisons a thread of two instructions: plain operations of 34 k IDs 68.7 -> 66.0 us.  With 128 ranges it is four times the
// work, and balancing 65 k samples took 101 us instead of 85.
__device__ __forceinline__ void own_cuts(const bucket_dev_job &job, uint32_t *sample, uint32_t *cut) {
    static_assert(1 << (kOwnCutsLog2 + kSamplesLog2) == kPartThreads, "an entry a thread");
    const int m_log2 = job.log2 + kSamplesLog2, m = 1 << m_log2, i = threadIdx.x;
    const uint32_t last_key = (uint32_t)(job.num_rows - 1);
    const uint32_t x = (uint32_t)job.ids[sample_place(i < m ? i : m - 1, m_log2, job.n)];
    const uint32_t key = x < last_key ? x : last_key;
    sample[i] = i < m ? key : 0xffffffffu;                   // behind every entry, and not below any
    __syncthreads();
    const int w0 = __builtin_amdgcn_readfirstlane(i & ~(kWave - 1));
    uint32_t rank = 0;
    auto count = [&](int from, int to, auto below) {
#pragma unroll 4
        for (int j = from; j < to; j += 4) {
            const u32x4 v = *reinterpret_cast<const u32x4 *>(sample + j);
#pragma unroll
            for (int q = 0; q < 4; ++q) rank += below(v[q], j + q) ? 1u : 0u;
        }
    };
    count(0, w0 < m ? w0 : m, [&](uint32_t v, int) { return v <= key; });
    count(w0, w0 + kWave, [&](uint32_t v, int j) { return v < key || (v == key && j < i); });
    count(w0 + kWave, m, [&](uint32_t v, int) { return v < key; });
    constexpr uint32_t kStep = 1u << kSamplesLog2;
    if (i < m && rank != 0 && rank % kStep == 0) {
        cut[rank / kStep - 1] = key;
        if (blockIdx.x == 0) job.cut[rank / kStep - 1] = key;
    }
    __syncthreads();
}

// ---- partition -----------------------------------------------------------------------------------------------------
// OWN: no sample has been sorted, the tiles find the cuts
template <bool OWN>
__global__ __launch_bounds__(kPartThreads, 8) void bucket_partition_kernel(const bucket_dev_batch batch,
                                                                          int *__restrict__ flags) {
    FS_WG_TRACE(14);
    const bucket_dev_job &job = batch.j[blockIdx.y];
    const int tile = blockIdx.x;
    if (tile >= job.tiles) return;
    extern __shared__ uint32_t lds[];                        // [waves][ranges] 16-bit counters
    __shared__ uint32_t bound[kMaxBuckets], start[kMaxBuckets];
    __shared__ uint32_t wave_sum[kPartWaves];
    __shared__ __align__(16) uint32_t s_key[kBucketTile];
    __shared__ __align__(16) uint16_t s_place[kBucketTile];
    uint16_t *cnt = reinterpret_cast<uint16_t *>(lds);
    const int log2 = job.log2, ranges = 1 << log2;
    const int lane = threadIdx.x & (kWave - 1);
    const int w = threadIdx.x / kWave;
    const int n = job.n, base = tile * kBucketTile, mine = w * (kWave * kPartKpt) + lane;
    const int64_t *__restrict__ ids = job.ids;
    uint32_t key[kPartKpt];
    bool bad = false;
#pragma unroll
    for (int r = 0; r < kPartKpt; ++r) {
        const int e = base + mine + r * kWave;
        const int64_t id = ids[e < n ? e : n - 1];
        bad |= id < 0 || id >= job.num_rows;
        key[r] = (uint32_t)id;
    }
    if constexpr (OWN) {
        own_cuts(job, s_key, start);
        for (int i = threadIdx.x; i < ranges - 1; i += kPartThreads) bound[i] = bound_at(start, i);
    } else {
        for (int i = threadIdx.x; i < ranges - 1; i += kPartThreads) bound[i] = bound_at(job.cut, i);
    }
    for (int i = threadIdx.x; i < (kPartWaves * ranges + 1) / 2; i += kPartThreads) lds[i] = 0u;
    if (bad) atomicOr(flags, kFlagRowRange);
    __syncthreads();
    uint32_t range[kPartKpt];                                // boundaries at or below the key
#pragma unroll
    for (int r = 0; r < kPartKpt; ++r) range[r] = 0;
    for (int step = ranges >> 1; step > 0; step >>= 1)
#pragma unroll
        for (int r = 0; r < kPartKpt; ++r) range[r] += bound[range[r] + step - 1] <= key[r] ? step : 0;
    uint32_t rank[kPartKpt];
#pragma unroll
    for (int r = 0; r < kPartKpt; ++r) {
        const bool valid = base + mine + r * kWave < n;
        const uint64_t peers = digit_peers<10>(range[r], valid);
        const uint32_t before = peers_before(peers);
        uint16_t *c = cnt + w * ranges + range[r];
        const uint32_t old = valid ? *c : 0u;                // all peers read ...
        wave_lds_order();
        if (valid && before == 0) *c = (uint16_t)(old + (uint32_t)__popcll(peers));      // ... then the first writes
        wave_lds_order();
        rank[r] = old + before;
    }
    __syncthreads();
    {
        // thread t has the ranges from per * t on: prefix over the waves, then over the ranges
        const int per = ranges > kPartThreads ? ranges / kPartThreads : 1, d0 = (int)threadIdx.x * per;
        uint32_t sum[kRangesPer], all = 0;
#pragma unroll
        for (int q = 0; q < kRangesPer; ++q) {
            sum[q] = all;
            if (q < per && d0 + q < ranges) {
                uint32_t run = 0;
#pragma unroll
                for (int i = 0; i < kPartWaves; ++i) {
                    uint16_t *c = cnt + i * ranges + d0 + q;
                    const uint32_t v = *c;
                    *c = (uint16_t)run;
                    run += v;
                }
                all += run;
            }
        }
        const uint32_t incl = wave_inclusive_scan<uint32_t>(all);
        if (lane == kWave - 1) wave_sum[w] = incl;
        __syncthreads();
        uint32_t before = incl - all;
#pragma unroll
        for (int i = 0; i < kPartWaves; ++i) before += i < w ? wave_sum[i] : 0u;
#pragma unroll
        for (int q = 0; q < kRangesPer; ++q)
            if (q < per && d0 + q < ranges) {
                start[d0 + q] = before + sum[q];
                job.table[(int64_t)tile * ranges + d0 + q] = (uint16_t)(before + sum[q]);
            }
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kPartKpt; ++r)
        if (base + mine + r * kWave < n) {
            const uint32_t pos = start[range[r]] + cnt[w * ranges + range[r]] + rank[r];
            s_key[pos] = key[r];
            s_place[pos] = (uint16_t)(mine + r * kWave);
        }
    __syncthreads();
    const int span = n - base < kBucketTile ? n - base : kBucketTile;
    if (span == kBucketTile) {
        static_assert(kPartKpt == 8, "sixteen bytes of places a thread");
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int q = (h * kPartThreads + threadIdx.x) * 4;
            *reinterpret_cast<u32x4 *>(job.part_keys + base + q) = *reinterpret_cast<const u32x4 *>(s_key + q);
        }
        const int q = threadIdx.x * 8;
        *reinterpret_cast<u32x4 *>(job.part_place + base + q) = *reinterpret_cast<const u32x4 *>(s_place + q);
    } else {
        for (int q = threadIdx.x; q < span; q += kPartThreads) {
            job.part_keys[base + q] = s_key[q];
            job.part_place[base + q] = s_place[q];
        }
    }
}

// ---- sort ----------------------------------------------------------------------------------------------------------
// the pieces of a range in the tiles, one after the other
struct range_pieces {
    const uint32_t *before;                                  // [tiles + 1] elements of the range before a tile
    const uint32_t *at;                                      // [tiles] where its elements in the tile start
    int tiles, steps;                                        // steps of a binary search over the tiles
    // places of elements i, i + step, ... of the range in part_keys, and their tiles: the searches side by side
    template <int N>
    __device__ __forceinline__ void places(uint32_t i, uint32_t step, uint32_t (&place)[N], int (&tile)[N]) const {
#pragma unroll
        for (int k = 0; k < N; ++k) tile[k] = 0;             // the last tile with before[tile] <= i
        for (int s = steps; s > 0; s >>= 1)
#pragma unroll
            for (int k = 0; k < N; ++k) {
                const int t = tile[k] + s;
                tile[k] = t < tiles && before[t < tiles ? t : 0] <= i + (uint32_t)k * step ? t : tile[k];
            }
#pragma unroll
        for (int k = 0; k < N; ++k) place[k] = at[tile[k]] + (i + (uint32_t)k * step - before[tile[k]]);
    }
};

// exclusive scan over the workgroup, total in every thread; contains two barriers
__device__ __forceinline__ uint32_t wide_exclusive_scan(uint32_t v, uint32_t *sh, uint32_t &total) {
    const int lane = threadIdx.x & (kWave - 1);
    const int w = threadIdx.x / kWave;
    const uint32_t inc = wave_inclusive_scan<uint32_t>(v);
    if (lane == kWave - 1) sh[w] = inc;
    __syncthreads();
    uint32_t base = 0, tot = 0;
#pragma unroll
    for (int i = 0; i < kBucketWaves; ++i) {
        const uint32_t x = sh[i];
        base += i < w ? x : 0u;
        tot += x;
    }
    __syncthreads();
    total = tot;
    return base + inc - v;
}

// where the occurrence of a sorted position goes, where the order alone is wanted
__device__ __forceinline__ uint32_t place_in_order(const bucket_dev_job &job, int p) {
    return job.deal.n > 0 ? job.deal.place32((uint32_t)p) : (uint32_t)p;
}

// one position of the sorted batch
__device__ __forceinline__ void emit(const bucket_dev_job &job, int first, int i, uint32_t key, uint32_t occurrence, bool head,
                                     int heads_before) {
    const int p = first + i;
    if (head) {
        job.row_key[first + heads_before] = key;
        job.row_seg[first + heads_before] = p;
    }
    job.perm[p] = (int32_t)occurrence;
    if (job.inverse != nullptr) job.rank[p] = heads_before + (head ? 1 : 0);
    if (job.sorted_ids != nullptr) job.sorted_ids[p] = (int64_t)key;
}

// A range that does not fit LDS: the same radix passes between two buffers in memory, a workgroup's width at a time.
template <bool ORDER>
__device__ __forceinline__ int sort_in_memory(const bucket_dev_job &job, const range_pieces &pieces, int first, int size,
                                              uint32_t lo, int bits, bucket_sort_shared &sh, uint32_t *wave_sum) {
    const int w = threadIdx.x / kWave;
    const int passes = (bits + kBucketBits - 1) / kBucketBits;
    const int per = (bits + passes - 1) / passes;
    const uint32_t mask = (1u << per) - 1u;
    int src = passes & 1;                                    // an odd number of passes starts in buffer 1: all end in 0
    for (int i = threadIdx.x; i < size; i += kBucketThreads) {
        int tile[1];
        uint32_t at[1];
        pieces.places<1>((uint32_t)i, 0u, at, tile);
        job.big_key[src][first + i] = job.part_keys[at[0]] - lo;
        job.big_idx[src][first + i] = tile[0] * kBucketTile + job.part_place[at[0]];
    }
    for (int pass = 0; pass < passes; ++pass, src ^= 1) {
        const uint32_t *ki = job.big_key[src] + first;
        const int32_t *vi = job.big_idx[src] + first;
        uint32_t *ko = job.big_key[src ^ 1] + first;
        int32_t *vo = job.big_idx[src ^ 1] + first;
        const int shift = pass * per;
        __syncthreads();
        const bool owner = threadIdx.x < kBucketRadix;        // a digit a thread
        if (owner) sh.base[threadIdx.x] = 0;
        clear_counters(sh);
        __syncthreads();
        for (int i = threadIdx.x; i < size; i += kBucketThreads) atomicAdd(&sh.base[(ki[i] >> shift) & mask], 1u);
        __syncthreads();
        uint32_t total;
        const uint32_t start = wide_exclusive_scan(owner ? sh.base[threadIdx.x] : 0u, wave_sum, total);
        if (owner) sh.base[threadIdx.x] = start;
        __syncthreads();
        for (int c0 = 0; c0 < size; c0 += kBucketThreads) {
            const int i = c0 + threadIdx.x;
            const bool valid = i < size;
            const uint32_t key = valid ? ki[i] : 0u;
            const int32_t val = valid ? vi[i] : 0;
            const uint32_t digit = (key >> shift) & mask;
            const uint64_t peers = digit_peers<kBucketBits>(digit, valid);
            const uint32_t before = peers_before(peers);
            if (valid && before == 0) sh.cnt[w][digit] = (uint32_t)__popcll(peers);
            __syncthreads();
            uint32_t run = 0;
            for (int q = 0; owner && q < kBucketWaves; ++q) {
                const uint32_t v = sh.cnt[q][threadIdx.x];
                sh.cnt[q][threadIdx.x] = run;
                run += v;
            }
            __syncthreads();
            if (valid) {
                const uint32_t pos = sh.base[digit] + sh.cnt[w][digit] + before;
                ko[pos] = key;
                vo[pos] = val;
            }
            __syncthreads();
            if (owner) sh.base[threadIdx.x] += run;
            for (int q = 0; owner && q < kBucketWaves; ++q) sh.cnt[q][threadIdx.x] = 0;
            __syncthreads();
        }
    }
    __syncthreads();
    if constexpr (ORDER) {
        for (int i = threadIdx.x; i < size; i += kBucketThreads) job.perm[place_in_order(job, first + i)] = job.big_idx[0][first + i];
        return 0;
    }
    uint32_t heads = 0;                                      // buffer 0 holds the result; its places are perm itself
    const uint32_t *k0 = job.big_key[0] + first;
    const int32_t *v0 = job.big_idx[0] + first;
    for (int c0 = 0; c0 < size; c0 += kBucketThreads) {
        const int i = c0 + threadIdx.x;
        const bool valid = i < size;
        const uint32_t key = valid ? k0[i] : 0u;
        const uint32_t val = valid ? (uint32_t)v0[i] : 0u;
        const bool head = valid && (i == 0 || k0[i - 1] != key);
        uint32_t total;
        const uint32_t before = wide_exclusive_scan(head ? 1u : 0u, wave_sum, total);
        if (valid) emit(job, first, i, key + lo, val, head, (int)(heads + before));
        heads += total;
    }
    return (int)heads;
}

// ORDER: of every job the order alone is wanted (a kernel of its own: the deal costs registers)
template <bool ORDER>
__global__ __launch_bounds__(kBucketThreads, 8) void bucket_sort_kernel(const bucket_dev_batch batch) {
    FS_WG_TRACE(15);
    const bucket_dev_job &job = batch.j[blockIdx.y];
    const int ranges = 1 << job.log2;
    // neighbouring ranges read neighbouring pieces of every tile: they go to one XCD
    const int e = ranges >= 8 ? ((int)blockIdx.x & 7) * (ranges >> 3) + ((int)blockIdx.x >> 3) : (int)blockIdx.x;
    if ((int)blockIdx.x >= ranges) return;
    extern __shared__ uint32_t lds[];
    uint32_t *skey = lds, *sval = lds + kBucketCap;
    __shared__ union {
        bucket_sort_shared sort;
        uint32_t pieces[2 * kBucketTiles + 1];
    } sh;
    __shared__ uint32_t wave_sum[kBucketWaves], wave_below[kBucketWaves];
    const int n = job.n, tiles = job.tiles;
    const int lane = threadIdx.x & (kWave - 1);
    const int w = threadIdx.x / kWave;
    if (ORDER && job.deal.n > 0)
        for (int64_t i = (int64_t)blockIdx.x * kBucketThreads + threadIdx.x; i <= job.deal.n; i += (int64_t)ranges * kBucketThreads)
            job.rank_offsets[i] = job.deal.rank_start(i);
    // boundaries, what there is to do, and the table's columns: one round of loads unless this range helps another
    uint32_t lo = e > 0 ? bound_at(job.cut, e - 1) : 0u;
    const uint32_t hi = e < ranges - 1 ? bound_at(job.cut, e) : (uint32_t)job.num_rows;
    uint32_t a, b;
    auto column = [&](int range) {
        a = b = 0;
        const int t = threadIdx.x;
        if (t < tiles) {
            const uint16_t *row = job.table + (int64_t)t * ranges;
            const int left = n - t * kBucketTile;
            a = row[range];
            b = range + 1 < ranges ? row[range + 1] : (uint32_t)(left < kBucketTile ? left : kBucketTile);
        }
    };
    column(e);
    // a range of one key, [v, v + 1), or an empty one behind it that helps: part `part` of `parts` of range `of`
    int of = e, part = 0, parts = 1;
    const bool one_key = e > 0 && e < ranges - 1 && hi - lo <= 1u;
    if (one_key) {
        of = bounds_below(job.cut, ranges - 1, hi);
        parts = bounds_below(job.cut, ranges - 1, hi + 1u) - of;
        part = e - of;
        if (of != e) column(of);
    }
    uint32_t *before = sh.pieces, *at = sh.pieces + kBucketTiles + 1;
    // where the pieces start in the range, and what the tiles hold of the ranges before it
    const uint32_t incl = wave_inclusive_scan<uint32_t>(b - a), incl_below = wave_inclusive_scan<uint32_t>(a);
    if (lane == kWave - 1) {
        wave_sum[w] = incl;
        wave_below[w] = incl_below;
    }
    __syncthreads();
    uint32_t run = incl - (b - a), all = 0, first32 = 0;
#pragma unroll
    for (int i = 0; i < kBucketWaves; ++i) {
        run += i < w ? wave_sum[i] : 0u;
        all += wave_sum[i];
        first32 += wave_below[i];
    }
    if ((int)threadIdx.x < tiles) {
        before[threadIdx.x] = run;
        at[threadIdx.x] = threadIdx.x * kBucketTile + a;
    }
    __syncthreads();
    int steps = 1;
    while (steps * 2 < tiles) steps *= 2;
    const range_pieces pieces = {before, at, tiles, steps};
    const int size = (int)all;
    const int first = (int)first32;
    // a range of one key is in order already, and the empty ranges behind it write their share of it
    if (one_key) {
        if (of != e) lo = lo - 1;                            // the boundary is v + 1 here
        const int i0 = (int)((int64_t)size * part / parts), i1 = (int)((int64_t)size * (part + 1) / parts);
        for (int i = i0 + threadIdx.x; i < i1; i += 4 * kBucketThreads) {
            int tile[4];
            uint32_t q[4], place[4];
            pieces.places<4>((uint32_t)i, kBucketThreads, q, tile);
#pragma unroll
            for (int k = 0; k < 4; ++k) place[k] = i + k * kBucketThreads < i1 ? job.part_place[q[k]] : 0u;
#pragma unroll
            for (int k = 0; k < 4; ++k)
                if (i + k * kBucketThreads < i1) {
                    const int p = first + i + k * kBucketThreads;
                    job.perm[ORDER ? place_in_order(job, p) : (uint32_t)p] = tile[k] * kBucketTile + (int)place[k];
                    if (job.inverse != nullptr) job.rank[p] = part == 0 ? 1 : 0;
                    if (job.sorted_ids != nullptr) job.sorted_ids[p] = (int64_t)lo;
                }
        }
        if (threadIdx.x == 0 && !ORDER) {
            const bool row = part == 0 && size > 0;
            if (row) {
                job.row_key[first] = lo;
                job.row_seg[first] = first;
            }
            job.first[e] = first + i0;
            job.size[e] = i1 - i0;
            job.heads[e] = row ? 1 : 0;
        }
        return;
    }
    const int bits = bits_of((hi > lo ? hi - 1u - lo : 0u) | 1u);
    int heads;
    if (size <= kBucketCap) {
        for (int i = threadIdx.x; i < size; i += 4 * kBucketThreads) {
            int tile[4];
            uint32_t q[4], key[4], place[4];
            pieces.places<4>((uint32_t)i, kBucketThreads, q, tile);
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const bool in = i + k * kBucketThreads < size;
                key[k] = in ? job.part_keys[q[k]] : 0u;
                place[k] = in ? job.part_place[q[k]] : 0u;
            }
#pragma unroll
            for (int k = 0; k < 4; ++k)
                if (i + k * kBucketThreads < size) {
                    skey[i + k * kBucketThreads] = key[k] - lo;
                    sval[i + k * kBucketThreads] = (uint32_t)(tile[k] * kBucketTile) + place[k];
                }
        }
        __syncthreads();                                     // the list of pieces gives way to the counters
        sort_any(size, bits, skey, sval, sh.sort);
        if constexpr (ORDER) {
            for (int i = threadIdx.x; i < size; i += kBucketThreads)
                job.perm[place_in_order(job, first + i)] = (int32_t)(sval[i] & kPlaceMask);
            return;
        }
        // the distinct rows, numbered: a wavefront has consecutive elements, G rounds side by side
        constexpr int G = 4;
        const int rounds = (size + kBucketThreads - 1) / kBucketThreads;
        const int e0 = w * (kWave * rounds) + lane;
        int found = 0;
        for (int r0 = 0; r0 < rounds; r0 += G) {
#pragma unroll
            for (int g = 0; g < G; ++g) {
                const int i = e0 + (r0 + g) * kWave;
                const bool in = r0 + g < rounds && i < size;
                const uint32_t key = in ? skey[i] : 0u, prev = in && i > 0 ? skey[i - 1] : ~key;
                found += __popcll(__ballot(in && prev != key));
            }
        }
        if (lane == 0) wave_sum[w] = (uint32_t)found;
        __syncthreads();
        int k = 0;
        heads = 0;
#pragma unroll
        for (int i = 0; i < kBucketWaves; ++i) {
            k += i < w ? (int)wave_sum[i] : 0;
            heads += (int)wave_sum[i];
        }
        for (int r0 = 0; r0 < rounds; r0 += G) {
            uint32_t key[G], val[G];
            uint64_t all[G];
            bool in[G];
#pragma unroll
            for (int g = 0; g < G; ++g) {
                const int i = e0 + (r0 + g) * kWave;
                in[g] = r0 + g < rounds && i < size;
                key[g] = in[g] ? skey[i] : 0u;
                val[g] = in[g] ? sval[i] & kPlaceMask : 0u;
                const uint32_t prev = in[g] && i > 0 ? skey[i - 1] : ~key[g];
                all[g] = __ballot(in[g] && prev != key[g]);
            }
#pragma unroll
            for (int g = 0; g < G; ++g) {
                if (in[g])
                    emit(job, first, e0 + (r0 + g) * kWave, key[g] + lo, val[g], ((all[g] >> lane) & 1ull) != 0, k + (int)peers_before(all[g]));
                k += __popcll(all[g]);
            }
        }
    } else {
        // the list of pieces moves out of the way of the counters
        uint32_t *before2 = lds, *at2 = lds + kBucketTiles;
        for (int t = threadIdx.x; t < tiles; t += kBucketThreads) {
            before2[t] = before[t];
            at2[t] = at[t];
        }
        __syncthreads();
        const range_pieces moved = {before2, at2, tiles, steps};
        heads = sort_in_memory<ORDER>(job, moved, first, size, lo, bits, sh.sort, wave_sum);
    }
    if (threadIdx.x == 0 && !ORDER) {
        job.first[e] = first;
        job.size[e] = size;
        job.heads[e] = heads;
    }
}

// ---- compact -------------------------------------------------------------------------------------------------------
__global__ __launch_bounds__(kScanThreads) void bucket_compact_kernel(const bucket_dev_batch batch) {
    FS_WG_TRACE(16);
    const bucket_dev_job &job = batch.j[blockIdx.y];
    const int ranges = 1 << job.log2;
    const int e = blockIdx.x;
    if (e >= ranges) return;
    __shared__ int sh[kScanThreads / kWave];
    const int first = job.first[e], heads = job.heads[e];
    int mine = 0;
    for (int t = threadIdx.x; t < e; t += kScanThreads) mine += job.heads[t];
    int before;
    (void)block_exclusive_scan<int>(mine, sh, before);
    for (int k = threadIdx.x; k < heads; k += kScanThreads) {
        job.unique[before + k] = (int64_t)job.row_key[first + k];
        job.seg_offsets[before + k] = job.row_seg[first + k];
    }
    if (job.inverse != nullptr) {
        const int size = job.size[e];
        for (int i = threadIdx.x; i < size; i += kScanThreads)
            job.inverse[job.perm[first + i]] = before + job.rank[first + i] - 1;
    }
    if (e == ranges - 1 && threadIdx.x == 0) {
        job.seg_offsets[before + heads] = job.n;
        *job.n_unique_dev = before + heads;
    }
}

// ---- host side -----------------------------------------------------------------------------------------------------
size_t bucket_table_size(int64_t max_ids) {
    const int64_t n = max_ids < kBucketIdsMax ? max_ids : kBucketIdsMax;
    return (size_t)ceil_div(n, kBucketTile) << ranges_log2(n);
}

int launch_bucket_unique(fs_ctx *ctx, int count, const fs_unique_job *jobs, hipStream_t s, int set0) {
    bucket_dev_batch batch;
    memset(&batch, 0, sizeof(batch));
    int tiles = 0, log2 = 0;
    bool dedup = false;                                      // else the order alone is wanted of every job
    for (int k = 0; k < count; ++k) {
        const fs_unique_job &in = jobs[k];
        const fs_sort_scratch &ws = ctx->sort[set0 + k];
        bucket_dev_job &j = batch.j[k];
        j.ids = in.ids; j.n = (int)in.n; j.num_rows = in.num_rows;
        j.tiles = (int)ceil_div(in.n, kBucketTile);
        j.log2 = ranges_log2(in.n);
        uint32_t *k0 = reinterpret_cast<uint32_t *>(ws.keys[0]), *k1 = reinterpret_cast<uint32_t *>(ws.keys[1]);
        j.part_keys = k0;
        j.row_seg = reinterpret_cast<int32_t *>(k0 + ctx->max_ids);
        j.part_place = reinterpret_cast<uint16_t *>(ws.idx[0]);
        j.table = ws.range_start;
        j.cut = ws.ranges;
        j.first = reinterpret_cast<int32_t *>(ws.ranges + kMaxBuckets);
        j.size = j.first + kMaxBuckets; j.heads = j.size + kMaxBuckets;
        j.row_key = k1;
        j.rank = ws.idx[1];
        // a range sorted in memory ends in buffer 0: keys beside the list of its rows, places where they belong
        j.big_key[0] = k1 + ctx->max_ids; j.big_key[1] = k1;
        // (dealt, they are spread over the output, and the list of first positions is not made)
        j.big_idx[0] = in.deal > 0 ? j.row_seg : in.perm; j.big_idx[1] = ws.idx[1];
        if (in.deal > 0) j.deal = fs_zigzag{in.deal, in.n / in.deal, in.n % in.deal};
        j.rank_offsets = in.rank_offsets;
        dedup = dedup || !in.order_only;
        j.unique = in.unique; j.seg_offsets = in.seg_offsets; j.perm = in.perm; j.inverse = in.inverse;
        j.n_unique_dev = in.n_unique_dev; j.sorted_ids = in.sorted_ids;
        tiles = j.tiles > tiles ? j.tiles : tiles;
        log2 = j.log2 > log2 ? j.log2 : log2;
    }
    // all batches of a launch are small: one launch less
    const bool own = log2 <= kOwnCutsLog2;
    const unsigned ranges = 1u << log2;
    const size_t part_lds = (size_t)kPartWaves * ranges * sizeof(uint16_t);
    if (!own)
        hipLaunchKernelGGL(log2 < 10 ? &bucket_sample_kernel<kSamplesMost / 2> : &bucket_sample_kernel<kSamplesMost>,
                           dim3((unsigned)count), dim3(kSampleThreads), 0, s, batch);
    if (tiles > 0)
        hipLaunchKernelGGL(own ? &bucket_partition_kernel<true> : &bucket_partition_kernel<false>,
                           dim3((unsigned)tiles, (unsigned)count), dim3(kPartThreads), part_lds, s, batch, ctx->d_flags);
    auto *sort = dedup ? &bucket_sort_kernel<false> : &bucket_sort_kernel<true>;
    hipLaunchKernelGGL(sort, dim3(ranges, (unsigned)count), dim3(kBucketThreads), 2 * kBucketCap * sizeof(uint32_t), s, batch);
    if (dedup)
        hipLaunchKernelGGL(bucket_compact_kernel, dim3(ranges, (unsigned)count), dim3(kScanThreads), 0, s, batch);
    FS_LAUNCH_CHECK(ctx, "bucket kernels");
    return FS_OK;
}

FS_TRACE_SETTER(bucket)

}  // namespace fs
