// compute_collision(I^i, I^{i+1}) of Algorithm 2 on ascending distinct row lists:
//   co = U_t & U_t1, ex = U_t \ U_t1, ex_next = U_t1 \ U_t, each ascending, each with the slot of
//   the row in its source list (the slot addresses the reduced-gradient row).
// Sorted-merge intersect by tiles: a tile of 1024 elements of one list only needs the window of
// the other list between its first and last element.  Two wavefronts find that window with a
// 64-ary search each, the workgroup stages it in LDS and every element binary-searches LDS (global
// binary search only if the window does not fit).  Membership flags are counted per tile and a
// second launch compacts with tile prefixes, the class order and the records of batch t with it where they are wanted.  Bound by dependent rounds, not bytes: the tile's own keys travel while the
// window is searched, the two ends are searched at once, and a thread's four keys take their steps through LDS side by
// side (the class order's positions and what their rows are likewise).  Plain operations of 34 k IDs 82.3 -> 80.5 us,
// self-contained step of 297 k 148.6 -> 146.4 against one search, one key and one position after the other.
// The list lengths are device scalars; the launch is sized by the host-side caps and tiles past the end do nothing.
#include <mutex>

#include "fs_common.h"
#include "fs_device.h"

namespace fs {

constexpr int kSplitWindow = 4096;       // elements of the other list staged in LDS (32 KB)

// number of elements of a[0, n) that are < key; executed by one whole wavefront (64-ary search)
__device__ __forceinline__ int wave_lower_bound(const int64_t *__restrict__ a, int n, int64_t key) {
    const int lane = threadIdx.x & (kWave - 1);
    int lo = 0, hi = n;                      // a[i] < key for i < lo, a[i] >= key for i >= hi
    while (lo < hi) {
        const int step = (hi - lo + kWave - 1) / kWave;
        const int probe = lo + (lane + 1) * step - 1;          // last element of my sub-block
        const bool less = (probe < hi) && (a[probe] < key);
        const int cnt = __popcll(__ballot(less));
        lo += cnt * step;
        const int nhi = lo + step - 1;
        hi = nhi < hi ? nhi : hi;
    }
    return lo;
}

__device__ __forceinline__ bool sorted_contains(const int64_t *__restrict__ a, int lo, int hi, int64_t key) {
    const int end = hi;
    while (lo < hi) {                        // first index with a[i] >= key
        const int mid = (lo + hi) >> 1;
        if (a[mid] < key) lo = mid + 1; else hi = mid;
    }
    return lo < end && a[lo] == key;
}

__device__ __forceinline__ int clamp_count(const int64_t *dev, int64_t cap) {
    if (dev == nullptr) return 0;
    int64_t v = *dev;
    if (v < 0) v = 0;
    if (v > cap) v = cap;
    return (int)v;
}

// One collision split + class order of a batch that shares its launches (blockIdx.y picks the job), as
// the kernels see it.
struct split_dev_job {
    const int64_t *u_t, *n_t_dev, *u_t1, *n_t1_dev;
    int64_t cap_t, cap_t1;
    int tiles_t, tiles_t1;        // tiles_t is at least 1: an empty U_t still has its counts written
    uint8_t *flag_t, *flag_t1;
    int32_t *tile_cnt;
    int64_t *co;
    int32_t *co_slot;
    int64_t *ex;
    int32_t *ex_slot;
    int64_t *ex_next;
    int32_t *ex_next_slot;
    int64_t *counts_dev;
    const int32_t *seg_offsets_t;
    int32_t *cstart_local, *tile_len, *cidx;
};
struct split_dev_batch {
    split_dev_job j[kMaxBatch];
};
// ... and what the class order takes and writes on top of it
struct class_dev_job {
    const int32_t *perm;
    const int64_t *n_unique_dev;
    int n, blocks;                // blocks is at least 1: an empty batch still has its counts and class extents written
    int32_t *cperm, *cslot, *cstart, *class_pos_dev, *short_rec;
};
struct class_dev_batch {
    split_dev_job split[kMaxBatch];
    class_dev_job cls[kMaxBatch];
};

constexpr int kRowIsCo = 1 << 16;        // of cidx; below it the place among the rows of the class in the tile
static_assert(kScanTile <= kRowIsCo, "a place in a tile");

// blocks [0, tiles_t) flag U_t against U_t1; blocks [tiles_t, tiles_t + tiles_t1) flag U_t1 against U_t
// CLASSES: with a class order (a kernel of its own: the split alone is over 0.8 us sooner without that code)
template <bool CLASSES>
__global__ __launch_bounds__(kScanThreads) void split_flag_kernel(const split_dev_batch batch, int *__restrict__ flags) {
    FS_WG_TRACE(5);
    const split_dev_job &job = batch.j[blockIdx.y];
    if ((int)blockIdx.x >= job.tiles_t + job.tiles_t1) return;
    const int64_t *__restrict__ u_t = job.u_t, *__restrict__ u_t1 = job.u_t1;
    const int64_t *__restrict__ n_t_dev = job.n_t_dev, *__restrict__ n_t1_dev = job.n_t1_dev;
    const int64_t cap_t = job.cap_t, cap_t1 = job.cap_t1;
    const int tiles_t = job.tiles_t;
    uint8_t *__restrict__ flag_t = job.flag_t, *__restrict__ flag_t1 = job.flag_t1;
    int32_t *__restrict__ tile_cnt = job.tile_cnt;
    __shared__ int sh[kScanThreads / kWave];
    __shared__ int win[2];
    __shared__ int64_t window[kSplitWindow];
    const int n_t = clamp_count(n_t_dev, cap_t), n_t1 = clamp_count(n_t1_dev, cap_t1);
    const bool side_t = (int)blockIdx.x < tiles_t;
    const int tile = side_t ? blockIdx.x : blockIdx.x - tiles_t;
    const int64_t *mine = side_t ? u_t : u_t1;
    const int64_t *other = side_t ? u_t1 : u_t;
    const int n_mine = side_t ? n_t : n_t1, n_other = side_t ? n_t1 : n_t;
    uint8_t *flag = side_t ? flag_t : flag_t1;
    const int t_lo = tile * kScanTile;
    if (t_lo >= n_mine) {                                    // whole workgroup: tile past the end
        if (threadIdx.x == 0) {
            tile_cnt[blockIdx.x] = 0;
            if (CLASSES && side_t) job.tile_len[tile] = job.tile_len[tiles_t + tile] = 0;
        }
        return;
    }
    const int t_hi = (t_lo + kScanTile < n_mine) ? t_lo + kScanTile : n_mine;
    const int p0 = t_lo + threadIdx.x * kScanIpt, w = threadIdx.x / kWave;
    int64_t key[kScanIpt];                                   // under way while the window is looked for
#pragma unroll
    for (int i = 0; i < kScanIpt; ++i) key[i] = p0 + i < t_hi ? mine[p0 + i] : 0;
    if (w < 2) {
        // upper end: the entries <= the tile's last element (a search for "last + 1" would wrap around at the
        // top of the ID range, which is legal when the table size is not given)
        const int j = w == 0 ? wave_lower_bound(other, n_other, mine[t_lo])
                             : wave_upper_bound<int64_t>(other, n_other, mine[t_hi - 1]);
        if ((threadIdx.x & (kWave - 1)) == 0) win[w] = j;
    }
    __syncthreads();
    const int j0 = win[0], j1 = win[1], in_win = j1 - j0;
    const bool staged = in_win <= kSplitWindow;
    if (staged)
        for (int i = threadIdx.x; i < in_win; i += kScanThreads) window[i] = other[j0 + i];
    __syncthreads();
    bool f[kScanIpt];
    if (staged) {
        int at[kScanIpt];                                    // entries of the window below the key
#pragma unroll
        for (int i = 0; i < kScanIpt; ++i) at[i] = 0;
        for (int step = in_win > 0 ? 1 << (31 - __builtin_clz(in_win)) : 0; step > 0; step >>= 1)
#pragma unroll
            for (int i = 0; i < kScanIpt; ++i) {
                const int q = at[i] + step;
                at[i] = q <= in_win && window[q <= in_win ? q - 1 : 0] < key[i] ? q : at[i];
            }
#pragma unroll
        for (int i = 0; i < kScanIpt; ++i) f[i] = at[i] < in_win && window[at[i] < in_win ? at[i] : 0] == key[i];
    } else {
#pragma unroll
        for (int i = 0; i < kScanIpt; ++i) f[i] = p0 + i < t_hi && sorted_contains(other, j0, j1, key[i]);
    }
    int found = 0;
#pragma unroll
    for (int i = 0; i < kScanIpt; ++i)
        if (p0 + i < t_hi) {
            if (!CLASSES || !side_t) flag[p0 + i] = f[i] ? 1 : 0;
            found += f[i] ? 1 : 0;
        }
    int total;
    const int found_before = block_exclusive_scan<int>(found, sh, total);
    if (threadIdx.x == 0) tile_cnt[blockIdx.x] = total;      // number of collisions in this tile
    if (!CLASSES || !side_t) return;
    // For the class order: the class and the place of every row among the rows of its class in this tile; for the rows with
    // more than FS_SHORT_SEGMENT occurrences those of the same-class rows that precede it in the tile, and the tile's
    // totals of them.
    const int32_t *__restrict__ seg_offsets_t = job.seg_offsets_t;
    int len[kScanIpt], co_len = 0, ex_len = 0;
    bool bad = false;                                        // a row without an occurrence
#pragma unroll
    for (int i = 0; i < kScanIpt; ++i) {
        len[i] = p0 + i < t_hi ? seg_offsets_t[p0 + i + 1] - seg_offsets_t[p0 + i] : 0;
        bad |= p0 + i < t_hi && len[i] < 1;
        if (len[i] <= FS_SHORT_SEGMENT) len[i] = 0;          // short segments are not part of the class order
        co_len += f[i] ? len[i] : 0;
        ex_len += f[i] ? 0 : len[i];
    }
    if (bad) atomicOr(flags, kFlagInternal);
    int co_total, ex_total;
    int co_before = block_exclusive_scan<int>(co_len, sh, co_total);
    int ex_before = block_exclusive_scan<int>(ex_len, sh, ex_total);
    int r_found = found_before;
#pragma unroll
    for (int i = 0; i < kScanIpt; ++i) {
        const int p = p0 + i;
        if (p < t_hi) {
            job.cidx[p] = f[i] ? r_found | kRowIsCo : p - t_lo - r_found;
            job.cstart_local[p] = f[i] ? co_before : ex_before;
        }
        r_found += f[i] ? 1 : 0;
        co_before += f[i] ? len[i] : 0;
        ex_before += f[i] ? 0 : len[i];
    }
    if (threadIdx.x == 0) {
        job.tile_len[tile] = co_total;
        job.tile_len[tiles_t + tile] = ex_total;
    }
}

// The rows of tile `tile` of U_t1 (n_t1 rows) that are not in U_t; `before`: collisions in the tiles before it.
__device__ __forceinline__ void list_ex_next(const split_dev_job &job, int n_t1, int tile, int before, int *sh) {
    const int p0 = tile * kScanTile + threadIdx.x * kScanIpt;
    bool f[kScanIpt];
    int found = 0;
#pragma unroll
    for (int i = 0; i < kScanIpt; ++i) {
        f[i] = p0 + i < n_t1 && job.flag_t1[p0 + i] != 0;
        found += f[i] ? 1 : 0;
    }
    int total;
    int r_found = before + block_exclusive_scan<int>(found, sh, total);
#pragma unroll
    for (int i = 0; i < kScanIpt; ++i) {
        const int p = p0 + i;
        if (p < n_t1 && !f[i]) {
            job.ex_next[p - r_found] = job.u_t1[p];
            job.ex_next_slot[p - r_found] = p;
        }
        r_found += f[i] ? 1 : 0;
    }
}

// The rows of tile `tile` of U_t (n_t rows), each in the list of its class; `before`: collisions in the tiles before it.
__device__ __forceinline__ void list_classes(const split_dev_job &job, int n_t, int tile, int before) {
#pragma unroll
    for (int i = 0; i < kScanIpt; ++i) {
        const int p = tile * kScanTile + i * kScanThreads + threadIdx.x;
        if (p < n_t) {
            const int at = job.cidx[p];
            const bool is_co = (at & kRowIsCo) != 0;
            const int li = (at & (kRowIsCo - 1)) + (is_co ? before : tile * kScanTile - before);
            (is_co ? job.co : job.ex)[li] = job.u_t[p];
            (is_co ? job.co_slot : job.ex_slot)[li] = p;
        }
    }
}

// collisions in the tiles of a side before `tile`
__device__ __forceinline__ int collisions_before(const int32_t *__restrict__ tile_cnt, int tile, int *sh) {
    int before = 0;
    for (int t = threadIdx.x; t < tile; t += kScanThreads) before += tile_cnt[t];
    int total;
    (void)block_exclusive_scan<int>(before, sh, total);
    return total;
}

// The lists of a split without a class order (with one, the launch that makes it writes them).
__global__ __launch_bounds__(kScanThreads) void split_compact_kernel(const split_dev_batch batch) {
    FS_WG_TRACE(6);
    const split_dev_job &job = batch.j[blockIdx.y];
    if ((int)blockIdx.x >= job.tiles_t + job.tiles_t1) return;
    __shared__ int sh[kScanThreads / kWave];
    const int n_t = clamp_count(job.n_t_dev, job.cap_t), n_t1 = clamp_count(job.n_t1_dev, job.cap_t1);
    const bool side_t = (int)blockIdx.x < job.tiles_t;
    const int tile = side_t ? blockIdx.x : blockIdx.x - job.tiles_t;
    const int found_before = collisions_before(job.tile_cnt + (side_t ? 0 : job.tiles_t), tile, sh);
    if (!side_t) {
        list_ex_next(job, n_t1, tile, found_before, sh);
        return;
    }
    const int p0 = tile * kScanTile + threadIdx.x * kScanIpt;
    bool f[kScanIpt];
    int found = 0;
#pragma unroll
    for (int i = 0; i < kScanIpt; ++i) {
        f[i] = p0 + i < n_t && job.flag_t[p0 + i] != 0;
        found += f[i] ? 1 : 0;
    }
    int tile_total;
    int r_found = found_before + block_exclusive_scan<int>(found, sh, tile_total);   // collisions before p0
#pragma unroll
    for (int i = 0; i < kScanIpt; ++i) {
        const int p = p0 + i;
        if (p < n_t) {
            const int64_t id = job.u_t[p];
            if (f[i]) { job.co[r_found] = id; job.co_slot[r_found] = p; }
            else { job.ex[p - r_found] = id; job.ex_slot[p - r_found] = p; }
            r_found += f[i] ? 1 : 0;
        }
    }
    // the last tile of side t knows |co|; |ex| and |ex_next| follow from the list lengths
    if (tile == job.tiles_t - 1 && threadIdx.x == 0) {
        const int n_co = found_before + tile_total;
        job.counts_dev[0] = n_co;
        job.counts_dev[1] = n_t - n_co;
        job.counts_dev[2] = n_t1 - n_co;
    }
}

// The lists, the records and the class order of batch t in one launch.  Records and class order are walked by sorted
// positions: the first position of a row writes the head of its record; every position of a row with at most FS_SHORT_SEGMENT
// occurrences goes to the record, of a longer one to the class order: sorted position q (row slot s, the j-th occurrence of
// that row) to [start of the class] + [occurrences of same-class rows before s] + j.
// The row slot of a sorted position is found in the segment boundaries themselves: a workgroup's 1024 consecutive sorted
// positions touch at most 1024 consecutive rows, whose boundaries it stages in LDS (the inverse map would
// give the same slot at the price of one random 4-byte read per occurrence).  They lie in at most two tiles of rows, so that
// what a workgroup needs of the tiles before them is three sums, taken while it looks for its rows.
// The workgroups behind those of the positions write the lists, a tile of U_t or of U_t1 each: those follow from the two lists
// of rows, whatever the layout (listed by their first positions, the rows of a layout that does not fit its batch came to be
// missing).  A layout whose rows have an occurrence each and lie between 0 and n is a consistent one; what is not is reported
// here and where the lengths are looked at.
// A launch of its own for the lists and the places of the rows cost 6 us of the self-contained step of 297 k IDs.
__global__ __launch_bounds__(kScanThreads) void class_scatter_kernel(const class_dev_batch batch,
                                                                     int *__restrict__ flags) {
    FS_WG_TRACE(7);
    const split_dev_job &job = batch.split[blockIdx.y];
    const class_dev_job &cls = batch.cls[blockIdx.y];
    if ((int)blockIdx.x >= cls.blocks + job.tiles_t + job.tiles_t1) return;
    __shared__ int sh[kScanThreads / kWave];
    if ((int)blockIdx.x >= cls.blocks) {
        int tile = blockIdx.x - cls.blocks;
        const int n_t = clamp_count(job.n_t_dev, job.cap_t), n_t1 = clamp_count(job.n_t1_dev, job.cap_t1);
        // (the launch is sized for occurrences, of which there are several to a row: most of these have nothing to list)
        if (tile < job.tiles_t ? tile * kScanTile >= n_t : (tile - job.tiles_t) * kScanTile >= n_t1) return;
        if (tile < job.tiles_t) {
            list_classes(job, n_t, tile, collisions_before(job.tile_cnt, tile, sh));
        } else {
            tile -= job.tiles_t;
            list_ex_next(job, n_t1, tile, collisions_before(job.tile_cnt + job.tiles_t, tile, sh), sh);
        }
        return;
    }
    const int32_t *__restrict__ perm = cls.perm;
    const int32_t *__restrict__ seg_offsets = job.seg_offsets_t;
    const int n = cls.n, tiles_t = job.tiles_t, cap = (int)job.cap_t;
    const int n_u = clamp_count(cls.n_unique_dev, cap);
    const int32_t *__restrict__ tile_cnt = job.tile_cnt, *__restrict__ tile_len = job.tile_len;
    const int64_t *__restrict__ u_t = job.u_t;
    __shared__ int sums[5][kScanThreads / kWave];
    __shared__ int32_t seg_win[kScanTile + 2];              // seg_offsets[slot_a .. slot_b + 1]
    __shared__ int win[2];
    const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
    const int qa = blockIdx.x * kScanTile;
    const int qb = (qa + kScanTile < n ? qa + kScanTile : n) - 1;          // last sorted position of the workgroup
    const int q0 = qa + threadIdx.x;
    int i[kScanIpt];                                         // under way while the rows are looked for
#pragma unroll
    for (int k = 0; k < kScanIpt; ++k) i[k] = q0 + k * kScanThreads < n ? perm[q0 + k * kScanThreads] : 0;
    // of a tile of rows: collision rows; occurrences of its long collision rows, of its long exclusive rows
    auto of_tile = [&](int t, int (&v)[3]) {
        v[0] = tile_cnt[t];
        v[1] = tile_len[t];
        v[2] = tile_len[tiles_t + t];
    };
    int mine[3] = {0, 0, 0};
    if (n > 0 && (int)threadIdx.x < tiles_t) of_tile(threadIdx.x, mine);
    if (w < 2) {
        // the row of a sorted position q: the last slot whose segment starts at or before q
        int k = 0;
        if (qa < n && n_u > 0) k = wave_upper_bound<int32_t>(seg_offsets, n_u + 1, w == 0 ? qa : qb) - 1;
        k = k < 0 ? 0 : (k > n_u - 1 ? n_u - 1 : k);
        if (lane == 0) win[w] = k;
    }
    __syncthreads();
    const int slot_a = win[0], tile_a = slot_a / kScanTile;
    int wn = (qa < n && n_u > 0) ? win[1] - slot_a + 2 : 0; // boundaries staged
    if (wn > kScanTile + 2 || wn < 0) {                     // cannot happen: every row has an occurrence
        if (threadIdx.x == 0) atomicOr(flags, kFlagInternal);
        wn = 0;
    }
    for (int j = threadIdx.x; j < wn; j += kScanThreads) seg_win[j] = seg_offsets[slot_a + j];
    int next[3] = {0, 0, 0};                                 // tile_a itself: what lies between it and the tile behind it
    if (n > 0) of_tile(tile_a, next);
    int part[5] = {0, 0, 0, 0, 0};                           // before tile_a; all collision rows, all their occurrences
    for (int t = threadIdx.x; n > 0 && t < tiles_t; t += kScanThreads) {
        if (t >= kScanThreads) of_tile(t, mine);
#pragma unroll
        for (int c = 0; c < 3; ++c) part[c] += t < tile_a ? mine[c] : 0;
        part[3] += mine[0];
        part[4] += mine[1];
    }
    int ex_all = 0;                                          // the first workgroup: occurrences of long exclusive rows
    if (blockIdx.x == 0) {
        int x = 0;
        for (int t = threadIdx.x; n > 0 && t < tiles_t; t += kScanThreads) x += tile_len[tiles_t + t];
        (void)block_exclusive_scan<int>(x, sh, ex_all);
    }
#pragma unroll
    for (int c = 0; c < 5; ++c) {
        const int x = wave_inclusive_scan<int>(part[c]);
        if (lane == kWave - 1) sums[c][w] = x;
    }
    __syncthreads();
    int total[5];
#pragma unroll
    for (int c = 0; c < 5; ++c) {
        total[c] = 0;
#pragma unroll
        for (int q = 0; q < kScanThreads / kWave; ++q) total[c] += sums[c][q];
    }
    const int n_co = total[3], n_co_pos = total[4];
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        const int n_t = clamp_count(job.n_t_dev, job.cap_t), n_t1 = clamp_count(job.n_t1_dev, job.cap_t1);
        cls.class_pos_dev[0] = n_co_pos;
        cls.class_pos_dev[1] = n_co_pos + ex_all;
        job.counts_dev[0] = n_co;
        job.counts_dev[1] = n_t - n_co;
        job.counts_dev[2] = n_t1 - n_co;
        if (n > 0 && n_u > 0 && (seg_offsets[0] != 0 || seg_offsets[n_u] != n)) atomicOr(flags, kFlagInternal);
    }
    // the first j with seg_win[j] > q, among the row starts, for all positions side by side
    int s[kScanIpt];
#pragma unroll
    for (int k = 0; k < kScanIpt; ++k) s[k] = 0;
    const int starts = wn - 1;
    for (int step = starts > 0 ? 1 << (31 - __builtin_clz(starts)) : 0; step > 0; step >>= 1)
#pragma unroll
        for (int k = 0; k < kScanIpt; ++k) {
            const int j = s[k] + step;
            s[k] = j <= starts && seg_win[j <= starts ? j - 1 : 0] <= q0 + k * kScanThreads ? j : s[k];
        }
    // what the rows of the positions are, again side by side
    bool ok[kScanIpt];
    int first[kScanIpt], len[kScanIpt], at[kScanIpt], local[kScanIpt];
    int64_t row[kScanIpt];
#pragma unroll
    for (int k = 0; k < kScanIpt; ++k) {
        const int q = q0 + k * kScanThreads;
        s[k] -= 1;                                           // place in the window, -1: before its first row
        ok[k] = q < n && s[k] >= 0 && q < seg_win[s[k] >= 0 ? s[k] + 1 : 0];
        first[k] = ok[k] ? seg_win[s[k]] : 0;
        len[k] = ok[k] ? seg_win[s[k] + 1] - first[k] : 0;
        const int slot = slot_a + s[k];
        at[k] = ok[k] ? job.cidx[slot] : 0;
        row[k] = ok[k] && q == first[k] ? u_t[slot] : 0;
        local[k] = len[k] > FS_SHORT_SEGMENT ? job.cstart_local[slot] : 0;
    }
#pragma unroll
    for (int k = 0; k < kScanIpt; ++k) {
        const int q = q0 + k * kScanThreads;
        if (q < n) {
            const int slot = slot_a + s[k], tile = slot / kScanTile;
            const bool is_co = (at[k] & kRowIsCo) != 0, behind = tile != tile_a;
            // place in the class list: the rows of its class in the tiles before, and in its own
            const int co_before = total[0] + (behind ? next[0] : 0);
            const int li = (at[k] & (kRowIsCo - 1)) + (is_co ? co_before : tile * kScanTile - co_before);
            if (!ok[k] || li < 0 || li >= cap) {             // layout and batch do not fit each other
                atomicOr(flags, kFlagInternal);
                continue;
            }
            // one record per row of the batch, at the row's place in its class list: header (row,
            // slot, occurrences) from the row's first position, occurrences only for short segments
            int32_t *rec = cls.short_rec + ((int64_t)(is_co ? 0 : cap) + li) * kShortRecInts;
            if (q == first[k]) {
                typedef int i32x4 __attribute__((ext_vector_type(4)));
                *reinterpret_cast<i32x4 *>(rec) =
                    i32x4{(int)(row[k] & 0xFFFFFFFFll), (int)(row[k] >> 32), slot, len[k]};
            }
            if (len[k] <= FS_SHORT_SEGMENT) {
                rec[4 + (q - first[k])] = i[k];
                continue;
            }
            const int before = is_co ? total[1] + (behind ? next[1] : 0) : n_co_pos + total[2] + (behind ? next[2] : 0);
            const int dest = before + local[k] + (q - first[k]);
            if (dest < 0 || dest >= n) {                     // cannot happen with a consistent layout and split
                atomicOr(flags, kFlagInternal);
                continue;
            }
            cls.cperm[dest] = i[k];
            cls.cslot[dest] = slot;
            if (q == first[k]) cls.cstart[slot] = dest;
        }
    }
}

__global__ void split_empty_kernel(const int64_t *n_t1_dev, int64_t cap_t1, int64_t *counts_dev) {
    counts_dev[0] = 0;
    counts_dev[1] = 0;
    counts_dev[2] = clamp_count(n_t1_dev, cap_t1);
}

static split_dev_job split_job(const fs_split_job &in, const fs_split_scratch &ws) {
    split_dev_job j;
    const int tiles_t = (int)ceil_div(in.cap_t, kScanTile);
    j.u_t = in.u_t; j.n_t_dev = in.n_t_dev; j.u_t1 = in.u_t1; j.n_t1_dev = in.n_t1_dev;
    j.cap_t = in.cap_t; j.cap_t1 = in.cap_t1;
    // With cap_t == 0 a single (empty) tile on side t keeps the count logic in one place.
    j.tiles_t = tiles_t > 0 ? tiles_t : 1;
    j.tiles_t1 = (int)ceil_div(in.cap_t1, kScanTile);
    j.flag_t = ws.flag_t; j.flag_t1 = in.flag_t1_out ? in.flag_t1_out : ws.flag_t1; j.tile_cnt = ws.cnt;
    j.co = in.co; j.co_slot = in.co_slot; j.ex = in.ex; j.ex_slot = in.ex_slot;
    j.ex_next = in.ex_next; j.ex_next_slot = in.ex_next_slot; j.counts_dev = in.counts_dev;
    j.seg_offsets_t = in.seg_offsets_t;
    j.cstart_local = ws.cstart_local; j.tile_len = ws.tile_len; j.cidx = ws.cidx;
    return j;
}

// one split, without a class order
static int launch_split_alone(fs_ctx *ctx, const fs_split_job &in, hipStream_t s, int set) {
    if (in.cap_t == 0 && in.cap_t1 == 0) {
        hipLaunchKernelGGL(split_empty_kernel, dim3(1), dim3(1), 0, s, in.n_t1_dev, in.cap_t1, in.counts_dev);
        FS_LAUNCH_CHECK(ctx, "split_empty_kernel");
        return FS_OK;
    }
    split_dev_batch batch;
    memset(&batch, 0, sizeof(batch));
    batch.j[0] = split_job(in, ctx->split[set]);
    const dim3 grid((unsigned)(batch.j[0].tiles_t + batch.j[0].tiles_t1), 1u);
    hipLaunchKernelGGL(split_flag_kernel<false>, grid, dim3(kScanThreads), 0, s, batch, ctx->d_flags);
    hipLaunchKernelGGL(split_compact_kernel, grid, dim3(kScanThreads), 0, s, batch);
    FS_LAUNCH_CHECK(ctx, "split kernels");
    return FS_OK;
}

int launch_split(fs_ctx *ctx, const int64_t *u_t, const int64_t *n_t_dev, const int64_t *u_t1,
                 const int64_t *n_t1_dev, int64_t cap_t, int64_t cap_t1, int64_t *co, int32_t *co_slot,
                 int64_t *ex, int32_t *ex_slot, int64_t *ex_next, int32_t *ex_next_slot, int64_t *counts_dev,
                 hipStream_t s) {
    const fs_split_job job = {u_t, n_t_dev, u_t1, n_t1_dev, cap_t, cap_t1, co, co_slot, ex, ex_slot,
                              ex_next, ex_next_slot, counts_dev, nullptr};
    if (small_split_fits(1, &job, nullptr, 0)) return launch_small_index(ctx, 1, nullptr, &job, nullptr, s);
    return launch_split_alone(ctx, job, s, 0);
}

int launch_split_class_batch(fs_ctx *ctx, int count, const fs_split_job *jobs, const fs_class_job *cls, hipStream_t s,
                             int set0) {
    if (small_split_fits(count, jobs, cls, set0)) return launch_small_index(ctx, count, nullptr, jobs, cls, s);
    if (count < 1 || count > kMaxBatch || set0 < 0 || set0 + count > kSortSets)
        return set_err(ctx, FS_EINVAL, "split: batch size");
    split_dev_batch batch;
    class_dev_batch order;
    memset(&batch, 0, sizeof(batch));
    memset(&order, 0, sizeof(order));
    int tiles = 0, blocks = 0;
    for (int k = 0; k < count; ++k) {
        const fs_class_job &in = cls[k];
        class_dev_job &j = order.cls[k];
        const split_dev_job sj = split_job(jobs[k], ctx->split[set0 + k]);
        if (sj.tiles_t > kClassOrderTiles)
            return set_err(ctx, FS_ERANGE, "class order: more than 7.8M distinct rows in one batch");
        batch.j[k] = order.split[k] = sj;
        j.perm = in.perm; j.n_unique_dev = in.n_unique_dev; j.n = (int)in.n;
        j.blocks = in.n > 0 ? (int)ceil_div(in.n, kScanTile) : 1;
        j.cperm = in.cperm; j.cslot = in.cslot; j.cstart = in.cstart; j.class_pos_dev = in.class_pos_dev;
        j.short_rec = in.short_rec;
        tiles = sj.tiles_t + sj.tiles_t1 > tiles ? sj.tiles_t + sj.tiles_t1 : tiles;
        const int mine = j.blocks + sj.tiles_t + sj.tiles_t1;
        blocks = mine > blocks ? mine : blocks;
    }
    hipLaunchKernelGGL(split_flag_kernel<true>, dim3((unsigned)tiles, (unsigned)count), dim3(kScanThreads), 0, s, batch,
                       ctx->d_flags);
    hipLaunchKernelGGL(class_scatter_kernel, dim3((unsigned)blocks, (unsigned)count), dim3(kScanThreads), 0, s, order,
                       ctx->d_flags);
    FS_LAUNCH_CHECK(ctx, "split and class order kernels");
    return FS_OK;
}

FS_TRACE_SETTER(split)

// ---- the collision split for callers that cannot allocate ----------------------------------------------------
// Same two kernels as launch_split_alone; the membership flags and per-tile counts live in a fixed device array
// instead of a context's slab.
constexpr int64_t kStaticSplitRows = FS_STATIC_SPLIT_MAX_ROWS;
constexpr size_t kStaticFlagBytes = ((size_t)kStaticSplitRows + 16 + 255) / 256 * 256;
constexpr size_t kStaticTiles = (size_t)(kStaticSplitRows / kScanTile) + 2;
constexpr size_t kStaticCntBytes = (2 * kStaticTiles * sizeof(int32_t) + 255) / 256 * 256;
constexpr size_t kStaticScratchBytes = 2 * kStaticFlagBytes + kStaticCntBytes;
static_assert(kStaticSplitRows % kScanTile == 0, "whole tiles");

static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

constexpr int kStaticMaxDevices = 64;
static std::mutex g_static_mu;
static unsigned char *g_static_ptr[kStaticMaxDevices];      // device address of `scratch` on each GPU, once asked for

// the address of this GPU's copy of `scratch` (each GPU holds its own); `device` must be current
static hipError_t static_scratch_for(int device, unsigned char **out) {
    std::lock_guard<std::mutex> lk(g_static_mu);
    if (g_static_ptr[device] == nullptr) {
        void *p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (p == nullptr) return hipErrorInvalidSymbol;
        g_static_ptr[device] = static_cast<unsigned char *>(p);
    }
    *out = g_static_ptr[device];
    return hipSuccess;
}

int static_split_prepare(int device) {
    if (device < 0 || device >= kStaticMaxDevices) return FS_EINVAL;
    unsigned char *p = nullptr;
    return static_scratch_for(device, &p) == hipSuccess ? FS_OK : FS_EHIP;
}

}  // namespace fs

extern "C" int fs_collision_split_static(const int64_t *u_t, const int64_t *n_t_dev, const int64_t *u_t1,
                                         const int64_t *n_t1_dev, int64_t cap_t, int64_t cap_t1, int64_t *co,
                                         int32_t *co_slot, int64_t *ex, int32_t *ex_slot, int64_t *ex_next,
                                         int32_t *ex_next_slot, int64_t *counts_dev, fs_stream stream) {
    using namespace fs;
    if (cap_t < 0 || cap_t1 < 0) return set_static_err(FS_EINVAL, "static split: negative capacity");
    if (cap_t > kStaticSplitRows || cap_t1 > kStaticSplitRows)
        return set_static_err(FS_ENOMEM, "static split: a list of more than FS_STATIC_SPLIT_MAX_ROWS rows does not fit "
                                         "the fixed scratch array; use fs_collision_split with a context");
    if (!counts_dev) return set_static_err(FS_EINVAL, "static split: null counts");
    if (cap_t > 0 && !(u_t && n_t_dev && co && co_slot && ex && ex_slot))
        return set_static_err(FS_EINVAL, "static split: null pointer (t side)");
    if (cap_t1 > 0 && !(u_t1 && n_t1_dev && ex_next && ex_next_slot))
        return set_static_err(FS_EINVAL, "static split: null pointer (t+1 side)");
    int device = -1;
    if (hipGetDevice(&device) != hipSuccess || device < 0 || device >= kStaticMaxDevices)
        return set_static_err(FS_EHIP, "static split: no current device");
    unsigned char *base = nullptr;
    const hipError_t se = static_scratch_for(device, &base);
    if (se != hipSuccess) return set_static_err(FS_EHIP, hipGetErrorString(se));
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    if (cap_t == 0 && cap_t1 == 0) {
        hipLaunchKernelGGL(split_empty_kernel, dim3(1), dim3(1), 0, s, (const int64_t *)nullptr, (int64_t)0, counts_dev);
    } else {
        // Nothing has to start at zero: the flag launch writes every flag and every per-tile count that the
        // compaction launch reads (tiles past the end of a list write a zero count).
        split_dev_batch batch;
        memset(&batch, 0, sizeof(batch));
        split_dev_job &j = batch.j[0];
        const int tiles_t = (int)ceil_div(cap_t, kScanTile);
        j.u_t = u_t; j.n_t_dev = cap_t > 0 ? n_t_dev : nullptr;
        j.u_t1 = u_t1; j.n_t1_dev = cap_t1 > 0 ? n_t1_dev : nullptr;
        j.cap_t = cap_t; j.cap_t1 = cap_t1;
        j.tiles_t = tiles_t > 0 ? tiles_t : 1;
        j.tiles_t1 = (int)ceil_div(cap_t1, kScanTile);
        j.flag_t = base;
        j.flag_t1 = base + kStaticFlagBytes;
        j.tile_cnt = reinterpret_cast<int32_t *>(base + 2 * kStaticFlagBytes);
        j.co = co; j.co_slot = co_slot; j.ex = ex; j.ex_slot = ex_slot;
        j.ex_next = ex_next; j.ex_next_slot = ex_next_slot; j.counts_dev = counts_dev;
        j.seg_offsets_t = nullptr; j.cstart_local = nullptr; j.tile_len = nullptr; j.cidx = nullptr;
        const dim3 grid((unsigned)(j.tiles_t + j.tiles_t1), 1u);
        hipLaunchKernelGGL(split_flag_kernel<false>, grid, dim3(kScanThreads), 0, s, batch, (int *)nullptr);
        hipLaunchKernelGGL(split_compact_kernel, grid, dim3(kScanThreads), 0, s, batch);
    }
    const hipError_t le = hipGetLastError();
    if (le != hipSuccess) return set_static_err(FS_EHIP, hipGetErrorString(le));
    return FS_OK;
}
