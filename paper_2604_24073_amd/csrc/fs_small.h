// Device code of the index half of a small batch on one workgroup; described in fs_small.hip.
#pragma once

#include "fs_common.h"
#include "fs_device.h"

namespace fs {

constexpr int kSmallThreads = 1024;
constexpr int kSmallWaves = kSmallThreads / kWave;
constexpr int kSmallRadix = 1 << kSmallBits;
static_assert(kSmallIds == kSmallThreads * 16, "KPT is at most 16");

struct small_dedup {
    const int64_t *ids;
    int n, bits, passes;
    int64_t num_rows;
    int64_t *unique;
    int32_t *seg_offsets, *perm, *inverse;
    int64_t *n_unique_dev, *sorted_ids;
};
struct small_split {
    const int64_t *u_t, *n_t_dev, *u_t1, *n_t1_dev;
    int cap_t, cap_t1;
    int64_t *co, *ex, *ex_next;
    int32_t *co_slot, *ex_slot, *ex_next_slot;
    int64_t *counts_dev;
    uint8_t *flag_t1;                                    // optional output
    const int32_t *seg_offsets, *perm;                   // layout of batch t; null: no class order wanted
    int n;                                               // occurrences of batch t
    int32_t *cperm, *cslot, *cstart, *class_pos_dev, *short_rec;
};
struct small_batch {
    small_dedup d[kMaxBatch];
    small_split s[kMaxBatch];
};

// what the phases keep in LDS; the arrays of one phase are dead in the next
struct small_shared {
    uint16_t cnt[kSmallWaves][kSmallRadix];
    uint32_t base[kSmallRadix];
    uint32_t part[kSmallRadix / kWave];
    int wave_a[kSmallWaves], wave_b[kSmallWaves], wave_c[kSmallWaves];
    int misfit;                                          // split: the layout of batch t does not fit its batch
    // ballots of the rounds of a wavefront (LDS, not registers: with loops over the rounds that are not unrolled the code
    // of a phase stays a few hundred instructions, and none of it is fetched for one use)
    uint64_t bal[2][kSmallWaves][kSmallIds / kSmallThreads];
};

// sum of v[0, w) and of all of v
__device__ __forceinline__ int small_prefix(const int *v, int w, int &total) {
    int before = 0, all = 0;
#pragma unroll
    for (int i = 0; i < kSmallWaves; ++i) {
        const int x = v[i];
        before += i < w ? x : 0;
        all += x;
    }
    total = all;
    return before;
}

// ---- dedup -----------------------------------------------------------------------------------------------------
template <int KPT>
__device__ __forceinline__ void small_dedup_body(const small_dedup &job, char *lds, small_shared &sh, int *flags) {
    uint32_t *keys = reinterpret_cast<uint32_t *>(lds);
    uint16_t *order = reinterpret_cast<uint16_t *>(lds + sizeof(uint32_t) * kSmallThreads * KPT);
    const int n = job.n;
    const int lane = threadIdx.x & (kWave - 1);
    const int w = threadIdx.x / kWave;
    const int e0 = w * (kWave * KPT) + lane;
    const uint64_t lt = (1ull << lane) - 1ull;
    uint32_t key[KPT];
    uint32_t at[KPT];                                    // place in the batch; while a pass ranks, the rank above it
    constexpr int kPlaceBits = 14;
    static_assert(kSmallIds == 1 << kPlaceBits, "a place and a rank share a register");
    bool bad = false;
#pragma unroll
    for (int r = 0; r < KPT; ++r) {
        // no branch around the registers of a round (here and below): they would be copied as a whole at its end
        const int e = e0 + r * kWave;
        const int64_t id = n > 0 ? job.ids[e < n ? e : n - 1] : 0;
        bad |= n > 0 && ((id < 0) || (job.num_rows > 0 && id >= job.num_rows));
        key[r] = (uint32_t)id;
        at[r] = (uint32_t)e;
    }
    if (bad) atomicOr(flags, kFlagRowRange);
    // stable LSD radix passes; the keys leave the registers only to change places
    for (int pass = 0; pass < job.passes; ++pass) {
        const int shift = pass * job.bits, bins = 1 << job.bits;
        for (int i = threadIdx.x; i < kSmallWaves * kSmallRadix / 2; i += kSmallThreads)
            reinterpret_cast<uint32_t *>(&sh.cnt[0][0])[i] = 0u;
        __syncthreads();
#pragma unroll
        for (int r = 0; r < KPT; ++r) {
            const bool valid = e0 + r * kWave < n;
            const uint32_t digit = (key[r] >> shift) & (bins - 1);
            const uint64_t all = __ballot(valid);
            uint32_t peers_lo = (uint32_t)all, peers_hi = (uint32_t)(all >> 32);
#pragma unroll
            for (int b = 0; b < kSmallBits; ++b) {               // bits a pass does not have are 0 in every lane
                const uint32_t m = (uint32_t)((int)(digit << (31 - b)) >> 31);       // my bit in every position
                const uint64_t bal = __ballot(m != 0);
                peers_lo &= ~((uint32_t)bal ^ m);
                peers_hi &= ~((uint32_t)(bal >> 32) ^ m);
            }
            const uint64_t peers = (uint64_t)peers_lo | ((uint64_t)peers_hi << 32);
            const uint32_t before = __builtin_amdgcn_mbcnt_hi(peers_hi, __builtin_amdgcn_mbcnt_lo(peers_lo, 0));
            const uint32_t old = valid ? sh.cnt[w][digit] : 0u;       // all peers read ...
            wave_lds_order();
            if (valid && before == 0) sh.cnt[w][digit] = (uint16_t)(old + (uint32_t)__popcll(peers));   // ... then the first writes
            wave_lds_order();
            at[r] |= (old + before) << kPlaceBits;
        }
        __syncthreads();
        if (threadIdx.x < kSmallRadix) {                          // digit d: prefix over the waves, then over the digits
            const int d = threadIdx.x;
            uint32_t run = 0;
#pragma unroll
            for (int i = 0; i < kSmallWaves; ++i) {
                const uint32_t v = sh.cnt[i][d];
                sh.cnt[i][d] = (uint16_t)run;
                run += v;
            }
            const uint32_t incl = wave_inclusive_scan<uint32_t>(run);
            sh.base[d] = incl - run;
            if (lane == kWave - 1) sh.part[w] = incl;
        }
        __syncthreads();
        uint32_t part[kSmallRadix / kWave];
        part[0] = 0;
#pragma unroll
        for (int i = 1; i < kSmallRadix / kWave; ++i) part[i] = part[i - 1] + sh.part[i - 1];
#pragma unroll
        for (int r = 0; r < KPT; ++r) {
            if (e0 + r * kWave < n) {
                const uint32_t digit = (key[r] >> shift) & (bins - 1);
                const uint32_t q = digit / kWave;
                const uint32_t pos = (q == 0 ? part[0] : q == 1 ? part[1] : q == 2 ? part[2] : part[3]) + sh.base[digit] +
                                     sh.cnt[w][digit] + (at[r] >> kPlaceBits);
                keys[pos] = key[r];
                order[pos] = (uint16_t)(at[r] & (kSmallIds - 1));
            }
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < KPT; ++r) {
            const int e = e0 + r * kWave;                        // past n: whatever the LDS holds, never used
            key[r] = keys[e];
            at[r] = order[e];
        }
    }
    // heads of the segments, numbered
    int mine = 0;
#pragma unroll
    for (int r = 0; r < KPT; ++r) {
        const int p = e0 + r * kWave;
        const uint64_t h = __ballot(p < n && (p == 0 || keys[p - 1] != key[r]));
        if (lane == 0) sh.bal[0][w][r] = h;
        mine += __popcll(h);
    }
    if (lane == 0) sh.wave_a[w] = mine;
    __syncthreads();
    int total;
    int run = small_prefix(sh.wave_a, w, total);
#pragma unroll
    for (int r = 0; r < KPT; ++r) {
        const int p = e0 + r * kWave;
        const uint64_t h = sh.bal[0][w][r];
        if (p < n) {
            const bool head = (h >> lane) & 1ull;
            const int k = run + __popcll(h & lt);                     // heads before p
            if (head) {
                job.unique[k] = (int64_t)key[r];
                job.seg_offsets[k] = p;
            }
            job.perm[p] = (int)at[r];
            if (job.inverse != nullptr) job.inverse[at[r]] = head ? k : k - 1;
            if (job.sorted_ids != nullptr) job.sorted_ids[p] = (int64_t)key[r];
        }
        run += __popcll(h);
    }
    if (threadIdx.x == 0) {
        job.seg_offsets[total] = n;
        *job.n_unique_dev = total;
    }
}

// ---- collision split and class order -------------------------------------------------------------------------------
__device__ __forceinline__ int small_count(const int64_t *dev, int cap) {
    if (dev == nullptr) return 0;
    const int64_t v = *dev;
    return v < 0 ? 0 : (v > cap ? cap : (int)v);
}

struct small_extent {
    int first, len;
};
// sorted positions of row e of batch t (none, and the flag, where the layout makes no sense)
__device__ __forceinline__ small_extent row_extent(const small_split &job, int e, bool &bad) {
    small_extent x = {job.seg_offsets[e], 0};
    x.len = job.seg_offsets[e + 1] - x.first;
    if (x.len < 1 || x.first < 0 || x.first > job.n - x.len) { bad = true; x = {0, 0}; }
    return x;
}

// maxn: rows the LDS is sized for.  A list of n rows takes ceil(n / 1024) rounds, whatever maxn is: the lists are much
// shorter than the batch, and all wavefronts should have a share.
__device__ __forceinline__ void small_split_body(const small_split &job, const int maxn, char *lds, small_shared &sh,
                                                 int *flags) {
    int64_t *other = reinterpret_cast<int64_t *>(lds);                       // U_t1
    uint32_t *mark = reinterpret_cast<uint32_t *>(lds + sizeof(int64_t) * maxn);   // a bit per row of U_t1: also in U_t
    uint16_t *found = reinterpret_cast<uint16_t *>(mark + maxn / 32);        // a bit per row of U_t that a thread looked up
    const int lane = threadIdx.x & (kWave - 1);
    const int w = threadIdx.x / kWave;
    const uint64_t lt = (1ull << lane) - 1ull;
    const int n_t = small_count(job.n_t_dev, job.cap_t), n_t1 = small_count(job.n_t1_dev, job.cap_t1);
    const bool classes = job.seg_offsets != nullptr;
    const int rounds_t = (n_t + kSmallThreads - 1) / kSmallThreads, rounds_t1 = (n_t1 + kSmallThreads - 1) / kSmallThreads;
    const int e0 = w * (kWave * rounds_t) + lane, f0 = w * (kWave * rounds_t1) + lane;       // first row of mine in either list
#pragma unroll 4
    for (int e = threadIdx.x; e < n_t1; e += kSmallThreads) other[e] = job.u_t1[e];
    if ((int)threadIdx.x < maxn / 32) mark[threadIdx.x] = 0;
    if (threadIdx.x == 0) sh.misfit = 0;
    __syncthreads();
    bool bad = false;
    // Both lists ascend: a thread takes a few consecutive rows of U_t, looks the first one up and walks on from there (a
    // search per row is 14 dependent LDS reads each); where U_t1 is much denser than U_t it searches again.
    {
        uint32_t bits = 0;
        int lo = 0;
        int64_t next = (int)threadIdx.x * rounds_t < n_t ? job.u_t[threadIdx.x * rounds_t] : 0;
        for (int i = 0; i < rounds_t; ++i) {
            const int e = threadIdx.x * rounds_t + i;
            if (e >= n_t) break;
            const int64_t id = next;
            if (i + 1 < rounds_t && e + 1 < n_t) next = job.u_t[e + 1];
            int hi = n_t1;                                   // entries before lo are < id
            if (i > 0)
                for (int step = 0; step < 6 && lo < hi; ++step) {
                    if (other[lo] < id) ++lo; else hi = lo;
                }
            while (lo < hi) {                                // first entry >= id
                const int mid = (lo + hi) >> 1;
                if (other[mid] < id) lo = mid + 1; else hi = mid;
            }
            if (lo < n_t1 && other[lo] == id) {
                bits |= 1u << i;
                atomicOr(&mark[lo / 32], 1u << (lo % 32));
            }
        }
        found[threadIdx.x] = (uint16_t)bits;
    }
    __syncthreads();
    int n_co_mine = 0, n_long_mine = 0, lens = 0;
    for (int r = 0; r < rounds_t; ++r) {
        const int e = e0 + r * kWave;
        bool f = false;
        int len = 0;
        if (e < n_t) {
            f = (found[e / rounds_t] >> (e % rounds_t)) & 1;
            if (classes) {
                const small_extent x = row_extent(job, e, bad);
                len = x.len;
                bad |= (e == 0 && x.first != 0) || (e == n_t - 1 && x.first + len != job.n);
            }
        }
        const uint64_t co_b = __ballot(f);
        const bool lg = len > FS_SHORT_SEGMENT;
        const uint64_t long_b = __ballot(lg);
        if (lane == 0) {
            sh.bal[0][w][r] = co_b;
            sh.bal[1][w][r] = long_b;
        }
        n_co_mine += __popcll(co_b);
        n_long_mine += __popcll(long_b);
        if (long_b != 0)                                     // wave-uniform
            lens += __shfl(wave_inclusive_scan<int>(lg ? (f ? len : len << 16) : 0), kWave - 1, kWave);
    }
    // With the ends of the layout right and every row at least one occurrence long, the boundaries ascend from 0 to n, so
    // the extents of the rows are disjoint: the long ones sum to at most n <= kSmallIds (the packed halves hold that), and
    // there are at most n / 9 of them.  A layout that does not fit its batch gets the flag and no class order: its extents
    // may overlap, and then nothing bounds their sum.
    bad |= classes && n_t == 0;
    if (lane == 0) {
        sh.wave_a[w] = n_co_mine;
        sh.wave_b[w] = lens;
        sh.wave_c[w] = n_long_mine;
    }
    if (bad) {
        sh.misfit = 1;
        atomicOr(flags, kFlagInternal);
    }
    __syncthreads();
    int n_co, len_all, n_long;
    int co_run = small_prefix(sh.wave_a, w, n_co);
    int len_run = small_prefix(sh.wave_b, w, len_all);     // occurrences of long rows before the round: co, ex << 16
    int long_run = small_prefix(sh.wave_c, w, n_long);
    const bool fits = sh.misfit == 0;
    const int n_co_pos = len_all & 0xffff, n_pos = n_co_pos + (int)((uint32_t)len_all >> 16);
    // the list of long rows: class position, sorted position, slot; U_t1 is not needed in LDS any more, but the marks are
    int32_t *l_dest = reinterpret_cast<int32_t *>(lds), *l_from = l_dest + maxn / 8, *l_slot = l_from + maxn / 8;
    for (int r = 0; r < rounds_t; ++r) {
        const int e = e0 + r * kWave;
        const uint64_t co_b = sh.bal[0][w][r], long_b = sh.bal[1][w][r];
        const bool f = (co_b >> lane) & 1ull;
        small_extent x = {0, 0};
        if (classes && e < n_t) x = row_extent(job, e, bad);
        int both = len_run;
        if (long_b != 0) {
            const int v = x.len > FS_SHORT_SEGMENT ? (f ? x.len : x.len << 16) : 0;
            const int inc = wave_inclusive_scan<int>(v);
            both += inc - v;
            len_run += __shfl(inc, kWave - 1, kWave);
        }
        if (e < n_t) {
            const int c = co_run + __popcll(co_b & lt);      // collision rows before this one
            const int64_t id = job.u_t[e];
            if (f) { job.co[c] = id; job.co_slot[c] = e; }
            else { job.ex[e - c] = id; job.ex_slot[e - c] = e; }
            if (classes) {
                typedef int i32x4 __attribute__((ext_vector_type(4)));
                int32_t *rec = job.short_rec + ((int64_t)(f ? 0 : job.cap_t) + (f ? c : e - c)) * kShortRecInts;
                *reinterpret_cast<i32x4 *>(rec) = i32x4{(int)(id & 0xFFFFFFFFll), (int)(id >> 32), e, x.len};
                if (x.len > FS_SHORT_SEGMENT) {
                    const int dest = f ? (both & 0xffff) : n_co_pos + (int)((uint32_t)both >> 16);
                    const int k = long_run + __popcll(long_b & lt);
                    if (k < maxn / 8) {                      // always, where the layout fits
                        l_dest[k] = dest;
                        l_from[k] = x.first;
                        l_slot[k] = f ? e : ~e;
                    }
                    job.cstart[e] = dest;
                } else {
                    // whole 16-byte pieces: one compute unit writes the records of the batch, and a store instruction
                    // costs it a cycle per line whatever it writes there
                    i32x4 o[2];
#pragma unroll
                    for (int j = 0; j < FS_SHORT_SEGMENT; ++j) o[j / 4][j % 4] = j < x.len ? job.perm[x.first + j] : 0;
                    *reinterpret_cast<i32x4 *>(rec + 4) = o[0];
                    if (x.len > 4) *reinterpret_cast<i32x4 *>(rec + 8) = o[1];
                }
            }
        }
        co_run += __popcll(co_b);
        long_run += __popcll(long_b);
    }
    if (threadIdx.x == 0) {
        job.counts_dev[0] = n_co;
        job.counts_dev[1] = n_t - n_co;
        job.counts_dev[2] = n_t1 - n_co;
        if (job.class_pos_dev != nullptr) {
            job.class_pos_dev[0] = classes && fits ? n_co_pos : 0;
            job.class_pos_dev[1] = classes && fits ? n_pos : 0;
        }
    }
    // the other side: rows of U_t1 that are not in U_t
    int mine = 0;
    for (int r = 0; r < rounds_t1; ++r) {
        const int e = f0 + r * kWave;
        const bool g = e < n_t1 && ((mark[e / 32] >> (e % 32)) & 1u) != 0;
        const uint64_t b = __ballot(g);
        if (lane == 0) sh.bal[0][w][r] = b;
        mine += __popcll(b);
        if (e < n_t1 && job.flag_t1 != nullptr) job.flag_t1[e] = g ? 1 : 0;
    }
    __syncthreads();                                         // wave_a has been read by everybody; the list is complete
    if (lane == 0) sh.wave_a[w] = mine;
    __syncthreads();
    int all;
    int run = small_prefix(sh.wave_a, w, all);
    for (int r = 0; r < rounds_t1; ++r) {
        const int e = f0 + r * kWave;
        const uint64_t b = sh.bal[0][w][r];
        if (e < n_t1 && !((b >> lane) & 1ull)) {
            const int k = e - (run + __popcll(b & lt));
            job.ex_next[k] = job.u_t1[e];
            job.ex_next_slot[k] = e;
        }
        run += __popcll(b);
    }
    if (!classes || !fits || n_long > maxn / 8) return;      // the last only tells the compiler how long the list can be
    // The class order, a thread per class position.  The list has the long rows in row order, both classes mixed:
    // inside a class the positions ascend with the list, so the row of a position is found by looking for the last row
    // of ITS class that starts at or before it - the rows of the class are separated first.
    int32_t *s_dest = l_slot + maxn / 8, *s_from = s_dest + maxn / 8, *s_slot = s_from + maxn / 8;
    // collision rows of the list keep their order in front, the others behind them
    int n_co_long = 0;
    {
        const int per = (n_long + kSmallThreads - 1) / kSmallThreads;        // at most two
        int c = 0;
        for (int i = 0; i < per; ++i) {
            const int k = threadIdx.x * per + i;
            c += (k < n_long && l_slot[k] >= 0) ? 1 : 0;
        }
        const int inc = wave_inclusive_scan<int>(c);
        if (lane == kWave - 1) sh.wave_b[w] = inc;
        __syncthreads();
        int before = small_prefix(sh.wave_b, w, n_co_long) + inc - c;
        for (int i = 0; i < per; ++i) {
            const int k = threadIdx.x * per + i;
            if (k < n_long) {
                const int s = l_slot[k];
                const int to = s >= 0 ? before : n_co_long + k - before;
                s_dest[to] = l_dest[k];
                s_from[to] = l_from[k];
                s_slot[to] = s >= 0 ? s : ~s;
                before += s >= 0 ? 1 : 0;
            }
        }
    }
    __syncthreads();
    for (int q = threadIdx.x; q < n_pos; q += kSmallThreads) {
        int lo = 0, hi = n_long;                             // first row that starts behind q
        while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            if (s_dest[mid] <= q) lo = mid + 1; else hi = mid;
        }
        if (lo == 0) continue;                               // cannot happen: row 0 of the list starts at 0
        const int j = lo - 1;
        const int p = s_from[j] + (q - s_dest[j]);
        job.cperm[q] = (p >= 0 && p < job.n) ? job.perm[p] : 0;
        job.cslot[q] = s_slot[j];
    }
}

// the device's view of a job (host side)
inline small_dedup small_dedup_job(const fs_unique_job &in) {
    small_dedup j;
    const int kb = key_bits_of(in.num_rows);
    j.passes = (kb + kSmallBits - 1) / kSmallBits;
    j.bits = (kb + j.passes - 1) / j.passes;
    j.ids = in.ids; j.n = (int)in.n; j.num_rows = in.num_rows; j.unique = in.unique;
    j.seg_offsets = in.seg_offsets; j.perm = in.perm; j.inverse = in.inverse; j.n_unique_dev = in.n_unique_dev;
    j.sorted_ids = in.sorted_ids;
    return j;
}
inline small_split small_split_job(const fs_split_job &in, const fs_class_job *cls) {
    small_split j;
    memset(&j, 0, sizeof(j));
    j.u_t = in.u_t; j.n_t_dev = in.n_t_dev; j.u_t1 = in.u_t1; j.n_t1_dev = in.n_t1_dev;
    j.cap_t = (int)in.cap_t; j.cap_t1 = (int)in.cap_t1;
    j.co = in.co; j.ex = in.ex; j.ex_next = in.ex_next;
    j.co_slot = in.co_slot; j.ex_slot = in.ex_slot; j.ex_next_slot = in.ex_next_slot;
    j.counts_dev = in.counts_dev; j.flag_t1 = in.flag_t1_out;
    if (cls) {
        j.class_pos_dev = cls->class_pos_dev;
        if (cls->n > 0) {
            j.seg_offsets = cls->seg_offsets; j.perm = cls->perm; j.n = (int)cls->n;
            j.cperm = cls->cperm; j.cslot = cls->cslot; j.cstart = cls->cstart; j.short_rec = cls->short_rec;
        }
    }
    return j;
}
// LDS of the split of up to `maxn` rows: the other list, a bit each, the rows found
constexpr size_t small_split_lds(size_t maxn) { return maxn * 8 + maxn / 8 + kSmallThreads * 2; }

}  // namespace fs
