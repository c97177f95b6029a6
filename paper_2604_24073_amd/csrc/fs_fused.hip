// update_embedding(I, G) of Algorithm 2 for ONE class of rows (collision rows = priority pass,
// exclusive rows = deferred pass) in a single launch: gradient segment reduce and row-wise
// Adagrad fused, so the summed gradient of a row never travels through HBM.
//
// The index half of the step has laid the occurrences of the batch out class by class
// ("class order": all occurrences of collision rows first, then those of exclusive rows; inside a
// class by ascending row, inside a row in batch order).  A launch walks the positions of its
// class only, so the priority pass reads exactly the gradient rows of collision rows.
//
// Rows with at most FS_SHORT_SEGMENT occurrences (the vast majority of rows) take the short path:
// one group of lanes per row requests all gradient rows of its segment and the table row at once,
// adds, updates, stores - four short dependent rounds, no LDS, nothing shared.  Only rows with more
// occurrences go through the class order and the position-cut path below.
//
// There work is cut by POSITION (row popularity is Zipf, the hottest row has tens of thousands of
// occurrences): one wavefront owns 64 consecutive class positions, streams their gradient rows
// (16 bytes per lane, 64/LPR rows per instruction) into fp64 accumulators and, whenever a segment
// ends, parks the finished sum (rounded once to fp32) in LDS.  The parked rows (a handful: every
// segment here is long) are updated together at the end of the chunk, so the dependent loads of
// the update (table row, accumulator) are in flight together.  A segment cut by a chunk border leaves fp64 partial rows; every
// wavefront that contributed one counts itself in at the segment's counter, and the one that
// arrives last adds the partials in chunk order and updates the row - in two levels for the hot
// rows (sixteen pieces at a time, then the sums of those), so that the last arriver of a row with
// tens of thousands of occurrences has two short rounds of loads to do, not dozens.  No wavefront
// ever waits for another, and the order of every floating-point sum depends on the layout alone.
//
// The pieces travel between wavefronts (possibly on different XCDs, each with its own L2) as
// device-scope relaxed atomic stores and loads, which go through to the coherent level, ordered
// against the counter by waiting for the stores to be acknowledged.  A device-scope fence would
// do the same but writes back the whole dirty L2 every time - measured 10x the kernel's time.
#include <algorithm>

#include "fs_common.h"
#include "fs_device.h"

namespace fs {

// build-time tuning knobs: row-group loads one wavefront issues per round
#ifndef FS_FUSED_UNR
#define FS_FUSED_UNR 8
#endif
#ifndef FS_FUSED_RU
#define FS_FUSED_RU 2                      // parked rows one group of lanes updates per round
#endif
#ifndef FS_SHORT_MAX_BLOCKS
#define FS_SHORT_MAX_BLOCKS 1280
#endif
#ifndef FS_SHORT_UNR
#define FS_SHORT_UNR 2                     // short path: rows one group of lanes takes per iteration
#endif
constexpr int kFusedSuper = 16;            // pieces of a cut segment that are added in one go (first level)

// Adagrad on `nrows` parked rows of one wavefront.  Group g of the wavefront takes rows g, g+GPW, ...
// stage: [row][LPR] fp32 sums (4 columns per lane), stage_row: table row, stage_slot: slot in U_t.
// What is done with a row's sum: Adagrad on a table of fp32 or of bf16 rows, or nothing but writing it down.
enum row_use { kUpdateF32, kUpdateBf16, kSumOnly };

template <row_use USE, int LPR, int RU>
__device__ __forceinline__ void update_parked(const f32x4 *stage, const int64_t *stage_row, const int *stage_slot,
                                              int nrows, void *table, float *state, int64_t num_rows, int gvec,
                                              float lr, float eps, f32x4 *reduced, bool &oob) {
#pragma clang fp contract(off)
    constexpr int GPW = kWave / LPR;
    constexpr bool BF16 = USE == kUpdateBf16;
    const int lane = threadIdx.x & (kWave - 1);
    const int grp = lane / LPR;
    const int lig = lane % LPR;
    const bool col_ok = lig < gvec;
    const int dim = gvec * 4;
    u32x4 *t4 = reinterpret_cast<u32x4 *>(table);
    u32x2 *t2 = reinterpret_cast<u32x2 *>(table);
    if constexpr (USE == kSumOnly) {
        for (int k = grp; k < nrows; k += GPW)
            if (col_ok) reduced[(int64_t)stage_slot[k] * gvec + lig] = stage[k * LPR + lig];
        return;
    }
    for (int base = 0; base < nrows; base += GPW * RU) {
        int64_t r[RU];
        int k[RU];
        bool live[RU];
        f32x4 g[RU];
        u32x4 w[RU];
        float s_old[RU];
#pragma unroll
        for (int u = 0; u < RU; ++u) {
            const int kk = base + u * GPW + grp;
            const bool in_list = kk < nrows;
            r[u] = in_list ? stage_row[kk] : 0;
            k[u] = in_list ? stage_slot[kk] : 0;
            g[u] = f32x4{0.f, 0.f, 0.f, 0.f};
            if (in_list && col_ok) g[u] = stage[kk * LPR + lig];
            const bool in_table = (r[u] >= 0) && (r[u] < num_rows);
            oob |= in_list && !in_table;
            live[u] = in_list && in_table;
        }
#pragma unroll
        for (int u = 0; u < RU; ++u) {
            w[u] = u32x4{0u, 0u, 0u, 0u};
            if (live[u] && col_ok) {
                if (BF16) {
                    const u32x2 h = t2[r[u] * gvec + lig];
                    w[u][0] = h[0];
                    w[u][1] = h[1];
                } else {
                    w[u] = t4[r[u] * gvec + lig];
                }
            }
            s_old[u] = live[u] ? state[r[u]] : 0.f;
        }
#pragma unroll
        for (int u = 0; u < RU; ++u) {
            double ss = 0.0;
#pragma unroll
            for (int c = 0; c < 4; ++c) ss += (double)g[u][c] * (double)g[u][c];
            ss = group_sum<LPR>(ss);
            const float m = (float)(ss / (double)dim);
            const float s_new = s_old[u] + m;
            const float c_step = __fdiv_rn(lr, sqrt_rn_f32(s_new) + eps);
            const bool mine = live[u] && col_ok;
            if (BF16) {
                const float c0 = bf16_lo(w[u][0]) - c_step * g[u][0];
                const float c1 = bf16_hi(w[u][0]) - c_step * g[u][1];
                const float c2 = bf16_lo(w[u][1]) - c_step * g[u][2];
                const float c3 = bf16_hi(w[u][1]) - c_step * g[u][3];
                const u32x2 o = {f32_to_bf16_bits(c0) | (f32_to_bf16_bits(c1) << 16),
                                 f32_to_bf16_bits(c2) | (f32_to_bf16_bits(c3) << 16)};
                if (mine) t2[r[u] * gvec + lig] = o;
            } else {
                u32x4 o;
#pragma unroll
                for (int c = 0; c < 4; ++c) o[c] = __float_as_uint(__uint_as_float(w[u][c]) - c_step * g[u][c]);
                if (mine) t4[r[u] * gvec + lig] = o;
            }
            if (live[u] && lig == 0) state[r[u]] = s_new;
            if (reduced != nullptr && mine) reduced[(int64_t)k[u] * gvec + lig] = g[u];
        }
    }
}

// A partial row in memory: four planes of gvec doubles (column 4*l + c of the row at plane c, place l), so
// that each of the four instructions of a group of lanes writes or reads one contiguous run instead of
// eight bytes out of every thirty-two (which the write-through stores paid for four times over).
__device__ __forceinline__ void store_piece(double *row, int gvec, int lig, const double (&t)[4]) {
#pragma unroll
    for (int c = 0; c < 4; ++c)
        __hip_atomic_store(row + c * gvec + lig, t[c], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ double load_piece(const double *row, int gvec, int lig, int c) {
    return __hip_atomic_load(row + c * gvec + lig, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// t += part[c] for c = c_begin, c_begin + stride, ... <= c_last (four rows requested per round)
__device__ __forceinline__ void add_partial_rows(double (&t)[4], const double *part, int dim, int lig, bool col_ok,
                                                 int c_begin, int c_last, int stride) {
    for (int c = c_begin; c <= c_last; c += 4 * stride) {
        double h[4][4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int cj = c + j * stride;
            const bool ok = col_ok && cj <= c_last;
            const double *src = part + (int64_t)(ok ? cj : c_begin) * dim;
#pragma unroll
            for (int i = 0; i < 4; ++i) h[j][i] = ok ? load_piece(src, dim / 4, lig, i) : 0.0;
        }
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int i = 0; i < 4; ++i) t[i] += h[j][i];
    }
}

// wave-private LDS hand-over between lanes: order the accesses for the compiler and the hardware
__device__ __forceinline__ void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// One wavefront's chunk of positions, wherever they come from (the class order, or the layout of a batch).  A lane
// stands for one position of the chunk: the occurrence there, the slot and the table row of its segment, whether it
// takes part.
struct chunk_view {
    int chunk, lo, n_chunks;       // number of the chunk, position of chunk 0, chunks there can be
    int log2;                      // positions of a chunk
    int pr, sl;
    int64_t rid;
    uint64_t live, tails;          // positions that take part; those that end a segment
    bool head_cut, rest;           // the first segment came in from the chunk before; the last one goes on
    int last;                      // the last position (its segment may go on)
    // extents of the first segment (lanes 0 to 2) and of the last one (3 to 5): its first position, and two numbers that
    // are as far apart as it is long.  Wanted at the end only: looked at in front, the gradient rows wait a round for them.
    int extents;
};

// Every segment of the position-cut path has more than FS_SHORT_SEGMENT positions, so only a few end inside one chunk:
// their sums wait in LDS and are all applied in one round at the end of the chunk.
constexpr int kParkedMost = kWave / (FS_SHORT_SEGMENT + 1) + 1;
template <int LPR>
struct parked_rows {
    f32x4 sum[kFusedWaves][kParkedMost * LPR];
    int64_t row[kFusedWaves][kParkedMost];
    int slot[kFusedWaves][kParkedMost];
};

template <row_use USE, int LPR, int UNR>
__device__ __forceinline__ void long_chunk(parked_rows<LPR> &sh, const chunk_view &ch, const f32x4 *__restrict__ grads,
                                           const int64_t *__restrict__ u_t, void *table, float *state, int64_t num_rows,
                                           int gvec, float lr, float eps, f32x4 *reduced, double *part_head,
                                           double *part_last, int *cnt_seg, int *cnt_sup, bool bad, int *flags) {
    constexpr int GPW = kWave / LPR;          // rows per wavefront instruction
    constexpr int BP = GPW * UNR;             // positions per batch
    constexpr int CAP = kParkedMost;
    constexpr int RU = FS_FUSED_RU;
    static_assert(BP <= kWave, "one tail word");
    auto &stage = sh.sum;
    auto &stage_row = sh.row;
    auto &stage_slot = sh.slot;

    const int lane = threadIdx.x & (kWave - 1);
    const int wib = threadIdx.x / kWave;
    const int grp = lane / LPR;
    const int lig = lane % LPR;
    const bool col_ok = lig < gvec;
    const int dim = gvec * 4;
    const int chunk = ch.chunk, lo = ch.lo, span = ch.last + 1;
    const uint64_t tails = ch.tails;
    const bool head_complete = !ch.head_cut;
    auto load_batch = [&](f32x4(&v)[UNR], int k) {
#pragma unroll
        for (int u = 0; u < UNR; ++u) {
            const int q = k * BP + u * GPW + grp;             // position inside the chunk
            const int p = __shfl(ch.pr, q, kWave);
            v[u] = f32x4{0.f, 0.f, 0.f, 0.f};
            if (col_ok && ((ch.live >> (q & 63)) & 1ull)) v[u] = __builtin_nontemporal_load(&grads[(int64_t)p * gvec + lig]);
        }
    };

    double acc[4] = {0.0, 0.0, 0.0, 0.0};
    int nflush = 0;
    int nparked = 0;
    bool oob = false;

    auto flush = [&](int q) {                                 // the segment that ends at chunk position q
        double t[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) t[c] = across_groups<LPR>(acc[c]);
        if (nflush == 0 && !head_complete) {
            if (grp == 0 && col_ok) store_piece(part_head + (int64_t)chunk * dim, gvec, lig, t);
        } else {
            if (nparked < CAP) {
                if (grp == 0 && col_ok)
                    stage[wib][nparked * LPR + lig] = f32x4{(float)t[0], (float)t[1], (float)t[2], (float)t[3]};
                const int s_q = __shfl(ch.sl, q, kWave);
                const int64_t r_q = __shfl(ch.rid, q, kWave);
                if (lane == 0) {
                    stage_slot[wib][nparked] = s_q;
                    stage_row[wib][nparked] = r_q;
                }
            }
            ++nparked;
        }
#pragma unroll
        for (int c = 0; c < 4; ++c) acc[c] = 0.0;
        ++nflush;
    };
    auto add_batch = [&](const f32x4(&vv)[UNR], int k) {
        const uint64_t shifted = tails >> ((k * BP) & 63);
        const uint64_t batch_tails = (BP == kWave) ? shifted : (shifted & ((1ull << (BP & 63)) - 1ull));
        if (batch_tails == 0) {                               // no segment ends in this batch
#pragma unroll
            for (int u = 0; u < UNR; ++u)
#pragma unroll
                for (int c = 0; c < 4; ++c) acc[c] += (double)vv[u][c];
            return;
        }
#pragma unroll
        for (int u = 0; u < UNR; ++u) {
            const uint64_t tb = (batch_tails >> (u * GPW)) & (GPW == kWave ? ~0ull : ((1ull << (GPW & 63)) - 1ull));
            if (tb == 0) {
#pragma unroll
                for (int c = 0; c < 4; ++c) acc[c] += (double)vv[u][c];
            } else {
                // narrow rows: written out for each of its positions the end of a segment is most of the kernel's code, and
                // took 187 registers of rows of 32 columns where the rolled loop takes 110
                constexpr int kUnrollGroups = GPW <= 4 ? GPW : 1;
#pragma unroll kUnrollGroups
                for (int g = 0; g < GPW; ++g) {
                    if (grp == g) {
#pragma unroll
                        for (int c = 0; c < 4; ++c) acc[c] += (double)vv[u][c];
                    }
                    if ((tb >> g) & 1ull) flush(k * BP + u * GPW + g);
                }
            }
        }
    };

    f32x4 v[UNR];
    for (int k = 0; k * BP < span; ++k) {
        // wave-uniform: nobody in this batch takes part
        if (((ch.live >> ((k * BP) & 63)) & (BP == kWave ? ~0ull : ((1ull << (BP & 63)) - 1ull))) == 0) continue;
        load_batch(v, k);
        add_batch(v, k);
    }
    if (nparked > CAP) {                                      // cannot happen with a consistent class order
        bad = true;
        nparked = 0;
    }
    if (nparked > 0) {
        wave_lds_sync();
        update_parked<USE, LPR, RU>(stage[wib], stage_row[wib], stage_slot[wib], nparked, table, state, num_rows,
                                     gvec, lr, eps, reduced, oob);
        wave_lds_sync();
    }

    // positions after the last segment end of the chunk (the chunk's last position is not a tail)
    const bool has_rest = ch.rest;
    if (has_rest) {
        double t[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) t[c] = across_groups<LPR>(acc[c]);
        if (grp == 0 && col_ok) {
            // a chunk wholly inside one segment is a middle piece (head buffer); otherwise this
            // chunk is the FIRST piece of the segment that continues (last buffer)
            store_piece(((nflush == 0 && !head_complete) ? part_head : part_last) + (int64_t)chunk * dim, gvec, lig, t);
        }
    }

    // Count this chunk in at every cut segment it holds a piece of (at most two: the one that came
    // in from the left, the one that leaves to the right).  A cut segment that starts in chunk f
    // and ends in chunk l has its first piece in part_last[f] and one piece in part_head[c] for
    // every c in (f, l].  Those are grouped sixteen at a time ("supers", the j-th starts at chunk
    // f+1+16j): the last piece of a super to arrive adds the super up (chunk order) and leaves the
    // sum in the super's first slot; the last of {first piece, supers} to arrive adds those up
    // (same order) and updates the row.
    // Both first arrivals are counted with ONE atomic instruction (lane 0:
    // the piece of a super, lane 1: the first piece of the segment that leaves to the right), so the
    // common case costs one store acknowledgement and one atomic round trip per chunk.
    const bool tail_cut = has_rest && (nflush > 0 || head_complete);
    int seg_s[2] = {__shfl(ch.sl, 0, kWave), __shfl(ch.sl, ch.last, kWave)}, c_first[2], c_last[2];
    bool valid[2] = {ch.head_cut, tail_cut};
#pragma unroll
    for (int which = 0; which < 2; ++which) {
        const int start = __shfl(ch.extents, which * 3, kWave);
        const int len = __shfl(ch.extents, which * 3 + 2, kWave) - __shfl(ch.extents, which * 3 + 1, kWave);
        c_first[which] = (start - lo) >> ch.log2;
        c_last[which] = (start + len - 1 - lo) >> ch.log2;
        if (valid[which] && (start < lo || c_first[which] > chunk || c_last[which] < chunk || c_last[which] >= ch.n_chunks ||
                             c_last[which] == c_first[which] || (which == 0) != (chunk > c_first[which]))) {
            bad = true;
            valid[which] = false;
        }
    }
    const int sup_first = c_first[0] + 1 + ((chunk - c_first[0] - 1) / kFusedSuper) * kFusedSuper;
    const int sup_last = (sup_first + kFusedSuper - 1 < c_last[0]) ? sup_first + kFusedSuper - 1 : c_last[0];
    int old = 0;
    if (valid[0] || valid[1]) {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");      // my pieces are acknowledged before I count myself in
        if (lane == 0 && valid[0])
            old = __hip_atomic_fetch_add(&cnt_sup[sup_first], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (lane == 1 && valid[1])
            old = __hip_atomic_fetch_add(&cnt_seg[c_first[1]], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    const int old_head = __shfl(old, 0, kWave), old_tail = __shfl(old, 1, kWave);

    // last arrival at a segment: first piece + the sums of the supers, in chunk order; update the row
    auto finish_segment = [&](int s, int cf, int cl) {
        if (lane == 0) __hip_atomic_store(&cnt_seg[cf], 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        double t[4] = {0.0, 0.0, 0.0, 0.0};
        if (grp == 0 && col_ok) {
            const double *x = part_last + (int64_t)cf * dim;
#pragma unroll
            for (int i = 0; i < 4; ++i) t[i] = load_piece(x, gvec, lig, i);
        }
        add_partial_rows(t, part_head, dim, lig, col_ok, cf + 1 + grp * kFusedSuper, cl, GPW * kFusedSuper);
#pragma unroll
        for (int i = 0; i < 4; ++i) t[i] = across_groups<LPR>(t[i]);
        if (grp == 0 && col_ok) stage[wib][lig] = f32x4{(float)t[0], (float)t[1], (float)t[2], (float)t[3]};
        if (lane == 0) {
            stage_slot[wib][0] = s;
            stage_row[wib][0] = USE == kSumOnly ? 0 : u_t[s];
        }
        wave_lds_sync();
        update_parked<USE, LPR, 1>(stage[wib], stage_row[wib], stage_slot[wib], 1, table, state, num_rows, gvec, lr,
                                    eps, reduced, oob);
        wave_lds_sync();
    };

    if (valid[0] && old_head == sup_last - sup_first) {       // wave-uniform: last piece of its super
        if (lane == 0) __hip_atomic_store(&cnt_sup[sup_first], 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        double t[4] = {0.0, 0.0, 0.0, 0.0};
        add_partial_rows(t, part_head, dim, lig, col_ok, sup_first + grp, sup_last, GPW);
#pragma unroll
        for (int i = 0; i < 4; ++i) t[i] = across_groups<LPR>(t[i]);
        if (grp == 0 && col_ok) store_piece(part_head + (int64_t)sup_first * dim, gvec, lig, t);
        const int n_sup = (c_last[0] - c_first[0] + kFusedSuper - 1) / kFusedSuper;
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        int o2 = 0;
        if (lane == 0) o2 = __hip_atomic_fetch_add(&cnt_seg[c_first[0]], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        o2 = __builtin_amdgcn_readfirstlane(o2);
        if (o2 == n_sup) finish_segment(seg_s[0], c_first[0], c_last[0]);   // 1 + n_sup arrivals in all
    }
    if (valid[1]) {
        const int n_sup = (c_last[1] - c_first[1] + kFusedSuper - 1) / kFusedSuper;
        if (old_tail == n_sup) finish_segment(seg_s[1], c_first[1], c_last[1]);
    }
    if (oob) atomicOr(flags, kFlagRowRange);
    if (bad) atomicOr(flags, kFlagInternal);
}

// The position-cut path over the class order: chunk `block * kFusedWaves + wavefront` of the class's positions.
template <row_use USE, int LPR, int UNR>
__device__ __forceinline__ void long_segments_body(
    parked_rows<LPR> &sh, const int block, const int log2, const f32x4 *__restrict__ grads, const int32_t *__restrict__ cperm,
    const int32_t *__restrict__ cslot, const int32_t *__restrict__ class_pos, int cls, int n,
    const int32_t *__restrict__ seg_offsets, const int32_t *__restrict__ cstart, const int64_t *__restrict__ u_t,
    void *table, float *state, int64_t num_rows, int gvec, float lr, float eps, f32x4 *reduced, double *part_head,
    double *part_last, int *cnt_seg, int *cnt_sup, int *flags) {
    const int lane = threadIdx.x & (kWave - 1);
    const int size = 1 << log2;
    // A consistent class order never trips the range checks below; they turn a corrupted one into
    // an error flag instead of a wild access.
    int lo = cls == 0 ? 0 : class_pos[0];
    if (lo < 0) lo = 0;
    chunk_view ch;
    ch.chunk = block * kFusedWaves + threadIdx.x / kWave;    // chunk number inside the class
    ch.lo = lo;
    ch.log2 = log2;
    ch.n_chunks = (n + size - 1) >> log2;
    const int64_t a64 = (int64_t)lo + ((int64_t)ch.chunk << log2);
    if (a64 >= n) return;                                    // wave-uniform; wavefronts share nothing
    const int a = (int)a64;
    // Asked for before the end of the class is known (a round of loads less in front of the priority pass); what lies
    // behind it is not looked at.  With that and the extents looked at last, ten steps of 297 k occurrences x 128 962 ->
    // 952 us, of eight tables 5161 -> 5037, of one hot bf16 row 1149 -> 1131.
    const bool maybe = lane < size && lane < n - a;
    ch.pr = maybe ? cperm[a + lane] : 0;
    ch.sl = maybe ? cslot[a + lane] : -1;
    int edge = -1;                                           // lane 0: slot of position a-1, lane 1: of position a + size
    if (lane == 0 && a > lo) edge = cslot[a - 1];
    if (lane == 1 && size < n - a) edge = cslot[a + size];
    int hi = class_pos[cls == 0 ? 0 : 1];
    if (hi > n) hi = n;
    if (a >= hi) return;
    const int b = (size < hi - a) ? a + size : hi;
    const int span = b - a;
    ch.last = span - 1;
    if (lane >= span) { ch.pr = 0; ch.sl = -1; }
    if (lane == 1 && b >= hi) edge = -1;
    const bool bad = (lane < span) && ((unsigned)ch.pr >= (unsigned)n || (unsigned)ch.sl >= (unsigned)n);
    if (bad) { ch.pr = 0; ch.sl = 0; }
    ch.live = span == kWave ? ~0ull : (1ull << span) - 1ull;
    ch.rid = (lane < span) ? u_t[ch.sl] : 0;                  // table row of every position (used where a segment ends)
    // class position of the first occurrence, sorted positions: only needed if the chunk border cuts the segment
    ch.extents = 0;
    {
        const int s_edge = __shfl(ch.sl, lane < 3 ? 0 : span - 1, kWave);
        if (lane < 6) {
            const int f = lane % 3;
            ch.extents = f == 0 ? cstart[s_edge] : seg_offsets[s_edge + (f - 1)];
        }
    }
    const int sl_prev = __shfl(edge, 0, kWave), sl_after = __shfl(edge, 1, kWave);
    int nxt = __shfl_down(ch.sl, 1, kWave);
    if (lane == span - 1) nxt = sl_after;
    ch.tails = __ballot(lane < span && nxt != ch.sl);
    ch.head_cut = a != lo && sl_prev == __builtin_amdgcn_readfirstlane(ch.sl);
    ch.rest = ((ch.tails >> (span - 1)) & 1ull) == 0;
    long_chunk<USE, LPR, UNR>(sh, ch, grads, u_t, table, state, num_rows, gvec, lr, eps, reduced, part_head, part_last,
                               cnt_seg, cnt_sup, bad, flags);
}

// The position-cut path straight over the layout of a batch (sorted positions, segment boundaries): positions of
// segments with at most FS_SHORT_SEGMENT occurrences take no part.  The wavefront finds the segment of its first
// position with a 64-ary search; its positions touch at most 64 consecutive segments, whose boundaries its lanes hold.
template <row_use USE, int LPR, int UNR>
__device__ __forceinline__ void long_segments_of_layout(
    parked_rows<LPR> &sh, const int block, const int log2, const f32x4 *__restrict__ grads, const int32_t *__restrict__ perm, int n,
    const int32_t *__restrict__ seg_offsets, const int64_t *__restrict__ u_t, int n_u, void *table, float *state,
    int64_t num_rows, int gvec, float lr, float eps, f32x4 *reduced, double *part_head, double *part_last, int *cnt_seg,
    int *cnt_sup, int *flags) {
    const int lane = threadIdx.x & (kWave - 1);
    const int size = 1 << log2;
    chunk_view ch;
    ch.chunk = block * kFusedWaves + threadIdx.x / kWave;
    ch.lo = 0;
    ch.log2 = log2;
    ch.n_chunks = (n + size - 1) >> log2;
    const int64_t a64 = (int64_t)ch.chunk << log2;
    if (a64 >= n || n_u <= 0) return;                        // wave-uniform; wavefronts share nothing
    const int a = (int)a64;
    const int span = (a + size < n) ? size : n - a;
    ch.last = span - 1;
    ch.pr = (lane < span) ? perm[a + lane] : 0;
    bool bad = (unsigned)ch.pr >= (unsigned)n;
    if (bad) ch.pr = 0;
    int s0 = wave_upper_bound<int32_t>(seg_offsets, n_u, a) - 1;   // the segment of position a (boundary 0 is 0)
    if (s0 < 0) { bad = true; s0 = 0; }
    const int k = s0 + lane;
    const int begin = k < n_u ? seg_offsets[k] : 0x7fffffff;
    const int end = k < n_u ? seg_offsets[k + 1] : 0x7fffffff;
    int idx = 0;                                             // the last of the 64 segments that starts at or before p
    const int p = a + lane;
#pragma unroll
    for (int step = kWave / 2; step >= 1; step >>= 1)
        if (__shfl(begin, idx + step, kWave) <= p) idx += step;
    const int my_begin = __shfl(begin, idx, kWave), my_end = __shfl(end, idx, kWave);
    ch.sl = s0 + idx;
    // what a consistent layout never trips
    if (lane < span && (my_begin < 0 || my_begin > p || my_end <= p || my_end > n || ch.sl >= n_u)) { bad = true; ch.sl = 0; }
    const bool in = lane < span && !bad && my_end - my_begin > FS_SHORT_SEGMENT;
    ch.live = __ballot(in);
    if (__ballot(bad) != 0) {
        if (lane == 0) atomicOr(flags, kFlagInternal);
        return;
    }
    if (ch.live == 0) return;
    ch.rid = USE != kSumOnly && in ? u_t[ch.sl] : 0;
    ch.tails = __ballot(in && my_end == p + 1);
    const int first_begin = __shfl(my_begin, 0, kWave), first_end = __shfl(my_end, 0, kWave);
    const int last_begin = __shfl(my_begin, ch.last, kWave), last_end = __shfl(my_end, ch.last, kWave);
    ch.extents = lane < 3 ? (lane == 2 ? first_end : first_begin) : (lane == 5 ? last_end : last_begin);
    ch.head_cut = (ch.live & 1ull) != 0 && first_begin < a;
    ch.rest = ((ch.live >> ch.last) & 1ull) != 0 && last_end > a + span;
    long_chunk<USE, LPR, UNR>(sh, ch, grads, u_t, table, state, num_rows, gvec, lr, eps, reduced, part_head, part_last,
                               cnt_seg, cnt_sup, false, flags);
}

// Short path: the rows of one class whose segment has at most FS_SHORT_SEGMENT occurrences.  The
// index half left one record per row of the class (row, slot, number of occurrences, the
// occurrences themselves), so a group of LPR lanes needs two dependent rounds per row: the record,
// then table row + accumulator + all gradient rows of the segment at once.  Rows with longer
// segments are skipped (the position-cut launch owns them).
// LAYOUT: there are no records; row, extent and occurrences of a row come straight from the layout of the batch (one
// dependent round more per row).
struct row_source {
    const int32_t *recs;           // records of a class, or
    const int64_t *u_t;            // the layout of a batch
    const int32_t *seg_offsets, *perm;
};

template <row_use USE, int LPR, int UNR, bool LAYOUT>
__device__ __forceinline__ void short_rows_body(
    const int block, const int nblocks, const f32x4 *__restrict__ grads, int n, const row_source src, int64_t n_rows,
    void *table, float *state, int64_t num_rows, int gvec, float lr, float eps, f32x4 *reduced, int *flags) {
#pragma clang fp contract(off)
    constexpr int GPW = kWave / LPR;
    constexpr bool BF16 = USE == kUpdateBf16;
    constexpr int T = FS_SHORT_SEGMENT;
    typedef int i32x4 __attribute__((ext_vector_type(4)));
    const int lane = threadIdx.x & (kWave - 1);
    const int grp = lane / LPR;
    const int lig = lane % LPR;
    const bool col_ok = lig < gvec;
    const int dim = gvec * 4;
    const int64_t waves = (int64_t)nblocks * kFusedWaves;
    const int64_t wave = (int64_t)block * kFusedWaves + (threadIdx.x / kWave);
    u32x4 *t4 = reinterpret_cast<u32x4 *>(table);
    u32x2 *t2 = reinterpret_cast<u32x2 *>(table);
    bool oob = false, bad = false;
    for (int64_t base = wave * (GPW * UNR); base < n_rows; base += waves * (GPW * UNR)) {
        i32x4 hd[UNR], pa[UNR], pb[UNR];
        if (LAYOUT) {
            int at[UNR], cnt[UNR];
#pragma unroll
            for (int u = 0; u < UNR; ++u) {
                const int64_t i = base + u * GPW + grp;
                hd[u] = i32x4{0, 0, 0, 0};
                at[u] = 0;
                if (i < n_rows) {
                    const int64_t row = USE == kSumOnly ? 0 : src.u_t[i];
                    at[u] = src.seg_offsets[i];
                    hd[u] = i32x4{(int)(row & 0xFFFFFFFFll), (int)(row >> 32), (int)i, src.seg_offsets[i + 1] - at[u]};
                }
                cnt[u] = hd[u][3] <= T ? hd[u][3] : 0;
                if (at[u] < 0 || at[u] > n - hd[u][3]) { bad = true; cnt[u] = 0; hd[u][3] = 0; }
            }
#pragma unroll
            for (int u = 0; u < UNR; ++u)
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    pa[u][j] = j < cnt[u] ? src.perm[at[u] + j] : 0;
                    pb[u][j] = 4 + j < cnt[u] ? src.perm[at[u] + 4 + j] : 0;
                }
        } else {
#pragma unroll
            for (int u = 0; u < UNR; ++u) {
                const int64_t i = base + u * GPW + grp;
                const i32x4 *rec = reinterpret_cast<const i32x4 *>(src.recs + i * kShortRecInts);
                hd[u] = i32x4{0, 0, 0, 0};
                pa[u] = i32x4{0, 0, 0, 0};
                pb[u] = i32x4{0, 0, 0, 0};
                if (i < n_rows) {
                    hd[u] = rec[0];
                    pa[u] = rec[1];
                    pb[u] = rec[2];
                }
            }
        }
        int64_t r[UNR];
        int len[UNR];
        bool mine[UNR];
        u32x4 w[UNR];
        float s_old[UNR];
        f32x4 g[UNR][4];
        bool any_more = false;
#pragma unroll
        for (int u = 0; u < UNR; ++u) {
            r[u] = ((int64_t)hd[u][1] << 32) | (uint32_t)hd[u][0];
            len[u] = hd[u][3];
            const bool in_list = base + u * GPW + grp < n_rows;
            const bool in_table = USE == kSumOnly || ((r[u] >= 0) && (r[u] < num_rows));
            oob |= in_list && !in_table;
            const bool is_short = len[u] >= 1 && len[u] <= T;
            const bool slot_ok = (unsigned)hd[u][2] < (unsigned)n;
            bad |= in_list && (len[u] < 1 || !slot_ok);
            const bool live = in_list && in_table && is_short && slot_ok;
            if (!live) len[u] = 0;
            mine[u] = live && col_ok;
            any_more |= len[u] > 4;
            w[u] = u32x4{0u, 0u, 0u, 0u};
            if (USE != kSumOnly && mine[u]) {
                if (BF16) {
                    const u32x2 h = t2[r[u] * gvec + lig];
                    w[u][0] = h[0];
                    w[u][1] = h[1];
                } else {
                    w[u] = t4[r[u] * gvec + lig];
                }
            }
            s_old[u] = USE != kSumOnly && live ? state[r[u]] : 0.f;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                g[u][j] = f32x4{0.f, 0.f, 0.f, 0.f};
                int p = pa[u][j];
                if ((unsigned)p >= (unsigned)n) { bad |= j < len[u]; p = 0; }
                if (mine[u] && j < len[u]) g[u][j] = __builtin_nontemporal_load(&grads[(int64_t)p * gvec + lig]);
            }
        }
        double acc[UNR][4];
#pragma unroll
        for (int u = 0; u < UNR; ++u)
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                acc[u][c] = (double)g[u][0][c];
#pragma unroll
                for (int j = 1; j < 4; ++j) acc[u][c] += (double)g[u][j][c];
            }
        if (__ballot(any_more) != 0) {                        // wave-uniform: some row has 5..8 occurrences
#pragma unroll
            for (int u = 0; u < UNR; ++u)
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    g[u][j] = f32x4{0.f, 0.f, 0.f, 0.f};
                    int p = pb[u][j];
                    if ((unsigned)p >= (unsigned)n) { bad |= 4 + j < len[u]; p = 0; }
                    if (mine[u] && 4 + j < len[u]) g[u][j] = __builtin_nontemporal_load(&grads[(int64_t)p * gvec + lig]);
                }
#pragma unroll
            for (int u = 0; u < UNR; ++u)
#pragma unroll
                for (int c = 0; c < 4; ++c)
#pragma unroll
                    for (int j = 0; j < 4; ++j) acc[u][c] += (double)g[u][j][c];
        }
#pragma unroll
        for (int u = 0; u < UNR; ++u) {
            const f32x4 gs = {(float)acc[u][0], (float)acc[u][1], (float)acc[u][2], (float)acc[u][3]};
            if constexpr (USE == kSumOnly) {
                if (mine[u]) reduced[(int64_t)hd[u][2] * gvec + lig] = gs;
                continue;
            }
            double ss = 0.0;
#pragma unroll
            for (int c = 0; c < 4; ++c) ss += (double)gs[c] * (double)gs[c];
            ss = group_sum<LPR>(ss);
            const float m = (float)(ss / (double)dim);
            const float s_new = s_old[u] + m;
            const float c_step = __fdiv_rn(lr, sqrt_rn_f32(s_new) + eps);
            if (BF16) {
                const float c0 = bf16_lo(w[u][0]) - c_step * gs[0];
                const float c1 = bf16_hi(w[u][0]) - c_step * gs[1];
                const float c2 = bf16_lo(w[u][1]) - c_step * gs[2];
                const float c3 = bf16_hi(w[u][1]) - c_step * gs[3];
                const u32x2 o = {f32_to_bf16_bits(c0) | (f32_to_bf16_bits(c1) << 16),
                                 f32_to_bf16_bits(c2) | (f32_to_bf16_bits(c3) << 16)};
                if (mine[u]) t2[r[u] * gvec + lig] = o;
            } else {
                u32x4 o;
#pragma unroll
                for (int c = 0; c < 4; ++c) o[c] = __float_as_uint(__uint_as_float(w[u][c]) - c_step * gs[c]);
                if (mine[u]) t4[r[u] * gvec + lig] = o;
            }
            if (len[u] > 0 && lig == 0) state[r[u]] = s_new;
            if (reduced != nullptr && mine[u]) reduced[(int64_t)hd[u][2] * gvec + lig] = gs;
        }
    }
    if (oob) atomicOr(flags, kFlagRowRange);
    if (bad) atomicOr(flags, kFlagInternal);
}

template <int LPR> constexpr int fused_unr() {
    return (kWave / (kWave / LPR)) < FS_FUSED_UNR ? kWave / (kWave / LPR) : FS_FUSED_UNR;
}

// One launch per class: the first `long_blocks` workgroups of a pass walk the class order (rows with many
// occurrences, position-cut), the others the records of the rows with few.  The long part goes
// first because its last arrivers have the longest dependent chains; workgroups past the end of
// either part leave at once, so an empty part costs nothing but their dispatch.
// A launch takes the class passes of up to kMaxBatch tables (blockIdx.y picks the pass): a pass is about one residency
// round of the chip however small it is, so the tables of a shard are better walked side by side than one after the
// other, of whatever widths: ten steps of three tables of 15 k IDs x 96, 32 and 200 columns, with their lookups, 635 us
// with a launch per width and 509 in shared ones; of eight tables of 64, 128 and 256 columns 5474 and 4938 (nine large
// launches a step against three, each of which ends in a tail of its own).
struct class_pass_job {
    const f32x4 *grads;
    int n, long_blocks, blocks, chunk_log2, gvec, cls, lpr;
    float lr, eps;
    const int32_t *cperm, *cslot, *class_pos, *seg_offsets, *cstart, *recs;
    const int64_t *u_t, *n_rows_dev;
    void *table;
    float *state;
    int64_t num_rows;
    f32x4 *reduced;
    double *part_head, *part_last;      // this table's stretch of the class's partial rows and counters
    int *cnt_seg, *cnt_sup;
};
struct class_pass_batch {
    class_pass_job j[kMaxBatch];
};

template <row_use USE, int LPR>
__device__ __forceinline__ void class_pass_body(parked_rows<LPR> &sh, const class_pass_job &job, int cls, int block, int *flags) {
    if (block < job.long_blocks)
        long_segments_body<USE, LPR, fused_unr<LPR>()>(sh, block, job.chunk_log2, job.grads, job.cperm, job.cslot, job.class_pos,
                                                        cls, job.n, job.seg_offsets, job.cstart, job.u_t, job.table, job.state,
                                                        job.num_rows, job.gvec, job.lr, job.eps, job.reduced, job.part_head,
                                                        job.part_last, job.cnt_seg, job.cnt_sup, flags);
    else {
        int64_t n_rows = *job.n_rows_dev;
        if (n_rows > job.n) n_rows = job.n;
        short_rows_body<USE, LPR, FS_SHORT_UNR, false>(block - job.long_blocks, job.blocks - job.long_blocks, job.grads, job.n,
                                                        row_source{job.recs, nullptr, nullptr, nullptr}, n_rows, job.table,
                                                        job.state, job.num_rows, job.gvec, job.lr, job.eps, job.reduced, flags);
    }
}

// CLS (0: priority pass, 1: deferred pass, 2: both of every table, one after the other in the grid) is a template
// parameter so that the passes are kernels of their own by name in a profile; the code is the same.
// LPR: the lanes of a row of every table of the launch, or 0: tables of different widths from kMixedFrom lanes on, each
// with its own (the order of a row's sums depends on it, so a table keeps its width whoever is beside it).
constexpr int kMixedFrom = 8;
template <bool BF16, int LPR, int CLS>
__global__ __launch_bounds__(kFusedWaves *kWave, 4) void class_pass_kernel(const class_pass_batch batch, int *flags) {
    FS_WG_TRACE(8 + CLS);
    __shared__ __align__(16) char lds[sizeof(parked_rows<LPR ? LPR : kWave>)];
    const class_pass_job &job = batch.j[blockIdx.y];
    const int block = blockIdx.x;
    if (block >= job.blocks) return;
    const int cls = CLS < 2 ? CLS : job.cls;
    constexpr row_use USE = BF16 ? kUpdateBf16 : kUpdateF32;
    if constexpr (LPR != 0) {
        class_pass_body<USE, LPR>(reinterpret_cast<parked_rows<LPR> &>(lds), job, cls, block, flags);
    } else {
#define FS_CASE(L) \
    case L: class_pass_body<USE, L>(reinterpret_cast<parked_rows<L> &>(lds), job, cls, block, flags); break;
        switch (job.lpr) { FS_CASE(8) FS_CASE(16) FS_CASE(32) FS_CASE(64) }
#undef FS_CASE
    }
}

// All rows of a batch in one launch, straight from its layout: what the self-contained step runs, which has no use for
// the two classes (nothing of it can start before the last update) and so needs neither split nor class order first.
struct batch_update_job {
    const f32x4 *grads;
    int n, long_blocks, chunk_log2, gvec;
    float lr, eps;
    const int32_t *perm, *seg_offsets;
    const int64_t *u_t, *n_unique_dev;
    void *table;
    float *state;
    int64_t num_rows;
    f32x4 *reduced;
    double *part_head, *part_last;
    int *cnt_seg, *cnt_sup;
};

template <row_use USE, int LPR>
__device__ __forceinline__ void batch_rows_body(const batch_update_job &job, int *flags) {
    __shared__ parked_rows<LPR> sh;
    int64_t n_u = *job.n_unique_dev;
    n_u = n_u < 0 ? 0 : (n_u > job.n ? job.n : n_u);
    if ((int)blockIdx.x < job.long_blocks)
        long_segments_of_layout<USE, LPR, fused_unr<LPR>()>(sh, (int)blockIdx.x, job.chunk_log2, job.grads, job.perm, job.n, job.seg_offsets,
                                                job.u_t, (int)n_u, job.table, job.state, job.num_rows, job.gvec, job.lr,
                                                job.eps, job.reduced, job.part_head, job.part_last, job.cnt_seg,
                                                job.cnt_sup, flags);
    else
        short_rows_body<USE, LPR, FS_SHORT_UNR, true>((int)blockIdx.x - job.long_blocks, (int)gridDim.x - job.long_blocks, job.grads,
                                             job.n, row_source{nullptr, job.u_t, job.seg_offsets, job.perm}, n_u, job.table,
                                             job.state, job.num_rows, job.gvec, job.lr, job.eps, job.reduced, flags);
}

template <bool BF16, int LPR>
__global__ __launch_bounds__(kFusedWaves *kWave) void batch_update_kernel(const batch_update_job job, int *flags) {
    FS_WG_TRACE(9);
    batch_rows_body<BF16 ? kUpdateBf16 : kUpdateF32, LPR>(job, flags);
}

// The segment reduce as an operation of its own (first half of update_embedding(I, G) of Algorithm 2): reduced[k, :] =
// sum of grads[perm[p], :] over the sorted positions p of distinct row k, in the order and with the rounding of the batch
// update.  It is bound as the passes are.  Against a chunk kernel of its own, 64 positions a wavefront whatever the batch, and
// a launch that adds the pieces of the cut segments: 33 k occurrences x 100 23.0 -> 9.7 us, 70 k x 64 28.5 -> 9.9, 300 k x
// 128 61.9 -> 47.5, 300 k x 8 105.6 -> 19.2, 600 k x 256 181 -> 161.
template <int LPR>
__global__ __launch_bounds__(kFusedWaves *kWave) void segment_reduce_kernel(const batch_update_job job, int *flags) {
    FS_WG_TRACE(9);
    batch_rows_body<kSumOnly, LPR>(job, flags);
}

// `idx[0..m)`: the jobs of `jobs` (all of one dtype, all with n > 0) that share this launch; kernel: for their width, or for any
static void fused_launch(fs_ctx *ctx, void (*kernel)(class_pass_batch, int *), int cls, const fs_class_pass_job *jobs,
                         const int *idx, int m, hipStream_t s) {
    const int per = cls < 2 ? 1 : 2;                          // passes of a table
    const size_t cap_chunks = (size_t)fused_chunk_space(ctx->max_ids);
    const size_t cap_doubles = cap_chunks * (size_t)ctx->max_dim;
    int at = 0;
    while (at < m) {
        // as many jobs as fit the class's partial-row and counter space, each with its own stretch of it
        class_pass_batch batch;
        memset(&batch, 0, sizeof(batch));
        size_t chunks = 0, doubles = 0;
        int k = 0;
        for (; at + k < m && (k + 1) * per <= kMaxBatch; ++k) {
            const fs_class_pass_job &in = jobs[idx[at + k]];
            const int n = (int)in.n;
            // Both parts are sized for the worst case the host can know (every occurrence in a long
            // segment / every occurrence a row of its own); the real sizes live on the device.
            const int log2 = chunk_log2(n);
            const int long_blocks = (int)ceil_div(ceil_div(n, 1 << log2), kFusedWaves);
            const size_t my_chunks = (size_t)long_blocks * kFusedWaves;
            if (k > 0 && (chunks + my_chunks > cap_chunks || doubles + my_chunks * (size_t)in.dim > cap_doubles)) break;
            for (int c = 0; c < per; ++c) {
                const int pass = per == 1 ? cls : c;
                class_pass_job &j = batch.j[k * per + c];
                j.grads = (const f32x4 *)in.grads;
                j.n = n; j.long_blocks = long_blocks; j.chunk_log2 = log2; j.cls = pass;
                j.gvec = in.dim / 4; j.lpr = lanes_per_row(j.gvec); j.lr = in.lr; j.eps = in.eps;
                j.cperm = in.cperm; j.cslot = in.cslot; j.class_pos = in.class_pos; j.seg_offsets = in.seg_offsets;
                j.cstart = in.cstart; j.u_t = in.u_t;
                // records and row count of class 1 lie behind those of class 0 (both passes: `in` names class 0)
                j.recs = in.short_rec + (int64_t)c * n * kShortRecInts;
                j.n_rows_dev = in.n_rows_dev + c;
                j.table = in.table; j.state = in.state; j.num_rows = in.num_rows; j.reduced = (f32x4 *)in.reduced;
                j.part_head = ctx->fpart_head[pass] + doubles;
                j.part_last = ctx->fpart_last[pass] + doubles;
                j.cnt_seg = ctx->fcounters[pass] + chunks;
                j.cnt_sup = ctx->fcounters_sup[pass] + chunks;
            }
            chunks += my_chunks;
            doubles += my_chunks * (size_t)in.dim;
        }
        // The short part walks its records with a grid stride: the tables of a launch share FS_SHORT_MAX_BLOCKS
        // workgroups (about five per compute unit, all resident from the start).  Measured on four workloads,
        // more and shorter-lived workgroups lose (16 k: +5 %, 64 k: +12 %), fewer than three per compute unit too.
        int blocks = 0;
        for (int q = 0; q < k * per; ++q) {
            class_pass_job &j = batch.j[q];
            int64_t short_blocks = ceil_div(j.n, (int64_t)(kWave / j.lpr) * FS_SHORT_UNR * kFusedWaves);
            const int64_t cap = FS_SHORT_MAX_BLOCKS / k > 256 ? FS_SHORT_MAX_BLOCKS / k : 256;
            if (short_blocks > cap) short_blocks = cap;
            j.blocks = j.long_blocks + (int)short_blocks;
            blocks = j.blocks > blocks ? j.blocks : blocks;
        }
        hipLaunchKernelGGL(kernel, dim3((unsigned)blocks, (unsigned)(k * per)), dim3(kFusedWaves * kWave), 0, s, batch, ctx->d_flags);
        at += k;
    }
}

// the kernel of a dtype, a class (2: both) and a row width (0: any)
template <bool BF16, int CLS>
static void (*class_pass_for(int lpr))(class_pass_batch, int *) {
    switch (lpr) {
        case 0: return &class_pass_kernel<BF16, 0, CLS>;
        case 1: return &class_pass_kernel<BF16, 1, CLS>;
        case 2: return &class_pass_kernel<BF16, 2, CLS>;
        case 4: return &class_pass_kernel<BF16, 4, CLS>;
        case 8: return &class_pass_kernel<BF16, 8, CLS>;
        case 16: return &class_pass_kernel<BF16, 16, CLS>;
        case 32: return &class_pass_kernel<BF16, 32, CLS>;
        case 64: return &class_pass_kernel<BF16, 64, CLS>;
        default: return nullptr;
    }
}

int launch_reduce_update_batch(fs_ctx *ctx, int cls, int count, const fs_class_pass_job *jobs, hipStream_t s) {
    // one launch (or as few as fit) per dtype, and for narrow rows per width
    if (count < 0 || count > FS_MAX_STEP_TABLES) return set_err(ctx, FS_EINVAL, "reduce+update: too many tables");
    bool done[FS_MAX_STEP_TABLES];
    for (int k = 0; k < count; ++k) {
        done[k] = jobs[k].n == 0;
        if (!done[k] && lanes_per_row(jobs[k].dim / 4) > kWave) return set_err(ctx, FS_EINVAL, "reduce+update: dim beyond 256");
    }
    for (int k0 = 0; k0 < count; ++k0) {
        if (done[k0]) continue;
        const bool bf = jobs[k0].dt == FS_BF16;
        int lpr = lanes_per_row(jobs[k0].dim / 4);
        const bool wide = lpr >= kMixedFrom;
        int idx[FS_MAX_STEP_TABLES], m = 0;
        for (int k = k0; k < count; ++k) {
            const int mine = lanes_per_row(jobs[k].dim / 4);
            if (done[k] || (jobs[k].dt == FS_BF16) != bf || (wide ? mine < kMixedFrom : mine != lpr)) continue;
            lpr = lpr == mine ? lpr : 0;
            idx[m++] = k;
            done[k] = true;
        }
        // the largest first: the smaller ones fill the end of the launch
        std::sort(idx, idx + m, [jobs](int a, int b) {
            const int64_t x = jobs[a].n * jobs[a].dim, y = jobs[b].n * jobs[b].dim;
            return x != y ? x > y : a < b;
        });
        auto *kernel = cls == 0 ? (bf ? class_pass_for<true, 0>(lpr) : class_pass_for<false, 0>(lpr))
                       : cls == 1 ? (bf ? class_pass_for<true, 1>(lpr) : class_pass_for<false, 1>(lpr))
                                  : (bf ? class_pass_for<true, 2>(lpr) : class_pass_for<false, 2>(lpr));
        fused_launch(ctx, kernel, cls, jobs, idx, m, s);
    }
    FS_LAUNCH_CHECK(ctx, "class_pass_kernel");
    return FS_OK;
}

int launch_reduce_update(fs_ctx *ctx, int cls, const float *grads, int64_t n, int32_t dim, const int32_t *cperm,
                         const int32_t *cslot, const int32_t *class_pos, const int32_t *seg_offsets,
                         const int32_t *cstart, const int64_t *u_t, void *table, int dt, float *state,
                         int64_t num_rows, float lr, float eps, float *reduced, hipStream_t s,
                         const int32_t *short_rec, const int64_t *n_rows_dev) {
    const fs_class_pass_job job = {grads, n, dim, cperm, cslot, class_pos, seg_offsets, cstart, u_t, table, dt, state,
                                   num_rows, lr, eps, reduced, short_rec, n_rows_dev};
    return launch_reduce_update_batch(ctx, cls, 1, &job, s);
}

// `set`: the partial rows and counters it works in
static batch_update_job batch_job(fs_ctx *ctx, const fs_batch_update_job &in, int set) {
    batch_update_job j;
    const int n = (int)in.n;
    j.grads = (const f32x4 *)in.grads;
    j.n = n; j.chunk_log2 = chunk_log2(n); j.gvec = in.dim / 4; j.lr = in.lr; j.eps = in.eps;
    j.long_blocks = (int)ceil_div(ceil_div(n, 1 << j.chunk_log2), kFusedWaves);
    j.perm = in.perm; j.seg_offsets = in.seg_offsets; j.u_t = in.u_t; j.n_unique_dev = in.n_unique_dev;
    j.table = in.table; j.state = in.state; j.num_rows = in.num_rows; j.reduced = (f32x4 *)in.reduced;
    j.part_head = ctx->fpart_head[set]; j.part_last = ctx->fpart_last[set];
    j.cnt_seg = ctx->fcounters[set]; j.cnt_sup = ctx->fcounters_sup[set];
    return j;
}
static dim3 batch_grid(const batch_update_job &j, int lpr) {
    const int64_t rows = ceil_div(j.n, (int64_t)(kWave / lpr) * FS_SHORT_UNR * kFusedWaves);
    return dim3((unsigned)(j.long_blocks + (rows < FS_SHORT_MAX_BLOCKS ? rows : FS_SHORT_MAX_BLOCKS)));
}

int launch_batch_update(fs_ctx *ctx, const fs_batch_update_job &job, hipStream_t s) {
    if (job.n == 0) return FS_OK;
    const batch_update_job j = batch_job(ctx, job, 0);
    const int lpr = lanes_per_row(j.gvec);
    const dim3 grid = batch_grid(j, lpr), block(kFusedWaves * kWave);
#define FS_CASE(L)                                                                                                \
    case L:                                                                                                       \
        if (job.dt == FS_BF16) hipLaunchKernelGGL((batch_update_kernel<true, L>), grid, block, 0, s, j, ctx->d_flags); \
        else hipLaunchKernelGGL((batch_update_kernel<false, L>), grid, block, 0, s, j, ctx->d_flags);            \
        break;
    switch (lpr) {
        FS_CASE(1) FS_CASE(2) FS_CASE(4) FS_CASE(8) FS_CASE(16) FS_CASE(32) FS_CASE(64)
        default: return set_err(ctx, FS_EINVAL, "update: dim beyond 256");
    }
#undef FS_CASE
    FS_LAUNCH_CHECK(ctx, "batch_update_kernel");
    return FS_OK;
}

int launch_reduce(fs_ctx *ctx, const float *grads, int64_t n, int32_t dim, const int32_t *perm,
                  const int32_t *seg_offsets, const int64_t *n_unique_dev, float *reduced, hipStream_t s) {
    if (n == 0) return FS_OK;
    const batch_update_job j = batch_job(ctx, fs_batch_update_job{grads, n, dim, perm, seg_offsets, nullptr, n_unique_dev,
                                                                  nullptr, FS_F32, nullptr, 0, 0.f, 0.f, reduced}, kReduceSet);
    const int lpr = lanes_per_row(j.gvec);
    const dim3 grid = batch_grid(j, lpr), block(kFusedWaves * kWave);
    switch (lpr) {
#define FS_CASE(L) \
    case L: hipLaunchKernelGGL((segment_reduce_kernel<L>), grid, block, 0, s, j, ctx->d_flags); break;
        FS_CASE(1) FS_CASE(2) FS_CASE(4) FS_CASE(8) FS_CASE(16) FS_CASE(32) FS_CASE(64)
#undef FS_CASE
        default: return set_err(ctx, FS_EINVAL, "reduce: dim beyond 256");
    }
    FS_LAUNCH_CHECK(ctx, "segment_reduce_kernel");
    return FS_OK;
}

FS_TRACE_SETTER(fused)

}  // namespace fs
