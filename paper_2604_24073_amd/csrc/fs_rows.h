// Device code of the passes over the rows of a batch: what one wavefront does with a chunk of positions, and with the rows of
// few occurrences.  Used by the class passes and the batch update (fs_fused.hip, where the design is described) and by the
// step of a small batch (fs_small_step.hip).
#pragma once

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
template <int LPR, int WAVES = kFusedWaves, int MOST = kParkedMost>
struct parked_rows {
    static constexpr int kWaves = WAVES, kMost = MOST;       // wavefronts of the workgroup, rows of a wavefront
    f32x4 sum[WAVES][MOST * LPR];
    int64_t row[WAVES][MOST];
    int slot[WAVES][MOST];
};

template <row_use USE, int LPR, int UNR, typename PARKED>
__device__ __forceinline__ void long_chunk(PARKED &sh, const chunk_view &ch, const f32x4 *__restrict__ grads,
                                           const int64_t *__restrict__ u_t, void *table, float *state, int64_t num_rows,
                                           int gvec, float lr, float eps, f32x4 *reduced, double *part_head,
                                           double *part_last, int *cnt_seg, int *cnt_sup, bool bad, int *flags) {
    constexpr int GPW = kWave / LPR;          // rows per wavefront instruction
    constexpr int BP = GPW * UNR;             // positions per batch
    constexpr int CAP = PARKED::kMost;
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
        } else if constexpr (USE == kSumOnly) {               // nothing to read first, so nothing to wait for
            const int s_q = __shfl(ch.sl, q, kWave);
            if (grp == 0 && col_ok) reduced[(int64_t)s_q * gvec + lig] = f32x4{(float)t[0], (float)t[1], (float)t[2], (float)t[3]};
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
template <row_use USE, int LPR, int UNR, typename PARKED>
__device__ __forceinline__ void long_segments_of_layout(
    PARKED &sh, const int block, const int log2, const f32x4 *__restrict__ grads, const int32_t *__restrict__ perm, int n,
    const int32_t *__restrict__ seg_offsets, const int64_t *__restrict__ u_t, int n_u, void *table, float *state,
    int64_t num_rows, int gvec, float lr, float eps, f32x4 *reduced, double *part_head, double *part_last, int *cnt_seg,
    int *cnt_sup, int *flags) {
    const int lane = threadIdx.x & (kWave - 1);
    const int size = 1 << log2;
    chunk_view ch;
    ch.chunk = block * PARKED::kWaves + threadIdx.x / kWave;
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

template <row_use USE, int LPR, int UNR, bool LAYOUT, int WAVES = kFusedWaves>
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
    const int64_t waves = (int64_t)nblocks * WAVES;
    const int64_t wave = (int64_t)block * WAVES + (threadIdx.x / kWave);
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

// `set`: the partial rows and counters it works in
inline batch_update_job batch_job(fs_ctx *ctx, const fs_batch_update_job &in, int set) {
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

}  // namespace fs
