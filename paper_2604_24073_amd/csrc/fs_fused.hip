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
#include "fs_rows.h"

namespace fs {

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
// with its own (the order of a row's sums depends on it, so a table keeps its width whoever is beside it).  With all of
// them it takes 123 to 125 registers, for the body of 8 lanes, where the kernels for 16, 32 and 64 lanes take 98 to 104, and
// always 33 KB of LDS: four wavefronts of it leave a SIMD nothing for the index kernels, which wait for some to end.
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

template <row_use USE, int LPR>
__device__ __forceinline__ void batch_rows_body(const batch_update_job &job, int *flags) {
    __shared__ parked_rows<LPR, kFusedWaves, USE == kSumOnly ? 1 : kParkedMost> sh;   // a sum is written where its segment ends
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
// update.  It is bound as the passes are.  A sum is written where its segment ends: without rows parked in LDS (33 KB of the
// widest, which is four workgroups to a compute unit) and with more workgroups of short rows than the passes, which end one
// by one while others read, 600 k occurrences x 144 146 -> 111 us, x 256 180 -> 149, x 128 98 -> 84, 100 k x 144 31 -> 25 (1280
// workgroups 117, 156, 88, 27; 65536 120, 157, 88, 25; four rows a round or one no better).  Against a chunk kernel of its own,
// 64 positions a wavefront whatever the batch, and a launch that adds the pieces of the cut segments: 33 k occurrences x 100
// 23.0 -> 9.9 us, 300 k x 8 121 -> 16, 100 k x 128 31.5 -> 19.2, x 144 26.9 -> 25.0, 600 k x 72 85 -> 71, x 144 119 -> 111, x 256
// 175 -> 149.
constexpr int kSumBlocks = 4096;
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

static dim3 batch_grid(const batch_update_job &j, int lpr, int64_t most) {
    const int64_t rows = ceil_div(j.n, (int64_t)(kWave / lpr) * FS_SHORT_UNR * kFusedWaves);
    return dim3((unsigned)(j.long_blocks + (rows < most ? rows : most)));
}

int launch_batch_update(fs_ctx *ctx, const fs_batch_update_job &job, hipStream_t s) {
    if (job.n == 0) return FS_OK;
    const batch_update_job j = batch_job(ctx, job, 0);
    const int lpr = lanes_per_row(j.gvec);
    const dim3 grid = batch_grid(j, lpr, FS_SHORT_MAX_BLOCKS), block(kFusedWaves * kWave);
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

// A layout that makes no sense can leave arrivals in the counters of a segment reduce (chunks that see it leave early), and
// the next call on the context is to be right all the same.  So every call has counters that no call has used since they were
// cleared: kReduceTurns sets in turn, all cleared by a launch when they have been used once, and a further one for launches
// that are recorded, which can run behind any other and clear it in front.
// Against a launch in front of every call it costs a thirty-second of one.  In the kernel itself it cost more: arrivals
// counted up from a number of the call's own, to which the counter is raised first, are two atomics each (400 k occurrences
// x 32 of one row 23.6 -> 26.8 us); clearing the set of the call before took registers from the sums (400 k x 32, 27.7 -> 34.1).
__global__ __launch_bounds__(256) void clear_counters_kernel(int *a, int *b, int n) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i < n) a[i] = b[i] = 0;
}

static int reduce_counters(fs_ctx *ctx, batch_update_job &j, hipStream_t s) {
    hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
    if (s != nullptr) FS_HIP(ctx, hipStreamIsCapturing(s, &status));
    const bool recorded = status != hipStreamCaptureStatusNone;
    const int64_t space = fused_chunk_space(ctx->max_ids, kReduceSet);
    const bool round = !recorded && ctx->reduce_turn == kReduceTurns;
    if (recorded || round) {
        const int64_t from = recorded ? kReduceTurns * space : 0, n = recorded ? space : kReduceTurns * space;
        hipLaunchKernelGGL(clear_counters_kernel, dim3((unsigned)ceil_div(n, 256)), dim3(256), 0, s, j.cnt_seg + from,
                           j.cnt_sup + from, (int)n);
        FS_LAUNCH_CHECK(ctx, "clear_counters_kernel");
    }
    if (round) ctx->reduce_turn = 0;
    const int64_t at = (recorded ? kReduceTurns : ctx->reduce_turn++) * space;
    j.cnt_seg += at;
    j.cnt_sup += at;
    return FS_OK;
}

int launch_reduce(fs_ctx *ctx, const float *grads, int64_t n, int32_t dim, const int32_t *perm,
                  const int32_t *seg_offsets, const int64_t *n_unique_dev, float *reduced, hipStream_t s) {
    if (n == 0) return FS_OK;
    batch_update_job j = batch_job(ctx, fs_batch_update_job{grads, n, dim, perm, seg_offsets, nullptr, n_unique_dev,
                                                            nullptr, FS_F32, nullptr, 0, 0.f, 0.f, reduced}, kReduceSet);
    const int rc = reduce_counters(ctx, j, s);
    if (rc != FS_OK) return rc;
    const int lpr = lanes_per_row(j.gvec);
    const dim3 grid = batch_grid(j, lpr, kSumBlocks), block(kFusedWaves * kWave);
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
