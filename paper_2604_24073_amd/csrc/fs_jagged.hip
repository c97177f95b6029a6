// Load-balancer data path on one GPU: the Fixed Batch Size partitioner (Section 4.1 of the paper,
// "Partitioning Algorithms") and the indexed permute of a jagged tensor (Section 4.2, "Triton Kernel
// Optimizations": the kernel that applies a partitioning to the gathered IDs).
//
// FBS: samples sorted by UIH length (the stable sort of the dedup, on the lengths), then dealt to
// the ranks in a zig-zag - rank i takes sorted positions i, 2n-1-i, 2n+i, 4n-1-i, ...  The deal is a
// closed form per sorted position, one thread each.
//
// Indexed permute: output sample k is input sample sample_of[k].  Up to 8192 samples two launches: one
// workgroup lays out the output offsets, then the copy; beyond, lengths summed per tile of samples, the
// output offsets by a scan with tile prefixes, and the copy.  The copy is driven
// by the OUTPUT (every lane writes consecutive pieces of the output, so a 16K-item sample costs per
// item what a short one costs): a workgroup takes 2048 to 8192 consecutive output pieces, looks up (up to 8192
// samples, where nothing is left in the context) or is told which samples they begin and end in, and marks the
// starts of its samples as bits in LDS.
//
// VBS: the same sort, then the sorted order is cut into n runs of about equal total weight.
//
// Keyed transpose, ranged dispatch and ranged combine (same section of the paper) are the same copy
// under a computed order of the F x B segments of a keyed jagged tensor, always told; the order is written down where
// the lengths are summed, beyond the 4096 segments of one workgroup.
#include "fs_common.h"
#include "fs_device.h"

namespace fs {

// ---- FBS: the deal ------------------------------------------------------------------------------------
// By ranges of keys the sort deals its positions itself and writes nothing that only a dedup needs: balancing 65 k samples
// three launches where sort, list of the distinct lengths and deal were five.
__global__ __launch_bounds__(256) void fbs_deal_kernel(const int32_t *__restrict__ sorted, int64_t B, const fs_zigzag deal,
                                                       int32_t *__restrict__ sample_of,
                                                       int64_t *__restrict__ rank_offsets) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    const int64_t gtid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    for (int64_t i = gtid; i <= deal.n; i += stride) rank_offsets[i] = deal.rank_start(i);
    for (int64_t s = gtid; s < B; s += stride) sample_of[deal.place(s)] = sorted[s];
}

int launch_partition_fbs(fs_ctx *ctx, const int64_t *lengths, int64_t B, int64_t max_len, int32_t n_ranks,
                         int32_t *sample_of, int64_t *rank_offsets, hipStream_t s) {
    if (B > 0) {
        fs_unique_job job = {lengths, B, max_len + 1, ctx->jag_unique, ctx->jag_seg, ctx->jag_sorted, nullptr, ctx->jag_n};
        job.order_only = true;
        const bool dealt = unique_by_ranges(1, &job, 0, true);
        if (dealt) {
            job.perm = sample_of;
            job.deal = n_ranks;
            job.rank_offsets = rank_offsets;
        }
        const int rc = launch_unique_batch(ctx, 1, &job, s, 0, true);
        if (rc != FS_OK || dealt) return rc;
    }
    const int64_t work = B > n_ranks ? B : (int64_t)n_ranks + 1;
    int64_t blocks = ceil_div(work, 256);
    if (blocks > 1024) blocks = 1024;
    hipLaunchKernelGGL(fbs_deal_kernel, dim3((unsigned)blocks), dim3(256), 0, s, ctx->jag_sorted, B,
                       fs_zigzag{n_ranks, B / n_ranks, B % n_ranks}, sample_of, rank_offsets);
    FS_LAUNCH_CHECK(ctx, "fbs_deal_kernel");
    return FS_OK;
}

// ---- indexed permute ------------------------------------------------------------------------------------
struct jagged_in {
    const int64_t *offsets;   // [B + 1]
    int64_t B, n_values;      // samples, elements behind them
};

// extent of input sample p (0 and a flag for a sample index out of range or a sample whose boundaries are not inside
// the values: such a sample is never read)
struct sample_extent {
    int64_t first, len;
};
__device__ __forceinline__ sample_extent extent_of(const jagged_in &in, int64_t p, bool &bad) {
    if (p < 0 || p >= in.B) { bad = true; return {0, 0}; }
    const int64_t a = in.offsets[p], b = in.offsets[p + 1];
    if (a < 0 || b < a || b > in.n_values) { bad = true; return {0, 0}; }
    return {a, b - a};
}

// What the copy wants to know of every output sample and every tile of the output, written down with the output
// offsets: a workgroup of the copy then opens its tile with two dependent rounds of loads, where a search for its first
// and last sample and a look at where they come from are six.
// It lies in the context, so that the calls that use it must not overlap.  The permute of up to kOwnPermute samples of a
// caller's list has no plan: its calls share nothing and may run side by side on several streams.
struct copy_plan {
    int64_t *delta;           // [n_out] first input element of a sample minus its first output element (null: no plan)
    int32_t *tile_first;      // [tiles] sample that the first piece of a tile belongs to (null: too many tiles)
    int64_t cap_out;          // elements of the output
    int ppe, tile_log2;       // pieces of an element, log2 of the pieces of a tile
};
// `mine`: this lane has a sample; met by whole wavefronts.  A lane writes the tiles of its sample down by itself, of a long one
// the wavefront together: one sample of 16.7 M IDs has 8192 tiles, and a lane alone was at them for 210 us.
constexpr int kLaneTiles = 64;
__device__ __forceinline__ void plan_sample(const copy_plan &plan, bool mine, int64_t k, int64_t start, const sample_extent &x) {
    if (plan.delta == nullptr) return;
    if (mine) plan.delta[k] = x.first - start;
    if (plan.tile_first == nullptr) return;
    int64_t end = start + x.len;
    if (end > plan.cap_out) end = plan.cap_out;
    const int64_t size = (int64_t)1 << plan.tile_log2;
    const int64_t t0 = (start * plan.ppe + size - 1) >> plan.tile_log2;
    const int64_t t1 = mine ? (end * plan.ppe + size - 1) >> plan.tile_log2 : t0;        // behind the last tile that starts in it
    const bool is_long = t1 - t0 > kLaneTiles;
    if (!is_long)
        for (int64_t t = t0; t < t1; ++t) plan.tile_first[t] = (int32_t)k;
    for (uint64_t left = __ballot(is_long); left != 0; left &= left - 1) {
        const int who = __ffsll((unsigned long long)left) - 1;
        const int64_t from = __shfl(t0, who, kWave), to = __shfl(t1, who, kWave);
        const int whose = __shfl((int)k, who, kWave);
        for (int64_t t = from + (threadIdx.x & (kWave - 1)); t < to; t += kWave) plan.tile_first[t] = whose;
    }
}

// ---- the order of the output samples ---------------------------------------------------------------------
// Segment (f, b) of a keyed jagged tensor with F keys and B samples is number f * B + b in feature-major
// form and b * F + f in batch-major form.  Ranks own sample ranges [ro[r], ro[r + 1]); what a rank is sent
// (dispatch) or has sent (combine) is a feature-major tensor over its own samples, rank after rank.
enum { kMapTranspose = 0, kMapDispatch = 1, kMapCombine = 2, kMapGiven = 3 };

// where the input sample of an output sample comes from: the caller's list, or computed from the keyed form
struct sample_order {
    int mode;
    const int32_t *given;     // kMapGiven
    int64_t F, B;             // the others
    const int64_t *ro;        // dispatch, combine
    int n_ranks;
    int64_t *splits;          // dispatch: elements each rank is sent
};

// the last r in [0, n) with scale * ro[r] <= x (ro ascending, ro[0] == 0)
__device__ __forceinline__ int last_rank_at_or_before(const int64_t *ro, int n, int64_t scale, int64_t x) {
    int lo = 0, hi = n;                      // first r with scale * ro[r] > x
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (scale * ro[mid] <= x) lo = mid + 1; else hi = mid;
    }
    return lo > 0 ? lo - 1 : 0;
}

// input segment of output segment j; -1 for ranges that make no sense: the copy skips and reports it
__device__ __forceinline__ int32_t ordered_segment(const sample_order &o, const int64_t *ro, int64_t j) {
    const int64_t F = o.F, B = o.B;
    int64_t in = -1;
    if (o.mode == kMapTranspose) {
        in = (j % F) * B + j / F;
    } else if (o.mode == kMapDispatch) {
        const int r = last_rank_at_or_before(ro, o.n_ranks, F, j);
        const int64_t first = ro[r], cnt = ro[r + 1] - first, local = j - F * first;
        if (cnt > 0 && local >= 0 && local < F * cnt) in = (local / cnt) * B + first + local % cnt;
    } else {
        const int64_t f = j / B, b = j % B;
        const int r = last_rank_at_or_before(ro, o.n_ranks, 1, b);
        const int64_t first = ro[r], cnt = ro[r + 1] - first;
        if (cnt > 0 && b >= first && b < first + cnt) in = F * first + f * cnt + (b - first);
    }
    return (in >= 0 && in < F * B) ? (int32_t)in : -1;
}

// what one workgroup sees wrong with the rank boundaries
__device__ __forceinline__ bool bad_ranks(const sample_order &o) {
    bool bad = false;
    if (o.mode == kMapDispatch || o.mode == kMapCombine) {
        for (int r = threadIdx.x; r < o.n_ranks; r += blockDim.x) bad |= o.ro[r + 1] < o.ro[r];
        if (threadIdx.x == 0) bad |= o.ro[0] != 0 || o.ro[o.n_ranks] != o.B;
    }
    return bad;
}

// elements rank r is sent: the extent of its F * count segments in the dispatched tensor
__device__ __forceinline__ int64_t rank_split(const sample_order &o, const int64_t *out_offsets, int64_t r) {
    int64_t a = o.ro[r], b = o.ro[r + 1];
    a = a < 0 ? 0 : (a > o.B ? o.B : a);
    b = b < a ? a : (b > o.B ? o.B : b);
    return out_offsets[o.F * b] - out_offsets[o.F * a];
}

// Everything the copy needs about a small number of output samples in ONE launch: their order, the output offsets
// and the splits.  The work is a few loads a sample; what it costs is launches, about 4 us each here (four keyed
// shuffles of 1024 segments spent three to four of them on it).  One workgroup, up to PER consecutive samples a thread.
// Beyond kPlanPer one compute unit takes longer than two launches over many (a permute of 8192 samples 17.5 us against 12.3,
// of 4096 10.8 against 11.6), but those leave sums in the context, and a permute without a plan leaves nothing there (its
// offsets in one launch over many, each adding up the lengths in front of its samples: 17.0).
constexpr int kPlanThreads = 1024;
constexpr int kPlanPer = 4, kOwnPer = 8;
constexpr int64_t kOwnPermute = (int64_t)kPlanThreads * kOwnPer;
constexpr int kPlanRanks = 1024;                 // rank boundaries kept in LDS

template <int PER>
__global__ __launch_bounds__(kPlanThreads) void jagged_plan_kernel(const jagged_in in, const sample_order order,
                                                                   int n_out, const copy_plan plan,
                                                                   int64_t *out_offsets, int *__restrict__ flags) {
    __shared__ int64_t s_ro[kPlanRanks + 1];
    __shared__ int64_t sh[kPlanThreads / kWave];
    const bool ranked = order.mode == kMapDispatch || order.mode == kMapCombine;
    const bool staged = ranked && order.n_ranks <= kPlanRanks;
    if (staged)
        for (int r = threadIdx.x; r <= order.n_ranks; r += kPlanThreads) s_ro[r] = order.ro[r];
    __syncthreads();
    const int64_t *ro = staged ? (const int64_t *)s_ro : order.ro;
    bool bad = n_out > 0 && bad_ranks(order);
    const int per = (n_out + kPlanThreads - 1) / kPlanThreads;           // at most PER
    const int k0 = (int)threadIdx.x * per;
    int32_t p[PER];
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        p[i] = -1;
        if (i < per && k0 + i < n_out) {
            p[i] = order.mode == kMapGiven ? order.given[k0 + i] : ordered_segment(order, ro, k0 + i);
        }
    }
    sample_extent x[PER];
    int64_t v = 0;
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        x[i] = {0, 0};
        if (i < per && k0 + i < n_out) x[i] = extent_of(in, p[i], bad);
        v += x[i].len;
    }
    const int64_t inc = wave_inclusive_scan<int64_t>(v);
    if ((threadIdx.x & (kWave - 1)) == kWave - 1) sh[threadIdx.x / kWave] = inc;
    __syncthreads();
    int64_t run = inc - v, total = 0;
#pragma unroll
    for (int w = 0; w < kPlanThreads / kWave; ++w) {
        if (w < (int)(threadIdx.x / kWave)) run += sh[w];
        total += sh[w];
    }
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        if (i < per) {                                                   // the same for all
            const bool mine = k0 + i < n_out;
            if (mine) out_offsets[k0 + i] = run;
            plan_sample(plan, mine, k0 + i, run, x[i]);
        }
        run += x[i].len;
    }
    if (threadIdx.x == 0) {
        out_offsets[n_out] = total;
        bad |= total > plan.cap_out;                                     // the copy stops there
    }
    if (bad) atomicOr(flags, kFlagOffsets);
    if (order.splits != nullptr) {
        __syncthreads();                                                 // the offsets above, by any thread
        for (int r = threadIdx.x; r < order.n_ranks; r += kPlanThreads) order.splits[r] = rank_split(order, out_offsets, r);
    }
}

// The same for more samples than one workgroup takes: order and lengths summed per tile, then the scan.
__global__ __launch_bounds__(kScanThreads) void permute_tile_sum_kernel(const jagged_in in, const sample_order order,
                                                                        int32_t *__restrict__ sel, int64_t n_out,
                                                                        int64_t *__restrict__ tile_sum,
                                                                        int *__restrict__ flags) {
    __shared__ int64_t sh[kScanThreads / kWave];
    const int64_t k0 = (int64_t)blockIdx.x * kScanTile + threadIdx.x * kScanIpt;
    bool bad = blockIdx.x == 0 && bad_ranks(order);
    int64_t v = 0;
#pragma unroll
    for (int i = 0; i < kScanIpt; ++i) {
        const int64_t k = k0 + i;
        if (k < n_out) {
            int32_t p;
            if (order.mode == kMapGiven) {
                p = order.given[k];
            } else {
                p = ordered_segment(order, order.ro, k);
                sel[k] = p;
            }
            v += extent_of(in, p, bad).len;
        }
    }
    int64_t total;
    (void)block_exclusive_scan<int64_t>(v, sh, total);
    if (threadIdx.x == 0) tile_sum[blockIdx.x] = total;
    if (bad) atomicOr(flags, kFlagOffsets);
}

__global__ __launch_bounds__(kScanThreads) void permute_offsets_kernel(const jagged_in in,
                                                                       const int32_t *__restrict__ sample_of,
                                                                       int64_t n_out,
                                                                       const int64_t *__restrict__ tile_sum,
                                                                       const copy_plan plan,
                                                                       int64_t *__restrict__ out_offsets,
                                                                       int *__restrict__ flags) {
    __shared__ int64_t sh[kScanThreads / kWave];
    int64_t before = 0;
    for (int t = threadIdx.x; t < (int)blockIdx.x; t += kScanThreads) before += tile_sum[t];
    int64_t tile_base;
    (void)block_exclusive_scan<int64_t>(before, sh, tile_base);
    const int64_t k0 = (int64_t)blockIdx.x * kScanTile + threadIdx.x * kScanIpt;
    bool bad = false;
    sample_extent x[kScanIpt];
    int64_t v = 0;
#pragma unroll
    for (int i = 0; i < kScanIpt; ++i) {
        x[i] = {0, 0};
        if (k0 + i < n_out) x[i] = extent_of(in, sample_of[k0 + i], bad);
        v += x[i].len;
    }
    int64_t tile_total;
    int64_t run = tile_base + block_exclusive_scan<int64_t>(v, sh, tile_total);
#pragma unroll
    for (int i = 0; i < kScanIpt; ++i) {
        const bool mine = k0 + i < n_out;
        if (mine) out_offsets[k0 + i] = run;
        plan_sample(plan, mine, k0 + i, run, x[i]);
        run += x[i].len;
    }
    if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) {
        const int64_t total = tile_base + tile_total;
        out_offsets[n_out] = total;
        if (total > plan.cap_out) atomicOr(flags, kFlagOffsets);     // the copy stops there
    }
}

__global__ __launch_bounds__(256) void dispatch_splits_kernel(const sample_order order,
                                                              const int64_t *__restrict__ out_offsets) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; r < order.n_ranks; r += stride)
        order.splits[r] = rank_split(order, out_offsets, r);
}

// Pieces per workgroup, and groups of sixteen bytes in flight per lane.  What bounds the copy of a large output is the rate of
// a plain copy; what bounds a small one is the life of a workgroup, so that short tiles, many at once, are the faster ones.
// One permute of the whole operation, tiles of 2048 pieces of 16 bytes (8 in flight) / of 8192 (4 in flight): 8 MB of output
// 10.1 / 14.8 us, 20 MB 16.0 / 19.8, 39 MB 23.1 / 26.5, 45 MB 20.9 / 23.4, 52 MB 24.8 / 24.3, 65 MB 28.6 / 27.8, 90 MB 36.8 /
// 36.3, 134 MB 52.9 / 50.4, 183 MB 72.2 / 71.6.  Large outputs with 8 / 4 / 2 in flight: dispatch, combine and transpose of
// 128 MB 169.6 / 166.7 / 159.7 (tiles of 2048, 8 in flight: 164.1).
// 8-byte pieces, tiles of 2048 (4 in flight) / of 4096: 100 k samples of 1 to 200 IDs 18.6 / 19.9, 65 k of 16 to 4096 60.8 /
// 60.5; two in flight 64.4.  4-byte pieces: a large output pays for opening its tiles with too few bytes each; tiles of 2048
// (2 in flight) / 4096 (4): 1 M pieces 14.4 / 14.8, 16.7 M 39.0 / 38.8.
constexpr int kCopyTile16 = 2048, kCopyTile16Large = 8192, kCopyTile8 = 2048, kCopyTile4 = 2048, kCopyTile4Large = 4096;
constexpr int64_t kCopyLarge16 = 3 << 20, kCopyLarge4 = 9 << 20;        // pieces of the output
constexpr int kCopyWindow = 2048 + 2;                           // sample boundaries staged in LDS

// sixteen bytes of pieces of type V, wherever a piece may lie
template <typename V>
struct piece_group {
    typedef V type __attribute__((ext_vector_type(16 / sizeof(V)), aligned(sizeof(V))));
};
template <>
struct piece_group<u32x4> {
    typedef u32x4 type;
};
// V: the piece, the widest of 4, 8, 16 bytes that divides the element; ppe pieces per element.  A lane moves sixteen bytes
// of consecutive output pieces at a time, in one access each way where they belong to one sample.
// Inside a tile everything is counted from the tile's first piece in 32 bits (a division per piece would cost more than
// the copy).  Where samples start is a bit per piece of the tile: the sample of a piece is a matter of counting bits,
// however short the samples are, where a walk over a list of boundaries takes a dependent step for each.
template <typename V, int kCopyTile, int GROUPS>
__global__ __launch_bounds__(kScanThreads) void permute_copy_kernel(const V *__restrict__ values, int64_t n_pieces,
                                                                    const jagged_in in, const int32_t *__restrict__ sample_of,
                                                                    int64_t n_out, const int64_t *__restrict__ out_offsets,
                                                                    const copy_plan plan, V *__restrict__ out) {
    typedef typename piece_group<V>::type G;
    constexpr int W = 16 / (int)sizeof(V);                      // pieces of a group
    constexpr int kWords = kCopyTile / 32;
    static_assert(kWords <= kScanThreads && kWords % kWave == 0, "a thread per word, whole wavefronts");
    __shared__ uint32_t starts[kWords];         // a bit per piece of the tile that is the first of a sample
    __shared__ uint32_t below[kWords];          // bits before a word
    __shared__ int64_t w_delta[kCopyWindow];    // per bit: first input piece of the sample minus its first output piece
    __shared__ int64_t win[2];
    __shared__ uint32_t wave_sum[kScanThreads / kWave];
    const int ppe = plan.ppe;
    // (without a plan: of a sample that is not empty, so that the plan kernel has found its extent inside the values)
    auto delta_of = [&](int64_t k) -> int64_t {
        if (plan.delta != nullptr) return plan.delta[k];
        const int64_t p = sample_of[k];
        return p >= 0 && p < in.B ? in.offsets[p] - out_offsets[k] : 0;
    };
    int64_t ka = 0, kb = n_out - 1;
    const bool planned = plan.tile_first != nullptr;
    if (planned) {
        ka = plan.tile_first[blockIdx.x];                       // of a tile past the end: whatever, nobody uses it
        if (blockIdx.x + 1 < gridDim.x) kb = plan.tile_first[blockIdx.x + 1];
    }
    int64_t total = out_offsets[n_out];
    if (total > plan.cap_out) total = plan.cap_out;
    const int64_t pieces = total * ppe;
    const int64_t q0 = (int64_t)blockIdx.x * kCopyTile;
    if (q0 >= pieces || n_pieces <= 0) return;                  // whole workgroup
    const int tile_pieces = (int)((q0 + kCopyTile < pieces ? q0 + kCopyTile : pieces) - q0);
    if (q0 + kCopyTile >= pieces) kb = n_out - 1;               // the last tile: nobody wrote down what follows it
    // What a plan says is a place only inside the lists and the input (here, and where pieces are read): of a call that
    // overlaps another one of its context, which is not allowed, the rows are wrong, but no access is out of range.
    ka = ka < 0 ? 0 : ka < n_out ? ka : n_out - 1;
    kb = kb < ka ? ka : kb < n_out ? kb : n_out - 1;
    auto piece = [&](int64_t from) {
        return __builtin_nontemporal_load(values + ((uint64_t)from < (uint64_t)n_pieces ? from : 0));
    };
    if (!planned || kb - ka + 1 > kCopyWindow) {
        if (threadIdx.x < 2 * kWave) {
            // sample of an element e: the last k with out_offsets[k] <= e (empty samples in between are skipped);
            // the first wavefront looks for the sample of the tile's first element, the second for that of its last
            const int w = threadIdx.x / kWave;
            const int64_t e = (w == 0 ? q0 : q0 + tile_pieces - 1) / ppe;
            const int64_t k = wave_upper_bound<int64_t>(out_offsets, (int)(n_out + 1), e) - 1;
            if ((threadIdx.x & (kWave - 1)) == 0) win[w] = k;
        }
        __syncthreads();
        ka = win[0];
        kb = win[1];
    }
    const int64_t last = n_pieces - W;                          // the last place to read sixteen bytes from
    if (kb - ka + 1 > kCopyWindow || last < 0) {
        // the samples between the tile's first and last do not fit: many empty ones, or more of them than the window has
        // places for in a tile of wide pieces (or there are no sixteen bytes).  A search per piece.
        for (int l = threadIdx.x; l < tile_pieces; l += kScanThreads) {
            const int64_t e = (q0 + l) / ppe;
            int64_t lo = ka, hi = kb + 1;                       // first sample that starts behind the element
            while (lo < hi) {
                const int64_t mid = (lo + hi) >> 1;
                if (out_offsets[mid] <= e) lo = mid + 1; else hi = mid;
            }
            out[q0 + l] = piece(q0 + l + delta_of(lo > ka ? lo - 1 : ka) * ppe);
        }
        return;
    }
    const int wn = (int)(kb - ka + 1);
    // first piece of sample ka + j in the tile; past its end: empty, or not in this tile
    auto first_in_tile = [&](int j) -> int {
        const int64_t start = out_offsets[ka + j], next = out_offsets[ka + j + 1], rel = start * ppe - q0;
        return next <= start || rel >= kCopyTile ? kCopyTile : rel > 0 ? (int)rel : 0;
    };
    int rel0 = kCopyTile;                                       // this thread's first sample of the window
    int64_t delta0 = 0;
    if ((int)threadIdx.x < wn) {
        rel0 = first_in_tile(threadIdx.x);
        delta0 = delta_of(ka + threadIdx.x);
    }
    if ((int)threadIdx.x < kWords) starts[threadIdx.x] = 0;
    __syncthreads();
    for (int j = threadIdx.x; j < wn; j += kScanThreads) {
        const int rel = j == (int)threadIdx.x ? rel0 : first_in_tile(j);
        if (rel < kCopyTile) atomicOr(&starts[rel >> 5], 1u << (rel & 31));
    }
    __syncthreads();
    {
        const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
        const uint32_t c = (int)threadIdx.x < kWords ? (uint32_t)__popc(starts[threadIdx.x]) : 0u;
        const uint32_t inc = wave_inclusive_scan<uint32_t>(c);
        if (lane == kWave - 1) wave_sum[w] = inc;
        __syncthreads();
        uint32_t before = inc - c;
#pragma unroll
        for (int i = 0; i < kScanThreads / kWave; ++i) before += i < w ? wave_sum[i] : 0u;
        if ((int)threadIdx.x < kWords) below[threadIdx.x] = before;
    }
    __syncthreads();
    // the number of the sample that piece l of the tile belongs to
    auto sample_at = [&](int l) { return (int)below[l >> 5] + __popc(starts[l >> 5] & ((2u << (l & 31)) - 1u)) - 1; };
    for (int j = threadIdx.x; j < wn; j += kScanThreads) {
        const bool held = j == (int)threadIdx.x;
        const int rel = held ? rel0 : first_in_tile(j);
        if (rel < kCopyTile) w_delta[sample_at(rel)] = (held ? delta0 : delta_of(ka + j)) * ppe;
    }
    __syncthreads();
    // Wavefront w copies the w-th quarter of the tile, 64 consecutive groups per instruction, front to back.
    constexpr int kWavePieces = kCopyTile / (kScanThreads / kWave);
    const int lane = threadIdx.x & (kWave - 1);
    const int w0 = (int)(threadIdx.x / kWave) * kWavePieces;
    static_assert(kWavePieces % (kWave * W * GROUPS) == 0, "a wavefront's quarter is a whole number of rounds");
#pragma unroll 1
    for (int r0 = 0; r0 < kWavePieces; r0 += kWave * W * GROUPS) {
        if (w0 + r0 >= tile_pieces) break;                      // whole wavefront
        G v[GROUPS];                                            // in flight per lane
        bool split[GROUPS];                                     // the group has the end of a sample or of the output
        // boundaries behind the first piece of a group: bit k - 1, piece k
        auto cuts_of = [&](int l) { return W == 1 ? 0u : (starts[l >> 5] >> (l & 31) >> 1) & ((1u << (W - 1)) - 1u); };
        // read once, written once: keeping either in the caches only pushes out the boundaries (three
        // shuffles of 250 k rows of 512 bytes: 202 us with plain accesses, 185 with the hint on the loads
        // only, 177 on both; at the rate of a plain copy now)
#pragma unroll
        for (int i = 0; i < GROUPS; ++i) {
            const int l = w0 + r0 + (i * kWave + lane) * W;     // first piece of the group
            const int at = l < tile_pieces ? l : tile_pieces - 1;
            // (every lane loads, from where sixteen bytes are: a load that only some lanes make waits for the one before)
            const int64_t from = q0 + at + w_delta[sample_at(at)];
            v[i] = __builtin_nontemporal_load(reinterpret_cast<const G *>(values + ((uint64_t)from < (uint64_t)last ? from : last)));
            split[i] = W > 1 && l < tile_pieces && (l + W > tile_pieces || cuts_of(l) != 0);
        }
        if constexpr (W > 1) {
            // the pieces of a divided group come one by one and are put together here: stored one by one they would leave
            // gaps in the lines that the rest of the wavefront writes
            V one[GROUPS][W];
#pragma unroll
            for (int i = 0; i < GROUPS; ++i)
                if (split[i]) {
                    const int l = w0 + r0 + (i * kWave + lane) * W;
#pragma unroll
                    for (int k = 0; k < W; ++k) {
                        const int at = l + k < tile_pieces ? l + k : tile_pieces - 1;
                        one[i][k] = piece(q0 + at + w_delta[sample_at(at)]);
                    }
                }
#pragma unroll
            for (int i = 0; i < GROUPS; ++i)
#pragma unroll
                for (int k = 0; k < W; ++k) v[i][k] = split[i] ? one[i][k] : v[i][k];
        }
#pragma unroll
        for (int i = 0; i < GROUPS; ++i) {
            const int l = w0 + r0 + (i * kWave + lane) * W;
            if (l + W <= tile_pieces) __builtin_nontemporal_store(v[i], reinterpret_cast<G *>(out + q0 + l));
            else if constexpr (W > 1) {
#pragma unroll
                for (int k = 0; k < W; ++k)
                    if (l + k < tile_pieces) __builtin_nontemporal_store((V)v[i][k], out + q0 + l + k);
            }
        }
    }
}

// output samples in the order `order`, whose list is `sample_of` (written here unless the caller gave it)
static int launch_ordered_copy(fs_ctx *ctx, const void *values, int64_t n_values, int32_t elem_bytes,
                               const int64_t *offsets, int64_t B, const sample_order &order, int64_t n_out,
                               void *out_values, int64_t cap_out, int64_t *out_offsets, hipStream_t s) {
    const jagged_in in = {offsets, B, n_values};
    const int32_t *sample_of = order.mode == kMapGiven ? order.given : ctx->jag_sel;
    const int piece = elem_bytes % 16 == 0 ? 16 : (elem_bytes % 8 == 0 ? 8 : 4);
    const int ppe = elem_bytes / piece;
    const bool large = piece != 8 && cap_out * ppe >= (piece == 16 ? kCopyLarge16 : kCopyLarge4);
    const int tile = piece == 16 ? (large ? kCopyTile16Large : kCopyTile16) : piece == 8 ? kCopyTile8
                                                                            : (large ? kCopyTile4Large : kCopyTile4);
    const int64_t blocks = n_out > 0 ? ceil_div(cap_out * ppe, tile) : 0;
    if (blocks > 0x7fffffffll) return set_err(ctx, FS_EINVAL, "indexed permute: output too large for one launch");
    const bool own = order.mode == kMapGiven && n_out <= kOwnPermute;
    const copy_plan plan = {own ? nullptr : ctx->jag_delta, own || blocks > 2 * ctx->max_ids ? nullptr : ctx->jag_tile_first,
                            cap_out, ppe, 31 - __builtin_clz(tile)};
    if (own || n_out <= (int64_t)kPlanThreads * kPlanPer) {
        auto *kernel = n_out <= (int64_t)kPlanThreads * kPlanPer ? &jagged_plan_kernel<kPlanPer> : &jagged_plan_kernel<kOwnPer>;
        hipLaunchKernelGGL(kernel, dim3(1), dim3(kPlanThreads), 0, s, in, order, (int)n_out, plan, out_offsets,
                           ctx->d_flags);
    } else {
        const int tiles = (int)ceil_div(n_out, kScanTile);
        hipLaunchKernelGGL(permute_tile_sum_kernel, dim3((unsigned)tiles), dim3(kScanThreads), 0, s, in, order,
                           ctx->jag_sel, n_out, ctx->jag_tile_sum, ctx->d_flags);
        hipLaunchKernelGGL(permute_offsets_kernel, dim3((unsigned)tiles), dim3(kScanThreads), 0, s, in, sample_of,
                           n_out, ctx->jag_tile_sum, plan, out_offsets, ctx->d_flags);
        if (order.splits != nullptr)
            hipLaunchKernelGGL(dispatch_splits_kernel, dim3((unsigned)ceil_div(order.n_ranks, 256)), dim3(256), 0, s, order,
                               out_offsets);
    }
    if (blocks > 0) {
        const dim3 grid((unsigned)blocks);
#define FS_COPY(V, TILE, GROUPS)                                                                                       \
    hipLaunchKernelGGL((permute_copy_kernel<V, TILE, GROUPS>), grid, dim3(kScanThreads), 0, s, (const V *)values,      \
                       n_values * ppe, in, sample_of, n_out, out_offsets, plan, (V *)out_values)
        if (piece == 16 && large) FS_COPY(u32x4, kCopyTile16Large, 2);
        else if (piece == 16) FS_COPY(u32x4, kCopyTile16, 8);
        else if (piece == 8) FS_COPY(uint64_t, kCopyTile8, 4);
        else if (large) FS_COPY(uint32_t, kCopyTile4Large, 4);
        else FS_COPY(uint32_t, kCopyTile4, 2);
#undef FS_COPY
    }
    FS_LAUNCH_CHECK(ctx, "indexed permute kernels");
    return FS_OK;
}

int launch_indexed_permute(fs_ctx *ctx, const void *values, int64_t n_values, int32_t elem_bytes,
                           const int64_t *offsets, int64_t B, const int32_t *sample_of, int64_t n_out, void *out_values,
                           int64_t cap_out, int64_t *out_offsets, hipStream_t s) {
    const sample_order order = {kMapGiven, sample_of, 0, 0, nullptr, 0, nullptr};
    return launch_ordered_copy(ctx, values, n_values, elem_bytes, offsets, B, order, n_out, out_values, cap_out, out_offsets, s);
}

// ---- VBS: cuts of about equal weight --------------------------------------------------------------------
// Sorted position s goes to rank min(n - 1, floor(n * w_before(s) / W)): weights are integers (a table per
// length), so every cut is exact.  Two launches after the sort: weights summed per tile of 1024 sorted
// positions; then every workgroup adds up the tile sums (the total W and its own start), scans its tile and
// writes the start of every rank whose first sample lies in it.
__device__ __forceinline__ int64_t vbs_weight(const int64_t *__restrict__ lengths, const int32_t *__restrict__ sorted,
                                              const int64_t *__restrict__ weight_of_len, int64_t max_len, int64_t s,
                                              int64_t B, bool &bad) {
    if (s < 0 || s >= B) return 0;
    const int64_t len = lengths[sorted[s]];
    if (len < 0 || len > max_len) return 0;              // the sort has reported it already
    const int64_t w = weight_of_len[len];
    if (w < 0) { bad = true; return 0; }
    return w;
}

__global__ __launch_bounds__(kScanThreads) void vbs_tile_sum_kernel(const int64_t *__restrict__ lengths,
                                                                    const int32_t *__restrict__ sorted, int64_t B,
                                                                    const int64_t *__restrict__ weight_of_len,
                                                                    int64_t max_len, int64_t *__restrict__ tile_sum,
                                                                    int *__restrict__ flags) {
    __shared__ int64_t sh[kScanThreads / kWave];
    const int64_t s0 = (int64_t)blockIdx.x * kScanTile + threadIdx.x * kScanIpt;
    bool bad = false;
    int64_t v = 0;
#pragma unroll
    for (int i = 0; i < kScanIpt; ++i) v += vbs_weight(lengths, sorted, weight_of_len, max_len, s0 + i, B, bad);
    int64_t total;
    (void)block_exclusive_scan<int64_t>(v, sh, total);
    if (threadIdx.x == 0) tile_sum[blockIdx.x] = total;
    if (bad) atomicOr(flags, kFlagRowRange);
}

__device__ __forceinline__ int64_t vbs_rank(int64_t before, int64_t total, int64_t n) {
    if (total <= 0) return 0;
    const int64_t q = (int64_t)((uint64_t)n * (uint64_t)before / (uint64_t)total);      // n * total < 2^63 (checked)
    return q >= n ? n - 1 : q;
}

__global__ __launch_bounds__(kScanThreads) void vbs_cut_kernel(const int64_t *__restrict__ lengths,
                                                               const int32_t *__restrict__ sorted, int64_t B,
                                                               const int64_t *__restrict__ weight_of_len, int64_t max_len,
                                                               const int64_t *__restrict__ tile_sum, int tiles, int64_t n,
                                                               int64_t *__restrict__ rank_offsets,
                                                               int *__restrict__ flags) {
    __shared__ int64_t sh[kScanThreads / kWave];
    if (B == 0) {                                          // one workgroup: every rank starts (and ends) at 0
        for (int64_t r = threadIdx.x; r <= n; r += kScanThreads) rank_offsets[r] = 0;
        return;
    }
    int64_t mine = 0, all = 0;
    for (int t = threadIdx.x; t < tiles; t += kScanThreads) {
        const int64_t v = tile_sum[t];
        all += v;
        if (t < (int)blockIdx.x) mine += v;
    }
    int64_t tile_base, total;
    (void)block_exclusive_scan<int64_t>(mine, sh, tile_base);
    (void)block_exclusive_scan<int64_t>(all, sh, total);
    if (total < 0 || total > INT64_MAX / n) {              // n * w_before would not fit: refuse, one rank takes all
        if (blockIdx.x == 0 && threadIdx.x == 0) atomicOr(flags, kFlagRowRange);
        total = 0;
    }
    const int64_t s0 = (int64_t)blockIdx.x * kScanTile + threadIdx.x * kScanIpt;
    bool bad = false;
    int64_t w[kScanIpt], v = 0;
#pragma unroll
    for (int i = 0; i < kScanIpt; ++i) {
        w[i] = vbs_weight(lengths, sorted, weight_of_len, max_len, s0 + i, B, bad);
        v += w[i];
    }
    const int64_t w_prev = vbs_weight(lengths, sorted, weight_of_len, max_len, s0 - 1, B, bad);
    int64_t tile_total;
    int64_t before = tile_base + block_exclusive_scan<int64_t>(v, sh, tile_total);
    // rank of the position before mine (-1 before the first: rank 0 starts at position 0)
    int64_t r_prev = s0 > 0 ? vbs_rank(before - w_prev, total, n) : -1;
#pragma unroll
    for (int i = 0; i < kScanIpt; ++i) {
        const int64_t s = s0 + i;
        if (s < B) {
            const int64_t r = vbs_rank(before, total, n);
            for (int64_t x = r_prev + 1; x <= r; ++x) rank_offsets[x] = s;
            r_prev = r;
            before += w[i];
            if (s == B - 1)
                for (int64_t x = r + 1; x <= n; ++x) rank_offsets[x] = B;
        }
    }
}

int launch_partition_vbs(fs_ctx *ctx, const int64_t *lengths, int64_t B, const int64_t *weight_of_len, int64_t max_len,
                         int32_t n_ranks, int32_t *sample_of, int64_t *rank_offsets, hipStream_t s) {
    const int tiles = (int)(B > 0 ? ceil_div(B, kScanTile) : 1);
    if (B > 0) {
        fs_unique_job job = {lengths, B, max_len + 1, ctx->jag_unique, ctx->jag_seg, sample_of, nullptr, ctx->jag_n};
        job.order_only = true;
        const int rc = launch_unique_batch(ctx, 1, &job, s, 0, true);
        if (rc != FS_OK) return rc;
        hipLaunchKernelGGL(vbs_tile_sum_kernel, dim3((unsigned)tiles), dim3(kScanThreads), 0, s, lengths, sample_of, B,
                           weight_of_len, max_len, ctx->jag_tile_sum, ctx->d_flags);
    }
    hipLaunchKernelGGL(vbs_cut_kernel, dim3((unsigned)tiles), dim3(kScanThreads), 0, s, lengths, sample_of, B,
                       weight_of_len, max_len, ctx->jag_tile_sum, tiles, (int64_t)n_ranks, rank_offsets, ctx->d_flags);
    FS_LAUNCH_CHECK(ctx, "vbs kernels");
    return FS_OK;
}

// ---- keyed transpose, ranged dispatch, ranged combine ---------------------------------------------------
int launch_keyed_shuffle(fs_ctx *ctx, int mode, const void *values, int64_t n_values, int32_t elem_bytes,
                         const int64_t *offsets, int64_t F, int64_t B, const int64_t *rank_offsets, int32_t n_ranks,
                         void *out_values, int64_t *out_offsets, int64_t *splits, hipStream_t s) {
    const int64_t segs = F * B;
    const sample_order order = {mode, nullptr, F, B, rank_offsets, (int)n_ranks, splits};
    return launch_ordered_copy(ctx, values, n_values, elem_bytes, offsets, segs, order, segs, out_values, n_values,
                               out_offsets, s);
}

}  // namespace fs
