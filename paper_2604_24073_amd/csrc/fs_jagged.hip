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
// item what a short one costs): a workgroup takes 2048 to 8192 consecutive output pieces, finds the samples
// they belong to with two 64-ary searches, stages their boundaries in LDS and lets every piece
// binary-search LDS.
//
// VBS: the same sort, then the sorted order is cut into n runs of about equal total weight.
//
// Keyed transpose, ranged dispatch and ranged combine (same section of the paper) are the same copy
// under a computed order of the F x B segments of a keyed jagged tensor, written down where the lengths
// are summed.
#include "fs_common.h"
#include "fs_device.h"

namespace fs {

// ---- FBS: the deal ------------------------------------------------------------------------------------
// full rounds R = B / n, m = B % n samples in the last, partial round (round R): forth if R is even
// (ranks 0..m-1 get one more), back if R is odd (ranks n-m..n-1 get one more)
__device__ __forceinline__ int64_t fbs_rank_start(int64_t i, int64_t n, int64_t R, int64_t m) {
    const int64_t extra = (R % 2 == 0) ? (i < m ? i : m) : (i > n - m ? i - (n - m) : 0);
    return i * R + extra;
}

__global__ __launch_bounds__(256) void fbs_deal_kernel(const int32_t *__restrict__ sorted, int64_t B, int64_t n,
                                                       int32_t *__restrict__ sample_of,
                                                       int64_t *__restrict__ rank_offsets) {
    const int64_t R = B / n, m = B % n;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    const int64_t gtid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    for (int64_t i = gtid; i <= n; i += stride) rank_offsets[i] = fbs_rank_start(i, n, R, m);
    for (int64_t s = gtid; s < B; s += stride) {
        const int64_t r = s / n, c = s % n;
        const int64_t i = (r % 2 == 0) ? c : n - 1 - c;
        sample_of[fbs_rank_start(i, n, R, m) + r] = sorted[s];
    }
}

int launch_partition_fbs(fs_ctx *ctx, const int64_t *lengths, int64_t B, int64_t max_len, int32_t n_ranks,
                         int32_t *sample_of, int64_t *rank_offsets, hipStream_t s) {
    if (B > 0) {
        const int rc = launch_unique(ctx, lengths, B, max_len + 1, ctx->jag_unique, ctx->jag_seg, ctx->jag_sorted,
                                     nullptr, ctx->jag_n, s, 0);
        if (rc != FS_OK) return rc;
    }
    const int64_t work = B > n_ranks ? B : (int64_t)n_ranks + 1;
    int64_t blocks = ceil_div(work, 256);
    if (blocks > 1024) blocks = 1024;
    hipLaunchKernelGGL(fbs_deal_kernel, dim3((unsigned)blocks), dim3(256), 0, s, ctx->jag_sorted, B, (int64_t)n_ranks,
                       sample_of, rank_offsets);
    FS_LAUNCH_CHECK(ctx, "fbs_deal_kernel");
    return FS_OK;
}

// ---- indexed permute ------------------------------------------------------------------------------------
struct jagged_in {
    const int64_t *offsets;   // [B + 1]
    int64_t B, n_values;      // samples, elements behind them
};

// length of input sample p (0 and a flag for a sample index out of range or a sample whose boundaries are not inside
// the values: such a sample is never read)
__device__ __forceinline__ int64_t sample_len(const jagged_in &in, int64_t p, bool &bad) {
    if (p < 0 || p >= in.B) { bad = true; return 0; }
    const int64_t a = in.offsets[p], b = in.offsets[p + 1];
    if (a < 0 || b < a || b > in.n_values) { bad = true; return 0; }
    return b - a;
}

// length of output sample k (0 past the end)
__device__ __forceinline__ int64_t out_len(const jagged_in &in, const int32_t *__restrict__ sample_of, int64_t k,
                                           int64_t n_out, bool &bad) {
    return k < n_out ? sample_len(in, sample_of[k], bad) : 0;
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
// shuffles of 1024 segments spent three to four of them on it).  One workgroup, up to kPlanPer consecutive samples
// a thread; beyond that one compute unit takes longer than two launches over many.
constexpr int kPlanThreads = 1024;
constexpr int kPlanPer = 8;
constexpr int kPlanRanks = 1024;                 // rank boundaries kept in LDS

__global__ __launch_bounds__(kPlanThreads) void jagged_plan_kernel(const jagged_in in, const sample_order order,
                                                                   int32_t *sel, int n_out, int64_t cap_out,
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
    const int per = (n_out + kPlanThreads - 1) / kPlanThreads;           // at most kPlanPer
    const int k0 = (int)threadIdx.x * per;
    int32_t p[kPlanPer];
#pragma unroll
    for (int i = 0; i < kPlanPer; ++i) {
        p[i] = -1;
        if (i < per && k0 + i < n_out) {
            if (order.mode == kMapGiven) {
                p[i] = order.given[k0 + i];
            } else {
                p[i] = ordered_segment(order, ro, k0 + i);
                sel[k0 + i] = p[i];
            }
        }
    }
    int64_t len[kPlanPer], v = 0;
#pragma unroll
    for (int i = 0; i < kPlanPer; ++i) {
        len[i] = (i < per && k0 + i < n_out) ? sample_len(in, p[i], bad) : 0;
        v += len[i];
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
    for (int i = 0; i < kPlanPer; ++i) {
        if (i < per && k0 + i < n_out) out_offsets[k0 + i] = run;
        run += len[i];
    }
    if (threadIdx.x == 0) {
        out_offsets[n_out] = total;
        bad |= total > cap_out;                                          // the copy stops at cap_out
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
            v += sample_len(in, p, bad);
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
                                                                       int64_t cap_out, int64_t *__restrict__ out_offsets,
                                                                       int *__restrict__ flags) {
    __shared__ int64_t sh[kScanThreads / kWave];
    int64_t before = 0;
    for (int t = threadIdx.x; t < (int)blockIdx.x; t += kScanThreads) before += tile_sum[t];
    int64_t tile_base;
    (void)block_exclusive_scan<int64_t>(before, sh, tile_base);
    const int64_t k0 = (int64_t)blockIdx.x * kScanTile + threadIdx.x * kScanIpt;
    bool bad = false;
    int64_t len[kScanIpt], v = 0;
#pragma unroll
    for (int i = 0; i < kScanIpt; ++i) {
        len[i] = out_len(in, sample_of, k0 + i, n_out, bad);
        v += len[i];
    }
    int64_t tile_total;
    int64_t run = tile_base + block_exclusive_scan<int64_t>(v, sh, tile_total);
#pragma unroll
    for (int i = 0; i < kScanIpt; ++i) {
        if (k0 + i < n_out) out_offsets[k0 + i] = run;
        run += len[i];
    }
    if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) {
        const int64_t total = tile_base + tile_total;
        out_offsets[n_out] = total;
        if (total > cap_out) atomicOr(flags, kFlagOffsets);     // the copy stops at cap_out
    }
}

__global__ __launch_bounds__(256) void dispatch_splits_kernel(const sample_order order,
                                                              const int64_t *__restrict__ out_offsets) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; r < order.n_ranks; r += stride)
        order.splits[r] = rank_split(order, out_offsets, r);
}

// Pieces per workgroup.  A copy of whole rows wants long stretches: the searches that open a tile are a chain of
// dependent loads that queue behind the rows of the other workgroups (250 k rows of 512 bytes, 16-byte pieces: 50 us
// with 128 KB a workgroup, 100 to 160 with 32 or 64 KB).  Where samples are short the walk over their boundaries
// counts, and more, shorter-lived wavefronts hide it: 16 KB of 8-byte pieces (eight in flight per lane) against 32 KB
// (sixteen), a whole balancer pass: samples of 1 to 200 IDs 198 -> 90 us, of 16 to 4096 IDs 108 -> 107.
// 4-byte pieces: a large output pays for the searches with too few bytes a tile, a small one fills the chip with short
// tiles only.  Tiles of 2048 (eight in flight) / 4096 (sixteen), one permute: 500 k pieces 22.3 / 31 us, 1 M 21.7 / 27.6,
// 8 M 38.5 / 38.3, 9 M 42.0 / 42.1, 10 M 48.5 / 43.0, 12.5 M 51.3 / 45.1, 32 M 99.8 / 87.3.
constexpr int kCopyTile16 = 8192, kCopyTile8 = 2048, kCopyTile4 = 2048, kCopyTile4Large = 4096;
constexpr int64_t kCopyLargeFrom = 9 << 20;                     // 4-byte pieces of the output
constexpr int kCopyWindow = 2048 + 2;                           // sample boundaries staged in LDS

// V: the piece, the widest of 4, 8, 16 bytes that divides the element; ppe pieces per element.
// Inside a tile everything is counted from the tile's first element in 32 bits (a 64-bit division per
// piece would cost more than the copy).
template <typename V, int kCopyTile, int PIECES>
__global__ __launch_bounds__(kScanThreads) void permute_copy_kernel(const V *__restrict__ values, const jagged_in in,
                                                                    const int32_t *__restrict__ sample_of,
                                                                    int64_t n_out, const int64_t *__restrict__ out_offsets,
                                                                    int64_t cap_out, int ppe, V *__restrict__ out) {
    __shared__ int32_t w_rel[kCopyWindow];      // out_offsets[ka + j] minus the tile's first element (at least -1)
    __shared__ int64_t w_delta[kCopyWindow];    // first input element of sample ka + j minus its first output element
    __shared__ int64_t win[2];
    const int64_t *__restrict__ offsets = in.offsets;
    int64_t total = out_offsets[n_out];
    if (total > cap_out) total = cap_out;
    const int64_t pieces = total * ppe;
    const int64_t q0 = (int64_t)blockIdx.x * kCopyTile;
    if (q0 >= pieces) return;                                   // whole workgroup
    const uint32_t tile_pieces = (uint32_t)((q0 + kCopyTile < pieces ? q0 + kCopyTile : pieces) - q0);
    const int64_t e0 = q0 / ppe;                                // first element of the tile
    const uint32_t rem0 = (uint32_t)(q0 - e0 * ppe);            // pieces of it that belong to the tile before
    const int64_t e1 = (q0 + tile_pieces - 1) / ppe;            // last element of the tile
    if (threadIdx.x < 2 * kWave) {
        // sample of an element e: the last k with out_offsets[k] <= e (empty samples in between are skipped);
        // the first wavefront looks for the sample of the tile's first element, the second for that of its last
        const int w = threadIdx.x / kWave;
        const int64_t k = wave_upper_bound<int64_t>(out_offsets, (int)(n_out + 1), w == 0 ? e0 : e1) - 1;
        if ((threadIdx.x & (kWave - 1)) == 0) win[w] = k;
    }
    __syncthreads();
    const int64_t ka = win[0], kb = win[1];
    const bool staged = kb - ka + 1 <= kCopyWindow;             // else: the samples touched by the tile do not fit
    const int wn = staged ? (int)(kb - ka + 1) : 0;
    if (staged)
        for (int j = threadIdx.x; j < wn; j += kScanThreads) {
            const int64_t start = out_offsets[ka + j];
            const int64_t p = sample_of[ka + j];
            w_rel[j] = start < e0 ? -1 : (int32_t)(start - e0);                // start - e0 <= kCopyTile
            w_delta[j] = (p >= 0 && p < in.B) ? offsets[p] - start : 0;        // a flagged sample is empty: never used
        }
    __syncthreads();
    // Wavefront w copies the w-th quarter of the tile, 64 consecutive pieces per instruction, front to back:
    // the sample of a lane's piece only moves forward, so after one binary search per lane the boundary
    // list is walked (a step every few instructions for samples of a few hundred elements; never more
    // steps per lane and tile than the list is long).
    const uint32_t uppe = (uint32_t)ppe;
    constexpr uint32_t kWavePieces = kCopyTile / (kScanThreads / kWave);
    const uint32_t lane = threadIdx.x & (kWave - 1);
    const uint32_t w0 = (threadIdx.x / kWave) * kWavePieces;
    const int64_t wn_all = kb - ka + 1;
    int64_t j = 0;                                              // sample ka + j holds the lane's current piece
    {
        const uint32_t t = rem0 + w0 + lane;
        const int64_t le = uppe == 1 ? t : t / uppe;
        int64_t lo = 0, hi = wn_all;                            // first j with start[j] > element
        while (lo < hi) {
            const int64_t mid = (lo + hi) >> 1;
            const bool le_mid = staged ? (w_rel[mid] <= (int32_t)le) : (out_offsets[ka + mid] <= e0 + le);
            if (le_mid) lo = mid + 1; else hi = mid;
        }
        j = lo - 1;
    }
    static_assert(kWavePieces % (kWave * PIECES) == 0, "a wavefront's quarter is a whole number of rounds");
    for (uint32_t r0 = 0; r0 < kWavePieces; r0 += kWave * PIECES) {
        if (w0 + r0 >= tile_pieces) break;                      // whole wavefront
        V v[PIECES];                                            // in flight per lane
        bool live[PIECES];
#pragma unroll
        for (int i = 0; i < PIECES; ++i) {
            const uint32_t l = w0 + r0 + (uint32_t)i * kWave + lane;                // piece of the tile
            live[i] = l < tile_pieces;
            if (live[i]) {
                const uint32_t t = rem0 + l;
                const uint32_t le = uppe == 1 ? t : t / uppe;                       // element of the tile
                const uint32_t pin = t - le * uppe;                                 // piece of the element
                int64_t delta;
                if (staged) {
                    while (j + 1 < wn_all && w_rel[j + 1] <= (int32_t)le) ++j;
                    delta = w_delta[j];
                } else {
                    const int64_t e = e0 + le;
                    while (j + 1 < wn_all && out_offsets[ka + j + 1] <= e) ++j;
                    delta = offsets[sample_of[ka + j]] - out_offsets[ka + j];
                }
                // read once, written once: keeping either in the caches only pushes out the boundaries (three
                // shuffles of 250 k rows of 512 bytes: 202 us with plain accesses, 185 with the hint on the loads
                // only, 177 on both; at the rate of a plain copy now)
                v[i] = __builtin_nontemporal_load(&values[(e0 + le + delta) * ppe + pin]);
            }
        }
#pragma unroll
        for (int i = 0; i < PIECES; ++i) {
            const uint32_t l = w0 + r0 + (uint32_t)i * kWave + lane;
            if (live[i]) __builtin_nontemporal_store(v[i], &out[q0 + l]);
        }
    }
}

// output samples in the order `order`, whose list is `sample_of` (written here unless the caller gave it)
static int launch_ordered_copy(fs_ctx *ctx, const void *values, int64_t n_values, int32_t elem_bytes,
                               const int64_t *offsets, int64_t B, const sample_order &order, int64_t n_out,
                               void *out_values, int64_t cap_out, int64_t *out_offsets, hipStream_t s) {
    const jagged_in in = {offsets, B, n_values};
    const int32_t *sample_of = order.mode == kMapGiven ? order.given : ctx->jag_sel;
    if (n_out <= (int64_t)kPlanThreads * kPlanPer) {
        hipLaunchKernelGGL(jagged_plan_kernel, dim3(1), dim3(kPlanThreads), 0, s, in, order, ctx->jag_sel, (int)n_out,
                           cap_out, out_offsets, ctx->d_flags);
    } else {
        const int tiles = (int)ceil_div(n_out, kScanTile);
        hipLaunchKernelGGL(permute_tile_sum_kernel, dim3((unsigned)tiles), dim3(kScanThreads), 0, s, in, order,
                           ctx->jag_sel, n_out, ctx->jag_tile_sum, ctx->d_flags);
        hipLaunchKernelGGL(permute_offsets_kernel, dim3((unsigned)tiles), dim3(kScanThreads), 0, s, in, sample_of,
                           n_out, ctx->jag_tile_sum, cap_out, out_offsets, ctx->d_flags);
        if (order.splits != nullptr)
            hipLaunchKernelGGL(dispatch_splits_kernel, dim3((unsigned)ceil_div(order.n_ranks, 256)), dim3(256), 0, s, order,
                               out_offsets);
    }
    if (cap_out > 0 && n_out > 0) {
        const int piece = elem_bytes % 16 == 0 ? 16 : (elem_bytes % 8 == 0 ? 8 : 4);
        const int ppe = elem_bytes / piece;
        const bool large = piece == 4 && cap_out * ppe >= kCopyLargeFrom;
        const int tile = piece == 16 ? kCopyTile16 : (piece == 8 ? kCopyTile8 : (large ? kCopyTile4Large : kCopyTile4));
        const int64_t blocks = ceil_div(cap_out * ppe, tile);
        if (blocks > 0x7fffffffll) return set_err(ctx, FS_EINVAL, "indexed permute: output too large for one launch");
        const dim3 grid((unsigned)blocks);
        if (piece == 16)
            hipLaunchKernelGGL((permute_copy_kernel<u32x4, kCopyTile16, 8>), grid, dim3(kScanThreads), 0, s, (const u32x4 *)values,
                               in, sample_of, n_out, out_offsets, cap_out, ppe, (u32x4 *)out_values);
        else if (piece == 8)
            hipLaunchKernelGGL((permute_copy_kernel<uint64_t, kCopyTile8, 8>), grid, dim3(kScanThreads), 0, s, (const uint64_t *)values,
                               in, sample_of, n_out, out_offsets, cap_out, ppe, (uint64_t *)out_values);
        else if (large)
            hipLaunchKernelGGL((permute_copy_kernel<uint32_t, kCopyTile4Large, 16>), grid, dim3(kScanThreads), 0, s, (const uint32_t *)values,
                               in, sample_of, n_out, out_offsets, cap_out, ppe, (uint32_t *)out_values);
        else
            hipLaunchKernelGGL((permute_copy_kernel<uint32_t, kCopyTile4, 8>), grid, dim3(kScanThreads), 0, s, (const uint32_t *)values,
                               in, sample_of, n_out, out_offsets, cap_out, ppe, (uint32_t *)out_values);
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
        const int rc = launch_unique(ctx, lengths, B, max_len + 1, ctx->jag_unique, ctx->jag_seg, sample_of, nullptr,
                                     ctx->jag_n, s, 0);
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
