// The self-contained step of a small batch in two launches instead of three: the index half (one workgroup, fs_small.h) and
// the update of the batch (fs_rows.h) depend on nothing of each other, so they are workgroups of one launch; the lookup
// follows.  Bound by the dependent rounds of the longer of the two, the index half (1 k IDs 11.8 us, where update and index
// half one after the other are 20).  Workgroups have 1024 threads because the index half needs them; the update keeps the
// chunks of sixteen positions that it has at these sizes, so its sums have the same order as in a launch of its own.
#include <atomic>

#include "fs_rows.h"
#include "fs_small.h"

namespace fs {

constexpr int kStepWaves = kSmallThreads / kWave;
constexpr int kStepChunk = 16;                            // positions of a chunk (chunk_log2 of a batch of this size)
constexpr int kStepParked = kStepChunk / (FS_SHORT_SEGMENT + 1) + 1;     // segments that can end in one
static_assert(kSmallIdsInline < 65536, "chunks of sixteen positions");

struct small_step_job {
    small_dedup d;
    small_split s;
    batch_update_job u;
    int lpr, short_blocks;
};

template <row_use USE, int LPR>
__device__ __forceinline__ void step_rows(const batch_update_job &job, int block, int short_blocks, char *lds, int *flags) {
    constexpr int GPW = kWave / LPR;
    constexpr int kRound = kStepChunk / GPW > 1 ? kStepChunk / GPW : 1;   // row-group loads that take a whole chunk
    constexpr int UNR = kRound < fused_unr<LPR>() ? kRound : fused_unr<LPR>();
    typedef parked_rows<LPR, kStepWaves, kStepParked> parked;
    int64_t n_u = *job.n_unique_dev;
    n_u = n_u < 0 ? 0 : (n_u > job.n ? job.n : n_u);
    if (block < job.long_blocks)
        long_segments_of_layout<USE, LPR, UNR>(*reinterpret_cast<parked *>(lds), block, job.chunk_log2, job.grads, job.perm, job.n,
                                               job.seg_offsets, job.u_t, (int)n_u, job.table, job.state, job.num_rows, job.gvec,
                                               job.lr, job.eps, job.reduced, job.part_head, job.part_last, job.cnt_seg,
                                               job.cnt_sup, flags);
    else
        short_rows_body<USE, LPR, FS_SHORT_UNR, true, kStepWaves>(block - job.long_blocks, short_blocks, job.grads, job.n,
                                                                  row_source{nullptr, job.u_t, job.seg_offsets, job.perm}, n_u,
                                                                  job.table, job.state, job.num_rows, job.gvec, job.lr, job.eps,
                                                                  job.reduced, flags);
}

template <int KPT, bool BF16>
__global__ __launch_bounds__(kSmallThreads) void small_step_kernel(const small_step_job job, int *__restrict__ flags) {
    FS_WG_TRACE(12);
    extern __shared__ __align__(16) char lds[];
    __shared__ small_shared sh;
    if (blockIdx.x == 0) {
        small_dedup_body<KPT>(job.d, lds, sh, flags);
        __syncthreads();                                     // U_t1 is written
        small_split_body(job.s, kSmallThreads * KPT, lds, sh, flags);
        return;
    }
    constexpr row_use USE = BF16 ? kUpdateBf16 : kUpdateF32;
    const int block = (int)blockIdx.x - 1;
#define FS_CASE(L) \
    case L: step_rows<USE, L>(job.u, block, job.short_blocks, lds, flags); break;
    switch (job.lpr) { FS_CASE(1) FS_CASE(2) FS_CASE(4) FS_CASE(8) FS_CASE(16) FS_CASE(32) FS_CASE(64) }
#undef FS_CASE
}

template <int KPT, bool BF16>
static hipError_t small_step_launch(fs_ctx *ctx, const small_step_job &job, unsigned blocks, hipStream_t s) {
    constexpr size_t index = small_split_lds((size_t)kSmallThreads * KPT), rows = sizeof(parked_rows<kWave, kStepWaves, kStepParked>);
    constexpr size_t lds = index > rows ? index : rows;
    auto *kernel = &small_step_kernel<KPT, BF16>;
    if (lds > 48 * 1024) {                                   // asked for once per GPU
        static std::atomic<uint64_t> asked{0};
        const uint64_t bit = 1ull << (ctx->device & 63);
        if (!(asked.load(std::memory_order_acquire) & bit)) {
            const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kernel),
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
            if (e != hipSuccess) return e;
            asked.fetch_or(bit, std::memory_order_release);
        }
    }
    hipLaunchKernelGGL(kernel, dim3(blocks), dim3(kSmallThreads), lds, s, job, ctx->d_flags);
    return hipGetLastError();
}

bool small_step_fits(const fs_unique_job &u, const fs_split_job &sp, const fs_class_job &cls) {
    return u.n > 0 && cls.n > 0 && small_unique_fits(1, &u, 0) && small_split_fits(1, &sp, &cls, 0, true);
}

int launch_small_step(fs_ctx *ctx, const fs_unique_job &u, const fs_split_job &sp, const fs_class_job &cls,
                      const fs_batch_update_job &up, hipStream_t s) {
    small_step_job job;
    job.d = small_dedup_job(u);
    job.s = small_split_job(sp, &cls);
    job.u = batch_job(ctx, up, 0);
    job.lpr = lanes_per_row(job.u.gvec);
    if (job.lpr > kWave) return set_err(ctx, FS_EINVAL, "update: dim beyond 256");
    job.u.long_blocks = (int)ceil_div(ceil_div(up.n, kStepChunk), kStepWaves);
    job.short_blocks = (int)ceil_div(up.n, (int64_t)(kWave / job.lpr) * FS_SHORT_UNR * kStepWaves);
    int64_t most = u.n;
    for (int64_t x : {sp.cap_t, sp.cap_t1, cls.n}) most = x > most ? x : most;
    const unsigned blocks = 1u + (unsigned)(job.u.long_blocks + job.short_blocks);
    const bool bf = up.dt == FS_BF16;
    hipError_t e;
    if (most <= 1024) e = bf ? small_step_launch<1, true>(ctx, job, blocks, s) : small_step_launch<1, false>(ctx, job, blocks, s);
    else if (most <= 2048) e = bf ? small_step_launch<2, true>(ctx, job, blocks, s) : small_step_launch<2, false>(ctx, job, blocks, s);
    else if (most <= 4096) e = bf ? small_step_launch<4, true>(ctx, job, blocks, s) : small_step_launch<4, false>(ctx, job, blocks, s);
    else e = bf ? small_step_launch<8, true>(ctx, job, blocks, s) : small_step_launch<8, false>(ctx, job, blocks, s);
    if (e != hipSuccess) return hip_err(ctx, e, "small_step_kernel");
    return FS_OK;
}

FS_TRACE_SETTER(small_step)

}  // namespace fs
