// The index half of a small batch on ONE workgroup: dedup, collision split and class order of up to kSmallIdsInline IDs
// (8192) on the caller's stream, of 10240 or 12288 ahead of time (small_index_ids in fs_dedup_rule.h).
//
// The kernels of fs_bucket.hip or fs_unique.hip and of fs_split.hip are a chain of up to six launches (ten of the radix
// sort); on a batch of a few thousand IDs each of them is a handful of workgroups and takes 2.5 to 9 us whatever it does, so
// a step that runs the chain takes 12 to 15 us longer up to 4 k IDs, and costs the host six launches (one workgroup,
// dedup, split and class order: 1 k IDs 14 us, 8 k 45 us, 16 k 96 us, three radix passes of 16 k keys on four SIMDs being
// most of that).  Here everything the launches exchange through memory stays in the LDS of one compute unit (160 KB: room
// for kSmallIds, 16384 IDs) and in registers, and a barrier takes the place of a launch.
//
// Elements are owned in the order (wavefront, round, lane): with R rounds, round r of wavefront w holds the 64 consecutive
// elements from w * 64 * R + 64 r on, so that ballots and popcounts number them in order.  Every output is what the
// chain of launches writes, bit for bit.
//
// Up to kMaxBatch independent jobs share a launch (blockIdx.x picks the job).
#include <atomic>

#include "fs_small.h"

namespace fs {

template <int KPT, bool DEDUP, bool SPLIT>
__global__ __launch_bounds__(kSmallThreads) void small_index_kernel(const small_batch batch, int *__restrict__ flags) {
    FS_WG_TRACE(12);
    extern __shared__ char lds[];
    __shared__ small_shared sh;
    if (DEDUP) small_dedup_body<KPT>(batch.d[blockIdx.x], lds, sh, flags);
    if (DEDUP && SPLIT) __syncthreads();                     // U_t1 is written
    if (SPLIT) small_split_body(batch.s[blockIdx.x], kSmallThreads * KPT, lds, sh, flags);
}

// ---- host side -----------------------------------------------------------------------------------------------------
template <int KPT, bool DEDUP, bool SPLIT>
static hipError_t small_launch(fs_ctx *ctx, const small_batch &batch, int count, hipStream_t s) {
    // sort: key and place of every element; split: the other list, a bit each, the rows found
    constexpr size_t maxn = (size_t)kSmallThreads * KPT;
    constexpr size_t lds = SPLIT ? small_split_lds(maxn) : maxn * 6;
    auto *kernel = &small_index_kernel<KPT, DEDUP, SPLIT>;
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
    hipLaunchKernelGGL(kernel, dim3((unsigned)count), dim3(kSmallThreads), lds, s, batch, ctx->d_flags);
    return hipGetLastError();
}

template <bool DEDUP, bool SPLIT>
static int small_dispatch(fs_ctx *ctx, const small_batch &batch, int count, int64_t most, hipStream_t s) {
    hipError_t e;
    if (most <= 1024) e = small_launch<1, DEDUP, SPLIT>(ctx, batch, count, s);
    else if (most <= 2048) e = small_launch<2, DEDUP, SPLIT>(ctx, batch, count, s);
    else if (most <= 4096) e = small_launch<4, DEDUP, SPLIT>(ctx, batch, count, s);
    else if (most <= 8192) e = small_launch<8, DEDUP, SPLIT>(ctx, batch, count, s);
    else e = small_launch<16, DEDUP, SPLIT>(ctx, batch, count, s);
    if (e != hipSuccess) return hip_err(ctx, e, "small_index_kernel");
    return FS_OK;
}

// scratch set 0 belongs to the caller's stream and the side stream, the others to the index streams
static int64_t small_limit(int set0, int key_bits) { return small_index_ids(set0 == 0, key_bits); }

bool small_unique_fits(int count, const fs_unique_job *jobs, int set0) {
    for (int k = 0; k < count; ++k) {
        const int kb = key_bits_of(jobs[k].num_rows);
        if (kb > 32 || jobs[k].n > small_limit(set0, kb)) return false;
    }
    return count >= 1 && count <= kMaxBatch;
}

bool small_split_fits(int count, const fs_split_job *jobs, const fs_class_job *cls, int set0, bool with_dedup) {
    for (int k = 0; k < count; ++k) {
        int64_t most = small_limit(set0, jobs[k].key_bits);
        if (set0 == 0 && !with_dedup) most = cls ? kSmallClassesInline : kSmallSplitInline;
        if (jobs[k].cap_t > most || jobs[k].cap_t1 > most || (cls && cls[k].n > most)) return false;
    }
    return count >= 1 && count <= kMaxBatch;
}

int launch_small_index(fs_ctx *ctx, int count, const fs_unique_job *u, const fs_split_job *sp, const fs_class_job *cls,
                       hipStream_t s) {
    small_batch batch;
    memset(&batch, 0, sizeof(batch));
    int64_t most = 1;
    for (int k = 0; k < count; ++k) {
        if (u) {
            batch.d[k] = small_dedup_job(u[k]);
            most = u[k].n > most ? u[k].n : most;
        }
        if (sp) {
            batch.s[k] = small_split_job(sp[k], cls ? &cls[k] : nullptr);
            most = sp[k].cap_t > most ? sp[k].cap_t : most;
            most = sp[k].cap_t1 > most ? sp[k].cap_t1 : most;
            if (cls && cls[k].n > most) most = cls[k].n;
        }
    }
    if (u && sp) return small_dispatch<true, true>(ctx, batch, count, most, s);
    if (u) return small_dispatch<true, false>(ctx, batch, count, most, s);
    return small_dispatch<false, true>(ctx, batch, count, most, s);
}

FS_TRACE_SETTER(small)

}  // namespace fs
