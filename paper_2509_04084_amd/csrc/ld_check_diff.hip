// ld_check_diff: does a differential read back from storage meet what the merges assume?
//
// The Recovery loop of Algorithm 1 (Sec. IV-B) loads differential checkpoints from storage
// and merges them. The merge kernels take for granted that a diff's indices lie in [0, n) and
// ascend strictly, and that no value is a NaN; a damaged file breaks that silently (the sweep
// would skip records, the scatter would write outside w). This pass counts the violations so
// that a caller can refuse the file before merging it. One read of the records, 8 bytes each.
#include <limits.h>

#include "ld_common.h"

namespace {

constexpr int kCheckPer = 4;  // 16-byte loads of indices per thread (and as many of values)

__global__ void k_check_zero(unsigned long long* out) {
    if (threadIdx.x < 3) out[threadIdx.x] = 0;
}

// Records up to which one workgroup (of 1024 threads, or of 256 where that is enough) checks them all in one round and writes the counts,
// which nothing has to clear for it then: check and merge of 501 records 6.0 -> 4.9 us, of 5001 6.6 -> 5.9, of 10,001 7.6 -> 6.1; a second
// round is 2 us. Where the records end, or an array is not 16-byte aligned, the vectors are read one by one, 100,001 records 8.8 -> 8.0 us,
// 333,334 17.9 -> 16.5, unaligned 1 M 23.2 -> 11.7; the workgroups inside load without a branch (1 M records, 256 MB written in between, 13.1 -> 11.5 us;
// 32,768 11.4 -> 10.2).
constexpr int64_t kCheckFew = 16384;

// A workgroup per THREADS * 16 records. ALONE: the only one; else they add to cleared counts.
template <int THREADS, bool ALONE>
__global__ __launch_bounds__(THREADS) void k_check_diff(const int32_t* __restrict__ idx,
                                                        const float* __restrict__ val, int64_t K, int64_t n,
                                                        unsigned long long* __restrict__ out) {
    __shared__ uint32_t part[3][THREADS / LD_WAVE];
    uint32_t range = 0, order = 0, nan = 0;
    // Records [e0, e0 + 4) of a thread's vectors; the record before them comes from the lane below, for
    // a wave's first lane from memory. As whole 16-byte vectors (4-byte loads and every index read
    // twice before): check and merge of a 0.5 M-record diff 26.5 -> 23.7 us. At 15.6 M records (54 us) it is
    // bound by what its reads evict.
    const bool vec = ((reinterpret_cast<uintptr_t>(idx) | reinterpret_cast<uintptr_t>(val)) & 15) == 0;
    const int64_t base = static_cast<int64_t>(blockIdx.x) * (THREADS * kCheckPer * 4);
    ld_u32x4 q[kCheckPer];
    ld_f32x4 x[kCheckPer];
    int32_t before[kCheckPer], have[kCheckPer];
    if (vec && base + THREADS * kCheckPer * 4 <= K) {  // uniform
#pragma unroll
        for (int u = 0; u < kCheckPer; ++u) {
            const int64_t e0 = base + (u * THREADS + threadIdx.x) * 4;
            have[u] = 4;
            q[u] = *reinterpret_cast<const ld_u32x4*>(idx + e0);  // cached: a merge of the same records follows
            x[u] = val ? *reinterpret_cast<const ld_f32x4*>(val + e0) : ld_f32x4{0.0f, 0.0f, 0.0f, 0.0f};
            before[u] = ld_lane() == 0 && e0 > 0 ? idx[e0 - 1] : INT_MIN;  // nothing precedes record 0
        }
    } else {
#pragma unroll
        for (int u = 0; u < kCheckPer; ++u) {
            const int64_t e0 = base + (u * THREADS + threadIdx.x) * 4, left = K - e0;
            have[u] = left < 0 ? 0 : left < 4 ? static_cast<int32_t>(left) : 4;
            q[u] = ld_u32x4{0u, 0u, 0u, 0u};
            x[u] = ld_f32x4{0.0f, 0.0f, 0.0f, 0.0f};
            if (vec && have[u] == 4) {
                q[u] = *reinterpret_cast<const ld_u32x4*>(idx + e0);
                if (val) x[u] = *reinterpret_cast<const ld_f32x4*>(val + e0);
            } else {
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    if (c < have[u]) {
                        q[u][c] = static_cast<uint32_t>(idx[e0 + c]);
                        if (val) x[u][c] = val[e0 + c];
                    }
                }
            }
            before[u] = ld_lane() == 0 && e0 > 0 && have[u] > 0 ? idx[e0 - 1] : INT_MIN;
        }
    }
#pragma unroll
    for (int u = 0; u < kCheckPer; ++u) {
        const int32_t i[4] = {static_cast<int32_t>(q[u].x), static_cast<int32_t>(q[u].y),
                              static_cast<int32_t>(q[u].z), static_cast<int32_t>(q[u].w)};
        const int32_t below = __builtin_amdgcn_update_dpp(0, i[3], 0x138 /* wave_shr:1 */, 0xf, 0xf, false);
        const int64_t e0 = base + (u * THREADS + threadIdx.x) * 4;
        const int32_t prev = ld_lane() == 0 ? before[u] : below;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const bool in = c < have[u];
            range += in && (i[c] < 0 || i[c] >= n);
            order += in && (c > 0 ? i[c] <= i[c - 1] : e0 > 0 && i[0] <= prev);
            nan += in && x[u][c] != x[u][c];
        }
    }
    range = ld_wave_sum(range);
    order = ld_wave_sum(order);
    nan = ld_wave_sum(nan);
    const int w = threadIdx.x >> 6;
    if (ld_lane() == 0) {
        part[0][w] = range;
        part[1][w] = order;
        part[2][w] = nan;
    }
    __syncthreads();
    if (threadIdx.x < 3) {
        uint32_t total = 0;
        for (int q = 0; q < THREADS / LD_WAVE; ++q) total += part[threadIdx.x][q];
        if (ALONE) out[threadIdx.x] = total;
        else if (total) atomicAdd(out + threadIdx.x, static_cast<unsigned long long>(total));
    }
}

}  // namespace

extern "C" ld_status ld_check_diff(const int32_t* idx, const float* val, int64_t K, int64_t n, int64_t* counts,
                                   ld_stream stream) {
    if (K < 0 || n < 0 || n > INT32_MAX) return LD_ERR_RANGE;
    if (!counts) return LD_ERR_NULL;
    if (K > 0 && !idx) return LD_ERR_NULL;
    if (!ld_aligned(idx, 4) || !ld_aligned(val, 4) || !ld_aligned(counts, 8)) return LD_ERR_ALIGN;
    constexpr int kThreads = 256;
    constexpr int64_t per = kThreads * kCheckPer * 4;
    const int64_t blocks = (K + per - 1) / per;
    if (blocks > INT32_MAX) return LD_ERR_RANGE;
    hipStream_t s = static_cast<hipStream_t>(stream);
    ld_begin_call();
    unsigned long long* out = reinterpret_cast<unsigned long long*>(counts);
    if (K <= kCheckFew) {
        if (K <= per) k_check_diff<kThreads, true><<<dim3(1), dim3(kThreads), 0, s>>>(idx, val, K, n, out);
        else k_check_diff<1024, true><<<dim3(1), dim3(1024), 0, s>>>(idx, val, K, n, out);
        return ld_launch_status();
    }
    k_check_zero<<<dim3(1), dim3(LD_WAVE), 0, s>>>(out);
    if (ld_launch_status() != LD_OK) return LD_ERR_HIP;
    k_check_diff<kThreads, false><<<dim3(static_cast<uint32_t>(blocks)), dim3(kThreads), 0, s>>>(idx, val, K, n, out);
    return ld_launch_status();
}
