// LowDiff+ dense path: layer snapshot and incremental Adam merge.
//
// ld_snapshot_layer(s): Snapshot(G^n_t) of Algorithm 2 (Sec. VI-B) - as soon as a
//   layer's synchronized gradient exists it is copied, bit for bit, into a
//   checkpoint-owned buffer so the backward pass may go on.  Here the copy stays
//   in HBM (streaming 16-byte loads/stores); the multi-layer entry packs many
//   small layers into one launch (Sec. VI-C, "Snapshotting module").
// ld_merge_dense_adam: "Merge in CPU" of Algorithm 2, M <- M + Adam(o_t, G_t)
//   (Eq. (4)), with the replica kept in HBM and the W steps of a window fused
//   into one pass: (24 + 2W) bytes per parameter instead of 26 per step.
#include <math.h>

#include "ld_common.h"

namespace {

// Consecutive 16 KB pieces of an array that an XCD is given at a time: runs of 1 MB, so that all
// XCDs stream the same neighbourhood. Against one contiguous eighth per XCD (two runs each): a copy of
// 202 M 16-bit elements 138 -> 130-134 us, 500 M 338-342 -> 324, 2 G 1345 -> 1322; the Adam replay of four
// steps on 20 M elements 113-115 -> 106 us, on 2 G 10.6-11.2 -> 10.3-10.6 ms, where it moves as much with the
// placement of the arrays. Runs of 1, 4, 8, 16 and 32 pieces: behind in one or the other.
constexpr uint32_t kXcdRun = 64;

// ----------------------------------------------------------------- snapshot

constexpr int kCopyThreads = 256;
constexpr int kCopyUnroll = 4;                                    // 16-byte vectors per thread
constexpr int64_t kCopyBlockBytes = kCopyThreads * kCopyUnroll * 16;  // 16 KB per block
// A launch takes as many layers as its 4 KB of arguments hold (128 in a table of addresses and 64-bit sizes: ResNet-50's 161 tensors were two
// launches). A workgroup finds its layer among them in two reads of 16 consecutive entries each: as a binary search it was eight dependent ones.
// ResNet-50's tensors 22.9 -> 19.4 us a call (102 MB: 5.3 TB/s with the launch). Up to 16 layers the search is the faster way: with 256 MB written in
// between, 2 to 8 layers of 100,000 elements 7.6 us in the two reads, 7.0 to 7.3 searched.
constexpr int kLayerGroup = 16;
constexpr int kLayerGroups = 11;
constexpr int kLayersPerLaunch = kLayerGroups * kLayerGroup;

// In the order of the reads: a line of the arguments' memory each, and next to one another what one read brings.
struct CopyBatch {
    int32_t first_of_group[kLayerGroup];        // [0]: all blocks; then every 16th of first_block, with at most 16 layers their number in [1]
    int32_t first_block[kLayersPerLaunch + 1];  // prefix of blocks per layer; entries past the last layer: all blocks
    struct Layer {
        const unsigned char* src;
        unsigned char* dst;
    } layer[kLayersPerLaunch];
    uint16_t last_elems[kLayersPerLaunch];      // 16-bit elements in the layer's last block, at most 8192
};
static_assert(sizeof(CopyBatch) <= 4096, "k_snapshot_batch's arguments must fit a kernel's 4 KB");
static_assert(kLayerGroups <= kLayerGroup, "one read finds the group");

typedef uint32_t ld_u32x4_any __attribute__((ext_vector_type(4), aligned(2)));  // 16 bytes at any even address

// One block of a layer: 16-byte stores on the destination's own 16-byte boundaries, 16-byte loads
// wherever the source then lies (global loads need no alignment), all of a thread's loads in flight
// together; the up to seven elements before and after go one by one. (Element by element, as ragged tails
// and unaligned layers went before, a block is up to 32 memory round trips: 40 layers of odd sizes, 40 M elements, 36.5 -> 31.3 us.)
__device__ __forceinline__ void copy_block(const unsigned char* __restrict__ src,
                                           unsigned char* __restrict__ dst, int32_t bytes) {
    int32_t head = static_cast<int32_t>(-reinterpret_cast<uintptr_t>(dst) & 15);
    if (head > bytes) head = bytes;
    const int32_t nv = (bytes - head) >> 4;
    const ld_u32x4_any* s = reinterpret_cast<const ld_u32x4_any*>(src + head);
    ld_u32x4* d = reinterpret_cast<ld_u32x4*>(dst + head);
    ld_u32x4 x[kCopyUnroll];
    if (nv == kCopyThreads * kCopyUnroll) {
#pragma unroll
        for (int u = 0; u < kCopyUnroll; ++u) x[u] = __builtin_nontemporal_load(s + u * kCopyThreads + threadIdx.x);
#pragma unroll
        for (int u = 0; u < kCopyUnroll; ++u) ld_nt_store(x[u], d + u * kCopyThreads + threadIdx.x);
        return;  // a whole block on a boundary
    }
#pragma unroll
    for (int u = 0; u < kCopyUnroll; ++u) {
        const int32_t at = u * kCopyThreads + static_cast<int32_t>(threadIdx.x);
        x[u] = ld_u32x4{0u, 0u, 0u, 0u};
        if (at < nv) x[u] = __builtin_nontemporal_load(s + at);
    }
    // the elements before the first boundary and after the last
    const int32_t h = head >> 1, rest = (bytes - head - 16 * nv) >> 1;
    const int32_t e = static_cast<int32_t>(threadIdx.x);
    if (e < h + rest) {
        const int32_t at = e < h ? 2 * e : head + 16 * nv + 2 * (e - h);
        *reinterpret_cast<uint16_t*>(dst + at) = *reinterpret_cast<const uint16_t*>(src + at);
    }
#pragma unroll
    for (int u = 0; u < kCopyUnroll; ++u) {
        const int32_t at = u * kCopyThreads + static_cast<int32_t>(threadIdx.x);
        if (at < nv) ld_nt_store(x[u], d + at);
    }
}

__global__ __launch_bounds__(kCopyThreads) void k_snapshot(const unsigned char* __restrict__ src,
                                                           unsigned char* __restrict__ dst,
                                                           int64_t bytes) {
    const int64_t blk = ld_xcd_piece<kXcdRun>(blockIdx.x, gridDim.x);
    const int64_t at = blk * kCopyBlockBytes, left = bytes - at;
    if (left > 0) copy_block(src + at, dst + at, static_cast<int32_t>(left < kCopyBlockBytes ? left : kCopyBlockBytes));
}

// FEW: at most a group of layers, found by a binary search.
template <bool FEW>
__global__ __launch_bounds__(kCopyThreads) void k_snapshot_batch(CopyBatch cb) {
    const int32_t blk = static_cast<int32_t>(ld_xcd_piece<kXcdRun>(blockIdx.x, gridDim.x));
    if (blk >= cb.first_of_group[0]) return;
    int l = 0;  // the last layer that begins at or before the block
    if (FEW) {
        for (int end = cb.first_of_group[1]; end - l > 1;) {
            const int mid = (l + end) >> 1;
            if (cb.first_block[mid] <= blk) l = mid; else end = mid;
        }
    } else {
        int group = 0;
#pragma unroll
        for (int i = 1; i < kLayerGroup; ++i) group += cb.first_of_group[i] <= blk;
        const int32_t* first = cb.first_block + group * kLayerGroup;
#pragma unroll
        for (int i = 1; i < kLayerGroup; ++i) l += first[i] <= blk;
        l += group * kLayerGroup;
    }
    const int64_t at = static_cast<int64_t>(blk - cb.first_block[l]) * kCopyBlockBytes;
    const bool last = blk + 1 == cb.first_block[l + 1];
    copy_block(cb.layer[l].src + at, cb.layer[l].dst + at, last ? 2 * cb.last_elems[l] : static_cast<int32_t>(kCopyBlockBytes));
}

// --------------------------------------------------------------------- Adam

struct AdamArgs {
    const uint16_t* grad[LD_MAX_ADAM_WINDOW];
    LdAdamSteps s;
    int32_t W;
};

constexpr int kAdamThreads = 256;
constexpr int kAdamH = 4;                          // 16-byte fp32 vectors per thread and array
constexpr int kAdamBlockElems = kAdamThreads * 4 * kAdamH; // elements per workgroup

// Replays steps [t0, t0 + WT) of the window (those below a.W). One workgroup per
// kAdamBlockElems consecutive elements; every load instruction of a wave covers
// one contiguous run (16 bytes of fp32 state or 8 bytes of bf16 gradient per
// lane), and all loads are issued before the first value is used.
template <int WT, bool GENERAL>
__global__ __launch_bounds__(kAdamThreads) void k_adam(float* __restrict__ w, float* __restrict__ m,
                                                       float* __restrict__ v, int64_t n, AdamArgs a, int t0) {
    const int64_t blk = ld_xcd_piece<kXcdRun>(blockIdx.x, gridDim.x);
    const int64_t b0 = blk * kAdamBlockElems;
    if (b0 >= n) return;
    if (b0 + kAdamBlockElems <= n) {
        const int64_t q0 = b0 / 4 + threadIdx.x;  // index of the thread's first 4-element vector
        ld_f32x4 wv[kAdamH], mv[kAdamH], vv[kAdamH];
        ld_u32x2 gq[WT][kAdamH];
#pragma unroll
        for (int t = 0; t < WT; ++t)
#pragma unroll
            for (int h = 0; h < kAdamH; ++h)
                gq[t][h] = (t0 + t < a.W) ? __builtin_nontemporal_load(reinterpret_cast<const ld_u32x2*>(a.grad[t0 + t]) +
                                                                       q0 + h * kAdamThreads)
                                          : ld_u32x2{0u, 0u};
        ld_f32x4* w4 = reinterpret_cast<ld_f32x4*>(w) + q0;
        ld_f32x4* m4 = reinterpret_cast<ld_f32x4*>(m) + q0;
        ld_f32x4* v4 = reinterpret_cast<ld_f32x4*>(v) + q0;
#pragma unroll
        for (int h = 0; h < kAdamH; ++h) {
            wv[h] = ld_nt_load(w4 + h * kAdamThreads);
            mv[h] = ld_nt_load(m4 + h * kAdamThreads);
            vv[h] = ld_nt_load(v4 + h * kAdamThreads);
        }
#pragma unroll
        for (int h = 0; h < kAdamH; ++h) {
            float ww[4] = {wv[h].x, wv[h].y, wv[h].z, wv[h].w};
            float mm[4] = {mv[h].x, mv[h].y, mv[h].z, mv[h].w};
            float v4_[4] = {vv[h].x, vv[h].y, vv[h].z, vv[h].w};
#pragma unroll
            for (int t = 0; t < WT; ++t) {
                if (t0 + t < a.W) {
                    const uint32_t gw[2] = {gq[t][h].x, gq[t][h].y};
                    const float lr_bc1 = a.s.lr_bc1[t0 + t], scale = a.s.root_scale[t0 + t], eps_s = a.s.eps_s[t0 + t];
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const uint32_t half = (e & 1) ? (gw[e >> 1] >> 16) : (gw[e >> 1] & 0xFFFFu);
                        float g1, g2;
                        ld_adam_terms(ld_bf16_widen(half), a.s.one_m_beta1, a.s.one_m_beta2, g1, g2);
                        ld_adam_step<GENERAL>(ww[e], mm[e], v4_[e], g1, g2, a.s.beta1, a.s.beta2, lr_bc1, scale, eps_s);
                    }
                }
            }
            ld_nt_store(ld_f32x4{ww[0], ww[1], ww[2], ww[3]}, w4 + h * kAdamThreads);
            ld_nt_store(ld_f32x4{mm[0], mm[1], mm[2], mm[3]}, m4 + h * kAdamThreads);
            ld_nt_store(ld_f32x4{v4_[0], v4_[1], v4_[2], v4_[3]}, v4 + h * kAdamThreads);
        }
    } else {
        // the last, ragged workgroup: element by element
        for (int64_t e = b0 + threadIdx.x; e < n; e += kAdamThreads) {
            float ww = w[e], mm = m[e], v1 = v[e];
            for (int t = t0; t < t0 + WT && t < a.W; ++t) {
                float g1, g2;
                ld_adam_terms(ld_bf16_widen(a.grad[t][e]), a.s.one_m_beta1, a.s.one_m_beta2, g1, g2);
                ld_adam_step<GENERAL>(ww, mm, v1, g1, g2, a.s.beta1, a.s.beta2, a.s.lr_bc1[t], a.s.root_scale[t],
                                      a.s.eps_s[t]);
            }
            w[e] = ww;
            m[e] = mm;
            v[e] = v1;
        }
    }
}

}  // namespace

extern "C" ld_status ld_snapshot_layer(const void* grad_bf16, void* snap_bf16, int64_t n_elems,
                                       ld_stream stream) {
    if (n_elems < 0) return LD_ERR_RANGE;
    if (n_elems == 0) return LD_OK;
    if (!grad_bf16 || !snap_bf16) return LD_ERR_NULL;
    if (!ld_aligned(grad_bf16, 2) || !ld_aligned(snap_bf16, 2)) return LD_ERR_ALIGN;
    const int64_t bytes = n_elems * 2;
    const int64_t blocks = (bytes + kCopyBlockBytes - 1) / kCopyBlockBytes;
    if (blocks > INT32_MAX - 8) return LD_ERR_RANGE;
    ld_begin_call();
    k_snapshot<<<dim3(static_cast<uint32_t>((blocks + 7) / 8 * 8)), dim3(kCopyThreads), 0,
                 static_cast<hipStream_t>(stream)>>>(static_cast<const unsigned char*>(grad_bf16),
                                                     static_cast<unsigned char*>(snap_bf16), bytes);
    return ld_launch_status();
}

extern "C" ld_status ld_snapshot_layers(const void* const* src, void* const* dst,
                                        const int64_t* n_elems, int32_t n_layers, ld_stream stream) {
    if (n_layers < 0) return LD_ERR_RANGE;
    if (n_layers == 0) return LD_OK;
    if (!src || !dst || !n_elems) return LD_ERR_NULL;
    for (int32_t l = 0; l < n_layers; ++l) {
        if (n_elems[l] < 0) return LD_ERR_RANGE;
        if (n_elems[l] > 0 && (!src[l] || !dst[l])) return LD_ERR_NULL;
        if (!ld_aligned(src[l], 2) || !ld_aligned(dst[l], 2)) return LD_ERR_ALIGN;
        if ((n_elems[l] * 2 + kCopyBlockBytes - 1) / kCopyBlockBytes > (1 << 30)) return LD_ERR_RANGE;
    }
    ld_begin_call();
    int32_t live = 0, l = 0;
    for (int32_t j = 0; j < n_layers; ++j) live += n_elems[j] > 0;
    if (live == 0) return LD_OK;
    // as many layers in every launch: 353 as 118, 118 and 117, not as 176, 176 and one (38.7 us instead of 39.8)
    const int32_t launches = (live + kLayersPerLaunch - 1) / kLayersPerLaunch, per = (live + launches - 1) / launches;
    while (l < n_layers) {
        CopyBatch cb;
        int32_t count = 0;
        int64_t blocks = 0;
        while (l < n_layers && count < per) {
            const int64_t bytes = n_elems[l] * 2;
            const int64_t nb = (bytes + kCopyBlockBytes - 1) / kCopyBlockBytes;
            if (nb == 0) { ++l; continue; }
            if (blocks + nb > (1 << 30)) break;
            cb.layer[count] = {static_cast<const unsigned char*>(src[l]), static_cast<unsigned char*>(dst[l])};
            cb.first_block[count] = static_cast<int32_t>(blocks);
            cb.last_elems[count] = static_cast<uint16_t>((bytes - (nb - 1) * kCopyBlockBytes) / 2);
            blocks += nb;
            ++count;
            ++l;
        }
        if (count == 0) continue;
        for (int32_t j = count; j < kLayersPerLaunch; ++j) {
            cb.layer[j] = {nullptr, nullptr};
            cb.last_elems[j] = 0;
        }
        for (int32_t j = count; j <= kLayersPerLaunch; ++j) cb.first_block[j] = static_cast<int32_t>(blocks);
        cb.first_of_group[0] = static_cast<int32_t>(blocks);
        for (int32_t g = 1; g < kLayerGroup; ++g)
            cb.first_of_group[g] = g < kLayerGroups ? cb.first_block[g * kLayerGroup] : static_cast<int32_t>(blocks);
        if (count <= kLayerGroup) cb.first_of_group[1] = count;
        const dim3 grid(static_cast<uint32_t>((blocks + 7) / 8 * 8));
        hipStream_t s = static_cast<hipStream_t>(stream);
        if (count <= kLayerGroup) k_snapshot_batch<true><<<grid, dim3(kCopyThreads), 0, s>>>(cb);
        else k_snapshot_batch<false><<<grid, dim3(kCopyThreads), 0, s>>>(cb);
        if (ld_launch_status() != LD_OK) return LD_ERR_HIP;
    }
    return LD_OK;
}

extern "C" ld_status ld_merge_dense_adam(float* w, float* m, float* v, int64_t n,
                                         const void* const* grads_bf16, int32_t W, int64_t step0,
                                         float lr, float beta1, float beta2, float eps,
                                         ld_stream stream) {
    if (n < 0 || W < 0 || W > LD_MAX_ADAM_WINDOW || step0 < 0) return LD_ERR_RANGE;
    if (!(beta1 >= 0.0f && beta1 < 1.0f) || !(beta2 >= 0.0f && beta2 < 1.0f)) return LD_ERR_RANGE;
    if (W == 0 || n == 0) return LD_OK;
    if (!w || !m || !v || !grads_bf16) return LD_ERR_NULL;
    if (!ld_aligned(w, 16) || !ld_aligned(m, 16) || !ld_aligned(v, 16)) return LD_ERR_ALIGN;
    static_assert(LD_MAX_ADAM_WINDOW <= LD_MAX_ADAM_STEPS, "step table too small");
    AdamArgs a;
    for (int32_t t = 0; t < LD_MAX_ADAM_WINDOW; ++t) a.grad[t] = nullptr;
    for (int32_t t = 0; t < W; ++t) {
        if (!grads_bf16[t]) return LD_ERR_NULL;
        if (!ld_aligned(grads_bf16[t], 16)) return LD_ERR_ALIGN;
        a.grad[t] = static_cast<const uint16_t*>(grads_bf16[t]);
    }
    const bool general = ld_adam_general(lr, beta2, eps);
    ld_fill_adam_steps(a.s, W, step0, lr, beta1, beta2, eps, general);
    a.W = W;
    const int64_t blocks = (n + kAdamBlockElems - 1) / kAdamBlockElems;
    if (blocks > INT32_MAX - 8) return LD_ERR_RANGE;
    const dim3 grid(static_cast<uint32_t>((blocks + 7) / 8 * 8)), block(kAdamThreads);
    hipStream_t s = static_cast<hipStream_t>(stream);
    ld_begin_call();
    // steps are fused four (or eight) at a time; the state round-trips through fp32
    // memory between passes, which is exactly what it does between two calls
    int t0 = 0;
    while (t0 < W) {
        const int left = W - t0;
        if (general) {
            if (left > 4) { k_adam<8, true><<<grid, block, 0, s>>>(w, m, v, n, a, t0); t0 += 8; }
            else if (left > 2) { k_adam<4, true><<<grid, block, 0, s>>>(w, m, v, n, a, t0); t0 += 4; }
            else if (left > 1) { k_adam<2, true><<<grid, block, 0, s>>>(w, m, v, n, a, t0); t0 += 2; }
            else { k_adam<1, true><<<grid, block, 0, s>>>(w, m, v, n, a, t0); t0 += 1; }
        } else {
            if (left > 4) { k_adam<8, false><<<grid, block, 0, s>>>(w, m, v, n, a, t0); t0 += 8; }
            else if (left > 2) { k_adam<4, false><<<grid, block, 0, s>>>(w, m, v, n, a, t0); t0 += 4; }
            else if (left > 1) { k_adam<2, false><<<grid, block, 0, s>>>(w, m, v, n, a, t0); t0 += 2; }
            else { k_adam<1, false><<<grid, block, 0, s>>>(w, m, v, n, a, t0); t0 += 1; }
        }
        if (ld_launch_status() != LD_OK) return LD_ERR_HIP;
    }
    return LD_OK;
}
