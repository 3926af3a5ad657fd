// Shared host/device helpers of the gfx950 LowDiff kernels (not part of the ABI).
#pragma once

#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "ld_map.h"
#include "lowdiff.h"

#define LD_WAVE 64

// An entry point calls this once, after its argument checks and before its first launch: an
// error that the caller's own earlier HIP calls left behind in this thread is dropped here, so
// that it is not taken for a failure of this call's launches.
static inline void ld_begin_call() { (void)hipGetLastError(); }

// Status of the launch just enqueued (reading it also clears the error). Checked after every
// launch: when it is not LD_OK the entry point returns at once, with earlier kernels of the
// call already enqueued - the outputs are then unspecified.
static inline ld_status ld_launch_status() {
    return hipGetLastError() == hipSuccess ? LD_OK : LD_ERR_HIP;
}

static inline bool ld_aligned(const void* p, size_t a) {
    return (reinterpret_cast<uintptr_t>(p) & (a - 1)) == 0;
}

static inline size_t ld_round_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

// Per-step scalars of an Adam replay window, prepared on the host in double. Folded (see
// ld_adam_step): root_scale = sqrt(1 / (1 - beta2^s)) / lr_bc1 and eps_s = eps / lr_bc1, with lr_bc1 =
// lr / (1 - beta1^s); general: root_scale = sqrt(1 / (1 - beta2^s)) and eps_s = eps.
#define LD_MAX_ADAM_STEPS 64
struct LdAdamSteps {
    float lr_bc1[LD_MAX_ADAM_STEPS];      // lr / (1 - beta1^s), general form only
    float root_scale[LD_MAX_ADAM_STEPS];
    float eps_s[LD_MAX_ADAM_STEPS];
    float beta1, one_m_beta1, beta2, one_m_beta2;
};

// Whether a replay runs the general form of ld_adam_step: an eps so small next to the roots that a
// denormal v must not count as zero (the root then misses up to 1.1e-19 times the root scale of the
// corrected moment, largest at step 1), or a learning rate or eps whose quotients leave the comfortable
// part of the float range. Decided without the step number, so that every way to cut a window into
// calls decides alike.
static inline bool ld_adam_general(float lr, float beta2, float eps) {
    const float mag = lr < 0.0f ? -lr : lr;
    return !(static_cast<double>(eps) * sqrt(1.0 - static_cast<double>(beta2)) >= 1e-12 && eps <= 1e3f &&
             mag >= 1e-10f && mag <= 1e3f);
}

// Scalars of steps step0+1 .. step0+W (W <= LD_MAX_ADAM_STEPS).
static inline void ld_fill_adam_steps(LdAdamSteps& a, int32_t W, int64_t step0, float lr, float beta1,
                                      float beta2, float eps, bool general) {
    for (int32_t t = 0; t < LD_MAX_ADAM_STEPS; ++t) a.lr_bc1[t] = a.root_scale[t] = a.eps_s[t] = 0.0f;
    for (int32_t t = 0; t < W; ++t) {
        const double s = static_cast<double>(step0 + 1 + t);
        const double bc1 = 1.0 - pow(static_cast<double>(beta1), s);
        const double bc2 = 1.0 - pow(static_cast<double>(beta2), s);
        const double lr_bc1 = static_cast<double>(lr) / bc1, fold = general ? 1.0 : lr_bc1;
        a.lr_bc1[t] = static_cast<float>(lr_bc1);
        a.root_scale[t] = static_cast<float>(1.0 / (sqrt(bc2) * fold));
        a.eps_s[t] = static_cast<float>(static_cast<double>(eps) / fold);
    }
    a.beta1 = beta1;
    a.one_m_beta1 = 1.0f - beta1;
    a.beta2 = beta2;
    a.one_m_beta2 = 1.0f - beta2;
}

#ifdef __HIPCC__

typedef float ld_f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t ld_u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t ld_u32x4 __attribute__((ext_vector_type(4)));

// Streaming (non-temporal) 16-byte accesses; p must be 16-byte aligned.
__device__ __forceinline__ ld_f32x4 ld_nt_load(const ld_f32x4* p) { return __builtin_nontemporal_load(p); }
__device__ __forceinline__ ld_u32x4 ld_nt_load(const ld_u32x4* p) { return __builtin_nontemporal_load(p); }
__device__ __forceinline__ void ld_nt_store(ld_f32x4 x, ld_f32x4* p) { __builtin_nontemporal_store(x, p); }
__device__ __forceinline__ void ld_nt_store(ld_u32x4 x, ld_u32x4* p) { __builtin_nontemporal_store(x, p); }

__device__ __forceinline__ int ld_lane() { return __lane_id(); }

__device__ __forceinline__ uint32_t ld_mbcnt(uint64_t mask) {  // set bits of `mask` below this lane
    return __builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(mask >> 32),
                                     __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(mask), 0u));
}

// |x| as an integer that orders like the magnitude (sign bit cleared).
__device__ __forceinline__ uint32_t ld_key(float x) { return __float_as_uint(x) & 0x7FFFFFFFu; }

// The lanes' values moved by a data-parallel-primitive control word within the vector unit; lanes without a source, and rows that
// the mask leaves out, get 0. All 64 lanes must be active. (As LDS permutes, which __shfl_up and its like compile to, a scan is six
// round trips to the LDS unit, some 100 cycles each, on chains of latencies that bound the small kernels. compress of flat 1 M
// elements 45.1 -> 42.0 us a call, ResNet-50 99.5 -> 96.5, GPT-2 small 303.5 -> 300.4; the combine of eight GPT-2 XL lists 538 -> 531.)
template <int CTRL, int ROWS = 0xf>
__device__ __forceinline__ uint32_t ld_dpp0(uint32_t x) {
    return static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(x), CTRL, ROWS, 0xf, false));
}
constexpr int kDppShr = 0x110;       // + n: from n lanes below in the row of 16
constexpr int kDppRor = 0x120;       // + n: rotated by n lanes in the row of 16
constexpr int kDppLast16 = 0x142;    // the last lane of a row to the row above it (rows 1 and 3 by their mask)
constexpr int kDppLast32 = 0x143;    // lane 31 to the rows above it (rows 2 and 3 by their mask)

// Inclusive scan over rows of ROW (16, 32 or 64) lanes.
template <int ROW>
__device__ __forceinline__ uint32_t ld_row_iscan(uint32_t x) {
    x += ld_dpp0<kDppShr + 1>(x);
    x += ld_dpp0<kDppShr + 2>(x);
    x += ld_dpp0<kDppShr + 4>(x);
    x += ld_dpp0<kDppShr + 8>(x);
    if (ROW >= 32) x += ld_dpp0<kDppLast16, 0xa>(x);
    if (ROW >= 64) x += ld_dpp0<kDppLast32, 0xc>(x);
    return x;
}

// Inclusive scan over the 64 lanes of a wave.
__device__ __forceinline__ uint32_t ld_wave_iscan(uint32_t x) { return ld_row_iscan<LD_WAVE>(x); }

// Inclusive maximum over the lanes up to each (x >= 0).
__device__ __forceinline__ uint32_t ld_wave_imax(uint32_t x) {
    const auto more = [&](uint32_t y) { x = y > x ? y : x; };
    more(ld_dpp0<kDppShr + 1>(x));
    more(ld_dpp0<kDppShr + 2>(x));
    more(ld_dpp0<kDppShr + 4>(x));
    more(ld_dpp0<kDppShr + 8>(x));
    more(ld_dpp0<kDppLast16, 0xa>(x));
    more(ld_dpp0<kDppLast32, 0xc>(x));
    return x;
}

// Sum over a row of 16 lanes, in every lane.
__device__ __forceinline__ uint32_t ld_row16_sum(uint32_t x) {
    x += ld_dpp0<kDppRor + 8>(x);
    x += ld_dpp0<kDppRor + 4>(x);
    x += ld_dpp0<kDppRor + 2>(x);
    x += ld_dpp0<kDppRor + 1>(x);
    return x;
}

__device__ __forceinline__ uint32_t ld_wave_sum(uint32_t x) {
    x = ld_row16_sum(x);
    x += ld_dpp0<kDppLast16, 0xa>(x);
    x += ld_dpp0<kDppLast32, 0xc>(x);
    return static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(x), LD_WAVE - 1));
}

// Exclusive scan over a 256-thread block. `sh` holds 4 words; returns the
// exclusive prefix of x and the block total. Ends with a barrier so `sh` may be
// reused right away.
__device__ __forceinline__ uint32_t ld_block_escan256(uint32_t x, uint32_t* sh, uint32_t& total) {
    const uint32_t inc = ld_wave_iscan(x);
    const int w = threadIdx.x >> 6;
    if (ld_lane() == LD_WAVE - 1) sh[w] = inc;
    __syncthreads();
    const uint32_t t0 = sh[0], t1 = sh[1], t2 = sh[2], t3 = sh[3];
    total = t0 + t1 + t2 + t3;
    uint32_t base = 0;
    if (w > 0) base += t0;
    if (w > 1) base += t1;
    if (w > 2) base += t2;
    __syncthreads();
    return base + inc - x;
}

__device__ __forceinline__ float ld_bf16_widen(uint32_t h) { return __uint_as_float(h << 16); }

// One Adam step on one element (Eq. (4); bias-corrected, eps added to the root of the
// corrected second moment). The only place the arithmetic is written: every replay
// kernel, fused window or single step, dense or sparse gradient, runs these operations.
//   g1 = (1 - beta1) g, g2 = ((1 - beta2) g) g  (ld_adam_terms)
// The folded form divides numerator and denominator of the update by lr / (1 - beta1^s): two
// moments, a square root, a fused multiply-add for the denominator, a reciprocal and a fused
// multiply-add for w - four full-rate operations and two of two issue slots each, and fewer
// roundings than the formula as written.
// The general form keeps the learning rate apart. The hardware square root takes a denormal
// argument for zero, which with eps = 0 (or tiny) would decide the result (a zero denominator):
// it scales such arguments into the normal range first: sqrt(x) = sqrt(x * 2^64) * 2^-32, exact
// scalings. ld_adam_general says which form a call runs.
__device__ __forceinline__ void ld_adam_terms(float g, float omb1, float omb2, float& g1, float& g2) {
    g1 = __fmul_rn(omb1, g);
    g2 = __fmul_rn(__fmul_rn(omb2, g), g);
}

template <bool GENERAL>
__device__ __forceinline__ void ld_adam_step(float& w, float& m, float& v, float g1, float g2, float b1, float b2,
                                             float lr_bc1, float root_scale, float eps_s) {
    m = __fmaf_rn(b1, m, g1);
    v = __fmaf_rn(b2, v, g2);
    if (GENERAL) {
        const bool tiny = v < 0x1p-96f;
        float root = __builtin_amdgcn_sqrtf(tiny ? __fmul_rn(v, 0x1p+64f) : v);
        root = tiny ? __fmul_rn(root, 0x1p-32f) : root;
        const float denom = __fmaf_rn(root, root_scale, eps_s);
        w = __fmaf_rn(-__fmul_rn(lr_bc1, m), __builtin_amdgcn_rcpf(denom), w);
    } else {
        const float denom = __fmaf_rn(__builtin_amdgcn_sqrtf(v), root_scale, eps_s);
        w = __fmaf_rn(-m, __builtin_amdgcn_rcpf(denom), w);
    }
}

// Device-scope load that is not served from a stale per-CU cache line.
__device__ __forceinline__ uint32_t ld_load_coherent(const uint32_t* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

#endif  // __HIPCC__
