// ld_merge_sparse_adam: ordered replay of a window of sparse diffs through Adam.
//
// Recovery loop of Algorithm 1 (Sec. IV-B) with the update the paper names there:
// for every diff j of the window, in iteration order, decompress it (Comp^-1: a dense
// gradient that is val at the recorded positions and zero elsewhere) and merge it with
// M_{j+1} = M_j + Adam(G_j) (Eq. (4)) into the model AND the optimizer state. Every
// element takes every step: a zero gradient still decays m and v and moves w.
//
// One streaming pass over (w, m, v): 24 n bytes + the records, whatever the window
// length. A wave owns a 1024-element sub-tile: its w, m, v live in registers (16
// elements per lane), the two terms that the current step's decompressed gradient adds to the
// moments in two 4 KB LDS tiles that are zero except where the step's records were
// scattered: the products are formed once per record instead of once per element. Per step:
// scatter the records that fall into the sub-tile, read the tiles back, apply the shared Adam
// step to all 16 elements, clear the scattered positions again. The records are found
// as in ld_merge_sparse: chunk table + interpolated record windows, verified.
// Bound by the vector ALUs for all but the shortest windows: an element's step is four full-rate
// operations and two of four issue slots each, 9.5 ms at 39.3 T slots/s for 20 diffs on 1.56 G
// elements (24 n bytes alone: 6.4 ms). Measured there: 9.6 ms (14.1 ms before, when the
// step took ten full-rate operations, the window of the next diff was waited for as soon as it
// was requested, and 2048-element sub-tiles left three waves per SIMD). 2048 elements with the
// present step: 11.7 ms, bound by latency at two waves per SIMD; 8 KB of LDS and 96 registers
// let five waves share a SIMD.
#include "ld_sparse_common.h"

namespace {

constexpr int kSub = 1024;                 // elements per wave sub-tile (two tiles: 8 KB of LDS, 20 waves per CU)
constexpr int kChunkSubs = 48;             // sub-tiles per chunk of the range table
static_assert(static_cast<int64_t>(kSub) * kChunkSubs == kChunk, "sub-tiles must tile a chunk");
constexpr int kRows = kSub / 4 / LD_WAVE;  // 16-byte vectors per lane and array: 4
constexpr int kMargin = 32;                // records the window starts before the interpolated position

// Writes (or clears) the records of [p, end) that fall into [lo, hi) into the gradient tiles.
__device__ __forceinline__ void scatter_from(float* tile1, float* tile2, const int32_t* __restrict__ idx,
                                             const float* __restrict__ val, int32_t p, int32_t end,
                                             int32_t lo, int32_t hi, bool clear, const LdAdamSteps& a, int lane) {
    for (; p < end; p += LD_WAVE) {
        const bool have = p + lane < end;
        const int32_t i = have ? idx[p + lane] : INT_MAX;
        const float v = (have && !clear) ? val[p + lane] : 0.0f;
        if (i >= lo && i < hi) ld_adam_terms(v, a.one_m_beta1, a.one_m_beta2, tile1[i - lo], tile2[i - lo]);
        if (__ballot(i >= hi)) break;
    }
}

// WIN 64-record windows per diff are loaded ahead.
template <bool GENERAL, int WIN>
__global__ __launch_bounds__(LD_WAVE, GENERAL || WIN > 1 ? 4 : 5) void k_sparse_adam(float* __restrict__ w, float* __restrict__ m,
                                                         float* __restrict__ v, int64_t n, int32_t nchunk,
                                                         DiffTable tb, int32_t W, LdAdamSteps a,
                                                         const int32_t* __restrict__ ctab) {
    __shared__ float tile1[kSub], tile2[kSub];  // the two terms of the step's gradient (ld_adam_terms)
    const int lane = threadIdx.x;
    // runs of 32 sub-tiles per XCD: 124 us for 10 diffs on 25.6 M elements, 132 us with eighths of the
    // arrays per XCD (the same on 1.56 G elements)
    const int64_t sub = ld_xcd_piece<32>(blockIdx.x, gridDim.x);
    if (sub * kSub >= n) return;
    const int64_t lo64 = sub * kSub;
    const int32_t len = static_cast<int32_t>((n - lo64) < kSub ? (n - lo64) : kSub);
    const int32_t lo = static_cast<int32_t>(lo64), hi = lo + len;  // n <= INT_MAX
    const bool full = (len == kSub);

    // state of the lane's 16 elements: vector j covers elements (j*64 + lane)*4 .. +3 of the sub-tile
    float ww[kRows][4], mm[kRows][4], vv[kRows][4];
    if (full) {
#pragma unroll
        for (int j = 0; j < kRows; ++j) {
            const int e = (j * LD_WAVE + lane) * 4;
            const ld_f32x4 a4 = ld_nt_load(reinterpret_cast<const ld_f32x4*>(w + lo64 + e));
            const ld_f32x4 b4 = ld_nt_load(reinterpret_cast<const ld_f32x4*>(m + lo64 + e));
            const ld_f32x4 c4 = ld_nt_load(reinterpret_cast<const ld_f32x4*>(v + lo64 + e));
            ww[j][0] = a4.x; ww[j][1] = a4.y; ww[j][2] = a4.z; ww[j][3] = a4.w;
            mm[j][0] = b4.x; mm[j][1] = b4.y; mm[j][2] = b4.z; mm[j][3] = b4.w;
            vv[j][0] = c4.x; vv[j][1] = c4.y; vv[j][2] = c4.z; vv[j][3] = c4.w;
            __builtin_amdgcn_sched_barrier(0);
        }
    } else {
#pragma unroll
        for (int j = 0; j < kRows; ++j) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int e = (j * LD_WAVE + lane) * 4 + q;
                const bool in = e < len;
                ww[j][q] = in ? w[lo64 + e] : 0.0f;
                mm[j][q] = in ? m[lo64 + e] : 0.0f;
                vv[j][q] = in ? v[lo64 + e] : 0.0f;
            }
        }
    }

    // lane t: where diff t's records of this chunk lie (requested first: the record windows wait for it)
    const int32_t chunk = static_cast<int32_t>(sub / kChunkSubs), part = static_cast<int32_t>(sub % kChunkSubs);
    int32_t c0 = 0, c1 = 0;
    if (lane < W) {
        const int32_t* row = ctab + static_cast<int64_t>(lane) * (nchunk + 1) + chunk;
        c0 = row[0];
        c1 = row[1];
    }
    // the guess for this sub-tile
    int32_t start = c0 + ((c1 - c0) * part) / kChunkSubs - kMargin;
    if (start < c0) start = c0;

#pragma unroll
    for (int j = 0; j < kRows; ++j) {
        reinterpret_cast<ld_f32x4*>(tile1)[j * LD_WAVE + lane] = ld_f32x4{0.0f, 0.0f, 0.0f, 0.0f};
        reinterpret_cast<ld_f32x4*>(tile2)[j * LD_WAVE + lane] = ld_f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    }
    __syncthreads();  // one wave: only orders the vector fill before the scalar scatters

    // One trip per diff; the record window of the next diff is requested before the current
    // one is applied (an Adam step over the sub-tile takes longer than a memory round trip).
    struct Window {
        int32_t s, e, b;        // first position of the window, end and begin of the chunk's records
        int32_t ri[WIN];
        float rv[WIN];
    };
    auto fetch = [&](int32_t t, Window& x) {
        const int tt = t < W ? t : 0;
        x.s = __builtin_amdgcn_readlane(start, tt);
        x.b = __builtin_amdgcn_readlane(c0, tt);
        x.e = t < W ? __builtin_amdgcn_readlane(c1, tt) : x.s;  // past W: an empty window
        const int32_t* __restrict__ ip = tb.idx[tt];
        const float* __restrict__ vp = tb.val[tt];
#pragma unroll
        for (int u = 0; u < WIN; ++u) {
            const int32_t p = x.s + u * LD_WAVE + lane;
            const bool h = p < x.e;
            x.ri[u] = h ? ip[p] : INT_MAX;
            x.rv[u] = h ? vp[p] : 0.0f;
        }
    };
    Window cur, nxt;
    fetch(0, cur);
    // The first window is waited for here: left pending, it would make the compiler wait at the top of
    // every trip, right after the next window was requested and for that window too.
#pragma unroll
    for (int u = 0; u < WIN; ++u) asm volatile("" : "+v"(cur.ri[u]), "+v"(cur.rv[u]));
#pragma unroll 1
    for (int32_t t = 0; t < W; ++t) {
        fetch(t + 1, nxt);
        // Scatter the step's records. rest: position from which records outside the window follow
        // (the window ended too early, or began too late), or the end when there are none.
        uint32_t at[WIN];  // where this lane's records went (kSub and above: nowhere)
        int32_t rest = cur.e;
        const int32_t first = __builtin_amdgcn_readfirstlane(cur.ri[0]);
        const bool hit = cur.s == cur.b || first <= lo;  // the window begins before the sub-tile's records do
#pragma unroll
        for (int u = 0; u < WIN; ++u) {
            at[u] = static_cast<uint32_t>(cur.ri[u]) - static_cast<uint32_t>(lo);
            if (!hit || at[u] >= static_cast<uint32_t>(len)) at[u] = kSub;
            if (at[u] < static_cast<uint32_t>(kSub))
                ld_adam_terms(cur.rv[u], a.one_m_beta1, a.one_m_beta2, tile1[at[u]], tile2[at[u]]);
        }
        if (!hit) rest = lower_bound_idx(tb.idx[t], cur.b, cur.s, lo);
        else if (!__ballot(cur.ri[WIN - 1] >= hi)) rest = cur.s + WIN * LD_WAVE;
        if (rest < cur.e) scatter_from(tile1, tile2, tb.idx[t], tb.val[t], rest, cur.e, lo, hi, false, a, lane);
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        const float lr_bc1 = a.lr_bc1[t], scale = a.root_scale[t], eps_s = a.eps_s[t];
#pragma unroll
        for (int j = 0; j < kRows; ++j) {
            const ld_f32x4 p4 = reinterpret_cast<const ld_f32x4*>(tile1)[j * LD_WAVE + lane];
            const ld_f32x4 q4 = reinterpret_cast<const ld_f32x4*>(tile2)[j * LD_WAVE + lane];
            const float g1[4] = {p4.x, p4.y, p4.z, p4.w}, g2[4] = {q4.x, q4.y, q4.z, q4.w};
#pragma unroll
            for (int q = 0; q < 4; ++q)
                ld_adam_step<GENERAL>(ww[j][q], mm[j][q], vv[j][q], g1[q], g2[q], a.beta1, a.beta2, lr_bc1, scale, eps_s);
            // at most two rows of the tiles in registers at a time (five waves per SIMD: 96 registers)
            if (j % 2 == 1) __builtin_amdgcn_sched_barrier(0);
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
        for (int u = 0; u < WIN; ++u)
            if (at[u] < static_cast<uint32_t>(kSub)) tile1[at[u]] = tile2[at[u]] = 0.0f;
        if (rest < cur.e) scatter_from(tile1, tile2, tb.idx[t], tb.val[t], rest, cur.e, lo, hi, true, a, lane);
        cur = nxt;
    }

    int back = lane;  // the addresses are made again here: kept across the loop they would spill
    asm volatile("" : "+v"(back));
    if (full) {
#pragma unroll
        for (int j = 0; j < kRows; ++j) {
            const int e = (j * LD_WAVE + back) * 4;
            ld_nt_store(ld_f32x4{ww[j][0], ww[j][1], ww[j][2], ww[j][3]}, reinterpret_cast<ld_f32x4*>(w + lo64 + e));
            ld_nt_store(ld_f32x4{mm[j][0], mm[j][1], mm[j][2], mm[j][3]}, reinterpret_cast<ld_f32x4*>(m + lo64 + e));
            ld_nt_store(ld_f32x4{vv[j][0], vv[j][1], vv[j][2], vv[j][3]}, reinterpret_cast<ld_f32x4*>(v + lo64 + e));
            __builtin_amdgcn_sched_barrier(0);
        }
    } else {
#pragma unroll
        for (int j = 0; j < kRows; ++j) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int e = (j * LD_WAVE + back) * 4 + q;
                if (e < len) {
                    w[lo64 + e] = ww[j][q];
                    m[lo64 + e] = mm[j][q];
                    v[lo64 + e] = vv[j][q];
                }
            }
        }
    }
}

}  // namespace

extern "C" size_t ld_merge_sparse_adam_workspace(int64_t n, int32_t W, const int64_t* K) {
    (void)K;
    if (n <= 0 || W <= 0) return 256;
    const int64_t group = W < kGroupMax ? W : kGroupMax;
    return ld_round_up(static_cast<size_t>(group) * (static_cast<size_t>(chunks(n)) + 1) * 4, 256);
}

extern "C" ld_status ld_merge_sparse_adam(float* w, float* m, float* v, int64_t n,
                                          const int32_t* const* idx, const float* const* val,
                                          const int64_t* K, int32_t W, int64_t step0, float lr,
                                          float beta1, float beta2, float eps, void* workspace,
                                          size_t workspace_bytes, ld_stream stream) {
    const ld_status st = check_diff_args(w, n, idx, val, K, W);
    if (st != LD_OK) return st;
    if (step0 < 0) return LD_ERR_RANGE;
    if (!(beta1 >= 0.0f && beta1 < 1.0f) || !(beta2 >= 0.0f && beta2 < 1.0f)) return LD_ERR_RANGE;
    if (W == 0 || n == 0) return LD_OK;
    if (!m || !v) return LD_ERR_NULL;
    if (!ld_aligned(m, 16) || !ld_aligned(v, 16)) return LD_ERR_ALIGN;
    if (!workspace || !ld_aligned(workspace, 256) ||
        workspace_bytes < ld_merge_sparse_adam_workspace(n, W, K))
        return LD_ERR_WORKSPACE;
    hipStream_t s = static_cast<hipStream_t>(stream);
    ld_begin_call();
    const int32_t nsub = static_cast<int32_t>((n + kSub - 1) / kSub), nchunk = chunks(n);
    int32_t* ctab = static_cast<int32_t*>(workspace);
    const bool general = ld_adam_general(lr, beta2, eps);
    static_assert(kGroupMax <= LD_MAX_ADAM_STEPS, "step table too small");
    for (int32_t g0 = 0; g0 < W; g0 += kGroupMax) {
        const int32_t gw = (W - g0) < kGroupMax ? (W - g0) : kGroupMax;
        DiffTable tb = {};
        int64_t most = 0;
        for (int32_t t = 0; t < kGroupMax; ++t) {
            const bool live = t < gw;
            if (live && K[g0 + t] > most) most = K[g0 + t];
            tb.idx[t] = live ? idx[g0 + t] : nullptr;
            tb.val[t] = live ? val[g0 + t] : nullptr;
            tb.K[t] = live ? static_cast<int32_t>(K[g0 + t]) : 0;
        }
        LdAdamSteps a;
        ld_fill_adam_steps(a, gw, step0 + g0, lr, beta1, beta2, eps, general);
        launch_chunks(tb, gw, n, nchunk, ctab, s);
        if (ld_launch_status() != LD_OK) return LD_ERR_HIP;
        const dim3 grid((nsub + 7) / 8 * 8), wave(LD_WAVE);
        // One window holds a sub-tile's records (margin included) up to 24 of them on average, 2.3 %;
        // the second window's registers leave four waves per SIMD instead of five.
        const bool one = most * kSub <= 24 * n;
        if (general) k_sparse_adam<true, 2><<<grid, wave, 0, s>>>(w, m, v, n, nchunk, tb, gw, a, ctab);
        else if (one) k_sparse_adam<false, 1><<<grid, wave, 0, s>>>(w, m, v, n, nchunk, tb, gw, a, ctab);
        else k_sparse_adam<false, 2><<<grid, wave, 0, s>>>(w, m, v, n, nchunk, tb, gw, a, ctab);
        if (ld_launch_status() != LD_OK) return LD_ERR_HIP;
    }
    return LD_OK;
}
