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
// Bound by the vector ALUs for all but the shortest windows. An element's step is four full-rate operations and two
// of two issue slots each (measured: v_sqrt_f32 and v_rcp_f32 take 2.1 slots of v_fma_f32; together with the tiles'
// reads the steps alone take 6.6 ms for 20 diffs on 1.56 G elements), about as long as its 24 n bytes take (6.7 ms
// without the steps); what a wave does per step and diff besides (addresses, window, scatter, clearing: some 25 vector
// instructions beside 96) and what of the two does not overlap make it 9.0-9.4 ms. The loop's order (a row of
// the tiles read while the row before is computed, scalars by lane reads instead of scalar loads, whose counter is
// the LDS's, windows without masks) took 9.4-9.7 ms to that. 8 KB of LDS and 96 registers let five waves share a SIMD; four
// run as fast, and so do other waves' priorities and other runs per XCD. 2048-element sub-tiles (two waves per SIMD): 11.7 ms before.
#include "ld_sparse_common.h"

namespace {

constexpr int kSub = 1024;                 // elements per wave sub-tile (two tiles: 8 KB of LDS, 20 waves per CU)
constexpr int kChunkSubs = 48;             // sub-tiles per chunk of the range table
static_assert(static_cast<int64_t>(kSub) * kChunkSubs == kChunk, "sub-tiles must tile a chunk");
constexpr int kRows = kSub / 4 / LD_WAVE;  // 16-byte vectors per lane and array: 4
constexpr int kMargin = 32;                // records the window starts before the interpolated position
constexpr int32_t kMany = 1 << 20;

// Adds the records of [p, end) that fall into [lo, hi) to the gradient tiles.
__device__ __forceinline__ void scatter_from(float* tile1, float* tile2, const int32_t* __restrict__ idx,
                                             const float* __restrict__ val, int32_t p, int32_t end,
                                             int32_t lo, int32_t hi, float omb1, float omb2, int lane) {
    for (; p < end; p += LD_WAVE) {
        const bool have = p + lane < end;
        const int32_t i = have ? idx[p + lane] : INT_MAX;
        const float v = have ? val[p + lane] : 0.0f;
        if (i >= lo && i < hi) ld_adam_terms(v, omb1, omb2, tile1[i - lo], tile2[i - lo]);
        if (__ballot(i >= hi)) break;
    }
}

__device__ __forceinline__ void clear_tiles(float* tile1, float* tile2, int lane) {
#pragma unroll
    for (int j = 0; j < kRows; ++j) {
        reinterpret_cast<ld_f32x4*>(tile1)[j * LD_WAVE + lane] = ld_f32x4{0.0f, 0.0f, 0.0f, 0.0f};
        reinterpret_cast<ld_f32x4*>(tile2)[j * LD_WAVE + lane] = ld_f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    }
}

// First record of the window for sub-tile `part` of a chunk of `len` elements whose records are [b, e): ahead of where the
// sub-tile's begin if the chunk's are evenly spread. Records of a neighbouring chunk that it reaches do not matter. The last chunk is
// short: its records lie in its first sub-tiles (as if they filled 48, its last windows ended too early, and its waves were what a
// call on a small array waited for: 450 K elements, 37 diffs of 0.5 %, 44 us instead of 33).
__device__ __forceinline__ int32_t window_begin(int32_t b, int32_t e, int32_t part, int32_t len) {
    const uint32_t of = e > b ? static_cast<uint32_t>(e - b) : 0u;  // at most an element's worth each: products below 2^32
    const uint32_t ahead = len == kChunk ? of * static_cast<uint32_t>(part) / kChunkSubs
                                         : of * static_cast<uint32_t>(part * kSub) / static_cast<uint32_t>(len);
    const int32_t p = static_cast<int32_t>(static_cast<uint32_t>(b) + ahead) - kMargin;
    return p < 0 ? 0 : p;
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

    // lane t: where diff t's records of this chunk lie, its record window's address and its step's
    // scalars. They are handed to the loop by lane reads: scalar loads there would share their counter
    // with the LDS reads, and every wait for one of those would be a wait for all.
    const int32_t chunk = static_cast<int32_t>(sub / kChunkSubs), part = static_cast<int32_t>(sub % kChunkSubs);
    int32_t c0 = 0, c1 = 0;
    const int32_t* ip = nullptr;
    const float* vp = nullptr;
    float lr_bc1_t = 0.0f, scale_t = 0.0f, eps_t = 0.0f;
    if (lane < W) {
        const int32_t* row = ctab + static_cast<int64_t>(lane) * (nchunk + 1) + chunk;
        c0 = row[0];
        c1 = row[1];
        ip = tb.idx[lane];
        vp = tb.val[lane];
        if (GENERAL) lr_bc1_t = a.lr_bc1[lane];
        scale_t = a.root_scale[lane];
        eps_t = a.eps_s[lane];
    }

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

    const int64_t chunk_left = n - static_cast<int64_t>(chunk) * kChunk;
    const int32_t chunk_len = static_cast<int32_t>(chunk_left < kChunk ? chunk_left : kChunk);
    const int32_t start = window_begin(c0, c1, part, chunk_len);
    const uint64_t ia = reinterpret_cast<uint64_t>(ip + start), va = reinterpret_cast<uint64_t>(vp + start);
    const uint32_t ia_lo = static_cast<uint32_t>(ia), ia_hi = static_cast<uint32_t>(ia >> 32);
    const uint32_t va_lo = static_cast<uint32_t>(va), va_hi = static_cast<uint32_t>(va >> 32);
    // records from the window's begin to the list's end (at most kMany), and whether it begins at or ahead of the chunk's
    int32_t count = lane < W ? tb.K[lane] - start : 0;
    if (count > kMany) count = kMany;
    const int32_t count_t = count * 2 + (start <= c0);
    clear_tiles(tile1, tile2, lane);
    __syncthreads();  // one wave: only orders the vector fill before the scalar scatters

    // The scalars are waited for here: left pending, every wait for an LDS read in the loop would be one for all of them.
    float beta1 = a.beta1, beta2 = a.beta2, omb1 = a.one_m_beta1, omb2 = a.one_m_beta2;
    asm volatile("" : "+s"(beta1), "+s"(beta2), "+s"(omb1), "+s"(omb2));

    struct Window {
        int32_t count;  // as count_t
        int32_t ri[WIN];
        float rv[WIN];
    };
    // Lanes beyond the list's end take its last record again: twice the same write of the same value. Past W: nothing.
    auto fetch = [&](int32_t t, Window& x) {
        x.count = t < W ? __builtin_amdgcn_readlane(count_t, t) : 1;
        const int32_t last = (x.count >> 1) - 1;
        if (last < 0) {
#pragma unroll
            for (int u = 0; u < WIN; ++u) {
                x.ri[u] = INT_MAX;
                x.rv[u] = 0.0f;
            }
        } else {
            const GlobalBytes i0 = lane_pointer(ia_lo, ia_hi, t), v0 = lane_pointer(va_lo, va_hi, t);
#pragma unroll
            for (int u = 0; u < WIN; ++u) {
                int32_t p = u * LD_WAVE + lane;
                if (p > last) p = last;
                const uint32_t o = static_cast<uint32_t>(p) * 4u;
                x.ri[u] = *reinterpret_cast<const __attribute__((address_space(1))) int32_t*>(i0 + o);
                x.rv[u] = *reinterpret_cast<const __attribute__((address_space(1))) float*>(v0 + o);
            }
        }
    };
    // Puts the step's records into the (zero) tiles; at: where this lane's went (len and above: nowhere).
    // True if some did not come from the window: it ended too early, or began too late.
    auto scatter = [&](int32_t t, const Window& x, uint32_t (&at)[WIN]) {
        const bool hit = (x.count & 1) || __builtin_amdgcn_readfirstlane(x.ri[0]) <= lo;
        const bool more = !hit || ((x.count >> 1) > WIN * LD_WAVE && __builtin_amdgcn_readlane(x.ri[WIN - 1], LD_WAVE - 1) < hi);
#pragma unroll
        for (int u = 0; u < WIN; ++u) {
            at[u] = static_cast<uint32_t>(x.ri[u]) - static_cast<uint32_t>(lo);
            if (at[u] < static_cast<uint32_t>(len))
                ld_adam_terms(x.rv[u], omb1, omb2, tile1[at[u]], tile2[at[u]]);
        }
        if (more) {  // the records ahead of the window too where it began too late: all there are
            const int32_t* row = ctab + static_cast<int64_t>(t) * (nchunk + 1) + chunk;
            const int32_t b = row[0], e = row[1];
            const int32_t from = hit ? window_begin(b, e, part, chunk_len) + WIN * LD_WAVE : lower_bound_idx(tb.idx[t], b, e, lo);
            scatter_from(tile1, tile2, tb.idx[t], tb.val[t], from, e, lo, hi, omb1, omb2, lane);
        }
        return more;
    };
    struct Row { ld_f32x4 g1, g2; };
    auto read_row = [&](int j) {
        return Row{reinterpret_cast<const ld_f32x4*>(tile1)[j * LD_WAVE + lane],
                   reinterpret_cast<const ld_f32x4*>(tile2)[j * LD_WAVE + lane]};
    };

    // One trip per diff. What the vector units need next is always on its way while they work: a row of
    // the tiles is read while the row before it is computed, the next step's records go into the tiles (cleared
    // at once behind the last read: LDS operations of a wave complete in order) before this step's last two
    // rows are computed, and their window was requested a whole step earlier.
    Window x0, x1;
    uint32_t at[WIN];
    fetch(0, x0);
    fetch(1, x1);
    bool more = scatter(0, x0, at);
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    Row r0 = read_row(0), r1;
    auto step = [&](int32_t t, Window& later, const Window& next) {
        fetch(t + 2, later);
        const float lr_bc1 = GENERAL ? __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(lr_bc1_t), t)) : 0.0f;
        const float scale = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(scale_t), t));
        const float eps_s = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(eps_t), t));
        auto compute = [&](int j, const Row& r) {
            const float g1[4] = {r.g1.x, r.g1.y, r.g1.z, r.g1.w}, g2[4] = {r.g2.x, r.g2.y, r.g2.z, r.g2.w};
#pragma unroll
            for (int q = 0; q < 4; ++q)
                ld_adam_step<GENERAL>(ww[j][q], mm[j][q], vv[j][q], g1[q], g2[q], beta1, beta2, lr_bc1, scale, eps_s);
            // keeps the row's work here (the compiler would sink it below the branches that follow) and the
            // moments out of the registers the row was read into (they would be moved back every trip)
            asm volatile("" : "+v"(ww[j][0]), "+v"(ww[j][1]), "+v"(ww[j][2]), "+v"(ww[j][3]) : "v"(r.g1), "v"(r.g2));
            __builtin_amdgcn_sched_barrier(0);
        };
        r1 = read_row(1);
        __builtin_amdgcn_sched_barrier(0);
        compute(0, r0);
        r0 = read_row(2);
        __builtin_amdgcn_sched_barrier(0);
        compute(1, r1);
        r1 = read_row(3);
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        __builtin_amdgcn_sched_barrier(0);
        if (more) {
            clear_tiles(tile1, tile2, lane);
        } else {
#pragma unroll
            for (int u = 0; u < WIN; ++u)
                if (at[u] < static_cast<uint32_t>(len)) tile1[at[u]] = tile2[at[u]] = 0.0f;
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        more = scatter(t + 1, next, at);
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_sched_barrier(0);
        compute(2, r0);
        r0 = read_row(0);
        __builtin_amdgcn_sched_barrier(0);
        compute(3, r1);
    };
#pragma unroll 1
    for (int32_t t = 0; t < W; t += 2) {
        step(t, x0, x1);
        if (t + 1 == W) break;
        step(t + 1, x1, x0);
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
