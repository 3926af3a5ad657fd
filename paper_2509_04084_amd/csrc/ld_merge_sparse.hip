// ld_merge_sparse: ordered replay of a window of sparse diffs onto w.
//
// Recovery loop of Algorithm 1 (Sec. IV-B) and Eq. (6): M_{j+1} = M_j + merge(diff j)
// for j in iteration order, with the diffs of a batch kept apart and replayed one
// after another (Sec. IV-C, "Batched write semantics").  Update rule per record:
// p = fl32(lr*val); w[idx] = fl32(w[idx] - p).
//
// Two strategies with identical results:
//  * sweep   - one streaming pass over w.  A wave owns a sub-tile of 2048 to 8192
//              elements held in LDS, pulls the records of every diff that fall into it and
//              applies them diff after diff.  LDS operations of one wave execute
//              in issue order, so the cross-diff order on an element needs no
//              barrier.  Where a diff's records for the sub-tile start is not
//              looked up in a table: a small kernel finds the record range of
//              every 49152-element chunk by binary search, the wave
//              interpolates inside its chunk, loads a window of 64 or 128 records a little
//              before the guess and keeps the records that fall into its
//              sub-tile.  The guess is checked (the window must begin before the
//              sub-tile does, and end after it); a miss costs a binary search
//              inside the chunk or one more window, never a wrong result.
//              HBM traffic: 8n + 8*sum(K) bytes + the chunk table. Long windows of
//              sparse diffs and small arrays know exactly where the records lie, from a table
//              that one pass over the index arrays makes (k_subtab), if the workspace holds it:
//              a lane per record (k_merge_thin), a window per diff (k_merge_rows).
//  * scatter - one kernel per diff, one thread per record; for windows that
//              touch only a small part of w.
#include <atomic>

#include "ld_sparse_common.h"
#include "ld_thin.h"

namespace {

constexpr int kSub = 8192;                 // elements of the largest sub-tile of a sweep (32 KB of LDS and the spare word: 4 waves per CU)
constexpr int64_t kFewSubs = 80000000;     // elements below which such sub-tiles are too few
constexpr int kMargin = 24;                // records the window starts before the interpolated position
constexpr int kSweepGroup = kTableMax;     // diffs per sweep: a lane keeps the chunk ranges of two of them
// Windows loaded ahead, as <diffs per batch, 64-record windows per diff>: 10 x 2 for the usual
// densities (~80 records per diff and 8192 elements at 1 %), 10 x 1 where a sub-tile's records fit one
// window, 20 x 1 for long windows of very sparse
// diffs (a handful of records each: half as many rounds of loads, each a memory round trip).

// N records per lane of ONE diff (so no two of the wave's 64 N records name the same element):
// all are read before any is written - one round trip to LDS instead of N. Records outside the
// sub-tile land on the spare word behind it (an unsigned minimum instead of two comparisons and a
// branch around every access: these waves are bound by the instructions they issue).
template <int SUB, int N>
__device__ __forceinline__ void apply_records(float* tile, const int32_t (&i)[N], const float (&v)[N], int32_t lo,
                                              float lr) {
    float cur[N];
    uint32_t at[N];
#pragma unroll
    for (int u = 0; u < N; ++u) {
        const uint32_t e = static_cast<uint32_t>(i[u]) - static_cast<uint32_t>(lo);
        at[u] = e < static_cast<uint32_t>(SUB) ? e : static_cast<uint32_t>(SUB);
        cur[u] = tile[at[u]];
    }
#pragma unroll
    for (int u = 0; u < N; ++u) tile[at[u]] = __fsub_rn(cur[u], __fmul_rn(lr, v[u]));   // rounded product: never fused
}

// Applies the records of one diff at positions [p, end) that fall into [lo, hi), up to the
// first record at or beyond hi. kDeep loads of 64 records are in flight together: a dense
// diff has many such batches per sub-tile, and one at a time would leave the wave waiting
// for memory once per batch.
constexpr int kDeep = 8;

template <int SUB>
__device__ __forceinline__ void apply_from(float* tile, const int32_t* __restrict__ idx,
                                           const float* __restrict__ val, int32_t p, int32_t end,
                                           int32_t lo, int32_t hi, float lr, int lane) {
    for (; p < end; p += kDeep * LD_WAVE) {
        int32_t i[kDeep];
        float v[kDeep];
#pragma unroll
        for (int u = 0; u < kDeep; ++u) {
            const int32_t q = p + u * LD_WAVE + lane;
            const bool have = q < end;
            i[u] = have ? idx[q] : INT_MAX;
            v[u] = have ? val[q] : 0.0f;
        }
        apply_records<SUB>(tile, i, v, lo, lr);
        if (__builtin_amdgcn_readlane(i[kDeep - 1], LD_WAVE - 1) >= hi) break;  // ascending
    }
}

// Chunk range [c0, c1) and guessed start of diff t (lanes 0..63) and, in sweeps of more than 64
// diffs (SETS = 2), of diff t + 64.
template <int SETS>
struct Ranges {
    int32_t c0[SETS], c1[SETS], start[SETS];
};

template <int SETS>
__device__ __forceinline__ int32_t of_diff(const int32_t (&x)[SETS], int t) {
    if (SETS == 1) return __builtin_amdgcn_readlane(x[0], t);
    return t < LD_WAVE ? __builtin_amdgcn_readlane(x[0], t) : __builtin_amdgcn_readlane(x[SETS - 1], t - LD_WAVE);
}

// The first WIN * 64 records of PRE consecutive diffs at and after the guessed positions.
template <int PRE, int WIN>
struct Batch {
    int32_t s[PRE], e[PRE], b[PRE];   // window start, end of the chunk's records, their begin (wave-uniform)
    int32_t ri[PRE][WIN];
    float rv[PRE][WIN];
};

template <int PRE, int WIN, int SETS>
__device__ __forceinline__ void load_batch(Batch<PRE, WIN>& X, const DiffTable& tb, int32_t W, int32_t t0,
                                           const Ranges<SETS>& R, int lane) {
#pragma unroll
    for (int g = 0; g < PRE; ++g) {
        const int t = (t0 + g < W) ? t0 + g : 0;
        X.s[g] = of_diff(R.start, t);
        X.b[g] = of_diff(R.c0, t);
        X.e[g] = (t0 + g < W) ? of_diff(R.c1, t) : X.s[g];  // past W: an empty window
        const int32_t* __restrict__ ip = tb.idx[t];
        const float* __restrict__ vp = tb.val[t];
#pragma unroll
        for (int u = 0; u < WIN; ++u) {
            const int32_t p = X.s[g] + u * LD_WAVE + lane;
            const bool h = p < X.e[g];
            X.ri[g][u] = h ? ip[p] : INT_MAX;
            X.rv[g][u] = h ? vp[p] : 0.0f;
        }
    }
}

template <int SUB, int PRE, int WIN, int SETS>
__global__ __launch_bounds__(LD_WAVE) void k_merge_sweep(float* __restrict__ w, int64_t n, int32_t nchunk,
                                                         DiffTable tb, int32_t W,
                                                         const int32_t* __restrict__ ctab, float lr) {
    constexpr int kParts = static_cast<int>(kChunk / SUB);  // sub-tiles per chunk of the range table
    static_assert(static_cast<int64_t>(SUB) * kParts == kChunk, "sub-tiles must tile a chunk");
    __shared__ float tile[SUB + 4];  // and the spare word
    const int lane = threadIdx.x;
    // consecutive workgroups go to different XCDs (each with an L2 of its own): give every XCD one
    // contiguous eighth of w, so that the overlapping record windows of neighbouring sub-tiles hit its L2
    const int64_t per = (static_cast<int64_t>(gridDim.x) + 7) / 8;
    const int64_t sub = static_cast<int64_t>(blockIdx.x % 8) * per + blockIdx.x / 8;
    if (sub * SUB >= n) return;
    const int64_t lo64 = sub * SUB;
    const int32_t len = static_cast<int32_t>((n - lo64) < SUB ? (n - lo64) : SUB);
    const int32_t lo = static_cast<int32_t>(lo64), hi = lo + len;  // n <= INT_MAX
    const bool full = (len == SUB);

    ld_f32x4 x[SUB / 4 / LD_WAVE];
    if (full) {
        const ld_f32x4* src = reinterpret_cast<const ld_f32x4*>(w + lo64);
#pragma unroll
        for (int j = 0; j < SUB / 4 / LD_WAVE; ++j) x[j] = ld_nt_load(src + j * LD_WAVE + lane);
    }

    // lane t: where the records of diffs t and t + 64 lie in this chunk, and the guesses for this sub-tile
    const int32_t chunk = static_cast<int32_t>(sub / kParts), part = static_cast<int32_t>(sub % kParts);
    Ranges<SETS> R;
#pragma unroll
    for (int h = 0; h < SETS; ++h) {
        const int t = h * LD_WAVE + lane;
        R.c0[h] = R.c1[h] = 0;
        if (t < W) {
            const int32_t* row = ctab + static_cast<int64_t>(t) * (nchunk + 1) + chunk;
            R.c0[h] = row[0];
            R.c1[h] = row[1];
        }
        R.start[h] = R.c0[h] + ((R.c1[h] - R.c0[h]) * part) / kParts - kMargin;
        if (R.start[h] < R.c0[h]) R.start[h] = R.c0[h];
    }

    // The windows of the first PRE diffs are requested before the tile goes to LDS. (Requesting
    // every next batch while the current one is applied made the sweep 10 % slower.)
    Batch<PRE, WIN> A;
    load_batch(A, tb, W, 0, R, lane);

    if (full) {
#pragma unroll
        for (int j = 0; j < SUB / 4 / LD_WAVE; ++j) reinterpret_cast<ld_f32x4*>(tile)[j * LD_WAVE + lane] = x[j];
    } else {
        for (int32_t e = lane; e < len; e += LD_WAVE) tile[e] = w[lo64 + e];
    }
    __syncthreads();  // one wave: only orders the vector fill before the scalar updates

    for (int32_t t0 = 0; t0 < W; t0 += PRE) {
        if (t0 > 0) load_batch(A, tb, W, t0, R, lane);
#pragma unroll
        for (int g = 0; g < PRE; ++g) {
            if (A.s[g] < A.e[g]) {
                const int t = t0 + g;
                const int32_t first = __builtin_amdgcn_readfirstlane(A.ri[g][0]);
                if (A.s[g] == A.b[g] || first <= lo) {
                    // the window begins before the sub-tile's records do; ascending indices: a record
                    // at or beyond hi (or the padding past the chunk's end) in the last window says
                    // that nothing of this sub-tile follows
                    apply_records<SUB>(tile, A.ri[g], A.rv[g], lo, lr);
                    const bool more = __builtin_amdgcn_readlane(A.ri[g][WIN - 1], LD_WAVE - 1) < hi;
                    if (more) apply_from<SUB>(tile, tb.idx[t], tb.val[t], A.s[g] + WIN * LD_WAVE, A.e[g], lo, hi, lr, lane);
                } else {
                    // guess too late: find the first record of the sub-tile inside the chunk
                    const int32_t p = lower_bound_idx(tb.idx[t], A.b[g], A.s[g], lo);
                    apply_from<SUB>(tile, tb.idx[t], tb.val[t], p, A.e[g], lo, hi, lr, lane);
                }
            }
            __builtin_amdgcn_wave_barrier();  // keep diff g's LDS traffic ahead of diff g+1's
        }
    }

    __syncthreads();
    if (full) {
        ld_f32x4* dst = reinterpret_cast<ld_f32x4*>(w + lo64);
#pragma unroll
        for (int j = 0; j < SUB / 4 / LD_WAVE; ++j)
            ld_nt_store(reinterpret_cast<const ld_f32x4*>(tile)[j * LD_WAVE + lane], dst + j * LD_WAVE + lane);
    } else {
        for (int32_t e = lane; e < len; e += LD_WAVE) w[lo64 + e] = tile[e];
    }
}

// ------------------------------------------------------- thin long windows: a lane per record
//
// A long window of very sparse diffs (config 3: 100 diffs of 0.1 %, eight records per diff and 8192
// elements) leaves the sweep above with a wave's 64 lanes serving eight records at a time, a
// hundred times in a row. Here the records of all diffs that fall into the wave's sub-tile form one
// list in diff order, and the lanes take 64 of it at a time. Where
// exactly a diff's records for a sub-tile begin comes from a table of its own (k_subtab: one
// streaming pass over the index arrays, which are small when diffs are this sparse); which diff a list position
// belongs to comes from marks where the diffs begin.
//
// Order: a list goes through in blocks of 512 records. Most elements are named by one record of the block: those are updated
// at once, all rows together. A record whose element was met before in the block, and the one it met, wait: they are lined
// up in list order and go through in rows of 64. There every pending record bids for its element's slot of a small owner
// table with its lane, the smallest lane wins the slot (atomic minimum), applies its update and leaves; lanes are in list order, so
// the updates of one element go through in list order whatever else shares the slot, and any number of records is
// served. Where many of the first 128 records meet (diffs that share their positions), and at the last 128 of a list, all rows bid,
// without lining up (short lists that went through all of it: 1 M elements, 11 diffs of 0.1 % 12.5 us instead of 11.5, 6 M, 100 of
// 1/3000 32.4 instead of 31.0, with 256 MB written in between).
// Sub-tiles where the diffs are dense go through diff after diff (kThinDense).
//
// Bound by w's bytes up to some 200 records a sub-tile (100 M elements, 20 diffs of 1/400: 6.1 TB/s), beyond by the records: pieces of
// 16 bytes of as many lists as there are diffs. us a call when all rows bid / now: 124 M elements, 100 diffs of 0.1 % 223 / 217 (without records
// 187, with their loads alone 212), 50 of 0.4 % 255 / 220, 100 M, 40 of 0.5 % 210 / 180, 5.9 M, 84 of 0.27 % 25 / 21; diffs that share half of their
// positions with the one before 265 / 263 (lined up 277). Waiting records of all rows bidding together instead of lined up: 244 for
// the second. A wave that loads its next tile while it serves one, eight waves per CU: 239 and 236 us for the first two (its waits are for the
// records requested last). Sub-tiles of 2048 / 8192 elements: slower.
constexpr int kThinSub = 4096;     // elements of a wave's sub-tile in this kernel
constexpr int kThinAhead = 8;      // rows of 64 records requested together
constexpr int kOwner = 256;        // slots of the owner table
constexpr int kThinAlike = 16;     // of a block's first 128 records, those of an element met before beyond which the diffs count as alike
static_assert(kOwner * 32 >= 2 * kThinSub, "two bits per element");
// Records per diff from which a sub-tile goes through diff after diff (rows of an embedding that every iteration
// touches) instead of in rows of the list, and the rows of 64 of one diff requested together there. 50 diffs of
// 0.4 % on 124 M elements, all of them the same dense rows of 64 / 192 / 768 / 8192 elements: 264 / 251 / 292 / 478 us, as
// a list 309 / 422 / 838 / 2031, and with the line at 64 or 256 records 347 / 251 and 295 / 297 for the first two.
constexpr uint32_t kThinDense = 128;
constexpr int kThinDeep = 16;
static_assert(kThinSub % (4 * LD_WAVE) == 0 && kThinSub <= 4096 && kOwner == 256, "whole rows of 16-byte accesses; see ld_thin_slot");

// tab[t * (nsub + 1) + s] = number of records of diff t with idx < s * SUB, s = 0 .. nsub.
// A thread looks at PER consecutive records (16-byte loads; the index arrays of these paths are
// 16-byte aligned) and at the one before them, and fills the entries between the sub-tiles of
// neighbouring records; the thread that meets record K closes the row.
// PER records per thread, by the records of the table's diffs: 4 / 8 / 16 67.1 / 65.3 / 67.8 us per call with 12.8 M of them,
// 307 / 298 / 312 with 60 M, but the work of a thread is a chain, and short lists leave most of the chip to few
// threads: 4 takes 3 to 9 % less of a call below 1 M records (up to 40 % where the lists are sparser than the sub-tiles), as much at 10 M.
constexpr int64_t kSubtabMany = 10000000;
// Sub-tiles without a record that a thread fills by itself; the lanes of its wave share longer stretches (12 diffs of
// 1 % in the first tenth of 110 M elements: 1890 us a call with one thread filling the other nine).
constexpr int32_t kSubtabWide = 16;

template <int SUB, int PER>
__global__ __launch_bounds__(256) void k_subtab(DiffTable tb, int32_t nsub, int32_t* __restrict__ tab) {
    const int t = blockIdx.y;
    const int32_t K = tb.K[t];
    const int32_t* __restrict__ idx = tb.idx[t];
    const int32_t j0 = (static_cast<int32_t>(blockIdx.x) * 256 + static_cast<int32_t>(threadIdx.x)) * PER;
    const int lane = ld_lane();
    // a block of four that begins at a record lies inside the array's last 16 bytes at worst
    ld_u32x4 q[PER / 4];
#pragma unroll
    for (int u = 0; u < PER / 4; ++u) {
        q[u] = ld_u32x4{0u, 0u, 0u, 0u};
        if (j0 + 4 * u < K) q[u] = *reinterpret_cast<const ld_u32x4*>(idx + j0 + 4 * u);
    }
    int32_t a = j0 == 0 || j0 > K ? -1 : idx[j0 - 1] / SUB;
    int32_t* row = tab + static_cast<int64_t>(t) * (nsub + 1);
#pragma unroll
    for (int c = 0; c < PER; ++c) {
        const int32_t j = j0 + c;
        const int32_t b = j >= K ? nsub : static_cast<int32_t>(q[c / 4][c % 4]) / SUB;
        LdThinEntries fill = ld_thin_entries(a, b, nsub);
        if (j > K) fill = LdThinEntries{0, -1};
        const bool wide = fill.last - fill.first >= kSubtabWide;
        if (!wide)
            for (int32_t s = fill.first; s <= fill.last; ++s) row[s] = j;
        for (uint64_t todo = __ballot(wide); todo; todo &= todo - 1) {  // a stretch without records: the wave's lanes share it
            const int l = __builtin_ctzll(todo);
            const int32_t first = __builtin_amdgcn_readlane(fill.first, l), last = __builtin_amdgcn_readlane(fill.last, l);
            const int32_t value = __builtin_amdgcn_readlane(j, l);
            for (int32_t s = first + lane; s <= last; s += LD_WAVE) row[s] = value;
        }
        a = b;
    }
}

__global__ __launch_bounds__(LD_WAVE) void k_merge_thin(float* __restrict__ w, int64_t n, int32_t nsub,
                                                        DiffTable tb, int32_t W, const int32_t* __restrict__ tab,
                                                        float lr) {
    __shared__ float tile[kThinSub + 4];                     // and the spare word of apply_records
    __shared__ const int32_t* ibase[kTableMax];              // diff t's record with list position k: ibase[t][k]
    __shared__ const float* vbase[kTableMax];
    // of a block: the diff whose records begin at a list position; then 64 records that wait for their turn
    __shared__ union { __align__(8) unsigned char whose[kThinAhead * LD_WAVE]; struct { uint32_t e; float p; } wait[LD_WAVE]; } line;
    __shared__ __align__(16) uint32_t mark[kOwner];          // elements seen / seen again (a bit each), then the owner table
    constexpr int kSets = kTableMax / LD_WAVE;
    const int lane = threadIdx.x;
    const int64_t per = (static_cast<int64_t>(gridDim.x) + 7) / 8;   // each XCD walks one contiguous eighth of w
    const int64_t sub = static_cast<int64_t>(blockIdx.x % 8) * per + blockIdx.x / 8;
    if (sub * kThinSub >= n) return;
    const int64_t lo64 = sub * kThinSub;
    const int32_t len = static_cast<int32_t>((n - lo64) < kThinSub ? (n - lo64) : kThinSub);
    const int32_t lo = static_cast<int32_t>(lo64);
    const bool full = (len == kThinSub);

    // lane t: the records of diffs t and t + 64 inside this sub-tile
    int32_t p0[kSets];
    uint32_t cnt[kSets];
#pragma unroll
    for (int h = 0; h < kSets; ++h) {
        const int t = h * LD_WAVE + lane;
        p0[h] = 0;
        cnt[h] = 0;
        if (t < W) {
            const int32_t* row = tab + static_cast<int64_t>(t) * (nsub + 1) + sub;
            p0[h] = row[0];
            cnt[h] = ld_thin_count(p0[h], row[1], kThinSub);
        }
    }
    ld_f32x4 x[kThinSub / 4 / LD_WAVE];
    if (full) {
        const ld_f32x4* src = reinterpret_cast<const ld_f32x4*>(w + lo64);
#pragma unroll
        for (int j = 0; j < kThinSub / 4 / LD_WAVE; ++j) x[j] = ld_nt_load(src + j * LD_WAVE + lane);
    }
    uint32_t total = 0, first[kSets];                        // first: list position of the diff's first record here
#pragma unroll
    for (int h = 0; h < kSets; ++h) {
        const int t = h * LD_WAVE + lane;
        const uint32_t inc = ld_wave_iscan(cnt[h]);
        first[h] = total + inc - cnt[h];
        // only positions first .. first + cnt - 1 are ever looked up through these
        ibase[t] = t < W ? tb.idx[t] + (static_cast<int64_t>(p0[h]) - first[h]) : nullptr;
        vbase[t] = t < W ? tb.val[t] + (static_cast<int64_t>(p0[h]) - first[h]) : nullptr;
        total += static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(inc), LD_WAVE - 1));
    }
    __syncthreads();  // one wave: orders the fills before what follows

    bool staged = false;
    auto stage = [&]() {
        staged = true;
        if (full) {
#pragma unroll
            for (int j = 0; j < kThinSub / 4 / LD_WAVE; ++j) reinterpret_cast<ld_f32x4*>(tile)[j * LD_WAVE + lane] = x[j];
        } else {
            for (int32_t e = lane; e < len; e += LD_WAVE) tile[e] = w[lo64 + e];
        }
        __syncthreads();
    };
    if (total >= kThinDense * static_cast<uint32_t>(W)) {
        // no two records of one diff name the same element: nothing is bid for
        total = 0;  // nothing left for the list
        stage();
#pragma unroll 1
        for (int t = 0; t < W; ++t) {
            static_assert(kSets == 2, "");
            const int32_t c = __builtin_amdgcn_readlane(static_cast<int32_t>(t < LD_WAVE ? cnt[0] : cnt[1]), t & (LD_WAVE - 1));
            const int32_t p = __builtin_amdgcn_readlane(t < LD_WAVE ? p0[0] : p0[1], t & (LD_WAVE - 1));
            const int32_t* __restrict__ ip = tb.idx[t];
            const float* __restrict__ vp = tb.val[t];
#pragma unroll 1
            for (int32_t q = 0; q < c; q += kThinDeep * LD_WAVE) {
                int32_t i[kThinDeep];
                float v[kThinDeep];
#pragma unroll
                for (int u = 0; u < kThinDeep; ++u) {
                    const int32_t k = q + u * LD_WAVE + lane;
                    i[u] = k < c ? ip[p + k] : INT_MAX;
                    v[u] = k < c ? vp[p + k] : 0.0f;
                }
                apply_records<kThinSub>(tile, i, v, lo, lr);
                __builtin_amdgcn_wave_barrier();
            }
        }
    }

    // The list's records in diff order, kThinAhead rows of 64 at a time.
    constexpr uint32_t kBlock = kThinAhead * LD_WAVE;
    const auto ordered = [] {  // the wave's own LDS operations complete in order
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    };
    // A row's records in lane order, which is list order, whatever they share: see above. The owner table is left as it was.
    const auto take_turns = [&](uint32_t e, float p, bool pend) {
        uint32_t* own = mark + ld_thin_slot(e);
        while (__ballot(pend)) {
            if (pend) atomicMin(own, static_cast<uint32_t>(lane));
            ordered();
            const bool won = pend && *own == static_cast<uint32_t>(lane);
            ordered();
            if (won) {
                tile[e] = __fsub_rn(tile[e], p);
                *own = 0xFFFFFFFFu;
            }
            ordered();
            pend = pend && !won;
        }
    };
#pragma unroll 1
    for (uint32_t k0 = 0; k0 < total || !staged; k0 += kBlock) {
        // Lane and row give the list position. The diff it belongs to is the last one that begins at or before it: every diff with
        // records in the block marks where they begin, and a running maximum carries the marks on.
        reinterpret_cast<ld_u32x2*>(line.whose)[lane] = ld_u32x2{0u, 0u};
        ordered();
#pragma unroll
        for (int h = 0; h < kSets; ++h)
            if (cnt[h] > 0 && first[h] < k0 + kBlock && first[h] + cnt[h] > k0)
                line.whose[first[h] > k0 ? first[h] - k0 : 0u] = static_cast<unsigned char>(h * LD_WAVE + lane);
        ordered();
        uint32_t t[kThinAhead], carry = 0;
#pragma unroll
        for (int u = 0; u < kThinAhead; ++u) t[u] = line.whose[u * LD_WAVE + lane];
        int32_t ri[kThinAhead];
        float rv[kThinAhead];
#pragma unroll
        for (int u = 0; u < kThinAhead; ++u) {
            const uint32_t k = k0 + u * LD_WAVE + lane;
            ri[u] = 0;
            rv[u] = 0.0f;
            if (k0 + u * LD_WAVE < total) {  // uniform
                const uint32_t reach = ld_wave_imax(t[u]);
                t[u] = reach > carry ? reach : carry;
                carry = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(t[u]), LD_WAVE - 1));
                if (k < total) {
                    ri[u] = ibase[t[u]][k];
                    rv[u] = vbase[t[u]][k];
                }
            }
        }
        const bool few = total - k0 <= 2 * LD_WAVE;  // uniform; the list ends here
        const uint32_t clear = few ? 0xFFFFFFFFu : 0u;
        reinterpret_cast<ld_u32x4*>(mark)[lane] = ld_u32x4{clear, clear, clear, clear};
        if (!staged) stage();  // the tile arrives while the first records travel
        ordered();
        if (few) {
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const uint32_t e = static_cast<uint32_t>(ri[u] - lo);
                take_turns(e, __fmul_rn(lr, rv[u]), k0 + u * LD_WAVE + lane < total && e < static_cast<uint32_t>(len));
            }
            break;
        }
        // Elements that only one record of the block names, most of them, are updated in any order, all rows at once: a bit per
        // element tells a record that it is not the first there, a second one tells the first.
        uint32_t e[kThinAhead], old[kThinAhead];
        bool in[kThinAhead];
        const auto meet = [&](int u) {
            if (in[u]) old[u] = atomicOr(&mark[e[u] >> 5], 1u << (e[u] & 31));
        };
        const auto met = [&](int u) { return in[u] && (old[u] >> (e[u] & 31) & 1u); };
#pragma unroll
        for (int u = 0; u < kThinAhead; ++u) {
            e[u] = static_cast<uint32_t>(ri[u] - lo);
            in[u] = k0 + u * LD_WAVE + lane < total && e[u] < static_cast<uint32_t>(len);
            rv[u] = __fmul_rn(lr, rv[u]);   // rounded product: never fused
        }
        meet(0);
        meet(1);
        if (__popcll(__ballot(met(0))) + __popcll(__ballot(met(1))) > kThinAlike) {
            // diffs that share their positions: row after row, every pending record bids for its element
            reinterpret_cast<ld_u32x4*>(mark)[lane] = ld_u32x4{0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu};
            ordered();
#pragma unroll
            for (int u = 0; u < kThinAhead; ++u) take_turns(e[u], rv[u], in[u]);
            continue;
        }
#pragma unroll
        for (int u = 2; u < kThinAhead; ++u) meet(u);
#pragma unroll
        for (int u = 0; u < kThinAhead; ++u)
            if (met(u)) atomicOr(&mark[kThinSub / 32 + (e[u] >> 5)], 1u << (e[u] & 31));
        ordered();
#pragma unroll
        for (int u = 0; u < kThinAhead; ++u) old[u] = in[u] ? mark[kThinSub / 32 + (e[u] >> 5)] : 0u;
        float cur[kThinAhead];
        uint32_t rank[kThinAhead], waiting = 0;  // among the records of the block that wait, in list order
#pragma unroll
        for (int u = 0; u < kThinAhead; ++u) {
            const bool again = met(u);
            const uint64_t all = __ballot(again);
            rank[u] = again ? waiting + ld_mbcnt(all) : 0xFFFFFFFFu;
            waiting += __popcll(all);
            old[u] = in[u] && !again ? e[u] : static_cast<uint32_t>(kThinSub);  // the spare word
            cur[u] = tile[old[u]];
        }
#pragma unroll
        for (int u = 0; u < kThinAhead; ++u) tile[old[u]] = __fsub_rn(cur[u], rv[u]);
        if (waiting == 0) continue;
        reinterpret_cast<ld_u32x4*>(mark)[lane] = ld_u32x4{0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu, 0xFFFFFFFFu};
#pragma unroll 1
        for (uint32_t r0 = 0; r0 < waiting; r0 += LD_WAVE) {
            ordered();
#pragma unroll
            for (int u = 0; u < kThinAhead; ++u)
                if (rank[u] - r0 < static_cast<uint32_t>(LD_WAVE)) {
                    line.wait[rank[u] - r0].e = e[u];
                    line.wait[rank[u] - r0].p = rv[u];
                }
            ordered();
            const bool mine = r0 + lane < waiting;
            take_turns(mine ? line.wait[lane].e : 0u, line.wait[lane].p, mine);
        }
    }

    __syncthreads();
    if (full) {
        ld_f32x4* dst = reinterpret_cast<ld_f32x4*>(w + lo64);
#pragma unroll
        for (int j = 0; j < kThinSub / 4 / LD_WAVE; ++j)
            ld_nt_store(reinterpret_cast<const ld_f32x4*>(tile)[j * LD_WAVE + lane], dst + j * LD_WAVE + lane);
    } else {
        for (int32_t e = lane; e < len; e += LD_WAVE) w[lo64 + e] = tile[e];
    }
}

// ------------------------------------------------ arrays that are a few rounds of the chip: windows from a table
//
// The sweep's windows hold three times the records that a small sub-tile needs: the margins of a guess. While w is not many
// times what the chip holds at once, that is what its time goes to (25.6 M elements, 50 diffs of 1 %: 87 us, without
// the windows 36). Here k_subtab says where every diff's records of every sub-tile lie, one pass over the index arrays;
// a window is those records and no more, and PRE diffs' windows are requested together.
// 25.6 M elements, 50 diffs of 1 %: 96 -> 72 us with the table's pass (13; 92 -> 66 on records that the last-level cache
// holds, as in what follows), 5 M, 20 diffs: 32 -> 16, 25 M, 100 diffs: 222 -> 163, 25 M, 50 diffs crowded in the first tenth
// 250 -> 85. Sub-tiles of 4096: 73 us for the first (nine waves per CU), of 2560: 65; 10 / 13 / 17 / 25 diffs a batch 67.6 / 66.8 /
// 66.8 / 67.5. The update left to the LDS unit's float add: 25 us more (sub-tiles of 4096).
constexpr int kRowSub = 2048;
constexpr int kRowBatch = 17;   // diffs whose windows are requested together (ten if they are two windows each)

template <int PRE, int WIN, int SETS>
__global__ __launch_bounds__(LD_WAVE) void k_merge_rows(float* __restrict__ w, int64_t n, int32_t nsub, DiffTable tb,
                                                        int32_t W, const int32_t* __restrict__ tab, float lr) {
    __shared__ float tile[kRowSub + 4];  // and the spare word of apply_records
    const int lane = threadIdx.x;
    // runs of 16 sub-tiles per XCD (4 / 64: 69.7 / 67.0 us against 66.3), not eighths of w: records crowd in places
    const int64_t sub = ld_xcd_piece<16>(blockIdx.x, gridDim.x);
    if (sub * kRowSub >= n) return;
    const int64_t lo64 = sub * kRowSub;
    const int32_t len = static_cast<int32_t>((n - lo64) < kRowSub ? (n - lo64) : kRowSub);
    const int32_t lo = static_cast<int32_t>(lo64);
    const bool full = (len == kRowSub);

    WindowTable rec[SETS];  // lane t: the records of diffs t and t + 64 inside this sub-tile
#pragma unroll
    for (int h = 0; h < SETS; ++h) {
        const int t = h * LD_WAVE + lane;
        rec[h] = WindowTable{0u, 0u, 0u, 0u, 0};
        if (t < W) {
            const int32_t* row = tab + static_cast<int64_t>(t) * (nsub + 1) + sub;
            rec[h] = window_at(tb, t, row[0], static_cast<int32_t>(ld_thin_count(row[0], row[1], kRowSub)));
        }
    }
    ld_f32x4 x[kRowSub / 4 / LD_WAVE];
    if (full) {
        const ld_f32x4* src = reinterpret_cast<const ld_f32x4*>(w + lo64);
#pragma unroll
        for (int j = 0; j < kRowSub / 4 / LD_WAVE; ++j) x[j] = ld_nt_load(src + j * LD_WAVE + lane);
    }
    Window<WIN> rows[PRE];
    auto load_rows = [&](int32_t t0) {
#pragma unroll
        for (int g = 0; g < PRE; ++g) {
            const int32_t t = t0 + g;
            if (SETS == 1 || t < LD_WAVE) load_window(rows[g], rec[0], t, t < W, lane);
            else load_window(rows[g], rec[SETS - 1], t - LD_WAVE, t < W, lane);
        }
    };
    load_rows(0);
    if (full) {
#pragma unroll
        for (int j = 0; j < kRowSub / 4 / LD_WAVE; ++j) reinterpret_cast<ld_f32x4*>(tile)[j * LD_WAVE + lane] = x[j];
    } else {
        for (int32_t e = lane; e < len; e += LD_WAVE) tile[e] = w[lo64 + e];
    }
    __syncthreads();  // one wave: only orders the vector fill before the scalar updates
#pragma unroll 1
    for (int32_t t0 = 0; t0 < W; t0 += PRE) {
        if (t0 > 0) load_rows(t0);
        bool crowded = false;
#pragma unroll
        for (int g = 0; g < PRE; ++g) crowded |= rows[g].count > WIN * LD_WAVE;
        if (!crowded) {
#pragma unroll
            for (int g = 0; g < PRE; ++g) {
                if (rows[g].count > 0) apply_records<kRowSub>(tile, rows[g].ri, rows[g].rv, lo, lr);
                __builtin_amdgcn_wave_barrier();  // keep diff g's LDS traffic ahead of diff g+1's
            }
        } else {  // diff after diff, eight times 64 records requested together
#pragma unroll 1
            for (int32_t t = t0; t < t0 + PRE && t < W; ++t) {
                const WindowTable& r = SETS == 1 || t < LD_WAVE ? rec[0] : rec[SETS - 1];
                const int l = t & (LD_WAVE - 1);
                const int32_t* ip = (const int32_t*)lane_pointer(r.idx_lo, r.idx_hi, l);
                const float* vp = (const float*)lane_pointer(r.val_lo, r.val_hi, l);
                apply_from<kRowSub>(tile, ip, vp, 0, __builtin_amdgcn_readlane(r.count, l), lo, INT_MAX, lr, lane);
                __builtin_amdgcn_wave_barrier();
            }
        }
    }
    __syncthreads();
    if (full) {
        ld_f32x4* dst = reinterpret_cast<ld_f32x4*>(w + lo64);
#pragma unroll
        for (int j = 0; j < kRowSub / 4 / LD_WAVE; ++j)
            ld_nt_store(reinterpret_cast<const ld_f32x4*>(tile)[j * LD_WAVE + lane], dst + j * LD_WAVE + lane);
    } else {
        for (int32_t e = lane; e < len; e += LD_WAVE) w[lo64 + e] = tile[e];
    }
}

__global__ __launch_bounds__(256) void k_merge_scatter(float* __restrict__ w,
                                                       const int32_t* __restrict__ idx,
                                                       const float* __restrict__ val, int32_t K,
                                                       float lr) {
    const int32_t j = blockIdx.x * 256 + threadIdx.x;
    if (j >= K) return;
    const int32_t i = idx[j];
    const float p = __fmul_rn(lr, val[j]);
    w[i] = __fsub_rn(w[i], p);
}

// A large diff scattered by granules of 64 bytes: four lanes read a granule that some record falls into, apply all of its
// records (at most 16, one after the other in the list) and write it back whole.
// What bounds the scatter of more records than the last-level cache takes granules for are the partial writes: 15.6 M updated
// words in 1.56 G elements take 294 us to read and 666 to write alone, as whole granules 259. Whole 128-byte lines
// are more bytes (676 us for both), plain loads or stores leave the granules in the caches (720).
// A wave whose records crowd into few granules (rows that every iteration touches) updates them word by word instead: its words
// are whole lines already, and a granule's records are a chain. kCrowded: granules of a wave's 64 records up to which it does.
// 15.6 M records in as many elements / 0.15 / 0.1 / 0.06 of theirs, us word by word 41 / 205 / 293 / 422, all by granules 470 / 241 /
// 241 / 297, now 41 / 204 / 230 / 294.
// Granules that hold records of two waves are updated word by word by both, so no wave reads another's records.
// A list that does not ascend or leaves [0, n) (a damaged file's) stays within the list and w here.
constexpr int kGran = 16;                    // elements
constexpr int kGranLanes = kGran / 4;        // lanes per granule
constexpr int kGranPer = LD_WAVE / kGranLanes;
constexpr int kCrowded = 32;

// Diffs that it is the faster way for, us word by word / by granules, and the same with another 0.8 GB written in between (a diff
// read back from storage finds neither itself nor its granules in the cache): 3 %, 15.6 M records 571 / 449 (565 / 507), 6 M 220 / 170 (212 /
// 192), 2 M 45 / 59 (79 / 68); 1 %, 15.6 M 718 / 650 (715 / 694), 6 M 279 / 249 (275 / 268), 5.1 M 1.2 % 228 / 200 (213 / 215); but
// 0.3-0.7 %, 5 to 8 M 270 / 255 (250 / 258), equidistant 6 M 308 / 301 (302 / 321), 9 M 407 / 394 (407 / 412).
bool granules_pay(int64_t n, int64_t k) { return k >= 9000000 || (k >= 5000000 && k * 80 >= n); }

__global__ __launch_bounds__(256) void k_merge_granules(float* __restrict__ w, int32_t n, const int32_t* __restrict__ idx,
                                                        const float* __restrict__ val, int32_t K, float lr) {
    __shared__ int32_t at[256 / LD_WAVE][LD_WAVE];
    __shared__ float by[256 / LD_WAVE][LD_WAVE];
    const int lane = threadIdx.x & (LD_WAVE - 1), wave = threadIdx.x / LD_WAVE;
    const int32_t base = static_cast<int32_t>(blockIdx.x) * 256 + wave * LD_WAVE;  // K <= n <= INT_MAX: the grid ends below 2^31
    if (base >= K) return;
    const int32_t left = K - base;           // >= 1
    const int32_t i = lane < left ? idx[base + lane] : -1;
    const float p = lane < left ? __fmul_rn(lr, val[base + lane]) : 0.0f;
    const int32_t g = i >= 0 && i < n ? i / kGran : -1;
    // the granule of the lane before (lane 0: none)
    const int32_t g_before = __builtin_amdgcn_update_dpp(-1, g, 0x138 /* wave_shr:1 */, 0xf, 0xf, false);
    const uint64_t first = __ballot(g >= 0 && g != g_before);  // the first record of its granule in the wave
    if (__popcll(first) <= kCrowded) {
        if (g >= 0) w[i] = __fsub_rn(w[i], p);
        return;
    }
    // lane 0: the record before the wave's, lane 63: the one behind (loaded ahead, a crowded wave would be a third slower)
    int32_t beside = -1;
    if (lane == 0 && base > 0) beside = idx[base - 1];
    if (lane == LD_WAVE - 1 && left > LD_WAVE) beside = idx[base + LD_WAVE];
    const int32_t g_beside = beside >= 0 && beside < n ? beside / kGran : -1;
    const int32_t shared0 = __builtin_amdgcn_readlane(g_beside, 0), shared1 = __builtin_amdgcn_readlane(g_beside, LD_WAVE - 1);
    // of a granule that a neighbouring wave has records of too, or one that w ends in
    const bool alone = g >= 0 && (g == shared0 || g == shared1 || g >= n / kGran);
    at[wave][lane] = alone ? -1 : g < 0 ? -1 : i;
    by[wave][lane] = p;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");  // the wave's own words: its LDS operations complete in order
    __builtin_amdgcn_wave_barrier();
    const int32_t* qi = at[wave];
    const float* qp = by[wave];

    const int part = lane % kGranLanes;
    ld_f32x4 x[kGranLanes];
    int32_t gran[kGranLanes];                // -1: nothing to do, its records are an earlier one's
#pragma unroll
    for (int t = 0; t < kGranLanes; ++t) {
        const int r = t * kGranPer + lane / kGranLanes;
        gran[t] = first >> r & 1u && qi[r] >= 0 ? qi[r] / kGran : -1;
        x[t] = ld_f32x4{0.0f, 0.0f, 0.0f, 0.0f};
        if (gran[t] >= 0) x[t] = ld_nt_load(reinterpret_cast<const ld_f32x4*>(w) + static_cast<int64_t>(gran[t]) * kGranLanes + part);
    }
    if (alone) w[i] = __fsub_rn(w[i], p);
#pragma unroll
    for (int t = 0; t < kGranLanes; ++t) {
        if (gran[t] < 0) continue;
        const int r = t * kGranPer + lane / kGranLanes;
        int32_t e = qi[r];
        int k = r;
        do {
            const float q = qp[k];
            const int c = e % kGran - part * 4;  // the lane's own elements: 0 to 3
            x[t].x = c == 0 ? __fsub_rn(x[t].x, q) : x[t].x;
            x[t].y = c == 1 ? __fsub_rn(x[t].y, q) : x[t].y;
            x[t].z = c == 2 ? __fsub_rn(x[t].z, q) : x[t].z;
            x[t].w = c == 3 ? __fsub_rn(x[t].w, q) : x[t].w;
            ++k;
            e = k < LD_WAVE ? qi[k] : -1;
        } while (e >= 0 && e / kGran == gran[t]);
        ld_nt_store(x[t], reinterpret_cast<ld_f32x4*>(w) + static_cast<int64_t>(gran[t]) * kGranLanes + part);
    }
}

template <int SUB, int PRE, int WIN>
void launch_sweep(float* w, int64_t n, int32_t nchunk, const DiffTable& tb, int32_t W, const int32_t* ctab, float lr,
                  hipStream_t s) {
    const int64_t nsub = (n + SUB - 1) / SUB;
    const dim3 grid(static_cast<uint32_t>((nsub + 7) / 8 * 8)), wave(LD_WAVE);
    if (W <= LD_WAVE) k_merge_sweep<SUB, PRE, WIN, 1><<<grid, wave, 0, s>>>(w, n, nchunk, tb, W, ctab, lr);
    else k_merge_sweep<SUB, PRE, WIN, 2><<<grid, wave, 0, s>>>(w, n, nchunk, tb, W, ctab, lr);
}

template <int SUB>
void launch_subtab(const DiffTable& tb, int32_t gw, int64_t most, int32_t nsub, int32_t* tab, hipStream_t s) {
    int64_t records = 0;
    for (int32_t t = 0; t < gw; ++t) records += tb.K[t];
    if (records < kSubtabMany) k_subtab<SUB, 4><<<dim3(static_cast<uint32_t>(most / (256 * 4) + 1), gw), dim3(256), 0, s>>>(tb, nsub, tab);
    else k_subtab<SUB, 8><<<dim3(static_cast<uint32_t>(most / (256 * 8) + 1), gw), dim3(256), 0, s>>>(tb, nsub, tab);
}

template <int PRE, int WIN>
void launch_rows(float* w, int64_t n, int32_t nsub, const DiffTable& tb, int32_t W, const int32_t* tab, float lr, hipStream_t s) {
    const dim3 grid(static_cast<uint32_t>((nsub + 7) / 8 * 8)), wave(LD_WAVE);
    if (W <= LD_WAVE) k_merge_rows<PRE, WIN, 1><<<grid, wave, 0, s>>>(w, n, nsub, tb, W, tab, lr);
    else k_merge_rows<PRE, WIN, 2><<<grid, wave, 0, s>>>(w, n, nsub, tb, W, tab, lr);
}

}  // namespace

namespace {

// Windows from a table (k_merge_rows), sweep / rows in us: 200 M elements, 4 diffs of 1 % 280 / 279, 100 M, 20 of 1 % 192 / 176,
// 60 of 1 % 361 / 298; but 170 M, 30 of 2 % 449 / 462, 300 M, 9 of 0.5 % 413 / 424 and 600 M, 20 of 1 % 996 / 1100: the pass
// over the index arrays costs what the windows save. Two windows where a sub-tile's records outgrow one (2 % a diff): 25 M, 50 of 3.3 %
// 170 / 127, 3 M, 20 of 2.5 % 29 / 18, but 100 M, 30 of 3.3 % 358 / 368. The larger the array the earlier: a sub-tile with more records than its
// window is served diff after diff, which few are of even records but many where layers differ in density. Sweep / one window / two,
// densities even and log-normal over 60 layers (sigma 0.7): 82 M elements, 18 diffs of 1.6 % 157 / 157 / 155 and 195 / 163 / 149, 72 of
// 1.25 % 401 / 314 / 340 and 550 / 361 / 356, 118 M, 18 of 1.25 % 211 / 207 / 199 and 250 / 211 / 197, 76 M, 40 of 1.6 % 273 / 229 / 232 and 333 / 236 /
// 232, 110 of 1.6 % 603 / 525 / 538 and 840 / 502 / 474: two windows are ten diffs a batch, which even records of many diffs lose by.
constexpr int64_t kRowsMost = 120000000;
int rows_windows(int64_t n, int32_t gw, int64_t most) {  // 64-record windows per diff, 0: another way
    if (n >= kRowsMost || most * kSub > 168 * n) return n < kFewSubs ? 2 : 0;
    if (n < 20000000) return 1;
    return n < kFewSubs ? (gw <= 64 && most * kSub > 120 * n ? 2 : 1) : (gw <= 32 && most * kSub > 100 * n ? 2 : 1);
}

// Up to which density a group of `gw` diffs runs a lane per record (k_merge_thin), in records of its largest diff per 8192 elements
// (0: not at all): that pays by the record, windows from a table and the sweep by the diff.
// Windows / a lane per record, us a call, densities even (and log-normal over 60 layers, sigma 0.7): 30 diffs of 1/200 49 / 62
// (49 / 62) on 25 M elements, 29 / 32 (28 / 37) on 10 M, 20 / 18 (20 / 27) on 6 M; 40 of 1/270 53 / 63 (53 / 63) on 25 M, 19 / 18
// (18 / 28) on 4 M, 159 / 161 (158 / 168) on 90 M, of 1/200 182 / 184 (180 / 206) on 100 M; 60 of 1/250 40 / 37 (40 / 48) on 10 M;
// 64 of 1/330 154 / 122 (153 / 134) on 60 M; 56 of 1/200 250 / 266 (250 / 301) on 118 M; 100 of 1/270 53 / 45 on 10 M, 338 / 294 on
// 118 M. Up to 24 diffs sparser than the line are scattered more often than not; below 2 M elements it is the launches.
// Sweep / a lane per record, where there is no table of windows: 150 M elements, 32 diffs of 1/120 343 / 313, 100 of 1/120 845 / 718;
// 400 M, 32 of 1/150 773 / 751, of 1/120 793 / 831, 64 of 1/150 1192 / 1107, 100 of 1/120 2035 / 1845. 11 to 24 diffs, sweep over a lane
// per record, densities even and log-normal (sigma 1): up to 74 records 1.01 to 1.15 and 1.05 to 1.30 on 130, 185 and 250 M elements (20
// diffs of 1/290 on 250 M 439 / 395 us, 24 of 1/300 on 185 M 326 / 301); 24 diffs on 400 to 800 M at 37 records 1.01 to 1.04 and 1.14 to
// 1.17, at 54 0.97 to 0.99 and 1.22; on 1.4 G at 28 1.00 and 1.13, at 37 1.00 and 1.14, 16 diffs there 0.98 and 1.05 to 1.07.
int thin_line(int64_t n, int32_t gw) {
    if (gw <= 10) return 0;
    if (n < 2000000) return gw > kRowBatch ? 48 : 20;
    if (n < kRowsMost) {
        if (gw <= 24) return 10;
        if (gw > LD_WAVE) return 48;
        return gw <= 32 || (n >= 20000000 && n < 45000000) ? 24 : 36;
    }
    if (gw <= 24) return n < 300000000 ? 60 : n < 1000000000 ? 48 : 27;
    return gw <= LD_WAVE ? 56 : 72;
}

size_t chunk_table_bytes(int64_t n, int32_t W) {
    const int64_t group = W < kSweepGroup ? W : kSweepGroup;
    return ld_round_up(static_cast<size_t>(group) * (static_cast<size_t>(chunks(n)) + 1) * 4, 256);
}

size_t sub_table_bytes(int64_t n, int32_t gw, int32_t sub) {
    return ld_round_up(static_cast<size_t>(gw) * (static_cast<size_t>((n + sub - 1) / sub) + 1) * 4, 256);
}

// The per-sub-tile table that a group runs with, if it fits the workspace.
struct GroupTable {
    int32_t sub;     // elements per sub-tile: kThinSub (a lane per record), kRowSub (windows); 0: none, it runs as a sweep
    size_t bytes;
};
GroupTable group_table(int64_t n, int32_t gw, int64_t most, size_t workspace_bytes) {
    const GroupTable none{0, 0}, thin{kThinSub, sub_table_bytes(n, gw, kThinSub)}, rows{kRowSub, sub_table_bytes(n, gw, kRowSub)};
    const int line = thin_line(n, gw);
    if (line > 0 && most * kSub <= line * n) return thin.bytes <= workspace_bytes ? thin : none;
    if (!rows_windows(n, gw, most)) return none;
    if (rows.bytes <= workspace_bytes) return rows;
    // half the table of the windows: still faster than the sweep (20 diffs of 1/400 on 100 M elements 148 / 164)
    return gw > 10 && most * kSub <= 48 * n && thin.bytes <= workspace_bytes ? thin : none;
}

// Whether a window that would be scattered runs faster in groups with tables, and can. What is certain of a scatter is 2.4 us a
// launch; its records cost up to 46 ps more, but next to nothing where they crowd or the diffs share them, which the table
// does not gain by: a group takes some 13 us and 2 ps per element of w (measured on 2900 windows of 1 to 128 diffs, up to 300 M
// elements: counting the records too, 8 diffs of 0.3 % that all lie in the first fiftieth of 53 M elements took 84 us instead of 22, 24 of 0.1 %
// of 836 M 1400 instead of 440. Where the rule takes the table the mean gain is 4.5-fold, none of the evenly spread windows lost).
bool tables_pay(const int32_t* const* idx, const int64_t* K, int32_t W, int64_t n, const void* workspace,
                size_t workspace_bytes) {
    const int32_t groups = (W + kSweepGroup - 1) / kSweepGroup;
    int32_t launches = 0;
    for (int32_t t = 0; t < W; ++t) launches += K[t] > 0;
    if (groups * (13.0 + 2e-6 * static_cast<double>(n)) >= 2.4 * launches) return false;
    if (!workspace || !ld_aligned(workspace, 256) || workspace_bytes < chunk_table_bytes(n, W)) return false;
    for (int32_t g0 = 0; g0 < W; g0 += kSweepGroup) {
        const int32_t gw = (W - g0) < kSweepGroup ? (W - g0) : kSweepGroup;
        int64_t most = 0;
        for (int32_t t = g0; t < g0 + gw; ++t) {
            most = K[t] > most ? K[t] : most;
            if (!ld_aligned(idx[t], 16)) return false;
        }
        if (group_table(n, gw, most, workspace_bytes).sub == 0) return false;
    }
    return true;
}

}  // namespace

// The chunk table always; for thin groups and small arrays (when K is given) the larger per-sub-tile table, without
// which they run as ordinary sweeps.
extern "C" size_t ld_merge_sparse_workspace(int64_t n, int32_t W, const int64_t* K) {
    if (n <= 0 || W <= 0) return 256;
    size_t need = chunk_table_bytes(n, W);
    if (K && n <= INT32_MAX && W <= LD_MAX_WINDOW) {
        for (int32_t g0 = 0; g0 < W; g0 += kSweepGroup) {
            const int32_t gw = (W - g0) < kSweepGroup ? (W - g0) : kSweepGroup;
            int64_t most = 0;
            for (int32_t t = g0; t < g0 + gw; ++t) most = K[t] > most ? K[t] : most;
            const size_t table = group_table(n, gw, most, SIZE_MAX).bytes;
            if (table > need) need = table;
        }
    }
    return need;
}

namespace {

ld_status merge_sparse_impl(float* w, int64_t n, const int32_t* const* idx, const float* const* val,
                            const int64_t* K, int32_t W, float lr, void* workspace, size_t workspace_bytes,
                            ld_stream stream, int32_t strategy) {
    const ld_status st = check_diff_args(w, n, idx, val, K, W);
    if (st != LD_OK) return st;
    if (strategy < LD_MERGE_AUTO || strategy > LD_MERGE_SCATTER) return LD_ERR_RANGE;
    if (W == 0 || n == 0) return LD_OK;
    hipStream_t s = static_cast<hipStream_t>(stream);
    ld_begin_call();

    int64_t total = 0;
    for (int32_t t = 0; t < W; ++t) total += K[t];
    if (total == 0) return LD_OK;
    // measured on 1.56 G elements: a scattered record costs 46 ps, the sweep 1.35 ps per element of w
    // plus little per record: they meet where the window holds n / 34 records
    if (strategy == LD_MERGE_AUTO)
        strategy = (total * 32 >= n || tables_pay(idx, K, W, n, workspace, workspace_bytes)) ? LD_MERGE_SWEEP
                                                                                                : LD_MERGE_SCATTER;

    if (strategy == LD_MERGE_SCATTER) {
        for (int32_t t = 0; t < W; ++t) {
            if (K[t] == 0) continue;
            const int32_t k = static_cast<int32_t>(K[t]);
            const dim3 grid((static_cast<uint32_t>(k) + 255) / 256);
            if (granules_pay(n, k) && ld_aligned(w, kGran * 4))
                k_merge_granules<<<grid, dim3(256), 0, s>>>(w, static_cast<int32_t>(n), idx[t], val[t], k, lr);
            else
                k_merge_scatter<<<grid, dim3(256), 0, s>>>(w, idx[t], val[t], k, lr);
            if (ld_launch_status() != LD_OK) return LD_ERR_HIP;
        }
        return LD_OK;
    }

    if (!workspace || !ld_aligned(workspace, 256) || workspace_bytes < chunk_table_bytes(n, W))
        return LD_ERR_WORKSPACE;
    const int32_t nchunk = chunks(n);
    int32_t* ctab = static_cast<int32_t*>(workspace);
    for (int32_t g0 = 0; g0 < W; g0 += kSweepGroup) {
        const int32_t gw = (W - g0) < kSweepGroup ? (W - g0) : kSweepGroup;
        DiffTable tb = {};
        int64_t most = 0;
        bool aligned16 = true;
        for (int32_t t = 0; t < kTableMax; ++t) {
            const bool live = t < gw;
            tb.idx[t] = live ? idx[g0 + t] : nullptr;
            tb.val[t] = live ? val[g0 + t] : nullptr;
            tb.K[t] = live ? static_cast<int32_t>(K[g0 + t]) : 0;
            if (live && K[g0 + t] > most) most = K[g0 + t];
            if (live && !ld_aligned(idx[g0 + t], 16)) aligned16 = false;
        }
        const dim3 wave(LD_WAVE);
        const GroupTable table = group_table(n, gw, most, workspace_bytes);
        if (table.sub > 0 && aligned16) {  // (else: the sweep below)
            const bool thin = table.sub == kThinSub;
            const int32_t nsub = static_cast<int32_t>((n + table.sub - 1) / table.sub);
            if (thin) launch_subtab<kThinSub>(tb, gw, most, nsub, ctab, s);
            else launch_subtab<kRowSub>(tb, gw, most, nsub, ctab, s);
            if (ld_launch_status() != LD_OK) return LD_ERR_HIP;
            if (thin) k_merge_thin<<<dim3((nsub + 7) / 8 * 8), wave, 0, s>>>(w, n, nsub, tb, gw, ctab, lr);
            else if (rows_windows(n, gw, most) == 1) launch_rows<kRowBatch, 1>(w, n, nsub, tb, gw, ctab, lr, s);
            else launch_rows<10, 2>(w, n, nsub, tb, gw, ctab, lr, s);
            if (ld_launch_status() != LD_OK) return LD_ERR_HIP;
            continue;
        }
        launch_chunks(tb, gw, n, nchunk, ctab, s);
        if (ld_launch_status() != LD_OK) return LD_ERR_HIP;
        // Sub-tile and record windows by the records of the densest diff in 8192 elements and by how many
        // sub-tiles there are. 2048 elements (19 waves per CU instead of 4) while the sub-tiles of 8192 make
        // only a few rounds of the chip, with one window per diff where its records fit: 25.6 M elements,
        // 50 diffs of 1 %: 124 -> 96 us, 20 diffs of 2 %: 118 -> 73; the same at 100 M. Beyond, a wave with
        // more records per diff than its windows hold fetches the rest by itself: smaller sub-tiles up to
        // where the windows fit again (400 M, 10 diffs of 2 %: 850 / 673 / 693 us with 8192 / 4096 / 2048,
        // of 4 %: 1007 / 915 / 836); else 8192, fewest windows (GPT-2 XL: 2555 / 2634 / 2746).
        const int64_t dense = most * kSub / n;
        if (gw > 10 && dense <= 16) launch_sweep<kSub, 20, 1>(w, n, nchunk, tb, gw, ctab, lr, s);
        else if (n < kFewSubs && dense <= 100) launch_sweep<2048, 10, 1>(w, n, nchunk, tb, gw, ctab, lr, s);
        else if (n < kFewSubs || dense > 200) launch_sweep<2048, 10, 2>(w, n, nchunk, tb, gw, ctab, lr, s);
        else if (dense > 100) launch_sweep<4096, 10, 2>(w, n, nchunk, tb, gw, ctab, lr, s);
        else launch_sweep<kSub, 10, 2>(w, n, nchunk, tb, gw, ctab, lr, s);
        if (ld_launch_status() != LD_OK) return LD_ERR_HIP;
    }
    return LD_OK;
}

}  // namespace

extern "C" ld_status ld_merge_sparse_strategy(float* w, int64_t n, const int32_t* const* idx,
                                              const float* const* val, const int64_t* K, int32_t W,
                                              float lr, void* workspace, size_t workspace_bytes,
                                              ld_stream stream, int32_t strategy) {
    return merge_sparse_impl(w, n, idx, val, K, W, lr, workspace, workspace_bytes, stream, strategy);
}

extern "C" ld_status ld_merge_sparse(float* w, int64_t n, const int32_t* const* idx,
                                     const float* const* val, const int64_t* K, int32_t W, float lr,
                                     void* workspace, size_t workspace_bytes, ld_stream stream) {
    return ld_merge_sparse_strategy(w, n, idx, val, K, W, lr, workspace, workspace_bytes, stream,
                                    LD_MERGE_AUTO);
}

// ------------------------------------------------ the entry point that allocates nothing
//
// The merge's only scratch memory is a group's table: the chunks' (k_chunks), or the sub-tiles' (k_subtab) where the
// window calls for that and it fits. Here it lives in a file-scope
// device array instead of a caller's workspace: one copy per GPU, held until the process
// ends, shared by every call on that GPU. Nothing in it has to start at zero (both kernels
// write every entry that is read), so nothing is cleared between calls.
static __device__ __align__(256) unsigned char scratch[LD_MERGE_STATIC_SCRATCH];

namespace {

constexpr int kMaxDevices = 64;
std::atomic<void*> scratch_ptr[kMaxDevices];  // per device: the address of ITS copy of `scratch`

// Device address of the current device's scratch array (looked up once per device; the array's
// name is only a host-side handle and is never passed to a kernel).
ld_status static_scratch(void** out) {
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return LD_ERR_HIP;
    void* p = scratch_ptr[dev].load(std::memory_order_acquire);
    if (!p) {
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return LD_ERR_HIP;
        scratch_ptr[dev].store(p, std::memory_order_release);  // every thread finds the same address
    }
    *out = p;
    return LD_OK;
}

}  // namespace

extern "C" size_t ld_merge_sparse_static_limit(void) { return LD_MERGE_STATIC_SCRATCH; }

extern "C" ld_status ld_merge_sparse_static(float* w, int64_t n, const int32_t* const* idx,
                                            const float* const* val, const int64_t* K, int32_t W, float lr,
                                            ld_stream stream) {
    const ld_status st = check_diff_args(w, n, idx, val, K, W);
    if (st != LD_OK) return st;
    if (chunk_table_bytes(n, W) > LD_MERGE_STATIC_SCRATCH) return LD_ERR_WORKSPACE;
    if (W == 0 || n == 0) return LD_OK;
    void* ptr = nullptr;
    const ld_status sp = static_scratch(&ptr);
    if (sp != LD_OK) return sp;
    return merge_sparse_impl(w, n, idx, val, K, W, lr, ptr, LD_MERGE_STATIC_SCRATCH, stream, LD_MERGE_AUTO);
}
