// ld_combine_sparse: N per-worker record lists combined into one.
//
// Sync of Algorithm 1 (Sec. IV-B; Eq. (3)) for compressed gradients: what an
// all-gather leaves on every rank is N ascending (idx, val) lists; the synchronized
// diff that is checkpointed holds every index recorded by at least one worker, with
// the workers' values added in worker order (one fp32 add each, starting from +0)
// and multiplied by `scale` (1 for a sum, 1/N for a mean).
//
// Two ways with the same result. Usually one pass over the records, a workgroup per 49152-element chunk (k_combine_chunk,
// below: as soon as it has counted its records it learns from the chunks before where its output begins). Where the lists
// are so dense that a chunk's records outgrow a workgroup (ld_combine_shape), the index space is cut
// into 8192-element sub-tiles, one wave each, in two passes:
//   k_combine_count  marks the sub-tile's recorded positions in an LDS bitmap, counts
//                    them and leaves the bitmap in the workspace (1 KB per sub-tile);
//   k_combine_groups / k_combine_scan   scan the counts (inside groups of 1024
//                    sub-tiles, then the at most 1024 group sums);
//   k_combine_emit   fetches the bitmap (marking the positions a second time cost more
//                    than the n / 8 bytes written and read), ranks every position among the
//                    recorded ones and adds the values at their rank in a small LDS array, list
//                    after list (LDS operations of one wave complete in order, and
//                    inside one list the indices are distinct), then writes the array
//                    out as one contiguous run at the sub-tile's offset. A dense tile
//                    of the sub-tile would cost 32 KB of LDS per wave and leave one
//                    wave per SIMD; the ranked array takes 7.5 KB.
// The records of a sub-tile are found as in ld_merge_sparse: chunk table +
// interpolated 128-record windows, verified. HBM traffic of the two passes: the indices twice, the values
// once, the bitmaps out and in, the output once; of the one pass: records and output once.
#include <type_traits>

#include "ld_combine_shape.h"
#include "ld_sparse_common.h"

namespace {

constexpr int kSub = 8192;                 // elements per wave sub-tile
constexpr int kChunkSubs = static_cast<int>(kChunk / kSub);  // sub-tiles per chunk of the range table
static_assert(static_cast<int64_t>(kSub) * kChunkSubs == kChunk, "sub-tiles must tile a chunk");
constexpr int kWin = 2;                    // 64-record windows per list loaded ahead (three: 6 % slower, the third is mostly unused)
constexpr int kPre = 8;                    // lists whose windows are loaded before any is used
constexpr int kMargin = 24;                // records the window starts before the interpolated position
constexpr int kWords = kSub / 32;          // bitmap words per sub-tile: 256
constexpr int kSubsPerGroup = 1024;        // n <= 2^31-1 gives at most 1024 groups
constexpr int kCap = 1024;                 // distinct indices of a sub-tile accumulated per round of the emission

// Lane t: where list t's records of a chunk lie, and where those of a part of it are looked for (at or ahead of the first).
struct Ranges {
    int32_t begin, end, start;
};
__device__ __forceinline__ Ranges sub_tile_ranges(int32_t W, const int32_t* __restrict__ ctab, int32_t nchunk, int64_t sub,
                                                  int lane) {
    const int32_t chunk = static_cast<int32_t>(sub / kChunkSubs), part = static_cast<int32_t>(sub % kChunkSubs);
    Ranges r = {0, 0, 0};
    if (lane < W) {
        const int32_t* row = ctab + static_cast<int64_t>(lane) * (nchunk + 1) + chunk;
        r.begin = row[0];
        r.end = row[1];
    }
    r.start = r.begin + ((r.end - r.begin) * part) / kChunkSubs - kMargin;  // the guess for this sub-tile
    if (r.start < r.begin) r.start = r.begin;
    return r;
}

// Calls f(t, i, v) for every record (i, v) of list t with lo <= i < hi, list after list
// (t ascending); all lanes of the wave take part, one record per lane and call.
// VAL: where the first record at or beyond hi of a list lies goes into `at`, for a sweep that begins at hi.
template <bool VAL, class F>
__device__ __forceinline__ void sweep_records(const DiffTable& tb, int32_t W, Ranges& at, int32_t lo, int32_t hi, int lane,
                                              F&& f) {
    auto from = [&](int t, int32_t p, int32_t end) {  // records [p, end) up to the first at or beyond hi; where that one is
        for (; p < end; p += LD_WAVE) {
            const bool have = p + lane < end;
            const int32_t i = have ? tb.idx[t][p + lane] : INT_MAX;
            const float v = (VAL && have) ? tb.val[t][p + lane] : 0.0f;
            if (i >= lo && i < hi) f(t, i, v);
            const uint64_t past = __ballot(i >= hi);
            if (past) return p + static_cast<int32_t>(__builtin_ctzll(past));
        }
        return end;
    };
#pragma unroll 1
    for (int32_t t0 = 0; t0 < W; t0 += kPre) {
        int32_t s_[kPre], e_[kPre], b_[kPre], ri[kPre][kWin];
        float rv[kPre][kWin];
#pragma unroll
        for (int g = 0; g < kPre; ++g) {
            const int t = (t0 + g < W) ? t0 + g : 0;
            s_[g] = __builtin_amdgcn_readlane(at.start, t);
            b_[g] = __builtin_amdgcn_readlane(at.begin, t);
            e_[g] = (t0 + g < W) ? __builtin_amdgcn_readlane(at.end, t) : s_[g];  // past W: an empty window
#pragma unroll
            for (int u = 0; u < kWin; ++u) {
                const int32_t p = s_[g] + u * LD_WAVE + lane;
                const bool h = p < e_[g];
                ri[g][u] = h ? tb.idx[t][p] : INT_MAX;
                rv[g][u] = (VAL && h) ? tb.val[t][p] : 0.0f;
            }
        }
#pragma unroll
        for (int g = 0; g < kPre; ++g) {
            if (s_[g] < e_[g]) {
                const int t = t0 + g;
                int32_t next;
                const int32_t first = __builtin_amdgcn_readfirstlane(ri[g][0]);
                if (s_[g] == b_[g] || first <= lo) {  // the window begins before the sub-tile's records do
                    uint64_t past = 0;
#pragma unroll
                    for (int u = 0; u < kWin; ++u) {
                        if (!past) {
                            if (ri[g][u] >= lo && ri[g][u] < hi) f(t, ri[g][u], rv[g][u]);
                            past = __ballot(ri[g][u] >= hi);
                            next = s_[g] + u * LD_WAVE;
                        }
                    }
                    if (past) next += static_cast<int32_t>(__builtin_ctzll(past));
                    else next = from(t, s_[g] + kWin * LD_WAVE, e_[g]);
                } else {  // guess too late: find the first record of the sub-tile inside the chunk
                    next = from(t, lower_bound_idx(tb.idx[t], b_[g], s_[g], lo), e_[g]);
                }
                if (VAL && lane == t) at.begin = at.start = next < e_[g] ? next : e_[g];
            }
            __builtin_amdgcn_wave_barrier();  // keep list g's LDS traffic ahead of list g+1's
        }
    }
}

struct SubTile {
    int64_t sub;
    int32_t lo, hi;
    bool live;
};

__device__ __forceinline__ SubTile sub_tile(int64_t n) {
    // consecutive workgroups go to different XCDs: each XCD walks one contiguous eighth of the index space
    SubTile s;
    const int64_t per = (static_cast<int64_t>(gridDim.x) + 7) / 8;
    s.sub = static_cast<int64_t>(blockIdx.x % 8) * per + blockIdx.x / 8;
    s.live = s.sub * kSub < n;
    const int64_t lo64 = s.sub * kSub;
    s.lo = static_cast<int32_t>(s.live ? lo64 : 0);
    s.hi = static_cast<int32_t>(s.live ? ((n - lo64) < kSub ? n : lo64 + kSub) : 0);  // n <= INT_MAX
    return s;
}

__global__ __launch_bounds__(LD_WAVE) void k_combine_count(int64_t n, int32_t nchunk, DiffTable tb, int32_t W,
                                                           const int32_t* __restrict__ ctab,
                                                           uint32_t* __restrict__ counts,
                                                           uint32_t* __restrict__ bitmaps) {
    __shared__ uint32_t bm[kWords];
    const int lane = threadIdx.x;
    const SubTile s = sub_tile(n);
    if (!s.live) return;
#pragma unroll
    for (int j = 0; j < kWords / LD_WAVE; ++j) bm[j * LD_WAVE + lane] = 0;
    __syncthreads();  // one wave: orders the fill before the marks
    Ranges at = sub_tile_ranges(W, ctab, nchunk, s.sub, lane);
    sweep_records<false>(tb, W, at, s.lo, s.hi, lane, [&](int, int32_t i, float) {
        const uint32_t q = static_cast<uint32_t>(i - s.lo);
        atomicOr(&bm[q >> 5], 1u << (q & 31));
    });
    __syncthreads();
    uint32_t c = 0;
#pragma unroll
    for (int j = 0; j < kWords / LD_WAVE; ++j) {
        const uint32_t word = bm[j * LD_WAVE + lane];
        c += __popc(word);
        bitmaps[s.sub * kWords + j * LD_WAVE + lane] = word;  // k_combine_emit takes it from here
    }
    c = ld_wave_sum(c);
    if (lane == 0) counts[s.sub] = c;
}

// One workgroup per group of kSubsPerGroup sub-tiles: counts -> exclusive prefix inside the group
// (in place), group total -> gsum.
__global__ __launch_bounds__(256) void k_combine_groups(uint32_t* __restrict__ counts, int32_t nsub,
                                                        uint32_t* __restrict__ gsum) {
    __shared__ uint32_t sh[4];
    constexpr int per = kSubsPerGroup / 256;
    const int32_t first = blockIdx.x * kSubsPerGroup + threadIdx.x * per;
    uint32_t x[per], sum = 0;
#pragma unroll
    for (int i = 0; i < per; ++i) {
        x[i] = first + i < nsub ? counts[first + i] : 0u;
        sum += x[i];
    }
    uint32_t total;
    uint32_t before = ld_block_escan256(sum, sh, total);
#pragma unroll
    for (int i = 0; i < per; ++i) {
        if (first + i < nsub) counts[first + i] = before;
        before += x[i];
    }
    if (threadIdx.x == 0) gsum[blockIdx.x] = total;
}

// Exclusive scan of the group sums (at most 1024 groups: n <= 2^31-1); total -> *out_count.
__global__ __launch_bounds__(1024) void k_combine_scan(const uint32_t* __restrict__ gsum, uint32_t* __restrict__ goff,
                                                       int32_t ngrp, int64_t* __restrict__ out_count) {
    __shared__ uint32_t sh[1024 / LD_WAVE];
    const uint32_t x = static_cast<int32_t>(threadIdx.x) < ngrp ? gsum[threadIdx.x] : 0u;
    const uint32_t inc = ld_wave_iscan(x);
    const int w = threadIdx.x >> 6;
    if (ld_lane() == LD_WAVE - 1) sh[w] = inc;
    __syncthreads();
    uint32_t base = 0, total = 0;
#pragma unroll
    for (int i = 0; i < 1024 / LD_WAVE; ++i) {
        const uint32_t t = sh[i];
        if (i < w) base += t;
        total += t;
    }
    if (static_cast<int32_t>(threadIdx.x) < ngrp) goff[threadIdx.x] = base + inc - x;
    if (threadIdx.x == 0) *out_count = static_cast<int64_t>(total);
}

__global__ __launch_bounds__(LD_WAVE) void k_combine_emit(int64_t n, int32_t nchunk, DiffTable tb, int32_t W,
                                                          const int32_t* __restrict__ ctab,
                                                          const uint32_t* __restrict__ prefix, int32_t nsub,
                                                          const uint32_t* __restrict__ gsum,
                                                          const uint32_t* __restrict__ goff,
                                                          const uint32_t* __restrict__ bitmaps, float scale,
                                                          int32_t* __restrict__ out_idx,
                                                          float* __restrict__ out_val, int64_t out_cap) {
    __shared__ uint32_t bm[kWords];      // recorded positions of the sub-tile
    __shared__ uint16_t wpre[kWords];    // recorded positions before each bitmap word
    __shared__ float acc[kCap];          // sums, at the rank of their position among the recorded ones
    __shared__ uint16_t accq[kCap];      // ... and the positions themselves
    const int lane = threadIdx.x;
    const SubTile s = sub_tile(n);
    if (!s.live) return;
    // records written before this sub-tile: its group's offset + its prefix inside the group; its own
    // count is the distance to the next prefix (or to the group's total)
    const int32_t grp = static_cast<int32_t>(s.sub / kSubsPerGroup);
    const uint32_t before = prefix[s.sub];
    const bool last_of_group = (s.sub + 1) % kSubsPerGroup == 0 || s.sub + 1 >= nsub;
    const uint32_t mine = (last_of_group ? gsum[grp] : prefix[s.sub + 1]) - before;
    if (mine == 0) return;  // nothing recorded in this sub-tile
    const int64_t off = static_cast<int64_t>(goff[grp]) + before;
#pragma unroll
    for (int j = 0; j < kWords / LD_WAVE; ++j) bm[j * LD_WAVE + lane] = bitmaps[s.sub * kWords + j * LD_WAVE + lane];
    __syncthreads();  // one wave: orders the fill before what reads it
    {  // lane l owns bitmap words 4l .. 4l+3
        uint32_t c[kWords / LD_WAVE], sum = 0;
#pragma unroll
        for (int j = 0; j < kWords / LD_WAVE; ++j) {
            c[j] = __popc(bm[lane * (kWords / LD_WAVE) + j]);
            sum += c[j];
        }
        uint32_t run = ld_wave_iscan(sum) - sum;
#pragma unroll
        for (int j = 0; j < kWords / LD_WAVE; ++j) {
            wpre[lane * (kWords / LD_WAVE) + j] = static_cast<uint16_t>(run);
            run += c[j];
        }
    }
    Ranges at = sub_tile_ranges(W, ctab, nchunk, s.sub, lane);
    __syncthreads();  // wpre is read across lanes
    // Rounds of as many whole bitmap words as hold at most kCap distinct indices (one round unless the sub-tile is crowded): the
    // values are added, list after list, at the rank of their position; then the round is written out as one run. Lists
    // ascend, so a round begins in each of them where the last one ended: 64 lists of 0.3 % of 119 M elements, all of them in the
    // first tenth, 3395 us with all lists read in every round, 1047 so; densities that differ between layers as a log-normal of
    // sigma 1 does 1105 / 460; even (two rounds) 300 either way.
    uint32_t r0 = 0;
#pragma unroll 1
    for (int32_t word = 0; word < kWords;) {
        int32_t end = 0;  // the word that the round ends before: those from `word` to it hold at most kCap positions
#pragma unroll
        for (int j = 0; j < kWords / LD_WAVE; ++j) {
            const int32_t e = j * LD_WAVE + lane + 1;
            const uint32_t upto = e < kWords ? wpre[e] : mine;
            end += static_cast<int32_t>(__popcll(__ballot(upto <= r0 + static_cast<uint32_t>(kCap))));
        }
        const uint32_t next = end < kWords ? __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(wpre[end])) : mine;
        const uint32_t cnt = next - r0;
        if (cnt > 0) {
#pragma unroll
            for (int j = 0; j < kCap / LD_WAVE; ++j) acc[j * LD_WAVE + lane] = 0.0f;
            __syncthreads();
            sweep_records<true>(tb, W, at, s.lo + word * 32, end < kWords ? s.lo + end * 32 : s.hi, lane, [&](int, int32_t i, float v) {
                const uint32_t q = static_cast<uint32_t>(i - s.lo);
                const uint32_t rank = wpre[q >> 5] + __popc(bm[q >> 5] & ((1u << (q & 31)) - 1u)) - r0;
                if (rank < static_cast<uint32_t>(kCap)) {
                    acc[rank] = __fadd_rn(acc[rank], v);
                    accq[rank] = static_cast<uint16_t>(q);
                }
            });
            __syncthreads();
            for (uint32_t i = lane; i < cnt; i += LD_WAVE) {
                const int64_t pos = off + r0 + i;
                if (pos < out_cap) {
                    out_idx[pos] = s.lo + static_cast<int32_t>(accq[i]);
                    out_val[pos] = __fmul_rn(scale, acc[i]);
                }
            }
            __syncthreads();
        }
        r0 = next;
        word = end;
    }
}

// ------------------------------------------------------------------ one pass, a workgroup per chunk
//
// Everything in one reading of the records. A workgroup takes a chunk of the range table, so that it knows exactly which
// records are its own: no guesses, and a list's records lie in one piece of some 2 KB. It marks the recorded positions in a
// bitmap, publishes how many there are, adds the values list after list at their ranks, and by then the counts of the
// chunks before it have been published too: it adds them up back to the nearest chunk that has published everything before
// itself (a word per chunk: the count and what it counts, so that no fence is needed), and writes its records.
// The wait for a count is bounded: a workgroup that has asked often enough counts that chunk itself, so it ends whatever
// order the workgroups run in.
// Measured, two passes / one, us per call: 8 lists of 1 % of 1.56 G elements 635 / 541 (439 with the places of the output given
// instead of found), of 0.1 % of 1.4 G 288 / 170, of 1.7 % of 400 M 397 / 243, of 1 % of 50 M 44 / 35, of 1.7 % of 5 M 46 / 24.
// What it took there (first cases, 1080 at first): the ranges by lane reads instead of scalar loads list after list and 64
// chunks asked at a time instead of 256, 660; LDS accesses that nothing branches around; the published words 64 bytes apart (in
// a row 790, 8 bytes apart 670, 16: 640; they are written and asked from all XCDs at once) and asked for only when the values
// are added (earlier, they mostly say nothing yet), 595; four waves to a workgroup, so that every SIMD has one, 540; the lists'
// addresses by lane reads too, no wait between the lists' loads, the sums cleared while these are on their way and
// written out in fours, 531 -> 522 (scans over lanes by data-parallel primitives before that, 538 -> 531). What bounds it: a workgroup waits for
// the slowest of the thousand before it that are running. Of its 27 K clocks 9 K go to the loads, 5 K to the sums and 5 K to that wait, which takes up
// whatever the others are shortened by: with waits for the indices alone 530, with the counts of 64 chunks summed in a word, so that one question
// finds the offset, no less, with the results kept in registers until the next chunk's loads have come 610 (three
// workgroups per CU then, or spills).
// Crowded chunks (much of the lists in little of the index space): their rounds take pieces of the lists, not all of them again,
// and what goes beyond the records that a workgroup loads at once is streamed. 8 lists of 0.4 % of 400 M elements, all
// in the first fiftieth: with every round reading all of it 2906 us, now 284; 8 lists of 13 K of 5 M 1680 / 226. Two passes take 490 for the first.
constexpr int kChunkWords = static_cast<int>(kChunk / 32);  // bitmap words: 1536
constexpr int32_t kPolls = 4096;
constexpr int kApart = 16;                                  // words between the chunks' published ones
// What a chunk publishes: 0 nothing yet, 1 + its own count, or kSummed + the count up to its end (at most n <= 2^31 - 1).
constexpr uint32_t kSummed = 1u << 31;

__global__ __launch_bounds__(256) void k_combine_clear(uint32_t* __restrict__ state, int32_t nchunk) {
    const int32_t c = static_cast<int32_t>(blockIdx.x * 256 + threadIdx.x);
    if (c < nchunk) state[static_cast<int64_t>(c) * kApart] = 0;
}

// Distinct positions recorded in a chunk, counted by one wave; bits: kChunkWords words of LDS.
__device__ __forceinline__ uint32_t count_chunk(const DiffTable& tb, int32_t N, const int32_t* __restrict__ ctab,
                                                int32_t nchunk, int64_t n, int32_t chunk, uint32_t* bits, int lane) {
    const int64_t lo64 = static_cast<int64_t>(chunk) * kChunk;
    const uint32_t lo = static_cast<uint32_t>(lo64), len = static_cast<uint32_t>(n - lo64 < kChunk ? n - lo64 : kChunk);
    for (int j = lane; j < kChunkWords; j += LD_WAVE) bits[j] = 0;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    for (int32_t t = 0; t < N; ++t) {
        const int32_t* row = ctab + static_cast<int64_t>(t) * (nchunk + 1) + chunk;
        const uint32_t end = static_cast<uint32_t>(row[1]);  // unsigned: positions may pass INT_MAX by a window
        for (uint32_t p = static_cast<uint32_t>(row[0]) + lane; p < end; p += LD_WAVE) {
            const uint32_t q = static_cast<uint32_t>(tb.idx[t][p]) - lo;
            if (q < len) atomicOr(&bits[q >> 5], 1u << (q & 31));
        }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    uint32_t c = 0;
    for (int j = lane; j < kChunkWords; j += LD_WAVE) c += __popc(bits[j]);
    return ld_wave_sum(c);
}

// Four words at any 4-byte address (global accesses need no more).
typedef int32_t I32x4Any __attribute__((ext_vector_type(4), aligned(4)));
typedef float F32x4Any __attribute__((ext_vector_type(4), aligned(4)));

// HELD: at most kPre lists, their records stay in registers between the marks and the sums.
// kDeep: records per thread and list loaded ahead.
template <int THREADS, int kDeep, int CAP, bool HELD>
__global__ __launch_bounds__(THREADS) void k_combine_chunk(int64_t n, int32_t nchunk, DiffTable tb, int32_t N,
                                                           const int32_t* __restrict__ ctab, uint32_t* state,
                                                           float scale, int32_t* __restrict__ out_idx,
                                                           float* __restrict__ out_val, int64_t out_cap,
                                                           int64_t* __restrict__ out_count, int32_t polls) {
    static_assert(CAP >= kChunkWords && kChunk <= 65536, "a bitmap in acc, 16-bit positions");
    constexpr int kWaves = THREADS / LD_WAVE;
    constexpr int kOwners = THREADS < 256 ? THREADS : 256;  // threads that own bitmap words
    constexpr int kOwn = kChunkWords / kOwners;
    static_assert(kOwn * kOwners == kChunkWords, "");
    // Lanes without a record work on a word of their own behind each array: nothing branches around an LDS access.
    __shared__ __align__(16) uint32_t bm[kChunkWords + LD_WAVE];  // recorded positions of the chunk
    __shared__ uint16_t wpre[kChunkWords + LD_WAVE]; // recorded positions before each bitmap word
    __shared__ __align__(16) float acc[CAP + LD_WAVE];      // sums, at the rank of their position among the recorded ones
    __shared__ __align__(16) uint16_t accq[CAP + LD_WAVE];  // ... and the positions themselves
    __shared__ uint32_t sums[kWaves];
    __shared__ uint32_t offset;
    __shared__ uint32_t used[LD_WAVE];               // crowded chunks: the records that a round takes of every list
    const int tid = threadIdx.x, lane = tid & (LD_WAVE - 1), wave = __builtin_amdgcn_readfirstlane(tid / LD_WAVE);
    const int32_t chunk = blockIdx.x;
    const int64_t lo64 = static_cast<int64_t>(chunk) * kChunk;
    const uint32_t lo = static_cast<uint32_t>(lo64), len = static_cast<uint32_t>(n - lo64 < kChunk ? n - lo64 : kChunk);

    // Lane t: where list t's records of this chunk lie (in the rounds of a crowded chunk: those still to come), and the list itself.
    // The loops take them by lane reads: scalar loads from the table would be waited for list after list.
    int32_t first = 0, have = 0;
    uint32_t idx_lo = 0, idx_hi = 0, val_lo = 0, val_hi = 0;
    if (lane < N) {
        const int32_t* row = ctab + static_cast<int64_t>(lane) * (nchunk + 1) + chunk;
        const uint64_t i = reinterpret_cast<uint64_t>(tb.idx[lane]), v = reinterpret_cast<uint64_t>(tb.val[lane]);
        first = row[0];
        have = row[1] > first ? row[1] - first : 0;
        idx_lo = static_cast<uint32_t>(i), idx_hi = static_cast<uint32_t>(i >> 32);
        val_lo = static_cast<uint32_t>(v), val_hi = static_cast<uint32_t>(v >> 32);
    }
    asm volatile("" : "+v"(idx_lo), "+v"(idx_hi), "+v"(val_lo), "+v"(val_hi));  // waited for here, not behind the first records
    // Records of kPre lists, kDeep per thread and list; at: their positions in the chunk (spare: none).
    const uint32_t spare = static_cast<uint32_t>(kChunk) + lane * 32u;
    uint32_t at[kPre][kDeep];
    float rv[kPre][kDeep];
    auto fetch = [&](int32_t t0, auto (&x)[kPre][kDeep], uint32_t list_lo, uint32_t list_hi) {
        typedef std::remove_reference_t<decltype(x[0][0])> T;
#pragma unroll
        for (int g = 0; g < kPre; ++g) {
            const int t = t0 + g;  // kPre divides 64: past N the count is 0
            const uint32_t count = static_cast<uint32_t>(__builtin_amdgcn_readlane(have, t));
            const GlobalBytes base = lane_pointer(list_lo, list_hi, t) + static_cast<int64_t>(__builtin_amdgcn_readlane(first, t)) * 4;
#pragma unroll
            for (int u = 0; u < kDeep; ++u) {
                asm volatile("" : "=v"(x[g][u]));  // anything: a value set here would be a wait for the loads of the lists before
                if (static_cast<uint32_t>(u * THREADS + wave * LD_WAVE) < count) {  // uniform in the wave
                    uint32_t p = u * THREADS + tid;
                    p = p < count ? p : count - 1;
                    x[g][u] = *reinterpret_cast<const __attribute__((address_space(1))) T*>(base + p * 4u);
                }
            }
        }
    };
    auto drop = [&]() {  // ends the registers' lifetime where the records will not be asked for again
#pragma unroll
        for (int g = 0; g < kPre; ++g)
#pragma unroll
            for (int u = 0; u < kDeep; ++u) at[g][u] = 0, rv[g][u] = 0.0f;
    };
    auto load = [&](int32_t t0, bool values) {
        fetch(t0, at, idx_lo, idx_hi);
        if (values) fetch(t0, rv, val_lo, val_hi);
    };
    auto place = [&](int32_t t0) {
#pragma unroll
        for (int g = 0; g < kPre; ++g) {
            const uint32_t count = static_cast<uint32_t>(__builtin_amdgcn_readlane(have, t0 + g));
#pragma unroll
            for (int u = 0; u < kDeep; ++u) {
                const uint32_t q = at[g][u] - lo;
                at[g][u] = static_cast<uint32_t>(u * THREADS + tid) < count && q < len ? q : spare;
            }
        }
    };
    // Crowded chunks (a list has more records than load() takes): list after list, kBatch records per thread, the next ones
    // requested while the present ones are applied.
    const bool crowded = __ballot(have > kDeep * THREADS) != 0;  // uniform in the workgroup
    constexpr int kBatch = 5;
    struct Batch {
        int32_t i[kBatch];
        float v[kBatch];
    };
    // Records [b, b + kBatch * THREADS) of list t; past its end its last one again, of no list or an empty one anything. The loads
    // are unconditional: around conditional ones every wait would be one for the next batch too.
    auto take = [&](Batch& x, int32_t t, uint32_t b, bool values) {
        const uint32_t count = t < N ? static_cast<uint32_t>(__builtin_amdgcn_readlane(have, t)) : 0u;
        const int32_t* ip = count ? tb.idx[t] + __builtin_amdgcn_readlane(first, t) : ctab;
        const float* vp = count ? tb.val[t] + __builtin_amdgcn_readlane(first, t) : reinterpret_cast<const float*>(ctab);
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
            uint32_t p = b + u * THREADS + tid;
            p = p < count ? p : (count ? count - 1 : 0u);
            x.i[u] = ip[p];
            if (values) x.v[u] = vp[p];
        }
    };
    // x.i: position in the chunk (spare: none) instead of the index
    auto place_batch = [&](Batch& x, uint32_t b, uint32_t count) {
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
            const uint32_t q = static_cast<uint32_t>(x.i[u]) - lo;
            x.i[u] = static_cast<int32_t>(b + u * THREADS + tid < count && q < len ? q : spare);
        }
    };
    auto mark = [&](uint32_t q) { atomicOr(&bm[q >> 5], 1u << (q & 31)); };
    load(0, HELD);
    for (int j = tid; j < kChunkWords / 4; j += THREADS) reinterpret_cast<ld_u32x4*>(bm)[j] = ld_u32x4{0u, 0u, 0u, 0u};
    static_assert(CAP % 4 == 0, "");
    for (int j = tid; j < CAP / 4; j += THREADS) reinterpret_cast<ld_f32x4*>(acc)[j] = ld_f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    // __syncthreads, but for LDS alone: the records stay on their way
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
#pragma unroll 1
    for (int32_t t0 = 0; t0 < (HELD ? 1 : N); t0 += kPre) {
        if (!HELD && t0 > 0) load(t0, false);
        place(t0);
#pragma unroll
        for (int g = 0; g < kPre; ++g)
#pragma unroll
            for (int u = 0; u < kDeep; ++u) mark(at[g][u]);
    }
    if (crowded) {
        auto next = [&](int32_t& t, uint32_t& b) {  // past the batch's end: the next list with more than load() took
            b += kBatch * THREADS;
            while (t < N && b >= static_cast<uint32_t>(__builtin_amdgcn_readlane(have, t))) {
                ++t;
                b = kDeep * THREADS;
            }
        };
        int32_t t = __builtin_ctzll(__ballot(have > kDeep * THREADS));
        uint32_t b = kDeep * THREADS;
        Batch now, later;
        take(now, t, b, false);
#pragma unroll 1
        while (t < N) {
            const uint32_t count = static_cast<uint32_t>(__builtin_amdgcn_readlane(have, t)), b0 = b;
            next(t, b);
            take(later, t, b, false);
            place_batch(now, b0, count);
#pragma unroll
            for (int u = 0; u < kBatch; ++u) mark(static_cast<uint32_t>(now.i[u]));
            now = later;
        }
        drop();
    }
    __syncthreads();

    uint32_t before = 0;  // of the thread's words
    uint32_t word[kOwn], sum = 0;
    if (tid < kOwners) {
#pragma unroll
        for (int j = 0; j < kOwn; ++j) {
            word[j] = __popc(bm[tid * kOwn + j]);
            sum += word[j];
        }
    }
    before = ld_wave_iscan(sum);
    if (lane == LD_WAVE - 1) sums[wave] = before;
    before -= sum;
    __syncthreads();
    uint32_t total = 0;
#pragma unroll
    for (int i = 0; i < kWaves; ++i) {
        if (i < wave) before += sums[i];
        total += sums[i];
    }
    if (tid < kOwners) {
#pragma unroll
        for (int j = 0; j < kOwn; ++j) {
            wpre[tid * kOwn + j] = static_cast<uint16_t>(before);  // below kChunk
            before += word[j];
        }
    }
    auto publish = [&](uint32_t x) { __hip_atomic_store(state + static_cast<int64_t>(chunk) * kApart, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); };
    if (tid == 0) publish(chunk > 0 ? total + 1 : kSummed + total);

    // Records before this chunk's; the first wave finds them, the others wait at the next barrier. bits: kChunkWords free words.
    auto ask = [&](int32_t c) {
        return c < 0 ? kSummed : __hip_atomic_load(state + static_cast<int64_t>(c) * kApart, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };
    auto find_offset = [&](uint32_t* bits) {
        if (wave != 0) return;
        uint32_t off = 0;
        bool found = chunk == 0;
        int32_t asked = 0;
#pragma unroll 1
        for (int32_t pos = chunk - 1; !found; pos -= LD_WAVE) {
            uint32_t told = ask(pos - lane);
            int last;  // lanes up to it count
            while (true) {
                const uint64_t summed = __ballot(told >= kSummed), none = __ballot(told == 0);
                last = summed ? __builtin_ctzll(summed) : LD_WAVE - 1;
                found = summed != 0;
                const uint64_t missing = none & (~0ull >> (LD_WAVE - 1 - last));
                if (!missing) break;
                if (asked < polls) {
                    ++asked;
                    __builtin_amdgcn_s_sleep(1);
                    if (told == 0) told = ask(pos - lane);
                } else {  // asked often enough: count the nearest one here
                    const int l = __builtin_ctzll(missing);
                    const uint32_t c = count_chunk(tb, N, ctab, nchunk, n, pos - l, bits, lane);
                    if (lane == l) told = c + 1;
                    else if (told == 0) told = ask(pos - lane);  // it may have been told meanwhile
                }
            }
            const uint32_t own = told >= kSummed ? told - kSummed : told - 1;
            off += ld_wave_sum(lane <= last ? own : 0u);
        }
        if (lane == 0) {
            publish(kSummed + (off + total));
            offset = off;
            if (chunk == nchunk - 1) *out_count = static_cast<int64_t>(off) + total;
        }
    };
    const bool once = total <= static_cast<uint32_t>(CAP);  // one round, unless the chunk is crowded
    if (!once) find_offset(reinterpret_cast<uint32_t*>(acc));
    __syncthreads();

    // Rounds of CAP distinct positions: the values are added, list after list, at the rank of their position; then
    // the round is written out as one run. Lists ascend, so a round takes a piece of every list: in a crowded chunk it begins
    // where the last round's ended, which the first record past the round tells.
#pragma unroll 1
    for (uint32_t r0 = 0; r0 == 0 || r0 < total; r0 += CAP) {
        const uint32_t cnt = total - r0 < static_cast<uint32_t>(CAP) ? total - r0 : static_cast<uint32_t>(CAP);
        if (!once)  // the only round's are cleared already
            for (uint32_t j = tid; j < cnt; j += THREADS) acc[j] = 0.0f;
        // at least CAP: of another round
        auto rank = [&](uint32_t q) {
            const uint32_t r = wpre[q >> 5] + __popc(bm[q >> 5] & ((1u << (q & 31)) - 1u)) - r0;
            return r < cnt && q < static_cast<uint32_t>(kChunk) ? r : static_cast<uint32_t>(CAP) + lane;
        };
        uint64_t over = 0;  // lists of a crowded chunk of which this round takes all that load() would and more
        if (crowded) {
            uint32_t end = static_cast<uint32_t>(kChunk);
            if (have > kDeep * THREADS) end = static_cast<uint32_t>(tb.idx[lane][first + kDeep * THREADS - 1]) - lo;
            over = __ballot(end < len && rank(end) < static_cast<uint32_t>(CAP));
            if (tid < LD_WAVE) used[tid] = static_cast<uint32_t>(have);
        }
        // the first of the wave's records past the round; p: a lane's, counted from the list's first
        auto past_round = [&](int32_t t, bool past, uint32_t p) {
            const uint64_t lanes = __ballot(past);
            if (lanes && lane == __builtin_ctzll(lanes)) atomicMin(&used[t], p);
            return lanes != 0;
        };
        __syncthreads();
#pragma unroll 1
        for (int32_t t0 = 0; t0 < (HELD ? 1 : N); t0 += kPre) {
            if (!(over >> t0 & ((1u << kPre) - 1u))) {
                if (!HELD || r0 > 0 || crowded) {
                    load(t0, true);
                    place(t0);
                }
                uint32_t to[kPre][kDeep];
#pragma unroll
                for (int g = 0; g < kPre; ++g)
#pragma unroll
                    for (int u = 0; u < kDeep; ++u) {
                        to[g][u] = rank(at[g][u]);
                        accq[to[g][u]] = static_cast<uint16_t>(at[g][u]);
                    }
#pragma unroll
                for (int g = 0; g < kPre; ++g) {
                    if (t0 + g < N) {  // uniform
                        // the positions of one list are distinct: all are read before any is written
                        float cur[kDeep];
#pragma unroll
                        for (int u = 0; u < kDeep; ++u) cur[u] = acc[to[g][u]];
#pragma unroll
                        for (int u = 0; u < kDeep; ++u) acc[to[g][u]] = __fadd_rn(cur[u], rv[g][u]);
                        __syncthreads();  // list after list
                    }
                }
                if (crowded) {
#pragma unroll
                    for (int g = 0; g < kPre; ++g)
#pragma unroll
                        for (int u = 0; u < kDeep; ++u)
                            past_round(t0 + g, to[g][u] >= static_cast<uint32_t>(CAP) && at[g][u] < static_cast<uint32_t>(kChunk), u * THREADS + tid);
                    drop();
                }
            } else {
                Batch now, later;
                take(now, t0, 0, true);
#pragma unroll 1
                for (int32_t t = t0; t < t0 + kPre && t < N; ++t) {
                    const uint32_t count = static_cast<uint32_t>(__builtin_amdgcn_readlane(have, t));
                    take(later, t + 1, 0, true);
                    bool past = false;  // the wave has seen a record past the round
#pragma unroll 1
                    for (uint32_t b = 0; b < count && !past; b += kBatch * THREADS) {
                        if (b > 0) take(now, t, b, true);
                        place_batch(now, b, count);
                        uint32_t to[kBatch];
                        float cur[kBatch];
#pragma unroll
                        for (int u = 0; u < kBatch; ++u) {
                            to[u] = rank(static_cast<uint32_t>(now.i[u]));
                            cur[u] = acc[to[u]];
                        }
#pragma unroll
                        for (int u = 0; u < kBatch; ++u) {
                            acc[to[u]] = __fadd_rn(cur[u], now.v[u]);
                            accq[to[u]] = static_cast<uint16_t>(now.i[u]);
                        }
#pragma unroll
                        for (int u = 0; u < kBatch; ++u)
                            past |= past_round(t, to[u] >= static_cast<uint32_t>(CAP) && now.i[u] < static_cast<int32_t>(kChunk), b + u * THREADS + tid);
                    }
                    if (count) __syncthreads();  // list after list
                    now = later;
                }
                drop();
            }
        }
        if (crowded) {
            __syncthreads();
            const int32_t took = static_cast<int32_t>(used[lane]);
            first += took;
            have -= took;
        }
        if (once) {
            find_offset(bm);
            __syncthreads();
        }
        const int64_t off = static_cast<int64_t>(offset) + r0;
        const uint32_t room = off >= out_cap ? 0u : out_cap - off < cnt ? static_cast<uint32_t>(out_cap - off) : cnt;
#pragma unroll 2
        for (uint32_t j = tid * 4; j < room; j += THREADS * 4) {  // four neighbours a thread, wherever the run begins
            const ld_f32x4 x = *reinterpret_cast<const ld_f32x4*>(acc + j);
            const ld_u32x2 q = *reinterpret_cast<const ld_u32x2*>(accq + j);
            const int32_t i[4] = {static_cast<int32_t>(lo + (q.x & 0xFFFFu)), static_cast<int32_t>(lo + (q.x >> 16)),
                                  static_cast<int32_t>(lo + (q.y & 0xFFFFu)), static_cast<int32_t>(lo + (q.y >> 16))};
            const float v[4] = {__fmul_rn(scale, x.x), __fmul_rn(scale, x.y), __fmul_rn(scale, x.z), __fmul_rn(scale, x.w)};
            if (j + 4 <= room) {
                *reinterpret_cast<I32x4Any*>(out_idx + off + j) = I32x4Any{i[0], i[1], i[2], i[3]};
                *reinterpret_cast<F32x4Any*>(out_val + off + j) = F32x4Any{v[0], v[1], v[2], v[3]};
            } else {
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    if (j + c < room) {
                        out_idx[off + j + c] = i[c];
                        out_val[off + j + c] = v[c];
                    }
                }
            }
        }
        if (once) return;
        __syncthreads();
    }
}

}  // namespace

namespace {
struct CombineLayout { size_t ctab, counts, gsum, goff, bitmaps, total; };
CombineLayout combine_layout(int64_t n, int32_t N) {
    CombineLayout L;
    size_t o = 0;
    auto take = [&](size_t bytes) { const size_t at = o; o += ld_round_up(bytes, 256); return at; };
    const size_t nsub = static_cast<size_t>((n + kSub - 1) / kSub);
    const size_t ngrp = (nsub + kSubsPerGroup - 1) / kSubsPerGroup;
    L.ctab = take(static_cast<size_t>(N) * (static_cast<size_t>(chunks(n)) + 1) * 4);
    L.counts = take(nsub * 4);
    L.gsum = take(ngrp * 4);
    L.goff = take(ngrp * 4);
    L.bitmaps = take(nsub * kWords * 4);  // recorded positions of every sub-tile: n / 8 bytes
    L.total = o;
    return L;
}
}  // namespace

extern "C" size_t ld_combine_sparse_workspace(int64_t n, int32_t N) {
    if (n <= 0 || N <= 0 || N > LD_MAX_WORKERS) return 256;
    return combine_layout(n, N).total;
}

extern "C" ld_status ld_combine_sparse(const int32_t* const* idx, const float* const* val, const int64_t* K,
                                       int32_t N, int64_t n, float scale, int32_t* out_idx, float* out_val,
                                       int64_t out_cap, int64_t* out_count, void* workspace,
                                       size_t workspace_bytes, ld_stream stream) {
    return ld_combine_sparse_strategy(idx, val, K, N, n, scale, out_idx, out_val, out_cap, out_count, workspace,
                                      workspace_bytes, stream, LD_COMBINE_AUTO);
}

extern "C" ld_status ld_combine_sparse_strategy(const int32_t* const* idx, const float* const* val, const int64_t* K,
                                                int32_t N, int64_t n, float scale, int32_t* out_idx, float* out_val,
                                                int64_t out_cap, int64_t* out_count, void* workspace,
                                                size_t workspace_bytes, ld_stream stream, int32_t strategy) {
    if (strategy < LD_COMBINE_AUTO || strategy > LD_COMBINE_ONE_PASS_ALONE) return LD_ERR_RANGE;
    if (n < 0 || n > INT32_MAX || N < 0 || N > LD_MAX_WORKERS || out_cap < 0) return LD_ERR_RANGE;
    if (!out_count) return LD_ERR_NULL;
    if (!ld_aligned(out_count, 8)) return LD_ERR_ALIGN;
    if (N > 0 && (!idx || !val || !K)) return LD_ERR_NULL;
    int64_t total = 0, most = 0;
    for (int32_t t = 0; t < N; ++t) {
        if (K[t] < 0 || K[t] > n) return LD_ERR_RANGE;
        if (K[t] > most) most = K[t];
        if (K[t] > 0 && (!idx[t] || !val[t])) return LD_ERR_NULL;
        if (!ld_aligned(idx[t], 4) || !ld_aligned(val[t], 4)) return LD_ERR_ALIGN;
        total += K[t];
    }
    if (out_cap > 0 && (!out_idx || !out_val)) return LD_ERR_NULL;
    if (!ld_aligned(out_idx, 4) || !ld_aligned(out_val, 4)) return LD_ERR_ALIGN;
    hipStream_t s = static_cast<hipStream_t>(stream);
    ld_begin_call();
    const int32_t nsub = static_cast<int32_t>((n + kSub - 1) / kSub);
    const int32_t ngrp = (nsub + kSubsPerGroup - 1) / kSubsPerGroup;
    if (n == 0 || N == 0 || total == 0) {  // an empty result: only the count is written
        static_assert(sizeof(uint32_t) == 4, "");
        k_combine_scan<<<dim3(1), dim3(1024), 0, s>>>(nullptr, nullptr, 0, out_count);
        return ld_launch_status();
    }
    const CombineLayout L = combine_layout(n, N);
    if (!workspace || !ld_aligned(workspace, 256) || workspace_bytes < L.total) return LD_ERR_WORKSPACE;
    char* ws = static_cast<char*>(workspace);
    int32_t* ctab = reinterpret_cast<int32_t*>(ws + L.ctab);
    uint32_t* counts = reinterpret_cast<uint32_t*>(ws + L.counts);
    uint32_t* gsum = reinterpret_cast<uint32_t*>(ws + L.gsum);
    uint32_t* goff = reinterpret_cast<uint32_t*>(ws + L.goff);
    uint32_t* bitmaps = reinterpret_cast<uint32_t*>(ws + L.bitmaps);
    static_assert(LD_MAX_WORKERS <= kGroupMax, "one launch must hold every list");
    DiffTable tb = {};
    for (int32_t t = 0; t < kGroupMax; ++t) {
        const bool live = t < N;
        tb.idx[t] = live ? idx[t] : nullptr;
        tb.val[t] = live ? val[t] : nullptr;
        tb.K[t] = live ? static_cast<int32_t>(K[t]) : 0;
    }
    const int32_t nchunk = chunks(n);
    const dim3 grid(static_cast<uint32_t>((nsub + 7) / 8 * 8)), wave(LD_WAVE);
    launch_chunks(tb, N, n, nchunk, ctab, s);
    if (ld_launch_status() != LD_OK) return LD_ERR_HIP;
    const LdCombineShape shape = ld_combine_shape(n, N, most, total, strategy);
    if (shape != kCombineTwoPasses) {
        static_assert(kCombineChunk == kChunk && kCombineHeld == kPre, "as the kernels have them");
        uint32_t* state = bitmaps;  // 64 bytes per chunk, where the two passes keep a bit per element
        const int32_t polls = strategy == LD_COMBINE_ONE_PASS_ALONE ? 0 : kPolls;
        k_combine_clear<<<dim3((nchunk + 255) / 256), dim3(256), 0, s>>>(state, nchunk);
        if (ld_launch_status() != LD_OK) return LD_ERR_HIP;
        auto launch = [&](auto kernel, uint32_t threads) {
            kernel<<<dim3(nchunk), dim3(threads), 0, s>>>(n, nchunk, tb, N, ctab, state, scale, out_idx, out_val, out_cap,
                                                        out_count, polls);
        };
        const bool held = N <= kPre;
        if (shape == kCombineNarrow) held ? launch(k_combine_chunk<128, 2, 2048, true>, 128) : launch(k_combine_chunk<128, 2, 2048, false>, 128);
        else if (shape == kCombineFew) launch(k_combine_chunk<192, 3, 2304, true>, 192);
        else if (shape == kCombineMiddle) held ? launch(k_combine_chunk<256, 3, 4608, true>, 256) : launch(k_combine_chunk<256, 3, 4608, false>, 256);
        else if (shape == kCombineLong) launch(k_combine_chunk<256, 4, 4608, true>, 256);
        else held ? launch(k_combine_chunk<512, 3, 9152, true>, 512) : launch(k_combine_chunk<512, 3, 9152, false>, 512);
        return ld_launch_status();
    }
    k_combine_count<<<grid, wave, 0, s>>>(n, nchunk, tb, N, ctab, counts, bitmaps);
    if (ld_launch_status() != LD_OK) return LD_ERR_HIP;
    k_combine_groups<<<dim3(ngrp), dim3(256), 0, s>>>(counts, nsub, gsum);
    if (ld_launch_status() != LD_OK) return LD_ERR_HIP;
    k_combine_scan<<<dim3(1), dim3(1024), 0, s>>>(gsum, goff, ngrp, out_count);
    if (ld_launch_status() != LD_OK) return LD_ERR_HIP;
    k_combine_emit<<<grid, wave, 0, s>>>(n, nchunk, tb, N, ctab, counts, nsub, gsum, goff, bitmaps, scale, out_idx,
                                         out_val,
                                         out_cap);
    return ld_launch_status();
}
