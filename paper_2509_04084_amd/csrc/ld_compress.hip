// ld_compress_topk: per-segment exact top-k sparsification with error feedback.
//
// Comp of Algorithm 1 (Sec. IV-B) at ratio rho (Sec. II-C, Sec. VII-A): the
// compressed gradient that is reused as the differential checkpoint.  The
// selection rule (|r+g| descending on the bit pattern, ties to the lower index,
// records ascending, selected residuals zeroed) is stated in lowdiff.h.
//
// Design: ONE streaming pass over gradient and residual, then three small passes
// over a candidate set of about 1.7 * k elements.
//
//   k_prep    one workgroup per segment. The segment table travels in its kernel arguments: as it is up
//             to 230 segments; beyond,
//             packed as a dictionary of the distinct (length, k) pairs plus one byte per
//             segment (a model has few distinct tensor shapes); every workgroup rebuilds the
//             prefix sums it needs from it. Tables that do not pack (more than 160 distinct
//             pairs or 2048 segments) go through k_upload launches first. From a 16K-element sample of |r+g| it
//             estimates three keys: a candidate threshold tau (the sample key at a
//             rank high enough that, with overwhelming probability, at least k
//             elements of the segment lie at or above it), the likeliest threshold
//             T_est (the sample key at the rank that corresponds to k), and the top
//             of the fine bins that the later passes lay over the keys above tau.
//             When the whole segment fits in the sample the three are exact.
//   k_main    the only full pass, 12 bytes per element. One wave per 4096-element
//             tile, the tiles dealt to the XCDs in short runs in address
//             order. Elements with key >= tau
//             go, in index order, into the tile's candidate slot. The residual is
//             written as if T_est were the threshold: +0 where key >= T_est, r + g
//             elsewhere - so that the scattered repair writes of the last pass touch
//             only the elements between T_est and the true threshold (a few percent
//             of k) instead of all k selected positions.
//   k_hist    histogram of the candidates over 2048 fine bins.
//   k_gather  finds the bin b holding the k-th largest key;
//             per tile: #candidates in bins above b; the (few) keys inside bin b are
//             gathered per segment.
//   k_emit    each workgroup selects the exact threshold T and tie count among the
//             gathered keys for itself and completes its tiles' counts with them
//             (tables with segments of more than 65 or 100 M elements: k_select before it);
//             ordered emission of (idx, val); repairs the residual where the
//             T_est guess and the true selection differ.
//
// The estimates can never make the result wrong, only slower:
//   * a tile with more candidates than its slot holds is marked, its residual is
//     stored unzeroed, and the later passes re-read that tile from the residual;
//   * a segment with fewer than k candidates, or with more keys in bin b than the
//     gather list holds, gets its residual restored from the slots and is handed to
//     k_full: a plain three-level radix select over the whole segment -
//     unless the overfull bin holds one value only (massive ties: zeros of a frozen
//     layer, values on a grid): then that value is the threshold and its ties are
//     taken in index order without leaving the candidate path.
//   * a segment whose sample holds the candidate threshold's own key hundreds of times (a
//     frozen layer's zeros, a constant) is "tied": its candidates are the keys above that
//     key, nothing is pre-zeroed, and if they are fewer than k the repeated key is the
//     threshold; its ties are counted per tile and taken in index order from the residual.
// The slot size (256 .. 2048 candidates per tile) and the lanes per tile of the candidate
// passes (16, 32 or 64) are chosen per call from the densities seg_k / n_s, so that calls
// at 5 or 10 % keep the same structure (the paper varies rho from 0.001 to 0.1, Exp. 10).
// Per-segment steps run as kernels of their own (a kernel boundary is the only
// device-wide hand-over the normal path needs). The full-segment path is ONE launch (k_full)
// that returns at once when no segment was handed to it; otherwise its five phases hand over
// through a barrier across the grid, which is kept small enough to be resident as a whole.
#include <math.h>

#include <atomic>

#include "ld_common.h"

namespace {

constexpr int kThreads = 256;
constexpr int kWaves = kThreads / LD_WAVE;
constexpr int kTile = 4096;                       // elements per k_main workgroup
#ifndef LD_SLOT_MIN
#define LD_SLOT_MIN 128
#endif
constexpr int kSlotMin = LD_SLOT_MIN;             // candidate slots per tile: 128 serve densities up to ~1 % (a denser
constexpr int kSlotMax = 2048;                    // layout of the slots made the candidate passes slower); denser calls get more (multiples of 64)
// Tiles per group, the unit of the passes over the candidates (a workgroup each): 64, or 16 for tables of
// fewer than kSmallGroups groups of 64, whose passes would leave most of the chip idle and whose small
// segments would cost k_main 64 tile slots each. Measured, us per call with 64 / 16: flat 1 M 59.9 /
// 50.6, ResNet-50 128 / 109, 5 M at 2 % 85 / 65, 64 M 193 / 186; the same at 128 M elements (500 groups of
// 64); GPT-2 XL 3268 / 3322.
constexpr int kTilesPerGroup = 64, kTilesPerSmallGroup = 16;
constexpr int64_t kSmallGroups = 512;
constexpr int kBins = 2048;
constexpr int kTopBin = kBins - 1;
constexpr int kShift1 = 20, kShift2 = 9;          // radix digits: [30:20] [19:9] [8:0]
constexpr int kSample = 16384;                        // sampled elements per segment
constexpr int kSampleRuns = kSample / LD_WAVE;        // as 256 runs of 64 consecutive elements
constexpr float kSampleZ = 6.5f;                  // safety margin of the rank estimate, in sigmas
constexpr int kGatherBase = 4096;                 // gather list of a segment: kGatherBase + n_s / kGatherPer keys
constexpr int kGatherPer = 4096;
constexpr int32_t kPrepWide = 256;                // segments up to which k_prep runs 1024 threads each
constexpr int kSegPerLaunch = 448;
constexpr int kFullGrid = 1024;                   // most workgroups of the (normally idle) k_full kernel
constexpr uint32_t kModeCand = 0, kModeFull = 1, kModeTies = 2;
constexpr uint32_t kTieSuspect = 512;             // sample keys equal to the candidate threshold (of 16384) that make a segment "tied"

constexpr uint32_t kOverflow = 0xFFFFFFFFu;       // tile count: slot too small, read the residual
constexpr int kSyncCount = 0, kSyncArrived = 1, kSyncGaveUp = 2, kSyncWords = 3;
constexpr int kDictMax = 160;                     // distinct (length, k) pairs of a packed segment table
constexpr int kDictSegs = 2048;                   // segments of a packed segment table

struct SegDesc {        // one per segment plus a sentinel
    int64_t off;        // first element
    int64_t out0;       // first output record
    int32_t k;          // records to keep; in the sentinel: the call's tiles per group
    int32_t group0;     // first group
};

struct GroupDesc {      // 64 bytes: all a workgroup needs to know about its group, in one fetch
    int64_t base;       // first element of the group's first tile (multiple of 4; may precede the segment)
    int64_t lo, hi;     // the segment's element range
    int64_t out0;       // the segment's first output record
    int32_t seg;
    int32_t k;          // records the segment keeps
    int32_t group0;     // the segment's first group
    int32_t ngroup;     // groups in the segment
    uint32_t tau;       // candidate threshold (see SegState)
    uint32_t sh;        // fine-bin shift
    uint32_t test;      // guessed threshold
    uint32_t tied;      // 1: the key tau - 1 is massively repeated (see SegState::tied)
};

struct SegState {       // 64 bytes
    uint32_t tau;       // candidate threshold (key); 0: every element, 0xFFFFFFFF: none
    uint32_t sh;        // fine bin of a candidate: min(kTopBin, (key - tau) >> sh)
    uint32_t test;      // guessed threshold T_est >= tau: k_main stores +0 where key >= T_est
    uint32_t prefix;    // k_gather: threshold bin, kModeTies: the threshold (k_full: radix prefix)
    uint32_t krem;      // rank left inside prefix, kModeTies: the number of ties to keep
    uint32_t mode;      // kModeCand | kModeFull | kModeTies
    uint32_t gcount;    // keys gathered from the threshold bin
    uint32_t fdone[4];  // tickets of the full-segment path: level 1, 2, 3, count
    uint32_t kmin, kmax;  // bounds of the threshold-bin keys that found no room in the gather list
    // A tied segment: the sample found one key repeated so often (a frozen layer's zeros, a constant)
    // that taking it as candidate threshold would make nearly every element a candidate. The
    // candidates are then the keys ABOVE it (tau = that key + 1) and nothing is pre-zeroed. If the
    // candidates turn out fewer than k, the threshold can only be that key or a smaller one:
    // k_gather counts the key per tile in the residual, k_emit checks that with those ties k is
    // reached (else: the full path), and k_emit takes the ties in index order (kModeTies).
    uint32_t tied;
    uint32_t late;      // 1: handed to the full path by k_emit, whose workgroups still read `mode`
    uint32_t pad;
};

struct Ctx {
    SegDesc* desc;          // [n_seg + 1]
    GroupDesc* gdesc;       // [n_group]
    SegState* state;        // [n_seg]
    uint32_t* hist;         // [n_seg][kBins]
    uint32_t* cnt;          // [n_group * tiles] candidates stored per tile, or kOverflow
    float* cval;            // [n_group * tiles][slot]
    uint16_t* cidx;         // [n_group * tiles][slot] element offset inside the tile
    uint32_t* tile_gt;      // [n_group * tiles] keys above the threshold bin
    uint32_t* tile_eq;      // [n_group * tiles] keys in it (kModeTies: equal to the threshold)
    uint32_t* group_gt;     // [n_group] sums over the group (full path: records emitted before the group)
    uint32_t* group_eq;     // [n_group]                       (ties before the group)
    uint32_t* gkey;         // per segment gather_cap entries from gather_first
    int32_t* gtile;         // per segment gather_cap entries from gather_first
    int32_t* fail_groups;   // [n_group] groups of segments in kModeFull
    uint32_t* fail_count;   // [kSyncWords]: groups listed; arrivals at k_full's grid barrier; its give-up flag
    int32_t n_seg;
    int32_t n_group;
    int32_t slot;           // candidates a tile can store (kSlotMin .. kSlotMax, multiple of 64)
    int32_t tiles;          // tiles per group: kTilesPerGroup or kTilesPerSmallGroup
};

struct UploadBatch {
    int32_t off[kSegPerLaunch + 1];
    int32_t k[kSegPerLaunch];
    int64_t out0;     // records before the first segment of the batch
    int32_t group0;   // groups before it
    int32_t first;    // index of the batch's first segment
    int32_t count;
    int32_t n_seg;
};

// The segment table as k_prep takes it in its arguments when it packs: n_seg = 0 says that it
// did not and that k_upload has written the descriptors.
struct PackedTable {
    uint32_t len[kDictMax];
    uint32_t k[kDictMax];
    uint32_t off0[kDictSegs / LD_WAVE];    // per bucket of 64 segments: elements,
    uint32_t out0[kDictSegs / LD_WAVE];    //   records
    uint32_t group0[kDictSegs / LD_WAVE];  //   and groups before it
    uint8_t code[kDictSegs];
    int32_t n_seg;
};
static_assert(sizeof(PackedTable) + sizeof(Ctx) + 24 <= 4096, "k_prep's arguments must fit a kernel's 4 KB");

// The segment table of up to kDirectSegs segments, as it is: a workgroup fetches its entry in one read
// instead of two dependent ones, three scans and a barrier: k_prep 15.7 -> 13.9 us for one segment, 16.5 ->
// 15.0 for ResNet-50's 161.
constexpr int kDirectSegs = 230;
struct DirectTable {
    struct Entry { uint32_t off, k, out0, group0; } seg[kDirectSegs + 1];  // entry n_seg: the totals
    int32_t n_seg;
};
static_assert(sizeof(DirectTable) + sizeof(Ctx) + 24 <= 4096, "k_prep's arguments must fit a kernel's 4 KB");

__host__ __device__ inline int64_t align_down4(int64_t x) { return x & ~static_cast<int64_t>(3); }

// Gather list of segment s = [lo, hi): first entry and capacity. Derived from the offsets alone,
// so that no table is needed: capacity >= kGatherBase + (hi - lo) / kGatherPer - 1.
__host__ __device__ inline int64_t gather_first(int32_t s, int64_t lo) {
    return static_cast<int64_t>(kGatherBase) * s + lo / kGatherPer;
}
__host__ __device__ inline uint32_t gather_cap(int64_t lo, int64_t hi) {
    return static_cast<uint32_t>(kGatherBase + hi / kGatherPer - lo / kGatherPer);
}

__host__ __device__ inline int32_t groups_of(int64_t off, int64_t end, int32_t tiles) {
    if (end <= off) return 0;
    const int64_t len = static_cast<int64_t>(tiles) * kTile;
    return static_cast<int32_t>((end - align_down4(off) + len - 1) / len);
}

// ------------------------------------------------------------ block helpers

// Exclusive scan over NT threads (NT = 256 or 1024); `sh` holds NT/64 words.
template <int NT>
__device__ __forceinline__ uint32_t block_escan(uint32_t x, uint32_t* sh, uint32_t& total) {
    constexpr int NW = NT / LD_WAVE;
    const uint32_t inc = ld_wave_iscan(x);
    const int w = threadIdx.x >> 6;
    if (ld_lane() == LD_WAVE - 1) sh[w] = inc;
    __syncthreads();
    uint32_t base = 0, tot = 0;
#pragma unroll
    for (int i = 0; i < NW; ++i) {
        const uint32_t t = sh[i];
        if (i < w) base += t;
        tot += t;
    }
    total = tot;
    __syncthreads();
    return base + inc - x;
}

// Ticket: true in exactly one workgroup per counter - the one that arrives last
// of `expected`. Everything the other workgroups wrote before taking their
// ticket is visible to it.
__device__ __forceinline__ bool last_block(uint32_t* counter, uint32_t expected) {
    __shared__ uint32_t ticket;
    __syncthreads();
    if (threadIdx.x == 0)
        ticket = __hip_atomic_fetch_add(counter, 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    const bool last = (ticket == expected - 1);
    if (last) {
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        __syncthreads();
    }
    return last;
}

// In a histogram of kBins counters (global or LDS), scanned from the top bin
// down, finds the bin d with #(bins above d) < krem <= #(bins above d) + h[d].
// The finder writes res[0] = d, res[1] = krem - #(above d), res[2] = h[d]; every thread gets the
// histogram total. NT threads, `sh` >= NT/64 words. res is unchanged if krem is
// 0 or exceeds the total.
template <int NT, bool GLOBAL>
__device__ __forceinline__ uint32_t find_bin(const uint32_t* h, uint32_t krem, uint32_t* sh, uint32_t* res) {
    constexpr int per = kBins / NT;
    const int top = kBins - 1 - threadIdx.x * per;  // this thread's highest bin
    uint32_t v[per], sum = 0;
#pragma unroll
    for (int i = 0; i < per; ++i) {
        v[i] = GLOBAL ? ld_load_coherent(h + top - i) : h[top - i];
        sum += v[i];
    }
    uint32_t total;
    uint32_t above = block_escan<NT>(sum, sh, total);
#pragma unroll
    for (int i = 0; i < per; ++i) {
        if (above < krem && krem <= above + v[i]) {
            res[0] = static_cast<uint32_t>(top - i);
            res[1] = krem - above;
            res[2] = v[i];
        }
        above += v[i];
    }
    __syncthreads();
    return total;
}

__device__ __forceinline__ void flush_hist(uint32_t* h, const uint32_t* lh) {
    for (int b = threadIdx.x; b < kBins; b += blockDim.x) {
        const uint32_t x = lh[b];
        if (x) atomicAdd(h + b, x);
    }
}

// In R histograms of kBins counters in LDS at h + own[i] * kBins: the bin of rank kr[i], counted from
// the top bin down, as in find_bin. With COPIES > 1 there is one, each counter in so many neighbouring words. The R scans share their
// barriers. `sh` holds 16 R words;
// res[3i], res[3i+1], res[3i+2] = bin, rank inside it, its count. The caller's counts are complete
// (a barrier has passed); ends with a barrier.
template <int NT, int R, int COPIES>
__device__ __forceinline__ void find_bins(const uint32_t* h, const int (&own)[R], const uint32_t (&kr)[R],
                                          uint32_t* sh, uint32_t* res) {
    constexpr int per = kBins / NT, NW = NT / LD_WAVE;
    static_assert(NW <= 16 && R * 16 <= LD_WAVE && (COPIES == 1 || COPIES == 4), "a row of lanes per rank");
    const int top = kBins - 1 - static_cast<int>(threadIdx.x) * per;  // this thread's highest bin
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    uint32_t v[R][per], sum[R], inc[R];
#pragma unroll
    for (int i = 0; i < R; ++i) {
        sum[i] = 0;
#pragma unroll
        for (int j = 0; j < per; ++j) {
            if (COPIES == 1) {
                v[i][j] = h[own[i] * kBins + top - j];
            } else {
                const ld_u32x4 x = *reinterpret_cast<const ld_u32x4*>(h + (top - j) * COPIES);
                v[i][j] = (x.x + x.y) + (x.z + x.w);
            }
            sum[i] += v[i][j];
        }
        inc[i] = ld_wave_iscan(sum[i]);
    }
#pragma unroll
    for (int i = 0; i < R; ++i)
        if (ld_lane() == LD_WAVE - 1) sh[i * 16 + w] = inc[i];
    __syncthreads();
    // row i of 16 lanes: the waves' sums for rank i
    const uint32_t part = ld_lane() < R * 16 && (ld_lane() & 15) < NW ? sh[ld_lane()] : 0u;
    const uint32_t waves_before = ld_row_iscan<16>(part) - part;
#pragma unroll
    for (int i = 0; i < R; ++i) {
        uint32_t above = inc[i] - sum[i] + static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(waves_before), i * 16 + w));
#pragma unroll
        for (int j = 0; j < per; ++j) {
            if (above < kr[i] && kr[i] <= above + v[i][j]) {
                res[3 * i] = static_cast<uint32_t>(top - j);
                res[3 * i + 1] = kr[i] - above;
                res[3 * i + 2] = v[i][j];
            }
            above += v[i][j];
        }
    }
    __syncthreads();
}

// The keys at R ranks (1 = largest, falling), each rounded DOWN to a multiple of
// 2^kShift2: two radix levels resolve the top 22 bits, which is all an estimate
// needs. Of a thread's keys the first `items` count (the same for all threads). The ranks share one pass over the keys per level; ranks whose prefixes
// coincide share a histogram. `lh` holds (1 + R) * kBins words and `listed` one, cleared, with a barrier since;
// `res` 3 * R, `sh` 16 * R. res[3i + 2] is left as the number of keys that round down to out[i].
// Each counter of the first level is four words that the lanes share out: a tail of keys falls into two dozen bins, and updates of one word go through
// one after another (4.5 K clocks of 27 K for one segment). The few keys of the ranks' bins are put into a list for the second level:
// asked for each of a thread's keys whether it is one of them, with few lanes active, it took 5.8 K. With the waves' sums added by lanes as well, k_prep
// takes 11.8 us instead of 13.9; a call on flat 1 M elements 37.8 -> 35.7 us, on ResNet-50 91.3 -> 88.7, on GPT-2 small 294.3 -> 293.
template <int NT, int ITEMS, int R>
__device__ __forceinline__ void block_select_multi(const uint32_t (&key)[ITEMS], int items, const uint32_t (&rank)[R], uint32_t* lh, uint32_t* sh,
                                                   uint32_t* res, uint32_t* listed, uint32_t (&out)[R]) {
    constexpr int kCopies = 4;
    static_assert(R + 1 >= kCopies, "the first level's counters");
    int own[R];
    uint32_t kr[R];
#pragma unroll
    for (int i = 0; i < R; ++i) {
        own[i] = 0;
        kr[i] = rank[i];
    }
#pragma unroll
    for (int q = 0; q < ITEMS; ++q)
        if (q < items) atomicAdd(&lh[(key[q] >> kShift1) * kCopies + (threadIdx.x & (kCopies - 1))], 1u);
    __syncthreads();
    find_bins<NT, R, kCopies>(lh, own, kr, sh, res);
    uint32_t p[R];
#pragma unroll
    for (int i = 0; i < R; ++i) {
        p[i] = res[3 * i];
        kr[i] = res[3 * i + 1];
        own[i] = i;  // the first rank with the same prefix: its histogram serves this one too
#pragma unroll
        for (int j = i - 1; j >= 0; --j)
            if (p[j] == p[i]) own[i] = j;
    }
    // the list takes the first kBins words, the second level's counters those behind
    uint32_t* l1 = lh + kBins;
    uint32_t mine = 0;
    const uint32_t least = p[0] << kShift1;  // those above belong to no rank's bin, or a higher one's
#pragma unroll
    for (int q = 0; q < ITEMS; ++q)
        if (q < items) mine |= static_cast<uint32_t>(key[q] >= least) << q;
    const uint32_t count = __popc(mine), inc = ld_wave_iscan(count);
    uint32_t at = 0;
    if (ld_lane() == LD_WAVE - 1) at = atomicAdd(listed, inc);
    at = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(at), LD_WAVE - 1)) + inc - count;
#pragma unroll
    for (int q = 0; q < ITEMS; ++q) {
        if ((mine >> q) & 1u) {
            if (at < static_cast<uint32_t>(kBins)) lh[at] = key[q];
            ++at;
        }
    }
    for (int b = threadIdx.x; b < R * kBins / 4; b += NT) reinterpret_cast<ld_u32x4*>(l1)[b] = ld_u32x4{0u, 0u, 0u, 0u};
    __syncthreads();
    const auto add = [&](uint32_t x) {
        const uint32_t d = (x >> kShift2) & 0x7FFu;
#pragma unroll
        for (int i = 0; i < R; ++i)
            if (own[i] == i && (x >> kShift1) == p[i]) atomicAdd(&l1[i * kBins + d], 1u);
    };
    const uint32_t n = *listed;
    if (n <= static_cast<uint32_t>(kBins)) {
        for (uint32_t j = threadIdx.x; j < n; j += NT) add(lh[j]);
    } else {
#pragma unroll
        for (int q = 0; q < ITEMS; ++q)
            if (q < items) add(key[q]);
    }
    __syncthreads();
    find_bins<NT, R, 1>(l1, own, kr, sh, res);
#pragma unroll
    for (int i = 0; i < R; ++i) out[i] = (p[i] << kShift1) | (res[3 * i] << kShift2);
}

__device__ __forceinline__ uint32_t umin(uint32_t a, uint32_t b) { return a < b ? a : b; }

__device__ __forceinline__ uint32_t fine_bin(uint32_t key, uint32_t tau, uint32_t sh) {
    return umin(static_cast<uint32_t>(kTopBin), (key - tau) >> sh);
}

// ------------------------------------------------------------------ geometry

typedef GroupDesc GroupRange;

__device__ __forceinline__ GroupRange group_range(const Ctx& c, int32_t g) {
    const ld_u32x4* p = reinterpret_cast<const ld_u32x4*>(c.gdesc + g);
    union { ld_u32x4 q[4]; GroupDesc d; } u;
#pragma unroll
    for (int i = 0; i < 4; ++i) u.q[i] = p[i];
    return u.d;
}

// Loads the 4 elements at e0..e0+3 that lie inside [lo, hi); returns the mask of
// valid components. e0 is a multiple of 4 and `p` is 16-byte aligned.
__device__ __forceinline__ uint32_t load4(const float* __restrict__ p, int64_t e0, int64_t lo, int64_t hi,
                                          float (&x)[4]) {
    if (e0 >= lo && e0 + 4 <= hi) {
        const ld_f32x4 q = *reinterpret_cast<const ld_f32x4*>(p + e0);
        x[0] = q.x; x[1] = q.y; x[2] = q.z; x[3] = q.w;
        return 0xF;
    }
    uint32_t mask = 0;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        x[c] = 0.0f;
        if (e0 + c >= lo && e0 + c < hi) {
            x[c] = p[e0 + c];
            mask |= 1u << c;
        }
    }
    return mask;
}

__device__ __forceinline__ void store4(float* __restrict__ p, int64_t e0, uint32_t mask, const float (&x)[4]) {
    if (mask == 0xF) {
        *reinterpret_cast<ld_f32x4*>(p + e0) = ld_f32x4{x[0], x[1], x[2], x[3]};
    } else {
#pragma unroll
        for (int c = 0; c < 4; ++c)
            if (mask & (1u << c)) p[e0 + c] = x[c];
    }
}

// -------------------------------------------------------------------- k_prep

__device__ __forceinline__ uint32_t hash32(uint32_t x) {
    x ^= x >> 16; x *= 0x7feb352dU; x ^= x >> 15; x *= 0x846ca68bU; x ^= x >> 16;
    return x;
}

// Segment tables of one batch: prefix sums over the batch entries before each one.
__global__ __launch_bounds__(512) void k_upload(UploadBatch ub, Ctx c) {
    __shared__ uint32_t sh[512 / LD_WAVE];
    const int j = threadIdx.x;
    const bool live = j < ub.count;
    const uint32_t my_groups = live ? static_cast<uint32_t>(groups_of(ub.off[j], ub.off[j + 1], c.tiles)) : 0u;
    const uint32_t my_k = live ? static_cast<uint32_t>(ub.k[j]) : 0u;  // the batch's sum is below 2^31
    uint32_t total;
    const uint32_t groups = block_escan<512>(my_groups, sh, total);
    const uint32_t ks = block_escan<512>(my_k, sh, total);
    if (!live) return;
    const int s = ub.first + j;
    c.desc[s] = SegDesc{ub.off[j], ub.out0 + ks, ub.k[j], ub.group0 + static_cast<int32_t>(groups)};
    if (s == ub.n_seg - 1)
        c.desc[s + 1] = SegDesc{ub.off[j + 1], ub.out0 + ks + my_k, c.tiles,
                                ub.group0 + static_cast<int32_t>(groups + my_groups)};
    if (s == 0)
        for (int i = 0; i < kSyncWords; ++i) c.fail_count[i] = 0;
}

// Descriptor of segment `s` and the end of its range from the packed table. The host has summed
// the segments of every bucket of 64; what is left is a prefix over the segments of the own
// bucket before `s`: one lane per segment, three scans across the first wave.
__device__ __forceinline__ SegDesc desc_from_table(const PackedTable& pt, int32_t s, int32_t tiles, int64_t& end) {
    __shared__ uint32_t found[5];
    if (threadIdx.x < LD_WAVE) {
        const int bucket = s / LD_WAVE, lane = threadIdx.x;
        const int j = bucket * LD_WAVE + lane;
        const bool live = j < pt.n_seg;
        const uint32_t code = live ? pt.code[j] : 0u;
        const uint32_t len = live ? pt.len[code] : 0u, kk = live ? pt.k[code] : 0u;
        const uint32_t off = pt.off0[bucket] + ld_wave_iscan(len) - len;   // n <= 2^31 - 1: the sums fit 32 bits
        const uint32_t out0 = pt.out0[bucket] + ld_wave_iscan(kk) - kk;
        const uint32_t groups = static_cast<uint32_t>(groups_of(off, static_cast<int64_t>(off) + len, tiles));
        const uint32_t group0 = pt.group0[bucket] + ld_wave_iscan(groups) - groups;
        if (j == s) {
            found[0] = off; found[1] = len; found[2] = out0; found[3] = kk; found[4] = group0;
        }
    }
    __syncthreads();
    end = static_cast<int64_t>(found[0]) + found[1];
    return SegDesc{static_cast<int64_t>(found[0]), static_cast<int64_t>(found[2]), static_cast<int32_t>(found[3]),
                   static_cast<int32_t>(found[4])};
}

__device__ __forceinline__ SegDesc desc_from_table(const DirectTable& dt, int32_t s, int32_t, int64_t& end) {
    const DirectTable::Entry e = dt.seg[s];
    end = dt.seg[s + 1].off;
    return SegDesc{static_cast<int64_t>(e.off), static_cast<int64_t>(e.out0), static_cast<int32_t>(e.k),
                   static_cast<int32_t>(e.group0)};
}

// NT threads: 1024 while every segment finds a CU of its own (the launch is then one chain of
// latencies: sixteen items per thread, all loads in flight at once), 512 beyond (two workgroups per CU:
// the sampled bytes bound it). Measured: one segment 20.2 -> 15.4 us, ResNet-50's 161 30.3 -> 16.1 (a
// segment that fits the sample waited for memory once per item), GPT-2 XL's 580 40.7 -> 31.9.
template <int NT, class Table>
__global__ __launch_bounds__(NT) void k_prep(const float* __restrict__ g, const float* __restrict__ r, Ctx c,
                                             int32_t no_estimate, Table pt) {
    constexpr int kItems = kSample / NT;
    static_assert(kItems <= 32 && kItems % 8 == 0, "a bit per item; loads go in batches of 8");
    __shared__ __align__(16) uint32_t lh[4 * kBins];
    __shared__ uint32_t sh[3 * 16];
    __shared__ uint32_t res[9], listed;
    // the barrier in the sampling below follows
    for (int b = threadIdx.x; b < kBins; b += NT) reinterpret_cast<ld_u32x4*>(lh)[b] = ld_u32x4{0u, 0u, 0u, 0u};
    if (threadIdx.x == 0) listed = 0;
    const int s = blockIdx.x;
    SegDesc d;
    int64_t end;
    if (pt.n_seg > 0) {
        d = desc_from_table(pt, s, c.tiles, end);
        if (threadIdx.x == 0) {
            c.desc[s] = d;
            if (s == pt.n_seg - 1)
                c.desc[s + 1] = SegDesc{end, d.out0 + d.k, c.tiles, d.group0 + groups_of(d.off, end, c.tiles)};
            if (s == 0)
                for (int i = 0; i < kSyncWords; ++i) c.fail_count[i] = 0;
        }
    } else {
        d = c.desc[s];
        end = c.desc[s + 1].off;
    }
    const int64_t off = d.off;
    const int32_t k = d.k;
    const int32_t ngroup = groups_of(off, end, c.tiles);
    if (threadIdx.x < sizeof(SegState) / 4) reinterpret_cast<uint32_t*>(&c.state[s])[threadIdx.x] = 0;
    for (int b = threadIdx.x; b < kBins; b += NT) c.hist[static_cast<int64_t>(s) * kBins + b] = 0;

    // candidate threshold, guessed threshold and bin width from a sample of |r + g|
    const int64_t ns = end - off;
    uint32_t tau = 0xFFFFFFFFu, test = 0xFFFFFFFFu, binsh = 0, tied = 0;
    if (k > 0 && !no_estimate) {
        uint32_t key[kItems];  // past the segment's end 0: the least, and no rank reaches beyond the segment's own
        const bool whole = ns <= kSample;
        const int lane = threadIdx.x & 63;
        const int64_t stride = ns / kSampleRuns;
        // no load depends on a lane's bounds: those of a batch are issued together (one memory
        // round trip per batch, not per item)
        constexpr int kLoadBatch = NT == 1024 ? 16 : 8;
        if (whole) {
            constexpr int kBatch = 4;
#pragma unroll
            for (int i0 = 0; i0 < kItems; i0 += kBatch) {
#pragma unroll
                for (int i = 0; i < kBatch; ++i) key[i0 + i] = 0;
                if (i0 * NT < ns) {  // uniform
                    float rv[kBatch], gv[kBatch];
#pragma unroll
                    for (int i = 0; i < kBatch; ++i) {
                        const int64_t e = off + (i0 + i) * NT + threadIdx.x;
                        const int64_t at = e < end ? e : end - 1;  // past the end: any element, not used
                        rv[i] = r[at];
                        gv[i] = g[at];
                    }
#pragma unroll
                    for (int i = 0; i < kBatch; ++i)
                        key[i0 + i] = off + (i0 + i) * NT + threadIdx.x < end ? ld_key(__fadd_rn(rv[i], gv[i])) : 0u;
                }
            }
        } else {
            // every run lies inside the segment: no bounds checks
#pragma unroll
            for (int i0 = 0; i0 < kItems; i0 += kLoadBatch) {
                float rv[kLoadBatch], gv[kLoadBatch];
#pragma unroll
                for (int i = 0; i < kLoadBatch; ++i) {
                    const int run = (i0 + i) * (NT / LD_WAVE) + (threadIdx.x >> 6);
                    const int64_t jitter = __umulhi(hash32(static_cast<uint32_t>(run) * 2654435761u + static_cast<uint32_t>(s)),
                                                    static_cast<uint32_t>(stride - LD_WAVE + 1));
                    const int64_t e = off + run * stride + jitter + lane;
                    rv[i] = r[e];
                    gv[i] = g[e];
                }
#pragma unroll
                for (int i = 0; i < kLoadBatch; ++i) key[i0 + i] = ld_key(__fadd_rn(rv[i], gv[i]));
            }
        }
        __syncthreads();  // the cleared counters, before the first count
        // Sample ranks (1 = largest). The selected keys are rounded down to 2^kShift2, which only
        // adds a few candidates.
        uint32_t rank[3], sel[3];
        bool estimate = true;
        if (whole) {
            // the sample is the segment: the exact threshold lies in [tau, tau + 2^kShift2); every key
            // above that range is certainly selected; bins of width 1
            rank[0] = rank[1] = rank[2] = static_cast<uint32_t>(k);
        } else {
            // expected sample hits a = k * kSample / ns. Candidates: sample rank x with x = a + z*sqrt(x),
            // so that fewer than k elements at or above tau is a z-sigma event. Bins span [tau, hi]
            // where hi is the sample key at rank a - z*sqrt(a): the k-th largest key lies below it, in
            // a fine bin, except in a z-sigma event.
            const float a = static_cast<float>(k) * (static_cast<float>(kSample) / static_cast<float>(ns));
            const float sq = 0.5f * (kSampleZ + sqrtf(kSampleZ * kSampleZ + 4.0f * a));
            rank[0] = static_cast<uint32_t>(sq * sq) + 2u;
            const float lo_rank = a - kSampleZ * sqrtf(a);
            rank[2] = lo_rank > 1.0f ? static_cast<uint32_t>(lo_rank) : 1u;
            const uint32_t mid = static_cast<uint32_t>(a + 0.5f);
            rank[1] = mid < rank[2] ? rank[2] : (mid > rank[0] ? rank[0] : mid);
            estimate = rank[0] < static_cast<uint32_t>(kSample);
        }
        if (!estimate) {
            tau = 0;  // k too large for an estimate: everything is a candidate, nothing is pre-zeroed
            binsh = kShift1;
        } else {
            block_select_multi<NT, kItems, 3>(key, whole ? static_cast<int>((ns + NT - 1) / NT) : kItems, rank, lh, sh, res, &listed, sel);
            tau = sel[0];
            if (whole) {
                test = tau + (1u << kShift2);
            } else {
                test = sel[1];
                // How often does the sample hold the candidate threshold's own key? (The selected keys
                // are rounded down to 2^kShift2: look at the sample keys of that bucket; if they are
                // many and all one value, that value is massively repeated in the segment.)
                if (res[2] >= kTieSuspect) {  // uniform
                    uint32_t kmin = 0xFFFFFFFFu, kmax = 0;
#pragma unroll
                    for (int i = 0; i < kItems; ++i) {
                        if ((key[i] >> kShift2) == (tau >> kShift2)) {
                            kmin = umin(kmin, key[i]);
                            kmax = key[i] > kmax ? key[i] : kmax;
                        }
                    }
                    __syncthreads();
                    if (threadIdx.x == 0) { res[0] = 0xFFFFFFFFu; res[1] = 0; }
                    __syncthreads();
                    if (kmin <= kmax) {
                        atomicMin(&res[0], kmin);
                        atomicMax(&res[1], kmax);
                    }
                    __syncthreads();
                    if (res[0] == res[1] && res[0] != 0x7FFFFFFFu) {
                        tied = 1;  // candidates: the keys above it; no pre-zeroing (see SegState::tied)
                        tau = res[0] + 1u;
                        test = 0xFFFFFFFFu;
                    }
                }
                const uint32_t top = sel[2] | ((1u << kShift2) - 1u);
                const uint32_t range = top > tau ? top - tau : 0u;
                while ((range >> binsh) > static_cast<uint32_t>(kTopBin - 1)) ++binsh;
            }
        }
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        c.state[s].tau = tau;
        c.state[s].sh = binsh;
        c.state[s].test = test;
        c.state[s].kmin = 0xFFFFFFFFu;
        c.state[s].tied = tied;
    }
    for (int32_t q = threadIdx.x; q < ngroup; q += NT)
        c.gdesc[d.group0 + q] = GroupDesc{align_down4(off) + static_cast<int64_t>(q) * c.tiles * kTile, off, end, d.out0,
                                          s, k, d.group0, ngroup, tau, binsh, test, tied};
}

// -------------------------------------------------------------------- k_main

// How the tiles are dealt to the XCDs: one by one in address order below kMainRunTiles
// (180 M elements), in runs of 16 tiles (256 KB per array) above. Measured, us per compress call with
// eighths of the arrays per XCD / single tiles / runs of 16: 48 M elements 180 / 169 / 174,
// 128 M 352 / 336 / 341, 160 M 433 / 407 / 409, 200 M 508 / 487 / 483, 512 M 1224 / 1184 / 1156, 1.2 G
// 2838 / 2782 / 2672; runs of 2, 8, 32 and 64 lie between or behind.
constexpr int64_t kMainRunTiles = 700 * 64;
constexpr int kMainRows = kTile / (LD_WAVE * 4);  // float4 rows per lane
// Tables with a quarter more tile slots than tiles (the groups of small or ragged segments are only begun): the XCDs
// take turns, or the first slots of all groups would be one's or two's. Measured, us per call without / with:
// 520 segments of up to 5000 elements 173 / 99, 3000 of up to 3000 508 / 292, 800 of 30,000 to 400,000 581 / 470,
// ResNet-50 (1.27 slots a tile) 106 / 99.5, GPT-2 small (1.23) 304 / 302; below the line they are the better
// unturned or the same (one segment of 160 M elements 485 / 489, GPT-2 XL, 1.09, 3267 / 3488).
constexpr int64_t kMainTurnQuarters = 5;

// SMALL: the slots have the minimum size (every call at the usual densities): a constant then.
// RUN: consecutive tiles an XCD is given at a time (see ld_xcd_piece and kMainRunTiles).
// A workgroup is one wave: with two, four and eight tiles per workgroup a call on 1.56 G elements took
// 3275, 3517 and 3546 us instead of 3255, on ResNet-50 136, 141 and 156 instead of 128 (a workgroup's
// registers are held until its last wave is done).
template <bool SMALL, uint32_t RUN>
__global__ __launch_bounds__(LD_WAVE) void k_main(const float* __restrict__ g, float* __restrict__ r, Ctx c,
                                              uint32_t turn) {
    const int32_t slot_size = SMALL ? kSlotMin : c.slot;
    const int32_t tile = static_cast<int32_t>(ld_xcd_piece<RUN>(blockIdx.x, gridDim.x, turn));
    const int shift = c.tiles == kTilesPerGroup ? 6 : 4;
    static_assert(kTilesPerGroup == 1 << 6 && kTilesPerSmallGroup == 1 << 4, "");
    const GroupDesc gd = group_range(c, tile >> shift);
    const int lane = ld_lane();
    const int64_t t = gd.base + static_cast<int64_t>(tile & (c.tiles - 1)) * kTile;
    const int64_t seg_lo = gd.lo, seg_hi = gd.hi;
    if (t >= seg_hi) {  // tile slot past the end of the segment
        if (lane == 0) c.cnt[tile] = 0;
        return;
    }
    const uint32_t tau = gd.tau, test = gd.test;
    const bool interior = t >= seg_lo && t + kTile <= seg_hi;
    float a[kMainRows][4];
    uint32_t mask[kMainRows];
    if (interior) {  // unconditional 16-byte streaming accesses
        const ld_f32x4* g4 = reinterpret_cast<const ld_f32x4*>(g + t) + lane;
        const ld_f32x4* r4 = reinterpret_cast<const ld_f32x4*>(r + t) + lane;
        ld_f32x4 gq[kMainRows], rq[kMainRows];
#pragma unroll
        for (int j = 0; j < kMainRows; ++j) gq[j] = ld_nt_load(g4 + j * LD_WAVE);
#pragma unroll
        for (int j = 0; j < kMainRows; ++j) rq[j] = ld_nt_load(r4 + j * LD_WAVE);
#pragma unroll
        for (int j = 0; j < kMainRows; ++j) {
            a[j][0] = __fadd_rn(rq[j].x, gq[j].x);
            a[j][1] = __fadd_rn(rq[j].y, gq[j].y);
            a[j][2] = __fadd_rn(rq[j].z, gq[j].z);
            a[j][3] = __fadd_rn(rq[j].w, gq[j].w);
            mask[j] = 0xF;
        }
    } else {
#pragma unroll
        for (int j = 0; j < kMainRows; ++j) {
            const int64_t e0 = t + (j * LD_WAVE + lane) * 4;
            float gv[4], rv[4];
            mask[j] = load4(g, e0, seg_lo, seg_hi, gv);
            load4(r, e0, seg_lo, seg_hi, rv);
#pragma unroll
            for (int q = 0; q < 4; ++q) a[j][q] = __fadd_rn(rv[q], gv[q]);
        }
    }
    // candidates, in element order (row, lane, component)
    uint32_t flag[kMainRows], zero[kMainRows], pos0[kMainRows], total = 0;
#pragma unroll
    for (int j = 0; j < kMainRows; ++j) {
        flag[j] = 0;
        zero[j] = 0;
        pos0[j] = total;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const uint32_t key = ld_key(a[j][q]);
            const bool f = ((mask[j] >> q) & 1u) && key >= tau;
            flag[j] |= static_cast<uint32_t>(f) << q;
            zero[j] |= static_cast<uint32_t>(f && key >= test) << q;
            const uint64_t m = __ballot(f);
            pos0[j] += ld_mbcnt(m);
            total += __popcll(m);
        }
    }
    const bool fits = total <= static_cast<uint32_t>(slot_size);  // else: the residual keeps r + g everywhere, the slot stays unused
    if (lane == 0) c.cnt[tile] = fits ? total : kOverflow;
    // residual: +0 where the guessed threshold selects, r + g elsewhere
#pragma unroll
    for (int j = 0; j < kMainRows; ++j) {
        float x[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) x[q] = (fits && ((zero[j] >> q) & 1u)) ? 0.0f : a[j][q];
        if (interior)
            ld_nt_store(ld_f32x4{x[0], x[1], x[2], x[3]}, reinterpret_cast<ld_f32x4*>(r + t) + j * LD_WAVE + lane);
        else
            store4(r, t + (j * LD_WAVE + lane) * 4, mask[j], x);
    }
    if (!fits || total == 0) return;
    float* sv = c.cval + static_cast<int64_t>(tile) * slot_size;
    uint16_t* si = c.cidx + static_cast<int64_t>(tile) * slot_size;
#pragma unroll
    for (int j = 0; j < kMainRows; ++j) {
        if (flag[j] == 0) continue;
        uint32_t pos = pos0[j];
        const uint32_t local = (j * LD_WAVE + lane) * 4;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            if ((flag[j] >> q) & 1u) {
                sv[pos] = a[j][q];
                si[pos] = static_cast<uint16_t>(local + q);
                ++pos;
            }
        }
    }
}

// ------------------------------------------------- passes over the candidates
//
// A wave of a small pass owns kTilesPerWave consecutive tiles of its group.
//
// Fast path, for tiles with at most ROW * 8 stored candidates (nearly all of them):
// 64 / ROW tiles at a time, one per row of ROW lanes (four tiles of up to 128 at the
// usual 1 % density). A lane holds 8 consecutive candidates of its row's tile (two
// 16-byte loads of values, one of in-tile offsets), so one trip through the loop body
// serves several tiles, and per-tile sums and prefixes are row operations. These
// passes are bound by instruction issue, not by memory: the body is kept small and
// rolled.
//
// Slow path (slow_tiles), for tiles with more stored candidates and for tiles whose
// slot overflowed (read back from the residual, which then holds r + g unzeroed,
// and filtered with the test k_main applied): begin(u); then item(have, val, local,
// stored) for batches of 64 candidates (one per lane, index order, called by all
// lanes together; `local` is the element's offset inside the tile, `stored` tells
// that the candidate comes from the slot); then end(u).
constexpr int kPerLane = 8;                   // candidates per lane

// Shape of the fast path: ROW lanes per tile (16, 32 or 64, chosen per call from the densities),
// so a trip serves 64 / ROW tiles of at most ROW * 8 candidates each; TILES tiles per group.
template <int ROW, int TILES>
struct Rows {
    static constexpr int kRow = ROW, kGroupTiles = TILES;
    static constexpr int kTilesPerWave = TILES / kWaves;
    static constexpr bool kSmall = TILES == kTilesPerSmallGroup;
    static constexpr int kTiles = LD_WAVE / ROW;                 // tiles per trip
    static constexpr uint32_t kFast = ROW * kPerLane;            // candidates a tile may hold
    static constexpr int kTrips = kTilesPerWave / kTiles;
    static constexpr int kAhead = kTrips < 4 ? kTrips : 4;       // trips requested together
};

// Slot size as the candidate passes see it: calls that run them with 16 lanes per tile expect at
// most 128 candidates per tile and always get the minimum slot, a constant.
template <class RW>
__device__ __forceinline__ int32_t slot_of(const Ctx& c) { return RW::kRow == 16 ? kSlotMin : c.slot; }

__device__ __forceinline__ int wave_in_group() { return static_cast<int>(threadIdx.x >> 6) & (kWaves - 1); }

// Lane u < RW::kTilesPerWave: the candidate count of the wave's tile u (k_main writes a
// count for every tile slot of every group, 0 past the end of a segment). Fetched
// first, so that it travels together with the group descriptor.
template <class RW>
__device__ __forceinline__ uint32_t wave_counts(const Ctx& c, int32_t group) {
    const int lane = ld_lane();
    const int32_t tile0 = group * RW::kGroupTiles + wave_in_group() * RW::kTilesPerWave;
    return lane < RW::kTilesPerWave ? c.cnt[tile0 + lane] : 0u;
}

template <int ROW>
__device__ __forceinline__ uint32_t row_sum(uint32_t x) {  // over a row of ROW lanes, in every lane
    if (ROW == LD_WAVE) return ld_wave_sum(x);
    x = ld_row16_sum(x);
    if (ROW == 32) x += __shfl_xor(x, 16, ROW);
    return x;
}

struct Trip {
    float v[kPerLane];      // candidate values (entries at or past `have` are stale)
    uint32_t x[kPerLane];   // their offsets inside the tile (IDX only)
    uint32_t have;          // valid entries of this lane: 0..kPerLane
    uint32_t cn;            // stored count of the row's tile (kOverflow, or > ROW * 8: not served here)
    int u;                  // the row's tile, counted inside the wave
};

// The lane's part of trip q (tiles kTiles*q .. of the wave) as it comes from memory: only the
// entries the tile's count says are there (these passes are bound by the bytes they pull from the
// scattered slots: reading whole slots regardless of the counts made them a third slower). The
// trips of a batch are requested together.
struct TripRaw { ld_f32x4 a, b; ld_u32x4 xi; };

template <bool IDX, class RW>
__device__ __forceinline__ void trip_issue(const Ctx& c, int32_t tile0, uint32_t mycnt, int q, TripRaw& R) {
    const int lane = ld_lane();
    const int u = RW::kTiles * q + lane / RW::kRow;
    const uint32_t cn = static_cast<uint32_t>(__shfl(static_cast<int>(mycnt), u, LD_WAVE));
    const uint32_t n = cn <= RW::kFast ? cn : 0u;
    const uint32_t first = static_cast<uint32_t>(lane & (RW::kRow - 1)) * kPerLane;
    const int64_t at = static_cast<int64_t>(tile0 + u) * slot_of<RW>(c) + first;
    R.a = ld_f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    R.b = R.a;
    R.xi = ld_u32x4{0u, 0u, 0u, 0u};
    if (first < n) R.a = *reinterpret_cast<const ld_f32x4*>(c.cval + at);
    if (first + 4 < n) R.b = *reinterpret_cast<const ld_f32x4*>(c.cval + at + 4);
    if (IDX && first < n) R.xi = *reinterpret_cast<const ld_u32x4*>(c.cidx + at);
}

template <bool IDX, class RW>
__device__ __forceinline__ void trip_finish(const TripRaw& R, uint32_t mycnt, int q, Trip& Q) {
    const int lane = ld_lane();
    const int u = RW::kTiles * q + lane / RW::kRow;
    const uint32_t cn = static_cast<uint32_t>(__shfl(static_cast<int>(mycnt), u, LD_WAVE));
    const uint32_t n = cn <= RW::kFast ? cn : 0u;
    const uint32_t first = static_cast<uint32_t>(lane & (RW::kRow - 1)) * kPerLane;
    Q.v[0] = R.a.x; Q.v[1] = R.a.y; Q.v[2] = R.a.z; Q.v[3] = R.a.w;
    Q.v[4] = R.b.x; Q.v[5] = R.b.y; Q.v[6] = R.b.z; Q.v[7] = R.b.w;
    if (IDX) {
        const uint32_t xw[4] = {R.xi.x, R.xi.y, R.xi.z, R.xi.w};
#pragma unroll
        for (int j = 0; j < kPerLane; ++j) Q.x[j] = (j & 1) ? (xw[j >> 1] >> 16) : (xw[j >> 1] & 0xFFFFu);
    }
    Q.have = first < n ? umin(n - first, static_cast<uint32_t>(kPerLane)) : 0u;
    Q.cn = cn;
    Q.u = u;
}

// Runs body(Q) for every trip of the wave, kAhead trips requested at a time. `first` holds the
// first batch, requested by the caller as early as it could.
template <bool IDX, class RW, class Body>
__device__ __forceinline__ void for_trips(const Ctx& c, int32_t tile0, uint32_t mycnt, TripRaw (&first)[RW::kAhead],
                                          Body&& body) {
    static_assert(RW::kTrips % RW::kAhead == 0, "trips come in whole batches");
#pragma unroll 1
    for (int q0 = 0; q0 < RW::kTrips; q0 += RW::kAhead) {
        if (q0 > 0) {
#pragma unroll
            for (int a = 0; a < RW::kAhead; ++a) trip_issue<IDX, RW>(c, tile0, mycnt, q0 + a, first[a]);
        }
#pragma unroll
        for (int a = 0; a < RW::kAhead; ++a) {
            Trip Q;
            trip_finish<IDX, RW>(first[a], mycnt, q0 + a, Q);
            body(Q, q0 + a);
        }
    }
}

template <bool IDX, class RW>
__device__ __forceinline__ void first_trips(const Ctx& c, int32_t tile0, uint32_t mycnt, TripRaw (&first)[RW::kAhead]) {
#pragma unroll
    for (int a = 0; a < RW::kAhead; ++a) trip_issue<IDX, RW>(c, tile0, mycnt, a, first[a]);
}

template <bool IDX, class RW, class Begin, class Item, class End>
__device__ __forceinline__ void slow_tiles(const Ctx& c, const float* __restrict__ r, const GroupRange& gr,
                                           int32_t group, uint32_t mycnt, uint32_t tau, Begin&& begin, Item&& item,
                                           End&& end) {
    const int lane = ld_lane();
    const int tl0 = wave_in_group() * RW::kTilesPerWave;
    const int32_t tile0 = group * RW::kGroupTiles + tl0;
    const int64_t tbase0 = gr.base + static_cast<int64_t>(tl0) * kTile;
    // tiles of the wave that are not served by the fast path
    uint64_t todo = __ballot(lane < RW::kTilesPerWave && mycnt > RW::kFast);
    while (todo) {
        const int u = __builtin_ctzll(todo);
        todo &= todo - 1;
        const uint32_t cn = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(mycnt), u));
        const bool stored = cn != kOverflow;
        const uint32_t total = stored ? cn : static_cast<uint32_t>(kTile);
        const int64_t slot = static_cast<int64_t>(tile0 + u) * slot_of<RW>(c);
        const int64_t tbase = tbase0 + static_cast<int64_t>(u) * kTile;
        begin(u);
        // kAhead batches of 64 are requested before the first is handed on: a tile read back from
        // the residual is 64 batches long, and one load at a time would wait for memory 64 times
        constexpr int kAhead = 4;
#pragma unroll 1
        for (uint32_t b0 = 0; b0 < total; b0 += kAhead * LD_WAVE) {
            bool have[kAhead];
            float v[kAhead];
            uint32_t x[kAhead];
#pragma unroll
            for (int a = 0; a < kAhead; ++a) {
                const uint32_t at = b0 + a * LD_WAVE + lane;
                have[a] = at < total;
                if (stored) {
                    v[a] = have[a] ? c.cval[slot + at] : 0.0f;
                    x[a] = (IDX && have[a]) ? c.cidx[slot + at] : 0u;
                } else {
                    const int64_t e = tbase + at;
                    have[a] = have[a] && e >= gr.lo && e < gr.hi;
                    v[a] = have[a] ? r[e] : 0.0f;
                    x[a] = at;
                }
            }
#pragma unroll
            for (int a = 0; a < kAhead; ++a) {
                if (b0 + a * LD_WAVE < total) {
                    const bool h = stored ? have[a] : (have[a] && ld_key(v[a]) >= tau);
                    item(h, v[a], x[a], stored);
                }
            }
        }
        end(u);
    }
}

__device__ __forceinline__ void mark_full(const Ctx& c, SegState* st, const GroupRange& gr, uint32_t* list0, bool late = false) {
    if (threadIdx.x == 0) {
        if (late) st->late = 1; else st->mode = kModeFull;
        *list0 = atomicAdd(c.fail_count + kSyncCount, static_cast<uint32_t>(gr.ngroup));
    }
    __syncthreads();
    for (int32_t q = threadIdx.x; q < gr.ngroup; q += blockDim.x) c.fail_groups[*list0 + q] = gr.group0 + q;
}

// Fine-bin histogram of the candidates of kHistGroups consecutive groups (256 threads each),
// added to their segments'. Updates of one counter from many workgroups queue up behind one
// another, and the largest segment has hundreds of groups: the groups of a workgroup that
// belong to the same segment are summed in LDS first and added once.
// With at most kFewGroups groups there is little to queue up and much of the chip idle: a workgroup per group
// then (us per call: flat 1 M elements 47.3 -> 45.0, 8 M 67.0 -> 65.3, 12 M 74.2 -> 73.0; 24 M and its 406 groups,
// where it was the slower one, 102.5 -> 104.1).
constexpr int kHistGroups = 4;
constexpr int32_t kFewGroups = 256;

template <class RW, int GROUPS>
__global__ __launch_bounds__(GROUPS * kThreads) void k_hist(const float* __restrict__ r, Ctx c) {
    __shared__ uint32_t lh[GROUPS][kBins];
    __shared__ int32_t qseg[GROUPS];
    const int q = threadIdx.x / kThreads, tid = threadIdx.x % kThreads;
    const int32_t group = blockIdx.x * GROUPS + q;
    const bool inside = group < c.n_group;
    const int32_t tile0 = group * RW::kGroupTiles + wave_in_group() * RW::kTilesPerWave;
    uint32_t mycnt = 0;
    GroupRange gr;
    gr.k = 0;
    TripRaw raw[RW::kAhead];
    if (inside) {
        mycnt = wave_counts<RW>(c, group);
        gr = group_range(c, group);
        first_trips<false, RW>(c, tile0, mycnt, raw);
    }
    const bool live = inside && gr.k != 0;
    const uint32_t tau = gr.tau, binsh = gr.sh;
    for (int b = tid; b < kBins; b += kThreads) lh[q][b] = 0;
    if (tid == 0) qseg[q] = live ? gr.seg : -1;
    __syncthreads();
    if (live) {
        // keys above the binned range all land in the top bin (a third of the candidates, more
        // at higher densities): counted in a register, added once per wave
        uint32_t top = 0;
        for_trips<false, RW>(c, tile0, mycnt, raw, [&](const Trip& Q, int) {
#pragma unroll
            for (int j = 0; j < kPerLane; ++j) {
                if (static_cast<uint32_t>(j) < Q.have) {
                    const uint32_t bin = fine_bin(ld_key(Q.v[j]), tau, binsh);
                    if (bin == static_cast<uint32_t>(kTopBin)) ++top; else atomicAdd(&lh[q][bin], 1u);
                }
            }
        });
        slow_tiles<false, RW>(
            c, r, gr, group, mycnt, tau, [](int) {},
            [&](bool have, float v, uint32_t, bool) {
                const uint32_t bin = fine_bin(ld_key(v), tau, binsh);
                const uint64_t any = __ballot(have);
                if (any == 0) return;
                // massive ties put a whole batch into one bin: one update instead of 64 on one counter
                const uint32_t lead = static_cast<uint32_t>(__shfl(static_cast<int>(bin), __builtin_ctzll(any), LD_WAVE));
                if (__ballot(have && bin == lead) == any) {
                    if (ld_lane() == 0) {
                        if (lead == static_cast<uint32_t>(kTopBin)) top += __popcll(any);
                        else atomicAdd(&lh[q][lead], static_cast<uint32_t>(__popcll(any)));
                    }
                } else if (have) {
                    if (bin == static_cast<uint32_t>(kTopBin)) ++top; else atomicAdd(&lh[q][bin], 1u);
                }
            },
            [](int) {});
        top = ld_wave_sum(top);
        if (ld_lane() == 0 && top) atomicAdd(&lh[q][kTopBin], top);
    }
    __syncthreads();
    if (!live || (q > 0 && qseg[q - 1] == gr.seg)) return;  // summed by the first group of the run
    int run = 1;
    while (q + run < GROUPS && qseg[q + run] == gr.seg) ++run;
    uint32_t* h = c.hist + static_cast<int64_t>(gr.seg) * kBins;
    for (int b = tid; b < kBins; b += kThreads) {
        uint32_t x = 0;
        for (int j = 0; j < run; ++j) x += lh[q + j][b];
        if (x) atomicAdd(h + b, x);
    }
}

// The fine bin that holds the segment's k-th largest key (res[0], res[1] = the rank inside it, res[2] = its keys),
// found in its histogram by a whole workgroup of kThreads; returns the mode the segment goes on in: the
// full path when the candidates are fewer than k. `note`: this workgroup writes it all to the
// segment's state and lists.
__device__ __forceinline__ uint32_t threshold_bin(const Ctx& c, const GroupRange& gr, SegState* st, bool note,
                                                  uint32_t* sh, uint32_t* res, uint32_t* list0) {
    const uint32_t* h = c.hist + static_cast<int64_t>(gr.seg) * kBins;
    if (threadIdx.x == 0) { res[0] = 0; res[1] = 0; }
    __syncthreads();
    const uint32_t total = find_bin<kThreads, false>(h, static_cast<uint32_t>(gr.k), sh, res);
    if (total >= static_cast<uint32_t>(gr.k)) {
        if (note && threadIdx.x == 0) { st->prefix = res[0]; st->krem = res[1]; }
        return kModeCand;
    }
    if (gr.tied) {
        // every candidate is selected; the rest must be ties of the repeated key (k_emit checks)
        if (note && threadIdx.x == 0) {
            st->mode = kModeTies;
            st->prefix = gr.tau - 1u;                           // T
            st->krem = static_cast<uint32_t>(gr.k) - total;     // m
        }
        return kModeTies;
    }
    if (note) mark_full(c, st, gr, list0);  // the candidate threshold was too high
    return kModeFull;
}

// Elements of the tile starting at tbase whose key is `key`, counted by the whole wave from the
// residual (which holds r + g wherever nothing was zeroed).
__device__ __forceinline__ uint32_t count_key_in_tile(const float* __restrict__ r, int64_t tbase, int64_t lo,
                                                      int64_t hi, uint32_t key) {
    uint32_t n = 0;
#pragma unroll 4
    for (int j = 0; j < kTile / (LD_WAVE * 4); ++j) {
        float x[4];
        const uint32_t mask = load4(r, tbase + (j * LD_WAVE + ld_lane()) * 4, lo, hi, x);
#pragma unroll
        for (int q = 0; q < 4; ++q) n += ((mask >> q) & 1u) && ld_key(x[q]) == key;
    }
    return ld_wave_sum(n);
}

// Keys of the threshold bin held by the lanes of a wave (bit j of `in`: candidate j of the lane)
// go to the segment's gather list: one reservation for the wave. Returns what found no room.
// Kept out of line: the loop around it is bound by instruction fetch, and this runs for a few
// keys per segment only.
struct Unplaced { uint32_t kmin, kmax; bool full; };

__device__ __attribute__((noinline)) Unplaced gather_lane_keys(SegState* st, uint32_t* gkey, int32_t* gtile,
                                                               uint32_t gcap, ld_f32x4 va, ld_f32x4 vb, uint32_t in,
                                                               int32_t tile, bool full) {
    const float v[kPerLane] = {va.x, va.y, va.z, va.w, vb.x, vb.y, vb.z, vb.w};
    Unplaced un{0xFFFFFFFFu, 0u, full};
    const int lane = ld_lane();
    const uint32_t n_in = __popc(in);
    const uint32_t inc = ld_wave_iscan(n_in);
    const uint32_t total = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(inc), LD_WAVE - 1));
    uint32_t base = gcap;
    if (!full) {
        if (lane == 0) base = atomicAdd(&st->gcount, total);
        base = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(base)));
        un.full = base + total > gcap;
    }
    uint32_t pos = base + inc - n_in;
#pragma unroll
    for (int j = 0; j < kPerLane; ++j) {
        if ((in >> j) & 1u) {
            const uint32_t key = ld_key(v[j]);
            if (pos < gcap) {
                gkey[pos] = key;
                gtile[pos] = tile;
            } else {
                un.kmin = umin(un.kmin, key);
                un.kmax = key > un.kmax ? key : un.kmax;
            }
            ++pos;
        }
    }
    return un;
}

// Small groups, keys of the threshold bin beyond which a workgroup of k_gather makes one reservation in the
// gather list for all of its waves. What the waves of a segment add to its counter queues up, 20 ns each, and small
// groups are as many waves as batches: 2 segments of 50 M elements with values on a coarse grid (keys of the bin
// in every wave) 183 -> 64 us, rounded to bf16 95 -> 23.5; the few keys of a small segment are placed
// 0.6 us sooner each by itself (flat 1 M elements).
constexpr uint32_t kFewKeys = 256;

// Per tile: candidates in bins above the threshold bin; the keys inside the bin
// are gathered per segment. The bin is found by each workgroup for itself: as a launch of one workgroup per segment ahead of this one it
// cost more, with any number of groups (GPT-2 small 299.2 -> 297.3 us a call, 520 segments of up to 5000 elements 82.2 -> 80.3, 3000 of up to
// 3000 258.7 -> 254, 800 of 30,000 to 400,000 489 -> 485; GPT-2 XL, 400 M, 1.2 G: the same).
template <class RW>
__global__ __launch_bounds__(kThreads) void k_gather(const float* __restrict__ r, Ctx c) {
    __shared__ uint32_t wsum[2][kWaves], wmin[kWaves], wmax[kWaves];
    const uint32_t mycnt = wave_counts<RW>(c, blockIdx.x);
    const GroupRange gr = group_range(c, blockIdx.x);
    TripRaw raw[RW::kAhead];
    first_trips<false, RW>(c, blockIdx.x * RW::kGroupTiles + (threadIdx.x >> 6) * RW::kTilesPerWave, mycnt, raw);
    SegState* st = c.state + gr.seg;
    if (gr.k == 0) return;
    // each workgroup finds the threshold bin for itself, the segment's first one notes it down
    __shared__ uint32_t sh[kWaves], res[3], list0;
    const uint32_t mode = threshold_bin(c, gr, st, static_cast<int32_t>(blockIdx.x) == gr.group0, sh, res, &list0);
    const uint32_t b1 = res[0];
    const bool many = RW::kSmall && mode == kModeCand && res[2] > kFewKeys;  // one reservation per workgroup (see below)
    if (mode == kModeFull) return;
    // kModeTies: every candidate lies above the threshold and nothing is gathered; the ties of a
    // tile are what k_main counted
    const bool ties_mode = mode == kModeTies;
    const uint32_t tau = gr.tau, binsh = gr.sh;
    const int lane = ld_lane();
    const int w = threadIdx.x >> 6;
    uint32_t* gkey = c.gkey + gather_first(gr.seg, gr.lo);
    int32_t* gtile = c.gtile + gather_first(gr.seg, gr.lo);
    const uint32_t gcap = gather_cap(gr.lo, gr.hi);
    const int32_t tile0 = blockIdx.x * RW::kGroupTiles + w * RW::kTilesPerWave;
    // Keys of the threshold bin go to the segment's gather list, one reservation per wave and
    // batch. When the list is full (massive ties: millions of equal keys) nothing more is
    // reserved (a wave learns that from its first reservation that comes back beyond the end);
    // the keys that found no room only widen the segment's [kmin, kmax]. With small groups a wave has
    // no second batch to profit from that: see kFewKeys.
    bool full = false;
    uint32_t lmin = 0xFFFFFFFFu, lmax = 0;
    uint32_t part_gt = 0, part_eq = 0;  // fast path: the first lane of a row sums the row's tiles
    uint32_t wave_ties = 0;
    if (ties_mode) {  // the repeated key tau - 1, counted per tile in the residual
        const int tl0 = w * RW::kTilesPerWave;
#pragma unroll 1
        for (int u = 0; u < RW::kTilesPerWave; ++u) {
            const int64_t tbase = gr.base + static_cast<int64_t>(tl0 + u) * kTile;
            const uint32_t t = tbase < gr.hi ? count_key_in_tile(r, tbase, gr.lo, gr.hi, tau - 1u) : 0u;
            if (lane == 0) c.tile_eq[tile0 + u] = t;
            wave_ties += t;
        }
    }
    uint32_t place = 0;  // small groups: where this lane's next key goes
    if (RW::kSmall && many) {  // uniform
        static_assert(!RW::kSmall || RW::kTrips == RW::kAhead, "all trips of a wave are in registers");
        __shared__ uint32_t wkeys[kWaves], first;
        uint32_t mine = 0, before = 0, total = 0;
#pragma unroll
        for (int a = 0; a < RW::kAhead; ++a) {
            Trip Q;
            trip_finish<false, RW>(raw[a], mycnt, a, Q);
#pragma unroll
            for (int j = 0; j < kPerLane; ++j)
                mine += static_cast<uint32_t>(j) < Q.have && fine_bin(ld_key(Q.v[j]), tau, binsh) == b1;
        }
        const uint32_t inc = ld_wave_iscan(mine);
        if (lane == LD_WAVE - 1) wkeys[w] = inc;
        __syncthreads();
#pragma unroll
        for (int u = 0; u < kWaves; ++u) {
            before += u < w ? wkeys[u] : 0u;
            total += wkeys[u];
        }
        if (total > 0) {  // uniform
            if (threadIdx.x == 0) first = atomicAdd(&st->gcount, total);
            __syncthreads();
            place = first + before + inc - mine;
            full = first + total > gcap;
        }
    }
    for_trips<false, RW>(c, tile0, mycnt, raw, [&](const Trip& Q, int) {
        uint32_t cnt = 0, in = 0;
#pragma unroll
        for (int j = 0; j < kPerLane; ++j) {
            const uint32_t bin = fine_bin(ld_key(Q.v[j]), tau, binsh);
            const bool valid = static_cast<uint32_t>(j) < Q.have;
            cnt += valid && (ties_mode || bin > b1);
            in |= static_cast<uint32_t>(valid && !ties_mode && bin == b1) << j;
        }
        const uint32_t n_in = __popc(in);
        const uint64_t who = __ballot(in != 0);
        if (who) {
            if (!RW::kSmall && (full || __popcll(who) >= 4)) {  // massive ties: one reservation for the wave, or none
                const Unplaced un = gather_lane_keys(st, gkey, gtile, gcap, ld_f32x4{Q.v[0], Q.v[1], Q.v[2], Q.v[3]},
                                                     ld_f32x4{Q.v[4], Q.v[5], Q.v[6], Q.v[7]}, in, tile0 + Q.u, full);
                lmin = umin(lmin, un.kmin);
                lmax = un.kmax > lmax ? un.kmax : lmax;
                full = un.full;
            } else {  // the usual case: a key or two; or the lane's own places
#pragma unroll
                for (int j = 0; j < kPerLane; ++j) {
                    if ((in >> j) & 1u) {
                        const uint32_t key = ld_key(Q.v[j]);
                        const uint32_t pos = many ? place++ : atomicAdd(&st->gcount, 1u);
                        if (pos < gcap) {
                            gkey[pos] = key;
                            gtile[pos] = tile0 + Q.u;
                        } else {
                            lmin = umin(lmin, key);
                            lmax = key > lmax ? key : lmax;
                        }
                    }
                }
            }
        }
        const uint32_t both = row_sum<RW::kRow>(cnt | (n_in << 16));  // a tile holds at most 512 here
        cnt = both & 0xFFFFu;
        const uint32_t eqc = both >> 16;
        if ((lane & (RW::kRow - 1)) == 0 && Q.cn <= RW::kFast) {
            c.tile_gt[tile0 + Q.u] = cnt;
            if (!ties_mode) c.tile_eq[tile0 + Q.u] = eqc;  // keys in the threshold bin: ties if the bin is overfull
            part_gt += cnt;
            part_eq += eqc;
        }
    });
    uint32_t slow_gt = 0, slow_eq = 0, gt = 0, eq = 0;
    int32_t tile_of_item = 0;
    slow_tiles<false, RW>(
        c, r, gr, blockIdx.x, mycnt, tau,
        [&](int u) {
            gt = 0;
            eq = 0;
            tile_of_item = tile0 + u;
        },
        [&](bool have, float v, uint32_t, bool) {
            const uint32_t key = ld_key(v);
            const uint32_t bin = have ? fine_bin(key, tau, binsh) : 0u;
            gt += __popcll(__ballot(have && (ties_mode || bin > b1)));
            const bool in = have && !ties_mode && bin == b1;
            const uint64_t min_ = __ballot(in);
            if (min_) {
                const uint32_t total = static_cast<uint32_t>(__popcll(min_));
                eq += total;
                uint32_t base = gcap;
                if (!full) {
                    if (lane == 0) base = atomicAdd(&st->gcount, total);
                    base = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(base)));
                    full = base + total > gcap;
                }
                const uint32_t pos = base + ld_mbcnt(min_);
                if (in) {
                    if (pos < gcap) {
                        gkey[pos] = key;
                        gtile[pos] = tile_of_item;
                    } else {
                        lmin = umin(lmin, key);
                        lmax = key > lmax ? key : lmax;
                    }
                }
            }
        },
        [&](int u) {
            if (lane == 0) {
                c.tile_gt[tile0 + u] = gt;
                if (!ties_mode) c.tile_eq[tile0 + u] = eq;
            }
            slow_gt += gt;
            slow_eq += eq;
        });
    if (__ballot(lmin <= lmax)) {  // some key of this wave found no room
#pragma unroll
        for (int d = LD_WAVE / 2; d > 0; d >>= 1) {
            lmin = umin(lmin, static_cast<uint32_t>(__shfl_xor(static_cast<int>(lmin), d, LD_WAVE)));
            const uint32_t o = static_cast<uint32_t>(__shfl_xor(static_cast<int>(lmax), d, LD_WAVE));
            lmax = o > lmax ? o : lmax;
        }
    }
    const uint32_t wave_gt = ld_wave_sum(part_gt) + slow_gt;
    const uint32_t wave_eq = ld_wave_sum(part_eq) + slow_eq + wave_ties;
    if (lane == 0) {
        wsum[0][w] = wave_gt;
        wsum[1][w] = wave_eq;
        wmin[w] = lmin;
        wmax[w] = lmax;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
#pragma unroll
        for (int u = 1; u < kWaves; ++u) {
            lmin = umin(lmin, wmin[u]);
            lmax = wmax[u] > lmax ? wmax[u] : lmax;
        }
        if (lmin <= lmax) {
            atomicMin(&st->kmin, lmin);
            atomicMax(&st->kmax, lmax);
        }
        c.group_gt[blockIdx.x] = wsum[0][0] + wsum[0][1] + wsum[0][2] + wsum[0][3];
        c.group_eq[blockIdx.x] = wsum[1][0] + wsum[1][1] + wsum[1][2] + wsum[1][3];
    }
}

// The exact threshold T of a segment and the number m of its ties to keep, selected among the gathered keys by every workgroup of
// k_emit for itself, and what lies before the workgroup's tiles: as a launch of its own between k_gather and k_emit (one workgroup per segment,
// which also completed the per-tile counts and scanned the groups' sums) it was a link more in the chain:
// flat 1 M elements 42.0 -> 37.7 us a call, ResNet-50 96.5 -> 91.0, GPT-2 small 300.4 -> 294.8, GPT-2 XL 3263 -> 3255.
// All gathered keys lie in one fine bin, so the select runs on (key - first key of the bin).
struct Picked {
    uint32_t T, m;
    uint32_t gt_before, eq_before;               // keys above T and equal to T in the segment's groups before this one
    uint32_t full;                               // 1: not to be decided here, the segment goes the full way
};
constexpr uint32_t kFewPicks = 512;              // keys that one wave selects among, in registers; 256 of them requested ahead

// By the first wave, among ng <= 64 R keys held by its lanes (row r: lane l holds key 64 r + l): bit by bit from the top, the
// keys still in question are a bit each.
template <int R>
__device__ __forceinline__ void pick_few(const uint32_t* key, const int32_t* tile, uint32_t ng, uint32_t base, int bits,
                                         uint32_t krem, int32_t tile0, int32_t tiles, Picked& out, uint32_t* own_gt, uint32_t* own_eq) {
    const int lane = ld_lane();
    uint64_t in[R];
#pragma unroll
    for (int r = 0; r < R; ++r) in[r] = __ballot(static_cast<uint32_t>(r * LD_WAVE + lane) < ng);
    uint32_t rel = 0;
#pragma unroll 1
    for (int b = bits - 1; b >= 0; --b) {
        uint64_t one[R];
        uint32_t ones = 0;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            one[r] = in[r] & __ballot((key[r] - base) >> b & 1u);
            ones += __popcll(one[r]);
        }
        const bool up = ones >= krem;
        if (up) rel |= 1u << b; else krem -= ones;
#pragma unroll
        for (int r = 0; r < R; ++r) in[r] = up ? one[r] : in[r] & ~one[r];
    }
    const uint32_t T = base + rel;
    uint32_t gt = 0, eq = 0;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const bool have = static_cast<uint32_t>(r * LD_WAVE + lane) < ng, above = have && key[r] > T, tie = have && key[r] == T;
        gt += __popcll(__ballot(above && tile[r] < tile0));
        eq += __popcll(__ballot(tie && tile[r] < tile0));
        const uint32_t t = static_cast<uint32_t>(tile[r] - tile0);
        if ((above || tie) && t < static_cast<uint32_t>(tiles)) atomicAdd((above ? own_gt : own_eq) + t, 1u);
    }
    if (lane == 0) out = Picked{T, krem, gt, eq, 0u};
}

// body(key, position) for every key of a list, eight of a thread requested together.
template <class Body>
__device__ __forceinline__ void for_keys(const uint32_t* __restrict__ gkey, uint32_t ng, Body&& body) {
    constexpr int kAhead = 8;
#pragma unroll 1
    for (uint32_t p0 = 0; p0 < ng; p0 += kAhead * kThreads) {
        uint32_t key[kAhead];
#pragma unroll
        for (int i = 0; i < kAhead; ++i) {
            const uint32_t p = p0 + i * kThreads + threadIdx.x;
            key[i] = gkey[p < ng ? p : ng - 1];
        }
#pragma unroll
        for (int i = 0; i < kAhead; ++i) {
            const uint32_t p = p0 + i * kThreads + threadIdx.x;
            if (p < ng) body(key[i], p);
        }
    }
}

// The threshold by the whole workgroup, among more keys, whole or (ng > gcap) more than the list holds. lh: kBins words. Ends with a
// barrier; every thread gets the result.
__device__ __attribute__((noinline)) Picked select_many(const uint32_t* gkey, uint32_t ng, uint32_t gcap, uint32_t kmin, uint32_t kmax,
                                                        uint32_t krem, uint32_t* lh, uint32_t* sh, uint32_t* res) {
    // More keys in the threshold bin than the list holds: if they are all one value (massive
    // ties: a frozen layer's zeros, values on a coarse grid) nothing has to be selected among
    // them: T is that value, and the rank left inside the bin is the number of ties to keep,
    // lowest index first. k_gather's per-tile counts of the bin are then the tie counts.
    if (threadIdx.x == 0) { res[0] = ng > gcap ? kmin : 0xFFFFFFFFu; res[1] = ng > gcap ? kmax : 0u; }
    __syncthreads();
    uint32_t lmin = 0xFFFFFFFFu, lmax = 0;
    for_keys(gkey, ng > gcap ? gcap : ng, [&](uint32_t key, uint32_t) {
        lmin = umin(lmin, key);
        lmax = key > lmax ? key : lmax;
    });
    atomicMin(&res[0], lmin);
    atomicMax(&res[1], lmax);
    __syncthreads();
    const uint32_t base = res[0], range = res[1] - base;
    __syncthreads();
    if (range == 0) return Picked{base, krem, 0u, 0u, 0u};
    if (ng > gcap) return Picked{base, krem, 0u, 0u, 1u};  // several values share an overfull bin: full
    const int bits = 32 - __builtin_clz(range);
    const int nlev = (bits + 10) / 11;  // one 11-bit radix level per 11 bits between the least and the largest
    uint32_t prefix = 0;
#pragma unroll 1
    for (int lev = 0; lev < nlev; ++lev) {
        const int shift = 11 * (nlev - 1 - lev);
        for (int b = threadIdx.x; b < kBins; b += kThreads) lh[b] = 0;
        __syncthreads();
        for_keys(gkey, ng, [&](uint32_t key, uint32_t) {
            const uint32_t rel = key - base;
            if (lev == 0 || ((rel ^ prefix) >> (shift + 11)) == 0) atomicAdd(&lh[(rel >> shift) & 0x7FFu], 1u);
        });
        __syncthreads();
        find_bin<kThreads, false>(lh, krem, sh, res);
        prefix |= res[0] << shift;
        krem = res[1];
        __syncthreads();
    }
    return Picked{base + prefix, krem, 0u, 0u, 0u};
}

// As pick_few, by the whole workgroup.
__device__ __attribute__((noinline)) void pick_many(const uint32_t* gkey, const int32_t* gtile, uint32_t ng, uint32_t gcap,
                                                    uint32_t kmin, uint32_t kmax, uint32_t krem, int32_t tile0, int32_t tiles,
                                                    Picked* out, uint32_t* own_gt, uint32_t* own_eq, uint32_t* lh, uint32_t* sh,
                                                    uint32_t* res) {
    const Picked x = select_many(gkey, ng, gcap, kmin, kmax, krem, lh, sh, res);
    if (threadIdx.x == 0) *out = x;
    __syncthreads();
    if (ng > gcap) return;
    uint32_t gt = 0, eq = 0;
    for_keys(gkey, ng, [&](uint32_t key, uint32_t p) {
        if (key < x.T) return;
        const int32_t tile = gtile[p];
        if (tile < tile0) ++(key > x.T ? gt : eq);
        else if (tile < tile0 + tiles) atomicAdd((key > x.T ? own_gt : own_eq) + (tile - tile0), 1u);
    });
    if (gt) atomicAdd(&out->gt_before, gt);
    if (eq) atomicAdd(&out->eq_before, eq);
    __syncthreads();
}

// Segments up to which k_emit's workgroups select for themselves. A larger one has more keys in the threshold bin than a wave
// selects among, and more groups before its last: one workgroup per segment does all that ahead of k_emit then (k_select). With small
// groups the line is where the segment's workgroups no longer all run at once and begin another round of reading the list (1024 of
// them, 67 M elements). us per call with / without that launch, small groups, one segment of 60 M elements 190 / 180, 70 M 213 / 210, 80 M
// 235 / 236, 99 M 281 / 283, at 5 % of values rounded to fp16 221 / 228, 250 / 269, 276 / 295, 332 / 361. Large groups: 140 M 365 / 366,
// at 5 % 434 / 425, of values rounded to fp16 579 / 594, 230 M 907 / 973, 400 M 916 / 915 and 1499 / 1609; ten of 80 M 1698 / 1708, at 5 %
// 2030 / 2021 and 2277 / 2334; GPT-2 XL, up to 80 M a segment, 3263 / 3255.
constexpr int64_t kOwnPick = 100000000, kOwnPickSmall = 65000000;

// One workgroup per segment: threshold and ties; per-tile counts completed; group sums scanned into output offsets.
__global__ __launch_bounds__(kThreads) void k_select(Ctx c) {
    __shared__ uint32_t lh[kBins];
    __shared__ uint32_t sh[kWaves];
    __shared__ uint32_t res[3];
    __shared__ uint32_t list0;
    const SegDesc d = c.desc[blockIdx.x];
    if (d.k == 0 || c.desc[blockIdx.x + 1].group0 == d.group0) return;
    const GroupRange gr = group_range(c, d.group0);
    SegState* st = c.state + gr.seg;
    const uint32_t mode = st->mode;
    if (mode == kModeFull) return;
    const uint32_t ng = st->gcount;
    const uint32_t* gkey = c.gkey + gather_first(gr.seg, gr.lo);
    const int32_t* gtile = c.gtile + gather_first(gr.seg, gr.lo);
    const uint32_t gcap = gather_cap(gr.lo, gr.hi);
    Picked x{st->prefix, st->krem, 0u, 0u, 0u};  // kModeTies: both were found with the threshold bin
    uint32_t seen = 0;
    if (mode != kModeTies) {
        x = select_many(gkey, ng, gcap, st->kmin, st->kmax, x.m, lh, sh, res);
        if (x.full) {
            mark_full(c, st, gr, &list0);
            return;
        }
        // k_gather counted every key of the bin as a tie: move those above T to the counts of the
        // selected, drop those below. The group sums are read back below by this same workgroup.
        // The updates return their old value, so each has been performed when its result arrives;
        // with the barrier that orders them before the reads. (A device-scope fence would do too,
        // but it writes back the whole L2 and costs 30 us here.)
        if (ng <= gcap)
            for_keys(gkey, ng, [&](uint32_t key, uint32_t p) {
                if (key == x.T) return;
                const int32_t tile = gtile[p];
                atomicSub(c.tile_eq + tile, 1u);
                seen |= atomicSub(c.group_eq + tile / c.tiles, 1u);
                if (key > x.T) {
                    atomicAdd(c.tile_gt + tile, 1u);
                    seen |= atomicAdd(c.group_gt + tile / c.tiles, 1u);
                }
            });
    }
    if (seen == 0xFFFFFFFFu) res[0] = seen;  // never true: keeps the results, and so the waits, alive
    __syncthreads();
    // exclusive scan over the segment's groups: records emitted / ties seen before each
    uint32_t carry_out = 0, carry_eq = 0;
#pragma unroll 1
    for (int32_t q0 = 0; q0 < gr.ngroup; q0 += kThreads) {
        const int32_t q = q0 + threadIdx.x;
        uint32_t cg = 0, ce = 0;
        if (q < gr.ngroup) {
            cg = ld_load_coherent(c.group_gt + gr.group0 + q);
            ce = ld_load_coherent(c.group_eq + gr.group0 + q);
        }
        uint32_t te, tg;
        const uint32_t eq_before = carry_eq + block_escan<kThreads>(ce, sh, te);
        const uint32_t take = umin(eq_before + ce, x.m) - umin(eq_before, x.m);  // ties kept: lowest index first
        const uint32_t out_before = carry_out + block_escan<kThreads>(cg + take, sh, tg);
        if (q < gr.ngroup) {
            c.group_gt[gr.group0 + q] = out_before;
            c.group_eq[gr.group0 + q] = eq_before;
        }
        carry_eq += te;
        carry_out += tg;
    }
    if (mode == kModeTies && carry_eq < x.m) {
        mark_full(c, st, gr, &list0);  // the repeated key does not fill k either: the threshold lies below it
        return;
    }
    if (threadIdx.x == 0) { st->prefix = x.T; st->krem = x.m; }
}

// Ordered emission of the records. k_main left +0 in the residual exactly where a
// stored candidate's key reaches T_est; only where that guess and the selection
// differ is the residual written again. A segment handed to the full path gets
// every pre-zeroed position back instead.
// OWN: the threshold is selected here. Four waves per SIMD: the selection's registers would leave three (GPT-2 XL 3225 us a call, so
// 3217; one segment of 60 M at 5 and 10 % 224 and 249 / 218 and 243); five spill them (3276). But large groups of tiles of 32 and 64 lanes,
// denser than 1.2 %, take 158 registers without the selection, and forced into 128 spill 20 to 32 of them: three waves there (20 segments of
// 60 M at 2 and 5 % 2729 and 3062 -> 2659 and 3035 us, 400 M at 5 % 1108 -> 1080, 160 M at 5 % 485 -> 477).
template <class RW>
constexpr int kEmitWaves = RW::kSmall || RW::kRow == 16 ? 4 : 3;

template <class RW, bool OWN>
__global__ __launch_bounds__(kThreads, kEmitWaves<RW>) void k_emit(float* __restrict__ r, int32_t* __restrict__ out_idx,
                                                   float* __restrict__ out_val, Ctx c) {
    __shared__ uint32_t tile_out[RW::kGroupTiles], tile_eqb[RW::kGroupTiles], tile_take[RW::kGroupTiles];
    __shared__ uint32_t own_gt[RW::kGroupTiles], own_eq[RW::kGroupTiles];  // gathered keys of the group's tiles: above T, equal to T
    __shared__ Picked picked;
    __shared__ uint32_t sums[3][kWaves], sh[kWaves], res[3], list0;
    constexpr int ROW = RW::kRow, kTiles = RW::kTiles, kTilesPerWave = RW::kTilesPerWave;
    constexpr uint32_t kFast = RW::kFast;
    __shared__ int32_t stage_i[kWaves][kTiles * kFast];
    __shared__ float stage_v[kWaves][kTiles * kFast];
    static_assert(sizeof(stage_i) >= kBins * 4, "a histogram in stage_i");
    const int lane = ld_lane();
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    uint32_t mycnt = wave_counts<RW>(c, blockIdx.x);
    const GroupRange gr = group_range(c, blockIdx.x);
    TripRaw raw[RW::kAhead];
    first_trips<true, RW>(c, blockIdx.x * RW::kGroupTiles + w * kTilesPerWave, mycnt, raw);
    SegState* st = c.state + gr.seg;
    if (gr.k == 0) return;
    uint32_t mode = st->mode;
    const uint32_t ng = st->gcount, bin = st->prefix, krem = st->krem;
    const uint32_t tau = gr.tau, test = gr.test;
    const int tl0 = w * kTilesPerWave;
    const int32_t group_tile0 = blockIdx.x * RW::kGroupTiles, tile0 = group_tile0 + tl0;
    int64_t tbase = 0;
    if (!OWN && mode != kModeFull) {
        if (w == 0) {  // offsets of the group's tiles
            const int32_t tile = group_tile0 + lane;
            const bool live = lane < RW::kGroupTiles && gr.base + static_cast<int64_t>(lane) * kTile < gr.hi;
            const uint32_t cg = live ? c.tile_gt[tile] : 0u, ce = live ? c.tile_eq[tile] : 0u;
            const uint32_t eq_before = c.group_eq[blockIdx.x] + ld_wave_iscan(ce) - ce;
            const uint32_t take = umin(eq_before + ce, krem) - umin(eq_before, krem);
            const uint32_t out_before = c.group_gt[blockIdx.x] + ld_wave_iscan(cg + take) - (cg + take);
            if (lane < RW::kGroupTiles) {
                tile_out[lane] = out_before;
                tile_eqb[lane] = eq_before;
                tile_take[lane] = take;
            }
        }
        __syncthreads();
    }
    if (OWN && mode != kModeFull) {
        // The first wave selects, the others add up what the segment's groups before this one count: keys above the
        // threshold bin, and where ties are counted per tile (kModeTies, an overfull bin) those too, before this group and in all.
        const uint32_t* gkey = c.gkey + gather_first(gr.seg, gr.lo);
        const int32_t* gtile = c.gtile + gather_first(gr.seg, gr.lo);
        const uint32_t gcap = gather_cap(gr.lo, gr.hi);
        const bool counted = mode == kModeTies || ng > gcap;  // uniform, as is what follows
        if (w == 0) {
            constexpr int kRows = kFewPicks / LD_WAVE;
            uint32_t key[kRows];
            int32_t tile[kRows];
#pragma unroll
            for (int i = 0; i < kRows / 2; ++i) {  // whatever the list holds there: it is longer
                key[i] = gkey[i * LD_WAVE + lane];
                tile[i] = gtile[i * LD_WAVE + lane];
            }
            static_assert(kGatherBase > kFewPicks, "");
            if (lane < RW::kGroupTiles) own_gt[lane] = own_eq[lane] = 0;
            const uint32_t base = tau + (bin << gr.sh);
            const int bits = bin == static_cast<uint32_t>(kTopBin) ? 31 : static_cast<int>(gr.sh);  // the top bin is open-ended
            if (mode == kModeTies) {  // both were found with the threshold bin: nothing to select
                if (lane == 0) picked = Picked{bin, krem, 0u, 0u, 0u};
            } else if (ng <= LD_WAVE) {
                pick_few<1>(key, tile, ng, base, bits, krem, group_tile0, RW::kGroupTiles, picked, own_gt, own_eq);
            } else if (ng <= kFewPicks / 2) {
                pick_few<kRows / 2>(key, tile, ng, base, bits, krem, group_tile0, RW::kGroupTiles, picked, own_gt, own_eq);
            } else if (ng <= kFewPicks) {
#pragma unroll
                for (int i = kRows / 2; i < kRows; ++i) {
                    key[i] = gkey[i * LD_WAVE + lane];
                    tile[i] = gtile[i * LD_WAVE + lane];
                }
                pick_few<kRows>(key, tile, ng, base, bits, krem, group_tile0, RW::kGroupTiles, picked, own_gt, own_eq);
            }
        } else {
            uint32_t gt = 0, eq = 0, all = 0;
            const int32_t before = static_cast<int32_t>(blockIdx.x) - gr.group0, upto = counted ? gr.ngroup : before;
#pragma unroll 4
            for (int32_t q = (w - 1) * LD_WAVE + lane; q < upto; q += (kWaves - 1) * LD_WAVE) {
                if (q < before) gt += c.group_gt[gr.group0 + q];
                if (counted) {
                    const uint32_t x = c.group_eq[gr.group0 + q];
                    all += x;
                    eq += q < before ? x : 0u;
                }
            }
            gt = ld_wave_sum(gt), eq = ld_wave_sum(eq), all = ld_wave_sum(all);
            if (lane == 0) { sums[0][w] = gt; sums[1][w] = eq; sums[2][w] = all; }
        }
        __syncthreads();
        if (mode == kModeCand && ng > kFewPicks)
            pick_many(gkey, gtile, ng, gcap, st->kmin, st->kmax, krem, group_tile0, RW::kGroupTiles, &picked, own_gt, own_eq,
                      reinterpret_cast<uint32_t*>(stage_i), sh, res);
        if (w == 0) {  // offsets of the group's tiles
            const Picked p = picked;
            const uint32_t m = p.m;
            const int32_t tile = group_tile0 + lane;
            const bool live = lane < RW::kGroupTiles && gr.base + static_cast<int64_t>(lane) * kTile < gr.hi;
            const uint32_t cg = live ? c.tile_gt[tile] + (counted ? 0u : own_gt[lane]) : 0u;
            const uint32_t ce = live ? (counted ? c.tile_eq[tile] : own_eq[lane]) : 0u;
            const uint32_t eq0 = counted ? sums[1][1] + sums[1][2] + sums[1][3] : p.eq_before;
            const uint32_t eq_before = eq0 + ld_wave_iscan(ce) - ce;
            const uint32_t take = umin(eq_before + ce, m) - umin(eq_before, m);  // ties kept: lowest index first
            const uint32_t out0 = sums[0][1] + sums[0][2] + sums[0][3] + p.gt_before + umin(eq0, m);
            const uint32_t out_before = out0 + ld_wave_iscan(cg + take) - (cg + take);
            if (lane < RW::kGroupTiles) {
                tile_out[lane] = out_before;
                tile_eqb[lane] = eq_before;
                tile_take[lane] = take;
            }
            // the repeated key does not fill k either: the threshold lies below it
            if (lane == 0 && mode == kModeTies && sums[2][1] + sums[2][2] + sums[2][3] < m) picked.full = 1;
        }
        __syncthreads();
    }
    if (mode == kModeFull || (OWN && picked.full)) {
        // handed to the full path: every pre-zeroed position back; the segment's first workgroup lists it, if k_gather's has not
        if (static_cast<int32_t>(blockIdx.x) == gr.group0) {
            for (int b = threadIdx.x; b < kBins; b += kThreads) c.hist[static_cast<int64_t>(gr.seg) * kBins + b] = 0;  // used again there
            // (not in `mode`: a wave that read it so would leave before the others have its part of the sums)
            if (OWN && mode != kModeFull) mark_full(c, st, gr, &list0, true);
        }
        for_trips<true, RW>(c, tile0, mycnt, raw, [&](const Trip& Q, int) {
            float* rt = r + gr.base + static_cast<int64_t>(tl0 + Q.u) * kTile;
#pragma unroll
            for (int j = 0; j < kPerLane; ++j)
                if (static_cast<uint32_t>(j) < Q.have && ld_key(Q.v[j]) >= test) rt[Q.x[j]] = Q.v[j];
        });
        slow_tiles<true, RW>(
            c, r, gr, blockIdx.x, mycnt, tau,
            [&](int u) { tbase = gr.base + static_cast<int64_t>(tl0 + u) * kTile; },
            [&](bool have, float v, uint32_t local, bool stored) {
                if (have && stored && ld_key(v) >= test) r[tbase + local] = v;
            },
            [](int) {});
        return;
    }
    const uint32_t T = OWN ? picked.T : bin, m = OWN ? picked.m : krem;  // (k_select's, where the bin and its rank were)
    // kModeTies: the ties are not among the stored candidates. A tile that keeps some of them is
    // read back from the residual (nothing was pre-zeroed in a tied segment), where candidates and
    // ties come in index order; keys at or above T pass the filter there.
    const uint32_t keep_from = mode == kModeTies ? T : tau;
    if (mode == kModeTies && lane < kTilesPerWave && tile_take[tl0 + lane] > 0) mycnt = kOverflow;
    for_trips<true, RW>(c, tile0, mycnt, raw, [&](const Trip& Q, int q) {
        const uint32_t out_tile = tile_out[tl0 + Q.u], eq_tile = tile_eqb[tl0 + Q.u];
        uint32_t gtm = 0, eqm = 0;
#pragma unroll
        for (int j = 0; j < kPerLane; ++j) {
            const uint32_t key = ld_key(Q.v[j]);
            const bool valid = static_cast<uint32_t>(j) < Q.have;
            gtm |= static_cast<uint32_t>(valid && key > T) << j;
            eqm |= static_cast<uint32_t>(valid && key == T) << j;
        }
        const uint32_t mine = __popc(gtm) | (__popc(eqm) << 16);  // a tile holds at most 512 here
        const uint32_t before = ld_row_iscan<ROW>(mine) - mine;
        uint32_t gt_before = before & 0xFFFFu;
        uint32_t eq_rank = eq_tile + (before >> 16);
        float* rt = r + gr.base + static_cast<int64_t>(tl0 + Q.u) * kTile;
        const int32_t e0 = static_cast<int32_t>(gr.base + static_cast<int64_t>(tl0 + Q.u) * kTile);
        // the records of a row's tile are staged in LDS at their rank inside the tile and then
        // written out as contiguous runs (stores of single records from scattered lanes cost
        // three times as much)
        int32_t* si = stage_i[w] + (lane / ROW) * kFast;
        float* sv = stage_v[w] + (lane / ROW) * kFast;
        uint32_t rank = 0;
#pragma unroll
        for (int j = 0; j < kPerLane; ++j) {
            const bool is_gt = (gtm >> j) & 1u, is_eq = (eqm >> j) & 1u;
            const bool selected = is_gt || (is_eq && eq_rank < m);
            rank = gt_before + (umin(eq_rank, m) - umin(eq_tile, m));
            if (selected) {
                si[rank] = e0 + static_cast<int32_t>(Q.x[j]);
                sv[rank] = Q.v[j];
            }
            const bool zeroed = ld_key(Q.v[j]) >= test;
            if (static_cast<uint32_t>(j) < Q.have && selected != zeroed) rt[Q.x[j]] = selected ? 0.0f : Q.v[j];
            gt_before += is_gt;
            eq_rank += is_eq;
        }
        rank = gt_before + (umin(eq_rank, m) - umin(eq_tile, m));  // in a row's last lane: records of the tile
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
#pragma unroll
        for (int row = 0; row < kTiles; ++row) {
            const uint32_t cnt = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(rank), row * ROW + ROW - 1));
            const int64_t o0 = gr.out0 + tile_out[tl0 + kTiles * q + row];
            for (uint32_t i = lane; i < cnt; i += LD_WAVE) {
                // streamed past the caches: the records are read much later, by another call
                __builtin_nontemporal_store(stage_i[w][row * kFast + i], out_idx + o0 + i);
                __builtin_nontemporal_store(stage_v[w][row * kFast + i], out_val + o0 + i);
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    });
    uint32_t run_out = 0;  // records of the segment emitted before this point
    uint32_t run_eq = 0;   // ties seen before this point
    slow_tiles<true, RW>(
        c, r, gr, blockIdx.x, mycnt, keep_from,
        [&](int u) {
            run_out = tile_out[tl0 + u];
            run_eq = tile_eqb[tl0 + u];
            tbase = gr.base + static_cast<int64_t>(tl0 + u) * kTile;
        },
        [&](bool have, float v, uint32_t local, bool stored) {
            const uint32_t key = ld_key(v);
            const bool is_gt = have && key > T;
            const bool is_eq = have && key == T;
            const uint64_t mg = __ballot(is_gt), me = __ballot(is_eq);
            const uint32_t eq_rank = run_eq + ld_mbcnt(me);
            const bool selected = is_gt || (is_eq && eq_rank < m);
            const int64_t e = tbase + local;
            if (selected) {
                const int64_t pos = gr.out0 + run_out + ld_mbcnt(mg) + (umin(eq_rank, m) - umin(run_eq, m));
                out_idx[pos] = static_cast<int32_t>(e);
                out_val[pos] = v;
            }
            const bool zeroed = stored && key >= test;
            if (have && selected != zeroed) r[e] = selected ? 0.0f : v;
            const uint32_t eq_end = run_eq + __popcll(me);
            run_out += __popcll(mg) + (umin(eq_end, m) - umin(run_eq, m));
            run_eq = eq_end;
        },
        [](int) {});
}

// ------------------------------------------ full-segment path (kModeFull only)
// Plain three-level radix select over every element of the listed groups.

struct FullRange { GroupRange gr; int64_t cs, ce; };

__device__ __forceinline__ FullRange full_range(const Ctx& c, int32_t g) {
    FullRange f;
    f.gr = group_range(c, g);
    f.cs = f.gr.base < f.gr.lo ? f.gr.lo : f.gr.base;
    const int64_t ge = f.gr.base + static_cast<int64_t>(c.tiles) * kTile;
    f.ce = ge > f.gr.hi ? f.gr.hi : ge;
    return f;
}

template <int LEVEL>
__device__ __forceinline__ void full_level(const float* __restrict__ r, const Ctx& c, uint32_t nlist, uint32_t* lh,
                                           uint32_t* sh, uint32_t* res) {
    constexpr int match_shift = (LEVEL == 1) ? 31 : (LEVEL == 2 ? kShift1 : kShift2);
    constexpr int digit_shift = (LEVEL == 1) ? kShift1 : (LEVEL == 2 ? kShift2 : 0);
    constexpr uint32_t digit_mask = (LEVEL == 3) ? 0x1FFu : 0x7FFu;
    for (uint32_t li = blockIdx.x; li < nlist; li += gridDim.x) {
        const FullRange fr = full_range(c, c.fail_groups[li]);
        SegState* st = c.state + fr.gr.seg;
        const uint32_t prefix = (LEVEL == 1) ? 0u : st->prefix;
        const uint32_t krem = (LEVEL == 1) ? static_cast<uint32_t>(fr.gr.k) : st->krem;
        for (int b = threadIdx.x; b < kBins; b += kThreads) lh[b] = 0;
        __syncthreads();
        for (int64_t t = fr.gr.base; t < fr.ce; t += kThreads * 4) {
            float x[4];
            const uint32_t mask = load4(r, t + threadIdx.x * 4, fr.cs, fr.ce, x);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const uint32_t key = ld_key(x[q]);
                if (((mask >> q) & 1u) && (key >> match_shift) == (prefix >> match_shift))
                    atomicAdd(&lh[(key >> digit_shift) & digit_mask], 1u);
            }
        }
        __syncthreads();
        uint32_t* h = c.hist + static_cast<int64_t>(fr.gr.seg) * kBins;
        flush_hist(h, lh);
        if (last_block(&st->fdone[LEVEL - 1], static_cast<uint32_t>(fr.gr.ngroup))) {
            find_bin<kThreads, true>(h, krem, sh, res);
            for (int b = threadIdx.x; b < kBins; b += kThreads) h[b] = 0;
            if (threadIdx.x == 0) {
                st->prefix = prefix | (res[0] << digit_shift);
                st->krem = res[1];
            }
        }
        __syncthreads();
    }
}

__device__ __forceinline__ void full_count(const float* __restrict__ r, const Ctx& c, uint32_t nlist, uint32_t* sh) {
    for (uint32_t li = blockIdx.x; li < nlist; li += gridDim.x) {
        const int32_t g = c.fail_groups[li];
        const FullRange fr = full_range(c, g);
        SegState* st = c.state + fr.gr.seg;
        const uint32_t T = st->prefix, m = st->krem;
        uint32_t gt = 0, eq = 0;
        for (int64_t t = fr.gr.base; t < fr.ce; t += kThreads * 4) {
            float x[4];
            const uint32_t mask = load4(r, t + threadIdx.x * 4, fr.cs, fr.ce, x);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const uint32_t key = ld_key(x[q]);
                if ((mask >> q) & 1u) { gt += (key > T); eq += (key == T); }
            }
        }
        uint32_t tot_gt, tot_eq;
        block_escan<kThreads>(gt, sh, tot_gt);
        block_escan<kThreads>(eq, sh, tot_eq);
        if (threadIdx.x == 0) { c.group_gt[g] = tot_gt; c.group_eq[g] = tot_eq; }
        if (last_block(&st->fdone[3], static_cast<uint32_t>(fr.gr.ngroup))) {
            uint32_t carry_out = 0, carry_eq = 0;
            for (int32_t q0 = 0; q0 < fr.gr.ngroup; q0 += kThreads) {
                const int32_t q = q0 + threadIdx.x;
                uint32_t cg = 0, ce = 0;
                if (q < fr.gr.ngroup) {
                    cg = ld_load_coherent(c.group_gt + fr.gr.group0 + q);
                    ce = ld_load_coherent(c.group_eq + fr.gr.group0 + q);
                }
                uint32_t te, tg;
                const uint32_t eq_before = carry_eq + block_escan<kThreads>(ce, sh, te);
                const uint32_t take = umin(eq_before + ce, m) - umin(eq_before, m);
                const uint32_t out_before = carry_out + block_escan<kThreads>(cg + take, sh, tg);
                if (q < fr.gr.ngroup) {
                    c.group_gt[fr.gr.group0 + q] = out_before;
                    c.group_eq[fr.gr.group0 + q] = eq_before;
                }
                carry_eq += te;
                carry_out += tg;
            }
        }
        __syncthreads();
    }
}

__device__ __forceinline__ void full_emit(float* __restrict__ r, int32_t* __restrict__ out_idx,
                                          float* __restrict__ out_val, const Ctx& c, uint32_t nlist,
                                          uint32_t (*part)[kWaves]) {  // part: packed (above | ties << 16) per wave
    const int lane = ld_lane();
    const int wv = threadIdx.x >> 6;
    for (uint32_t li = blockIdx.x; li < nlist; li += gridDim.x) {
        const int32_t g = c.fail_groups[li];
        const FullRange fr = full_range(c, g);
        const SegState* st = c.state + fr.gr.seg;
        const uint32_t T = st->prefix, m = st->krem;
        uint32_t run_out = c.group_gt[g], run_eq = c.group_eq[g];
        int buf = 0;
        // element order inside a step of 1024: (thread, component)
        for (int64_t t = fr.gr.base; t < fr.ce; t += kThreads * 4, buf ^= 1) {
            const int64_t e0 = t + threadIdx.x * 4;
            float x[4];
            const uint32_t mask = load4(r, e0, fr.cs, fr.ce, x);
            uint32_t fg = 0, fe = 0;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const uint32_t key = ld_key(x[q]);
                if ((mask >> q) & 1u) {
                    fg |= static_cast<uint32_t>(key > T) << q;
                    fe |= static_cast<uint32_t>(key == T) << q;
                }
            }
            const uint32_t cg = __popc(fg), ce = __popc(fe);
            const uint32_t inc = ld_wave_iscan(cg | (ce << 16));
            if (lane == LD_WAVE - 1) part[buf][wv] = inc;
            __syncthreads();
            uint32_t base_gt = 0, base_eq = 0, tot_gt = 0, tot_eq = 0;
#pragma unroll
            for (int u = 0; u < kWaves; ++u) {
                const uint32_t p = part[buf][u];
                if (u < wv) { base_gt += p & 0xFFFFu; base_eq += p >> 16; }
                tot_gt += p & 0xFFFFu;
                tot_eq += p >> 16;
            }
            uint32_t gt_before = base_gt + (inc & 0xFFFFu) - cg;
            uint32_t eq_rank = run_eq + base_eq + (inc >> 16) - ce;
            bool touched = false;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const bool is_gt = (fg >> q) & 1u, is_eq = (fe >> q) & 1u;
                if (is_gt || (is_eq && eq_rank < m)) {
                    const int64_t pos = fr.gr.out0 + run_out + gt_before + (umin(eq_rank, m) - umin(run_eq, m));
                    out_idx[pos] = static_cast<int32_t>(e0 + q);
                    out_val[pos] = x[q];
                    x[q] = 0.0f;
                    touched = true;
                }
                gt_before += is_gt;
                eq_rank += is_eq;
            }
            if (touched) store4(r, e0, mask, x);
            const uint32_t eq_end = run_eq + tot_eq;
            run_out += tot_gt + (umin(eq_end, m) - umin(run_eq, m));
            run_eq = eq_end;
        }
        __syncthreads();
    }
}

// Barrier across the grid of k_full: every workgroup adds one arrival and waits until `target`
// have come. Needs every workgroup of the grid resident at once (the host sizes the grid for
// that). The wait is bounded: a workgroup that has polled kSpinLimit times (seconds; a barrier
// takes microseconds) raises the give-up flag, and every workgroup that sees the flag leaves the
// kernel, so the grid always drains. Returns false when the kernel is to be left.
constexpr uint32_t kSpinLimit = 1u << 21;

__device__ __forceinline__ bool grid_barrier(uint32_t* sync, uint32_t target) {
    __shared__ uint32_t go;
    __syncthreads();
    if (threadIdx.x == 0) {
        __hip_atomic_fetch_add(sync + kSyncArrived, 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
        uint32_t ok = 1, spins = 0;
        while (__hip_atomic_load(sync + kSyncArrived, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_AGENT) < target) {
            if (__hip_atomic_load(sync + kSyncGaveUp, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0 ||
                ++spins > kSpinLimit) {
                __hip_atomic_store(sync + kSyncGaveUp, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                ok = 0;
                break;
            }
            __builtin_amdgcn_s_sleep(64);
        }
        go = ok;
    }
    __syncthreads();
    const bool ok = go != 0;
    if (ok) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    __syncthreads();
    return ok;
}

// The whole full-segment path in one launch: nothing listed (the usual case), nothing done.
__global__ __launch_bounds__(kThreads) void k_full(float* __restrict__ r, int32_t* __restrict__ out_idx,
                                                   float* __restrict__ out_val, Ctx c) {
    __shared__ uint32_t lh[kBins];
    __shared__ uint32_t sh[kWaves];
    __shared__ uint32_t res[3];
    __shared__ uint32_t part[2][kWaves];
    const uint32_t nlist = c.fail_count[kSyncCount];
    if (nlist == 0) return;
    full_level<1>(r, c, nlist, lh, sh, res);
    if (!grid_barrier(c.fail_count, 1 * gridDim.x)) return;
    full_level<2>(r, c, nlist, lh, sh, res);
    if (!grid_barrier(c.fail_count, 2 * gridDim.x)) return;
    full_level<3>(r, c, nlist, lh, sh, res);
    if (!grid_barrier(c.fail_count, 3 * gridDim.x)) return;
    full_count(r, c, nlist, sh);
    if (!grid_barrier(c.fail_count, 4 * gridDim.x)) return;
    full_emit(r, out_idx, out_val, c, nlist, part);
}

// ---------------------------------------------------------------- host side

struct Layout {
    size_t desc, gdesc, state, hist, cnt, cval, cidx, tile_gt, tile_eq, group_gt, group_eq, gkey, gtile,
        fail_groups, fail_count, total;
};

Layout layout(int32_t n_seg, int64_t n_group, int32_t tiles, int32_t slot) {
    Layout L;
    size_t o = 0;
    const size_t ns = static_cast<size_t>(n_seg), ng = static_cast<size_t>(n_group), nt = ng * static_cast<size_t>(tiles);
    auto take = [&](size_t bytes) { const size_t at = o; o += ld_round_up(bytes, 256); return at; };
    L.desc = take(sizeof(SegDesc) * (ns + 1));
    L.gdesc = take(sizeof(GroupDesc) * ng);
    L.state = take(sizeof(SegState) * ns);
    L.hist = take(sizeof(uint32_t) * kBins * ns);
    L.cnt = take(4 * nt);
    L.tile_gt = take(4 * nt);
    L.tile_eq = take(4 * nt);
    L.group_gt = take(4 * ng);
    L.group_eq = take(4 * ng);
    const size_t gather_entries = static_cast<size_t>(kGatherBase) * ns + nt * (kTile / kGatherPer) + 1;
    L.gkey = take(4 * gather_entries);
    L.gtile = take(4 * gather_entries);
    L.fail_groups = take(4 * ng);
    L.fail_count = take(4 * kSyncWords);
    L.cval = take(4 * nt * static_cast<size_t>(slot));  // the two arrays whose size depends on `slot` come last
    L.cidx = take(2 * nt * static_cast<size_t>(slot));
    L.total = o;
    return L;
}

// Counts groups; returns -1 on a malformed offset table.
int64_t count_groups(int32_t n_seg, const int64_t* seg_off, int32_t tiles) {
    if (n_seg < 0 || (n_seg > 0 && !seg_off)) return -1;
    if (n_seg > 0 && seg_off[0] != 0) return -1;
    int64_t total = 0;
    for (int32_t s = 0; s < n_seg; ++s) {
        if (seg_off[s + 1] < seg_off[s]) return -1;
        total += groups_of(seg_off[s], seg_off[s + 1], tiles);
    }
    return total;
}

// How a segment table is cut into groups.
struct Cut {
    int32_t tiles;      // tiles per group
    int64_t n_group;    // -1: malformed table
};

// The cut that a table runs fastest with (see kSmallGroups).
Cut wanted_cut(int32_t n_seg, const int64_t* seg_off) {
    const Cut large{kTilesPerGroup, count_groups(n_seg, seg_off, kTilesPerGroup)};
    if (large.n_group < 0 || large.n_group >= kSmallGroups) return large;
    return Cut{kTilesPerSmallGroup, count_groups(n_seg, seg_off, kTilesPerSmallGroup)};
}

// Slot size that holds the candidates of a tile in all but a few tiles: the candidate threshold
// of k_prep sits at sample rank x = a + z*sqrt(x) (a = k * kSample / n_s expected hits), i.e. a
// fraction x / kSample of the elements are candidates, plus five sigmas of a tile's own count.
// Taken over the segments of at least 16 tiles (the tiles of smaller ones may overflow into the
// residual re-read: there are few of them).
int32_t wanted_slot(int32_t n_seg, const int64_t* seg_off, const int32_t* seg_k, int32_t* per_tile = nullptr) {
    double most = 0.0;
    for (int32_t s = 0; s < n_seg; ++s) {
        const int64_t ns = seg_off[s + 1] - seg_off[s];
        if (ns < 16 * kTile || seg_k[s] <= 0) continue;
        const double a = static_cast<double>(seg_k[s]) * kSample / static_cast<double>(ns);
        const double sq = 0.5 * (kSampleZ + sqrt(kSampleZ * kSampleZ + 4.0 * a));
        const double x = sq * sq + 2.0;
        if (x >= kSample) continue;  // no estimate for this segment: every element is a candidate
        const double per_tile = x * kTile / kSample;
        const double need = per_tile + 5.0 * sqrt(per_tile) + 8.0;
        if (need > most) most = need;
    }
    if (per_tile) *per_tile = static_cast<int32_t>(most);
    int64_t slot = (static_cast<int64_t>(most) + 63) / 64 * 64;
    if (slot < kSlotMin) slot = kSlotMin;
    if (slot > kSlotMax) slot = kSlotMax;
    return static_cast<int32_t>(slot);
}

size_t layout_bytes(int32_t n_seg, const Cut& cut, int32_t slot) { return layout(n_seg, cut.n_group, cut.tiles, slot).total; }

// The cut of a call with this workspace and these slots: the wanted one unless only groups of 64 fit. The
// descriptors of four times the groups make the layout of large segments in small groups up to 66 KB
// larger, so without this a workspace sized for a table just above kSmallGroups would not serve one just below it.
Cut call_cut(int32_t n_seg, const int64_t* seg_off, int32_t slot, size_t workspace_bytes) {
    const Cut cut = wanted_cut(n_seg, seg_off);
    if (cut.n_group < 0 || cut.tiles == kTilesPerGroup || workspace_bytes >= layout_bytes(n_seg, cut, slot)) return cut;
    const Cut large{kTilesPerGroup, count_groups(n_seg, seg_off, kTilesPerGroup)};
    const bool small_fits = workspace_bytes >= layout_bytes(n_seg, cut, kSlotMin);
    return workspace_bytes >= layout_bytes(n_seg, large, small_fits ? slot : kSlotMin) ? large : cut;
}

Ctx make_ctx(void* workspace, const Layout& L, int32_t n_seg, int64_t n_group, int32_t tiles, int32_t slot) {
    char* ws = static_cast<char*>(workspace);
    Ctx c;
    c.desc = reinterpret_cast<SegDesc*>(ws + L.desc);
    c.gdesc = reinterpret_cast<GroupDesc*>(ws + L.gdesc);
    c.state = reinterpret_cast<SegState*>(ws + L.state);
    c.hist = reinterpret_cast<uint32_t*>(ws + L.hist);
    c.cnt = reinterpret_cast<uint32_t*>(ws + L.cnt);
    c.cval = reinterpret_cast<float*>(ws + L.cval);
    c.cidx = reinterpret_cast<uint16_t*>(ws + L.cidx);
    c.tile_gt = reinterpret_cast<uint32_t*>(ws + L.tile_gt);
    c.tile_eq = reinterpret_cast<uint32_t*>(ws + L.tile_eq);
    c.group_gt = reinterpret_cast<uint32_t*>(ws + L.group_gt);
    c.group_eq = reinterpret_cast<uint32_t*>(ws + L.group_eq);
    c.gkey = reinterpret_cast<uint32_t*>(ws + L.gkey);
    c.gtile = reinterpret_cast<int32_t*>(ws + L.gtile);
    c.fail_groups = reinterpret_cast<int32_t*>(ws + L.fail_groups);
    c.fail_count = reinterpret_cast<uint32_t*>(ws + L.fail_count);
    c.n_seg = n_seg;
    c.n_group = static_cast<int32_t>(n_group);
    c.slot = slot;
    c.tiles = tiles;
    return c;
}

// One workgroup per segment: the path the last call took for it, and how many of its tiles
// overflowed their candidate slot.
__global__ __launch_bounds__(kThreads) void k_paths(Ctx wanted, Ctx large, int32_t* __restrict__ paths,
                                                    int32_t* __restrict__ overflowed) {
    __shared__ uint32_t sh[kWaves];
    const int32_t s = blockIdx.x;
    // the descriptors lie at the same place whatever the cut; the sentinel tells which one the call ran with
    const Ctx c = large.desc[large.n_seg].k == wanted.tiles ? wanted : large;
    const SegDesc d = c.desc[s], dn = c.desc[s + 1];
    uint32_t over = 0;
    if (d.k > 0) {
        const int64_t t0 = static_cast<int64_t>(d.group0) * c.tiles, t1 = static_cast<int64_t>(dn.group0) * c.tiles;
        for (int64_t t = t0 + threadIdx.x; t < t1; t += kThreads) over += c.cnt[t] == kOverflow;
    }
    uint32_t total;
    block_escan<kThreads>(over, sh, total);
    if (threadIdx.x == 0) {
        const SegState st = c.state[s];
        paths[s] = static_cast<int32_t>((st.late ? kModeFull : st.mode) | (st.tied ? 0x100u : 0u) |
                                        (c.fail_count[kSyncGaveUp] ? 0x10000u : 0u));
        if (overflowed) overflowed[s] = static_cast<int32_t>(total);
    }
}

// Packs the segment table for k_prep's arguments; false when it has too many segments or too
// many distinct (length, k) pairs.
bool pack_table(int32_t n_seg, const int64_t* seg_off, const int32_t* seg_k, int32_t tiles, PackedTable& pt) {
    pt.n_seg = 0;
    if (n_seg > kDictSegs) return false;
    int used = 0, last = 0;
    for (int32_t s = 0; s < n_seg; ++s) {
        const uint32_t len = static_cast<uint32_t>(seg_off[s + 1] - seg_off[s]), k = static_cast<uint32_t>(seg_k[s]);
        int code = -1;
        if (used > 0 && pt.len[last] == len && pt.k[last] == k) code = last;  // runs of equal tensors are common
        for (int d = 0; code < 0 && d < used; ++d)
            if (pt.len[d] == len && pt.k[d] == k) code = d;
        if (code < 0) {
            if (used == kDictMax) return false;
            code = used++;
            pt.len[code] = len;
            pt.k[code] = k;
        }
        pt.code[s] = static_cast<uint8_t>(code);
        last = code;
    }
    int64_t out0 = 0, group0 = 0;
    for (int32_t b = 0; b < kDictSegs / LD_WAVE; ++b) {
        const int32_t s0 = b * LD_WAVE < n_seg ? b * LD_WAVE : n_seg;
        pt.off0[b] = static_cast<uint32_t>(seg_off[s0]);
        pt.out0[b] = static_cast<uint32_t>(out0);
        pt.group0[b] = static_cast<uint32_t>(group0);
        for (int32_t s = s0; s < n_seg && s < s0 + LD_WAVE; ++s) {
            out0 += seg_k[s];
            group0 += groups_of(seg_off[s], seg_off[s + 1], tiles);
        }
    }
    for (int d = used; d < kDictMax; ++d) pt.len[d] = pt.k[d] = 0;
    for (int32_t s = n_seg; s < kDictSegs; ++s) pt.code[s] = 0;
    pt.n_seg = n_seg;
    return true;
}

void fill_direct(int32_t n_seg, const int64_t* seg_off, const int32_t* seg_k, int32_t tiles, DirectTable& dt) {
    int64_t out0 = 0, group0 = 0;
    for (int32_t s = 0; s <= n_seg; ++s) {
        const uint32_t k = s < n_seg ? static_cast<uint32_t>(seg_k[s]) : 0u;
        dt.seg[s] = DirectTable::Entry{static_cast<uint32_t>(seg_off[s]), k, static_cast<uint32_t>(out0),
                                       static_cast<uint32_t>(group0)};
        out0 += k;
        if (s < n_seg) group0 += groups_of(seg_off[s], seg_off[s + 1], tiles);
    }
    for (int32_t s = n_seg + 1; s <= kDirectSegs; ++s) dt.seg[s] = dt.seg[n_seg];
    dt.n_seg = n_seg;
}

// Workgroups of k_full that the current device keeps resident at once, halved to leave room for
// whatever else runs (looked up once per device: a property of the device and of the kernel, not
// state of a call). 0 on failure.
int32_t full_grid_limit() {
    constexpr int kMaxDevices = 64;
    static std::atomic<int32_t> limit[kMaxDevices];
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return 0;
    int32_t v = limit[dev].load(std::memory_order_acquire);
    if (v == 0) {
        int cus = 0, per_cu = 0;
        if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_full, kThreads, 0) != hipSuccess) return 0;
        if (cus <= 0 || per_cu <= 0) return 0;
        const int64_t all = static_cast<int64_t>(cus) * per_cu / 2;
        v = static_cast<int32_t>(all < 1 ? 1 : (all > kFullGrid ? kFullGrid : all));
        limit[dev].store(v, std::memory_order_release);
    }
    return v;
}

// The passes over the candidates.
template <class RW>
ld_status candidate_passes(const Ctx& c, bool own, float* residual, int32_t* out_idx, float* out_val, hipStream_t st) {
    const dim3 groups(static_cast<uint32_t>(c.n_group)), segments(static_cast<uint32_t>(c.n_seg)), block(kThreads);
    const dim3 hgroups(static_cast<uint32_t>((c.n_group + kHistGroups - 1) / kHistGroups));
    if (c.n_group <= kFewGroups) k_hist<RW, 1><<<groups, block, 0, st>>>(residual, c);
    else k_hist<RW, kHistGroups><<<hgroups, dim3(kHistGroups * kThreads), 0, st>>>(residual, c);
    if (ld_launch_status() != LD_OK) return LD_ERR_HIP;
    k_gather<RW><<<groups, block, 0, st>>>(residual, c);
    if (ld_launch_status() != LD_OK) return LD_ERR_HIP;
    if (!own) {
        k_select<<<segments, block, 0, st>>>(c);
        if (ld_launch_status() != LD_OK) return LD_ERR_HIP;
        k_emit<RW, false><<<groups, block, 0, st>>>(residual, out_idx, out_val, c);
    } else {
        k_emit<RW, true><<<groups, block, 0, st>>>(residual, out_idx, out_val, c);
    }
    return ld_launch_status();
}

}  // namespace

extern "C" size_t ld_compress_topk_workspace(int32_t n_seg, const int64_t* seg_off) {
    const Cut cut = wanted_cut(n_seg, seg_off);
    if (cut.n_group < 0) return 0;
    return layout_bytes(n_seg, cut, kSlotMin);
}

extern "C" size_t ld_compress_topk_workspace_for(int32_t n_seg, const int64_t* seg_off, const int32_t* seg_k) {
    const Cut cut = wanted_cut(n_seg, seg_off);
    if (cut.n_group < 0 || (n_seg > 0 && !seg_k)) return 0;
    return layout_bytes(n_seg, cut, wanted_slot(n_seg, seg_off, seg_k));
}

extern "C" ld_status ld_compress_topk_strategy(const float* grad, float* residual, const int64_t* seg_off,
                                               const int32_t* seg_k, int32_t n_seg, int32_t* out_idx,
                                               float* out_val, void* workspace, size_t workspace_bytes,
                                               ld_stream stream, int32_t strategy) {
    if (n_seg < 0 || (strategy != LD_COMPRESS_AUTO && strategy != LD_COMPRESS_FULL)) return LD_ERR_RANGE;
    if (n_seg == 0) return LD_OK;
    if (!seg_off || !seg_k) return LD_ERR_NULL;
    const Cut wanted = wanted_cut(n_seg, seg_off);
    if (wanted.n_group < 0 || wanted.n_group > INT32_MAX / wanted.tiles) return LD_ERR_RANGE;
    const int64_t n = seg_off[n_seg];
    if (n > INT32_MAX) return LD_ERR_RANGE;
    int64_t K = 0;
    for (int32_t s = 0; s < n_seg; ++s) {
        if (seg_k[s] < 0 || seg_k[s] > seg_off[s + 1] - seg_off[s]) return LD_ERR_RANGE;
        K += seg_k[s];
    }
    if (n == 0) return LD_OK;
    if (!grad || !residual) return LD_ERR_NULL;
    if (K > 0 && (!out_idx || !out_val)) return LD_ERR_NULL;
    if (!ld_aligned(grad, 16) || !ld_aligned(residual, 16) || !ld_aligned(out_idx, 4) ||
        !ld_aligned(out_val, 4))
        return LD_ERR_ALIGN;
    int32_t per_tile = 0;
    int32_t slot = wanted_slot(n_seg, seg_off, seg_k, &per_tile);
    const Cut cut = call_cut(n_seg, seg_off, slot, workspace_bytes);
    if (!workspace || !ld_aligned(workspace, 256) || workspace_bytes < layout_bytes(n_seg, cut, kSlotMin))
        return LD_ERR_WORKSPACE;
    const int32_t tiles = cut.tiles;
    const int64_t n_group = cut.n_group;
    // the largest slot, up to the one this call's densities ask for, that the workspace holds
    while (slot > kSlotMin && layout(n_seg, n_group, tiles, slot).total > workspace_bytes) slot -= 64;
    const Layout L = layout(n_seg, n_group, tiles, slot);

    hipStream_t st = static_cast<hipStream_t>(stream);
    const Ctx c = make_ctx(workspace, L, n_seg, n_group, tiles, slot);

    ld_begin_call();
    // The segment table travels as kernel arguments: in k_prep's own as it is when it is short, packed when
    // it has few distinct (length, k) pairs, else through k_upload launches of kSegPerLaunch segments each.
    PackedTable pt;
    if (n_seg > kDirectSegs && !pack_table(n_seg, seg_off, seg_k, tiles, pt)) {
        int64_t out0 = 0;
        int32_t group0 = 0;
        for (int32_t s0 = 0; s0 < n_seg; s0 += kSegPerLaunch) {
            UploadBatch ub;
            const int32_t cnt = (n_seg - s0) < kSegPerLaunch ? (n_seg - s0) : kSegPerLaunch;
            ub.out0 = out0;
            ub.group0 = group0;
            ub.first = s0;
            ub.count = cnt;
            ub.n_seg = n_seg;
            for (int32_t j = 0; j <= kSegPerLaunch; ++j) {
                const int32_t q = (s0 + j <= n_seg) ? (s0 + j) : n_seg;
                ub.off[j] = static_cast<int32_t>(seg_off[q]);
                if (j < kSegPerLaunch) ub.k[j] = (s0 + j < n_seg) ? seg_k[s0 + j] : 0;
            }
            for (int32_t j = 0; j < cnt; ++j) {
                out0 += seg_k[s0 + j];
                group0 += groups_of(seg_off[s0 + j], seg_off[s0 + j + 1], tiles);
            }
            k_upload<<<dim3(1), dim3(512), 0, st>>>(ub, c);
            if (ld_launch_status() != LD_OK) return LD_ERR_HIP;
        }
    }
    const dim3 sgrid(static_cast<uint32_t>(n_seg));
    const int32_t no_estimate = strategy == LD_COMPRESS_FULL ? 1 : 0;
    if (n_seg <= kDirectSegs) {
        DirectTable dt;
        fill_direct(n_seg, seg_off, seg_k, tiles, dt);
        k_prep<1024, DirectTable><<<sgrid, dim3(1024), 0, st>>>(grad, residual, c, no_estimate, dt);
    } else if (n_seg <= kPrepWide) {
        k_prep<1024, PackedTable><<<sgrid, dim3(1024), 0, st>>>(grad, residual, c, no_estimate, pt);
    } else {
        k_prep<512, PackedTable><<<sgrid, dim3(512), 0, st>>>(grad, residual, c, no_estimate, pt);
    }
    if (ld_launch_status() != LD_OK) return LD_ERR_HIP;
    if (n_group == 0) return LD_OK;
    const dim3 mgrid(static_cast<uint32_t>(n_group * tiles)), mblock(LD_WAVE);
    const bool runs = n_group * tiles >= kMainRunTiles;
    const uint32_t turn = n_group * tiles * 4 >= (n / kTile + n_seg) * kMainTurnQuarters ? 7u : 0u;
    if (slot == kSlotMin) {
        if (runs) k_main<true, 16><<<mgrid, mblock, 0, st>>>(grad, residual, c, turn);
        else k_main<true, 1><<<mgrid, mblock, 0, st>>>(grad, residual, c, turn);
    } else {
        if (runs) k_main<false, 16><<<mgrid, mblock, 0, st>>>(grad, residual, c, turn);
        else k_main<false, 1><<<mgrid, mblock, 0, st>>>(grad, residual, c, turn);
    }
    if (ld_launch_status() != LD_OK) return LD_ERR_HIP;
    if (K == 0) return LD_OK;
    // lanes per tile in the candidate passes: enough for the candidates a tile is expected to hold
    const int row = (per_tile <= 128 && slot == kSlotMin) ? 16 : (per_tile <= 256 ? 32 : 64);  // 16 implies the minimum slot
    int64_t largest = 0;
    for (int32_t s = 0; s < n_seg; ++s) largest = seg_off[s + 1] - seg_off[s] > largest ? seg_off[s + 1] - seg_off[s] : largest;
    const bool own = largest <= (tiles == kTilesPerGroup ? kOwnPick : kOwnPickSmall);
    ld_status passes;
    if (tiles == kTilesPerGroup) {
        if (row == 16) passes = candidate_passes<Rows<16, kTilesPerGroup>>(c, own, residual, out_idx, out_val, st);
        else if (row == 32) passes = candidate_passes<Rows<32, kTilesPerGroup>>(c, own, residual, out_idx, out_val, st);
        else passes = candidate_passes<Rows<64, kTilesPerGroup>>(c, own, residual, out_idx, out_val, st);
    } else {
        if (row == 16) passes = candidate_passes<Rows<16, kTilesPerSmallGroup>>(c, own, residual, out_idx, out_val, st);
        else if (row == 32) passes = candidate_passes<Rows<32, kTilesPerSmallGroup>>(c, own, residual, out_idx, out_val, st);
        else passes = candidate_passes<Rows<64, kTilesPerSmallGroup>>(c, own, residual, out_idx, out_val, st);
    }
    if (passes != LD_OK) return passes;
    // segments handed to the full path (normally none: the launch returns at once). Its grid must be
    // resident as a whole (the phases hand over through a barrier across it).
    const int32_t resident = full_grid_limit();
    if (resident <= 0) return LD_ERR_HIP;
    const dim3 fgrid(static_cast<uint32_t>(n_group < resident ? n_group : resident));
    k_full<<<fgrid, dim3(kThreads), 0, st>>>(residual, out_idx, out_val, c);
    return ld_launch_status();
}

extern "C" ld_status ld_compress_topk_paths(const void* workspace, size_t workspace_bytes, int32_t n_seg,
                                            const int64_t* seg_off, int32_t* paths, int32_t* overflowed_tiles,
                                            ld_stream stream) {
    if (n_seg < 0) return LD_ERR_RANGE;
    if (n_seg == 0) return LD_OK;
    if (!seg_off || !paths) return LD_ERR_NULL;
    const Cut wanted = wanted_cut(n_seg, seg_off);
    if (wanted.n_group < 0 || wanted.n_group > INT32_MAX / wanted.tiles) return LD_ERR_RANGE;
    if (!ld_aligned(paths, 4) || !ld_aligned(overflowed_tiles, 4)) return LD_ERR_ALIGN;
    const Cut large{kTilesPerGroup, count_groups(n_seg, seg_off, kTilesPerGroup)};
    // the slot size only moves the candidate arrays
    const Layout L = layout(n_seg, wanted.n_group, wanted.tiles, kSlotMin), G = layout(n_seg, large.n_group, large.tiles, kSlotMin);
    if (!workspace || !ld_aligned(workspace, 256) || (workspace_bytes < L.total && workspace_bytes < G.total))
        return LD_ERR_WORKSPACE;
    void* ws = const_cast<void*>(workspace);
    ld_begin_call();
    k_paths<<<dim3(static_cast<uint32_t>(n_seg)), dim3(kThreads), 0, static_cast<hipStream_t>(stream)>>>(
        make_ctx(ws, L, n_seg, wanted.n_group, wanted.tiles, kSlotMin),
        make_ctx(ws, G, n_seg, large.n_group, large.tiles, kSlotMin), paths, overflowed_tiles);
    return ld_launch_status();
}

extern "C" ld_status ld_compress_topk(const float* grad, float* residual, const int64_t* seg_off,
                                      const int32_t* seg_k, int32_t n_seg, int32_t* out_idx,
                                      float* out_val, void* workspace, size_t workspace_bytes,
                                      ld_stream stream) {
    return ld_compress_topk_strategy(grad, residual, seg_off, seg_k, n_seg, out_idx, out_val, workspace,
                                     workspace_bytes, stream, LD_COMPRESS_AUTO);
}
