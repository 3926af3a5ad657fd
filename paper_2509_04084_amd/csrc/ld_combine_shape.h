// How a combine runs, apart from its kernels so that host code can be built from it as well: the tests look there whether
// the inputs that they make for a kernel reach it.
#pragma once

#include <stdint.h>

#include "lowdiff.h"

// Shapes of the one pass (k_combine_chunk): threads x records per thread and list loaded at once, distinct positions a round.
enum LdCombineShape {
    kCombineTwoPasses,
    kCombineNarrow,  // 128 x 2, 2048
    kCombineFew,     // 192 x 3, 2304; up to kCombineHeld lists
    kCombineMiddle,  // 256 x 3, 4608
    kCombineLong,    // 256 x 4, 4608; up to kCombineHeld lists
    kCombineWide     // 512 x 3, 9152
};

constexpr int64_t kCombineChunk = 49152;  // elements per workgroup
constexpr int32_t kCombineHeld = 8;       // lists whose records a workgroup keeps in registers

// list, all: mean records of a chunk, of the longest list and of all lists. The threads hold a list's records of a chunk with
// room above their mean, and the distinct positions of a chunk fit one round. Two passes / one, us per call of 400 M elements:
// narrow 8 lists of 0.25 % 101 / 70, few 2 of 1 % 81 / 79 (1.4 G: 272 / 249) and 4 of 1 % 117 / 91, middle 8 of 1 % 179 / 157, long
// 2 of 2 % 135 / 131, wide 8 of 1.7 % 397 / 243. Large arrays with two lists of 1.7 %: two passes (117 / 129, though
// 24.6 / 21.7 at 5 M elements). Five lists and more of 0.25-0.4 % on up to 100 M elements: middle, which is as fast as narrow
// where the records are even (20 M, 8 lists of 0.35 %: 4 % slower) and takes fewer rounds where they are not (layers whose
// densities differ as a log-normal of sigma 1.5: 12 % faster).
inline LdCombineShape ld_combine_shape_held(int64_t n, int32_t N, double list, double all) {
    if (n > 100000000 && N <= 2 && list > 500) return kCombineTwoPasses;
    const double narrow = N <= 4 || n > 100000000 ? 190 : 120;
    if (list <= narrow && all <= 1850) return kCombineNarrow;
    if (list <= 500 && all <= 2100 && (N <= 4 || list > 190)) return kCombineFew;
    if (list <= 640 && all <= 4300) return kCombineMiddle;
    if (list <= 1000 && all <= 4300) return kCombineLong;
    if (list <= 1350 && all <= 17000) return kCombineWide;
    return kCombineTwoPasses;
}

// More lists: their records are read twice by the one pass too, group after group of eight with a barrier per list, so that
// threads without a record and barriers cost the more the more lists there are. Geometric means of two passes over one, of a
// sweep of 1700 even inputs: narrow 1.5 for 16 lists of up to 0.2 % on more than 100 M elements, 1.1 below 50 M; middle 1.05 up to 50 M
// (16 lists of 0.4 %) and on larger arrays 0.96 to 1 while a chunk is one round (it stays there: lists that crowd cost two passes
// up to twice as much); wide 1.3-1.9 where the lists have more than 640 records a chunk (1.3 %) and, on small arrays, whose
// workgroups all run at once, from 200 on. Elsewhere the one pass lost: middle 0.76 in two rounds, wide 0.6 to
// 0.73 with 16 to 32 lists of 0.3-0.8 % on more than 100 M elements (330 M, 12 lists of 0.8 %: two passes 186 us, one 295; 119 M, 64
// of 0.3 %: 300 / 502), 0.84 with 64 lists of 0.3 % on 30 M. Lists of very different lengths: wide 0.7, middle 0.91 to 1.2.
inline LdCombineShape ld_combine_shape_many(int64_t n, int32_t N, double list, double all) {
    const bool large = n > 50000000, one_each = n <= 12600000;  // at most a workgroup per CU
    const bool even = one_each || all >= 0.7 * N * list;
    if (list <= (!large ? 120 : N <= 12 ? 270 : 190) && all <= (large ? 3600 : 1850)) return kCombineNarrow;
    if (list > 1350 || all > 17000) return kCombineTwoPasses;
    const LdCombineShape dense = even ? kCombineWide : kCombineMiddle;
    if (N > 16) return list > (large ? 640 : N <= 32 || one_each ? 190 : 270) ? dense : kCombineTwoPasses;
    if (list <= 400 && all <= 4300) return kCombineMiddle;
    if (!large || list > 640) return dense;
    return !even || (list > 400 && N > 12 && n <= 100000000) ? kCombineMiddle : kCombineTwoPasses;
}

// most, total: records of the longest list and of all
inline LdCombineShape ld_combine_shape(int64_t n, int32_t N, int64_t most, int64_t total, int32_t strategy) {
    if (strategy == LD_COMBINE_TWO_PASSES) return kCombineTwoPasses;
    const double list = static_cast<double>(most) * kCombineChunk / static_cast<double>(n);
    const double all = static_cast<double>(total) * kCombineChunk / static_cast<double>(n);
    const LdCombineShape shape = N <= kCombineHeld ? ld_combine_shape_held(n, N, list, all) : ld_combine_shape_many(n, N, list, all);
    return shape == kCombineTwoPasses && strategy != LD_COMBINE_AUTO ? kCombineWide : shape;
}
