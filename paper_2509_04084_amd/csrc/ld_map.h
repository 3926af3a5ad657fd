// Which piece of its work a workgroup takes, apart from the kernels so that host code can be built from it as well (the maps
// are checked there for being permutations).
#pragma once

#include <stdint.h>

#ifdef __HIPCC__
#define LD_HD __host__ __device__ __forceinline__
#else
#define LD_HD inline
#endif

// The piece of work of workgroup `b` of a grid of `grid` workgroups (a multiple of 8). Consecutive
// workgroups go to the 8 XCDs in turn: every XCD is given runs of CHUNK consecutive pieces, so that
// all XCDs together walk the arrays in address order; the pieces past the last whole round of
// 8 CHUNK are dealt out in eighths.
template <uint32_t CHUNK>
LD_HD uint32_t ld_xcd_piece(uint32_t b, uint32_t grid) {
    const uint32_t whole = grid / (8u * CHUNK) * (8u * CHUNK);
    if (b < whole) {
        const uint32_t q = b / 8u;
        return q / CHUNK * (8u * CHUNK) + (b % 8u) * CHUNK + q % CHUNK;
    }
    const uint32_t rest = b - whole;
    return whole + (rest % 8u) * ((grid - whole) / 8u) + rest / 8u;
}

// The same, with `turn` = 7 the XCDs taking their runs of a round in another order every round (0: as above).
// For pieces that come in groups of 16 or 64 of which only the first few are work (small segments): unturned,
// all of that work would be one XCD's, or two's.
template <uint32_t CHUNK>
LD_HD uint32_t ld_xcd_piece(uint32_t b, uint32_t grid, uint32_t turn) {
    const uint32_t round = b / (8u * CHUNK);
    return ld_xcd_piece<CHUNK>((b & ~7u) | ((b + ((round + (round >> 3)) & turn)) & 7u), grid);
}
