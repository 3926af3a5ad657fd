// Index arithmetic of the lane-per-record merge, apart from its kernels so that host code can be built
// from it as well: what it has to withstand are lists that break the caller's contract (a damaged
// file's), and those are tried on the host.
#pragma once

#include "ld_map.h"

// Entries [first, last] of a diff's row of the sub-tile table that one record fills, `before` and `sub` being
// the sub-tiles of the record ahead of it (-1: none) and its own (nsub: it is the end of the list). Indices
// outside the array give sub-tiles outside [0, nsub): the entries stay inside the row of nsub + 1, and every
// entry is filled by some record whatever the order of the list.
struct LdThinEntries { int32_t first, last; };
LD_HD LdThinEntries ld_thin_entries(int32_t before, int32_t sub, int32_t nsub) {
    const int32_t a = before >= nsub ? nsub - 1 : (before < -1 ? -1 : before);
    return LdThinEntries{a + 1, sub > nsub ? nsub : sub};
}

// Records of one diff in a sub-tile of `elements` elements, from its two entries of the table. The entries of a list
// that does not ascend may descend or lie any number of records apart; a strictly ascending list has at
// most one record per element. With this bound every position begin .. begin + count - 1 is a record
// of the list (entries lie in [0, K]) and the work of a sub-tile is bounded.
LD_HD uint32_t ld_thin_count(int32_t begin, int32_t end, int32_t elements) {
    if (end <= begin) return 0;
    const uint32_t count = static_cast<uint32_t>(end) - static_cast<uint32_t>(begin);
    return count < static_cast<uint32_t>(elements) ? count : static_cast<uint32_t>(elements);
}

// Owner slot, one of 256, of element `e` of a sub-tile of at most 4096. Positions at a fixed stride (a column of a weight
// matrix) have to fall on different slots as well: with the low bits of `e` as the slot, 16 elements 256
// apart shared one (50 diffs of 0.4 %, one column of 124 M elements: 3654 us, now 292). The product's bits 12 to 19
// keep 64 equidistant elements apart (two to a slot at most; multiples of 233 excepted).
LD_HD uint32_t ld_thin_slot(uint32_t e) { return ((e & 4095u) * 0x9E37u >> 12) & 255u; }
