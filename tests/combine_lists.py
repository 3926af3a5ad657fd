"""Inputs of the combine's strategies: index space, records per list, the span that they lie in (None: all of it), and how the
one pass runs them: the shape that the library picks, or "" where it picks two passes and the one pass is wide."""

COMBINE_LISTS = {
    "one record": (49152 * 3 + 5, [1], None, "narrow"),
    "sparse, 3 of 70 chunks": (49152 * 70 + 1, [2000, 1, 0, 1900], (0, 140000), "narrow"),
    "narrow": (49152 * 9 + 77, [1500] * 8, None, "middle"),
    "middle": (49152 * 300, [147000] * 8, None, "middle"),
    "wide": (49152 * 11 + 4096, [11000, 10000, 9000], None, "long"),
    "more than 8 lists": (49152 * 6 + 1, [2500] * 17, None, "wide"),
    "crowded chunk": (49152 * 4, [9000] * 5, (60000, 75000), ""),
    "all of it": (49152 * 2 + 3, [98307] * 3, None, ""),
    "64 lists": (200000, [700] * 64, None, ""),
    # even lists, up to 8 and more of them
    "even, narrow": (49152 * 20 + 3, [2000] * 8, None, "narrow"),
    "even, narrow, 9 lists": (49152 * 20, [1500] * 8 + [1], None, "narrow"),
    "even, few": (49152 * 20 - 1, [8000] * 4, None, "few"),
    "even, middle, 12 lists": (49152 * 20 + 1, [6000] * 12, None, "middle"),
    "even, long": (49152 * 20, [15000] * 3, None, "long"),
    "even, wide": (49152 * 20 + 7, [22000] * 5, None, "wide"),
    "even, wide, 9 lists": (49152 * 20 - 7, [15000] * 9, None, "wide"),
    # a few chunks crowded in lists that are sparse all in all: the workgroups are made for few records and take the chunk in
    # many rounds, each a piece of every list (lists that end early or begin late among them)
    "crowded, narrow": (49152 * 60, [11000] * 4, (50000, 110000), "narrow"),
    "crowded, narrow, 9 lists": (49152 * 75, [8000] * 8 + [100], (49000, 100000), "narrow"),
    "crowded, few": (49152 * 50, [20000, 300, 20000], (0, 60000), "few"),
    "crowded, middle, 9 lists": (49152 * 50, [11000] * 9, (49152, 49152 * 2), "middle"),
    "crowded, middle": (49152 * 50, [30000, 29000, 0, 30000, 1], (100000, 160000), "middle"),
    "crowded, middle, 10 lists": (49152 * 50, [20000] * 10, (49152 * 50 - 60000, 49152 * 50), "middle"),
    "crowded, long": (49152 * 50, [45000] * 3, (49152 * 7 + 1000, 49152 * 8), "long"),
    "crowded, wide, 9 lists": (49152 * 50, [40000] + [15000] * 8, (49152 * 7 - 100, 49152 * 8), "wide"),
    "crowded, wide": (49152 * 50, [60000] * 8, (49152 * 10, 49152 * 13), "wide"),
    "crowded, wide, 17 lists": (49152 * 50, [40000] * 17, (49152 * 10, 49152 * 11 + 2), "wide"),
    "crowded, wide, 64 lists": (49152 * 40, [7000] * 60 + [0, 1, 300, 49000], (49152 * 3 - 20, 49152 * 5), "wide"),
}
