"""Index arithmetic that kernels share with the host, built with g++: tried over its whole range, and on what no GPU
run may be given (record lists that break the contract of the merges, as a damaged file's)."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

from combine_lists import COMBINE_LISTS

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2509_04084_amd", "csrc")

SHIM = """
#include "ld_combine_shape.h"
#include "ld_map.h"
#include "ld_thin.h"
extern "C" {
int32_t combine_shape(int64_t n, int32_t N, int64_t most, int64_t total, int32_t strategy) {
    return ld_combine_shape(n, N, most, total, strategy);
}
// the table row of one diff, each entry taken by the first (order 0) or the last (1) of the records that fill it
void thin_row(const int32_t* idx, int32_t K, int32_t sub, int32_t nsub, int32_t order, int32_t* row) {
    for (int32_t s = 0; s <= nsub; ++s) row[s] = -1;
    for (int32_t j = 0; j <= K; ++j) {
        const LdThinEntries f = ld_thin_entries(j == 0 ? -1 : idx[j - 1] / sub, j == K ? nsub : idx[j] / sub, nsub);
        for (int32_t s = f.first; s <= f.last; ++s)
            if (order == 1 || row[s] < 0) row[s] = j;
    }
}
uint32_t thin_count(int32_t begin, int32_t end, int32_t elements) { return ld_thin_count(begin, end, elements); }
uint32_t thin_slot(uint32_t e) { return ld_thin_slot(e); }
// the piece of every workgroup of a grid
void xcd_pieces(uint32_t run, int32_t turned, uint32_t grid, uint32_t* piece) {
    for (uint32_t b = 0; b < grid; ++b) {
        if (run == 1) piece[b] = turned ? ld_xcd_piece<1>(b, grid, 7) : ld_xcd_piece<1>(b, grid);
        if (run == 16) piece[b] = turned ? ld_xcd_piece<16>(b, grid, 7) : ld_xcd_piece<16>(b, grid, 0);
        if (run == 32) piece[b] = turned ? ld_xcd_piece<32>(b, grid, 7) : ld_xcd_piece<32>(b, grid, 0);
        if (run == 64) piece[b] = turned ? ld_xcd_piece<64>(b, grid, 7) : ld_xcd_piece<64>(b, grid, 0);
    }
}
}
"""


@pytest.fixture(scope="module")
def shim(tmp_path_factory):
    d = tmp_path_factory.mktemp("index")
    src, lib = str(d / "shim.cpp"), str(d / "shim.so")
    with open(src, "w") as f:
        f.write(SHIM)
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-fPIC", "-shared", "-fsanitize=undefined",
                    "-fno-sanitize-recover", "-I", CSRC, "-I", os.path.join(ROOT, "include"), src, "-o", lib], check=True)
    L = ctypes.CDLL(lib)
    L.thin_count.restype = L.thin_slot.restype = ctypes.c_uint32
    return L


def rows(shim, idx, n, sub):
    nsub = (n + sub - 1) // sub
    for order in (0, 1):
        row = np.full(nsub + 3, -7, np.int32)  # a word either side of the row
        shim.thin_row(ctypes.c_void_p(idx.ctypes.data), idx.size, sub, nsub, order, ctypes.c_void_p(row.ctypes.data + 4))
        assert row[0] == -7 and row[-1] == -7
        yield row[1:-1]


@pytest.mark.parametrize("kind", ["ascending", "descending", "random", "zeros", "repeated", "outside", "two_runs"])
@pytest.mark.parametrize("n,K", [(5, 3), (40960, 500), (100003, 4096), (100003, 60000)])
def test_sub_tile_counts_stay_inside_any_list(shim, kind, n, K):
    sub = 4096
    rs = np.random.RandomState(K)
    up = np.sort(rs.choice(n, min(K, n), replace=False))
    idx = {"ascending": up, "descending": up[::-1], "random": rs.permutation(up), "zeros": np.zeros(K, np.int64),
           "repeated": np.full(K, n - 1), "outside": rs.randint(-2 ** 31, 2 ** 31, K),
           "two_runs": np.concatenate([up, up])}[kind]
    idx = np.ascontiguousarray(idx, np.int32)
    for row in rows(shim, idx, n, sub):
        assert row.min() >= 0 and row.max() <= idx.size      # every entry filled, and with a position of the list
        for b, e in zip(row[:-1], row[1:]):
            count = shim.thin_count(int(b), int(e), sub)
            assert 0 <= count <= sub and b + count <= idx.size
            if kind == "ascending":
                assert count == e - b
        if kind == "ascending":
            np.testing.assert_array_equal(row, np.searchsorted(up, np.minimum(np.arange(row.size) * sub, n)))


def test_sub_tile_count_of_any_two_entries(shim):
    ends = [0, 1, 5, 4095, 4096, 4097, 2 ** 31 - 1]
    for b in ends:
        for e in ends:
            assert shim.thin_count(b, e, 4096) == min(max(e - b, 0), 4096)


def test_owner_slots_keep_equidistant_elements_apart(shim):
    # a row of 64 records of one diff bids once per record that shares a slot: columns of a matrix must not pile up
    slot = np.array([shim.thin_slot(e) for e in range(4096)])
    assert slot.min() >= 0 and slot.max() <= 255
    assert np.bincount(slot, minlength=256).max() <= 18            # 4096 elements over 256 slots
    for stride in range(1, 4096):
        if stride % 233 == 0:                                      # 233 * 0x9E37 = 9 * 2^20 + 15: no matrix is that wide
            continue
        for first in (0, 5, 77):
            e = np.arange(first, 4096, stride)[:64]
            assert np.bincount(slot[e], minlength=256).max() <= 2, stride
    for e in (4096, 2 ** 31, 2 ** 32 - 1):                         # records outside the sub-tile bid for nothing, but look
        assert shim.thin_slot(ctypes.c_uint32(e)) <= 255


@pytest.mark.parametrize("run", [1, 16, 32, 64])
def test_xcd_maps_are_permutations(shim, run):
    for grid in (8, 16, 64, 120, 128, 136, 512, 520, 1024, 1032, 4096, 44800, 44808):
        for turned in (0, 1):
            piece = np.zeros(grid, np.uint32)
            shim.xcd_pieces(run, turned, grid, ctypes.c_void_p(piece.ctypes.data))
            np.testing.assert_array_equal(np.sort(piece), np.arange(grid))


@pytest.mark.parametrize("tiles,run", [(16, 1), (64, 1), (64, 16)])
@pytest.mark.parametrize("used", [1, 2, 3])
def test_small_segments_are_spread_over_the_xcds(shim, tiles, run, used):
    # one group per segment, of whose tile slots only the first are work: no XCD (workgroup number modulo 8) may be given
    # much more than its eighth of them
    for n_seg in (64, 500, 520, 3000):
        grid = n_seg * tiles
        piece = np.zeros(grid, np.uint32)
        shim.xcd_pieces(run, 1, grid, ctypes.c_void_p(piece.ctypes.data))
        work = np.bincount(np.arange(grid)[piece % tiles < used] % 8, minlength=8)
        assert work.max() <= 1.25 * used * n_seg / 8 + 4 * used, (n_seg, work)


def test_bare_barriers_are_fenced_on_both_sides():
    # s_barrier alone does not order memory accesses for the compiler: a release fence has to stand before it and an acquire
    # fence behind it, next to it (as __syncthreads has them), whatever they are restricted to
    bare = 0
    for name in sorted(os.listdir(CSRC)):
        if not name.endswith((".hip", ".h")):
            continue
        with open(os.path.join(CSRC, name)) as f:
            lines = [line.split("//")[0].strip() for line in f]
        lines = [line for line in lines if line]
        for i, line in enumerate(lines):
            if "__builtin_amdgcn_s_barrier()" in line:
                bare += 1
                for fence, kinds in ((lines[i - 1], ("__ATOMIC_RELEASE", "__ATOMIC_ACQ_REL")),
                                     (lines[i + 1], ("__ATOMIC_ACQUIRE", "__ATOMIC_ACQ_REL"))):
                    assert "__builtin_amdgcn_fence(" in fence and any(k in fence for k in kinds), f"{name}: {line}"
    assert bare == 1  # the rule above looks at lines: a barrier written in another way would pass it unseen


TWO, NARROW, FEW, MIDDLE, LONG, WIDE = range(6)


def combine_shape(shim, n, counts, strategy=0):
    return shim.combine_shape(ctypes.c_int64(n), len(counts), ctypes.c_int64(max(counts)), ctypes.c_int64(sum(counts)), strategy)


@pytest.mark.parametrize("n,N,rho,shape", [
    (1_557_611_200, 8, 100, MIDDLE), (1_400_000_000, 8, 1000, NARROW), (5_000_000, 8, 1000, NARROW), (400_000_000, 8, 60, WIDE),
    # where one pass was the slower one: 300 us two passes / 502 one, 187 / 291, 66 / 88, 119 / 210, 612 / 1043, 258 / 411, 53 / 76
    (119_177_435, 64, 313, TWO), (329_999_869, 12, 129, TWO), (76_868_857, 16, 150, TWO), (31_779_675, 64, 294, TWO),
    (1_087_848_157, 16, 170, TWO), (445_490_825, 16, 175, TWO), (65_608_085, 9, 120, TWO),
    # and where two are: 288 / 170, 84 / 65, 1185 / 709, 8 lists of 0.35 % whose layers differ in density 50 / 46 (narrow 58)
    (1_400_000_000, 16, 1000, NARROW), (10_000_000, 16, 100, WIDE), (400_000_000, 16, 50, WIDE), (20_000_000, 8, 290, MIDDLE)])
def test_combine_takes_the_way_that_measured_faster(shim, n, N, rho, shape):
    assert combine_shape(shim, n, [n // rho] * N) == shape


def test_combine_strategies_are_what_the_caller_says(shim):
    for n, N, rho in ((1000, 1, 2), (10 ** 6, 64, 3), (2 ** 31 - 1, 64, 2), (2 ** 31 - 1, 2, 1), (400_000_000, 12, 129)):
        assert combine_shape(shim, n, [n // rho] * N, 1) == TWO
        for strategy in (2, 3):
            assert combine_shape(shim, n, [n // rho] * N, strategy) != TWO
        for k in range(N):  # shapes without a kernel for more than 8 lists are not chosen for them
            assert k < 8 or combine_shape(shim, n, [n // rho] * (k + 1)) not in (FEW, LONG)


def test_combine_lists_reach_the_kernels_that_they_are_made_for(shim):
    names = ["two", "narrow", "few", "middle", "long", "wide"]
    ran = set()
    for name, (n, counts, span, shape) in COMBINE_LISTS.items():
        assert names[combine_shape(shim, n, counts)] == (shape or "two"), name
        one = names[combine_shape(shim, n, counts, 2)]
        assert one == (shape or "wide"), name
        ran.add((one, len(counts) > 8, name.startswith("crowded")))
    for many in (False, True):
        for crowded in (False, True):
            for shape in ("narrow", "middle", "wide") + (() if many else ("few", "long")):
                assert (shape, many, crowded) in ran, (shape, many, crowded)
