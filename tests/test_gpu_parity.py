"""GPU parity: the HIP library (through its C ABI) against the CPU oracle,
element by element on the same seeded inputs.

Bars: bit-exact for indices, values, residuals, snapshots and sparse merges;
|x - y| <= 1e-7 + 1e-6 |y| for the dense Adam replay (and a relative-only check
on v, which never cancels).
"""
import ctypes

import numpy as np
import pytest
import torch

import oracle
from combine_lists import COMBINE_LISTS
from paper_2509_04084_amd import lowdiff as ld
from paper_2509_04084_amd import synth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def bits(a):
    return np.ascontiguousarray(a, dtype=np.float32).view(np.uint32)


def to_gpu(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to(DEV)


def compress_paths(ws, seg_off):
    """(path, tied flag, overflowed tiles) per segment of the last call on workspace `ws`; also checks
    that the full-segment pass never gave up."""
    paths, over = ld.ld_compress_topk_paths(ws, seg_off)
    torch.cuda.synchronize()
    paths, over = paths.cpu().numpy(), over.cpu().numpy()
    assert not np.any(paths & 0x10000), "the full-segment pass gave up at its barrier"
    return paths & 0xFF, (paths & 0x100) != 0, over


def check_compress(g, r, seg_off, seg_k, select=True, tag="",
                   strategies=(ld.LD_COMPRESS_AUTO, ld.LD_COMPRESS_FULL), want=None, large_groups=False):
    """Runs one compress call per strategy on the GPU and once on the oracle;
    returns (idx, val, r_new) of the oracle. `want(path, tied, overflowed)` is called with what
    the AUTO call reports about the way each segment went. With `large_groups` all of it once more
    with 520 segments of one element behind the others: every segment is a group at least, and from 512 groups of
    64 tiles on a call runs with those (and other kernels) instead of groups of 16; and with a large segment
    behind them, whose size has the thresholds of all selected in a launch of their own."""
    alone = large_groups
    if large_groups:
        more = 520
        rs = np.random.RandomState(more)
        ext = lambda a: np.concatenate([a, rs.standard_normal(more).astype(np.float32)])
        check_compress(ext(g), ext(r), np.concatenate([seg_off, seg_off[-1] + 1 + np.arange(more)]),
                       np.concatenate([seg_k, np.arange(more) % 2]).astype(np.int32), select, tag + " large groups",
                       strategies, want)
    print(f"[compress] {tag} n={len(g)} n_seg={len(seg_k)}", flush=True)
    oi, ov, orr = oracle.topk_ef(g, r, seg_off, seg_k, select=select)
    g_gpu = to_gpu(g)
    seg_k = np.asarray(seg_k, np.int32)
    ws = torch.empty(max(256, ld.ld_compress_topk_workspace(seg_off, seg_k)), dtype=torch.uint8, device=DEV)
    for strategy in strategies:
        r_gpu = to_gpu(r)
        idx, val = ld.ld_compress_topk(g_gpu, r_gpu, seg_off, seg_k, workspace=ws, strategy=strategy)
        torch.cuda.synchronize()
        tg = f"{tag} strategy={strategy}"
        np.testing.assert_array_equal(idx.cpu().numpy(), oi, err_msg=f"idx {tg}")
        np.testing.assert_array_equal(bits(val.cpu().numpy()), bits(ov), err_msg=f"val {tg}")
        np.testing.assert_array_equal(bits(r_gpu.cpu().numpy()), bits(orr), err_msg=f"residual {tg}")
        if len(seg_k) and int(np.asarray(seg_off)[-1]) > 0:
            path, tied, over = compress_paths(ws, seg_off)
            if strategy == ld.LD_COMPRESS_FULL:  # every segment that keeps anything went the full way
                assert np.all(path[seg_k > 0] == ld.LD_PATH_FULL), tg
            elif want is not None:
                want(path, tied, over)
    if alone:
        check_compress_before_a_large_segment(g_gpu, r, seg_off, seg_k, (oi, ov, orr), tag, want)
    return oi, ov, orr


_large = {}


def check_compress_before_a_large_segment(g, r, seg_off, seg_k, expected, tag, want):
    """The same segments once more with one of 66 M elements behind them (groups of 16 tiles) or of 135 M (groups of 64), that keeps one
    element, 2 % or 6 % (which has 16, 32 and 64 lanes serve a tile): k_select, and k_emit without a selection of its own. The large
    segment's records are checked by what holds at any size."""
    oi, ov, orr = expected
    n, K = int(seg_off[-1]), len(oi)
    if "g" not in _large:
        gen = torch.Generator(device=DEV).manual_seed(66)
        _large["g"] = torch.randn(135_000_001, generator=gen, device=DEV)
    for size in (66_000_001, 135_000_001):
        for k in (1, size // 50, size * 6 // 100):
            tg = f"{tag}, before {size} elements of which {k} are kept"
            gx, rx = torch.cat([g, _large["g"][:size]]), torch.cat([to_gpu(r), torch.zeros(size, device=DEV)])
            off, kk = np.append(seg_off, n + size), np.append(seg_k, k).astype(np.int32)
            ws = torch.empty(ld.ld_compress_topk_workspace(off, kk), dtype=torch.uint8, device=DEV)
            idx, val = ld.ld_compress_topk(gx, rx, off, kk, workspace=ws)
            torch.cuda.synchronize()
            np.testing.assert_array_equal(idx[:K].cpu().numpy(), oi, err_msg=f"idx {tg}")
            np.testing.assert_array_equal(bits(val[:K].cpu().numpy()), bits(ov), err_msg=f"val {tg}")
            np.testing.assert_array_equal(bits(rx[:n].cpu().numpy()), bits(orr), err_msg=f"residual {tg}")
            li, lv, left = idx[K:].long(), val[K:], gx
            assert li.numel() == k and bool((li[1:] > li[:-1]).all()) and int(li[0]) >= n and int(li[-1]) < n + size, tg
            assert torch.equal(lv.view(torch.int32), left[li].view(torch.int32)), tg
            left[li] = 0.0
            assert torch.equal(left[n:].view(torch.int32), rx[n:].view(torch.int32)), tg
            assert float(left[n:].abs().max()) <= float(lv.abs().min()), tg
            path, tied, over = compress_paths(ws, off)
            assert path[-1] == ld.LD_PATH_CANDIDATES, tg
            if want is not None:
                want(path[:-1], tied[:-1], over[:-1])


# ------------------------------------------------------------------ compress

def test_compress_flat_1m_chained():
    wl = synth.workload("flat1m")
    off, k = wl.seg_off, wl.seg_k
    r = np.zeros(wl.n, np.float32)
    for t in range(3):
        g = synth.gradient(wl, t).numpy()
        def usual(path, tied, over):
            assert path[0] == ld.LD_PATH_CANDIDATES and not tied[0] and over[0] == 0
        _, _, r = check_compress(g, r, off, k, select=(t > 0), tag=f"flat1m t={t}", want=usual)


def test_compress_ragged_segments():
    sizes = [1, 3, 64, 0, 4095, 4097, 65535, 65537, 2, 70001, 0, 200000, 131072, 5]
    off = synth.seg_offsets(sizes)
    rs = np.random.RandomState(1)
    n = int(off[-1])
    g = rs.standard_normal(n).astype(np.float32)
    r = (rs.standard_normal(n) * 0.3).astype(np.float32)
    check_compress(g, r, off, synth.seg_topk(sizes, 1, 100) * (np.array(sizes) > 0), tag="rho=1%")
    check_compress(g, r, off, np.array(sizes, np.int32), tag="k=n")
    check_compress(g, r, off, np.zeros(len(sizes), np.int32), tag="k=0")
    check_compress(g, r, off, np.minimum(np.array(sizes), 1).astype(np.int32), tag="k=1")
    check_compress(g, r, off, (np.array(sizes) // 2).astype(np.int32), tag="k=n/2")


def test_compress_thousands_of_small_segments():
    # 3,000 segments (a model of many small tensors): the segment table travels in seven launches,
    # most segments are smaller than the sample and a tile, a few span several tiles
    rs = np.random.RandomState(11)
    sizes = [int(x) for x in rs.randint(0, 2000, size=3000)]
    for j in range(0, 3000, 250):
        sizes[j] = int(rs.randint(5000, 40000))
    off = synth.seg_offsets(sizes)
    n = int(off[-1])
    g = (rs.standard_t(3, n) * 1e-3).astype(np.float32)
    r = (rs.standard_normal(n) * 1e-3).astype(np.float32)
    k = synth.seg_topk(sizes, 1, 100) * (np.array(sizes) > 0)
    check_compress(g, r, off, k, tag="3000 segments rho=1%")
    k2 = np.array([int(rs.randint(0, s + 1)) for s in sizes], np.int32)
    check_compress(g, r, off, k2, tag="3000 segments random k")


@pytest.mark.parametrize("n_seg", [229, 230, 231, 255, 257, 511, 512, 513])
def test_compress_segment_counts_around_the_launch_rules(n_seg):
    # either side of the segment counts where k_prep's workgroups and the groups' size change (every
    # segment is at least one group), with segments around the sample size and the tile edges
    rs = np.random.RandomState(n_seg)
    sizes = list(rs.randint(1, 3000, n_seg))
    for at, size in ((0, 16383), (1, 16384), (2, 16385), (3, 4097), (4, 65537), (n_seg - 1, 70001)):
        sizes[at] = size
    off, k = synth.seg_offsets(sizes), synth.seg_topk(sizes, 1, 50)
    n = int(off[-1])
    g = (rs.standard_t(3, n) * 1e-3).astype(np.float32)
    r = (rs.standard_normal(n) * 1e-3).astype(np.float32)
    check_compress(g, r, off, k, tag=f"n_seg={n_seg}")


@pytest.mark.parametrize("n_seg", [231, 255, 256, 257, 511, 512])
def test_compress_packed_tables(n_seg):
    # more segments than travel as they are, of few distinct sizes (a model's): the packed table, with 1024 and 512
    # threads in k_prep and groups of 16 and (512 segments) of 64 tiles
    rs = np.random.RandomState(n_seg)
    sizes = [int(x) for x in rs.choice([1, 3, 64, 768, 4095, 4097, 16383, 16385, 65537, 70001], n_seg,
                                       p=[.1, .1, .2, .2, .1, .1, .08, .08, .02, .02])]
    off, k = synth.seg_offsets(sizes), synth.seg_topk(sizes, 1, 50)
    assert len(set(zip(sizes, k.tolist()))) <= 160
    n = int(off[-1])
    check_compress((rs.standard_t(3, n) * 1e-3).astype(np.float32), (rs.standard_normal(n) * 1e-3).astype(np.float32),
                   off, k, tag=f"packed n_seg={n_seg}")


def test_compress_dense_call_of_many_tiles():
    # 5 % of 184 M elements: slots beyond the smallest and tiles dealt out in runs of 16. The result is shown to be the
    # top k by its properties (the order is total, so they fix it).
    n = 184_000_003
    off, k = np.array([0, n], np.int64), np.array([n // 20], np.int32)
    gen = torch.Generator(device=DEV).manual_seed(9)
    g = torch.randn(n, device=DEV, generator=gen)
    r = torch.zeros(n, device=DEV)
    ws = torch.empty(ld.ld_compress_topk_workspace(off, k), dtype=torch.uint8, device=DEV)
    idx, val = ld.ld_compress_topk(g, r, off, k, workspace=ws)
    torch.cuda.synchronize()
    path, tied, over = compress_paths(ws, off)
    assert path[0] == ld.LD_PATH_CANDIDATES and not tied[0]
    i = idx.long()
    assert bool((i[1:] > i[:-1]).all()) and int(i[0]) >= 0 and int(i[-1]) < n
    assert torch.equal(val.view(torch.int32), g[i].view(torch.int32))
    kept = torch.ones(n, dtype=torch.bool, device=DEV)
    kept[i] = False
    assert torch.equal(torch.where(kept, g, 0.0).view(torch.int32), r.view(torch.int32))
    least = val.abs().min()
    assert float(r.abs().max()) <= float(least)
    left = torch.nonzero(kept & (g.abs() == least)).flatten()   # ties at the threshold: the lowest indices were taken
    assert left.numel() == 0 or int(left[0]) > int(i[val.abs() == least][-1])


@pytest.mark.parametrize("rho", [(1, 100), (10, 100)])
def test_compress_workspace_that_holds_only_groups_of_64(rho):
    # The query for a table of few groups counts groups of 16 tiles, whose descriptors take more room than those
    # of 64 when the segments are large (a workspace sized for a larger table can be smaller): the call then runs
    # with groups of 64, and the paths hook reads what it left whichever size it is given.
    sizes = [262144] * 39 + [262143]
    off, k = synth.seg_offsets(sizes), synth.seg_topk(sizes, *rho)
    rs = np.random.RandomState(rho[0])
    n = int(off[-1])
    g = (rs.standard_t(3, n) * 1e-3).astype(np.float32)
    r = (rs.standard_normal(n) * 1e-3).astype(np.float32)
    oi, ov, orr = oracle.topk_ef(g, r, off, k, select=True)
    # 160 and 40 groups: descriptors of 64 bytes, three words each; pieces of 256 bytes
    pieces = lambda groups: -(-groups * 64 // 256) + 3 * -(-groups * 4 // 256)
    gap = (pieces(160) - pieces(40)) * 256
    least, best = ld.ld_compress_topk_workspace(off), ld.ld_compress_topk_workspace(off, k)
    whole = torch.empty(best, dtype=torch.uint8, device=DEV)
    over = {}
    for size in (best, best - 256, best - gap, least, least - 256, least - gap):
        r_gpu = to_gpu(r)
        idx, val = ld.ld_compress_topk(to_gpu(g), r_gpu, off, k, workspace=whole[:size])
        torch.cuda.synchronize()
        np.testing.assert_array_equal(idx.cpu().numpy(), oi)
        np.testing.assert_array_equal(bits(val.cpu().numpy()), bits(ov))
        np.testing.assert_array_equal(bits(r_gpu.cpu().numpy()), bits(orr))
        for ws in (whole[:size], whole):
            path, tied, over[size] = compress_paths(ws, off)
            assert np.all(path == ld.LD_PATH_CANDIDATES) and not np.any(tied)
    assert not np.any(over[best - gap]), "slots of the size that the call asks for"
    np.testing.assert_array_equal(over[least], over[least - gap])   # the same tiles overflow in either cut
    assert rho[0] == 1 or np.all(over[least] > 0)
    with pytest.raises(ld.LowDiffError, match="WORKSPACE"):
        ld.ld_compress_topk(to_gpu(g), to_gpu(r), off, k, workspace=whole[:least - gap - 1])


def test_compress_takes_a_workspace_sized_for_a_larger_table():
    # one segment either side of the size where the groups change: the larger table asks for fewer bytes, and what
    # it asks for serves the smaller one
    n = 511 * 262144
    off, k = np.array([0, n], np.int64), np.array([n // 1000], np.int32)
    size = ld.ld_compress_topk_workspace(np.array([0, n + 262144], np.int64))
    own = ld.ld_compress_topk_workspace(off, k)
    assert size < own
    gen = torch.Generator(device=DEV).manual_seed(5)
    g = torch.randn(n, device=DEV, generator=gen)
    outs = []
    for nbytes in (size, own):
        r = torch.zeros(n, device=DEV)
        idx, val = ld.ld_compress_topk(g, r, off, k, workspace=torch.empty(nbytes, dtype=torch.uint8, device=DEV))
        outs.append((idx, val.view(torch.int32), r.view(torch.int32)))
    torch.cuda.synchronize()
    assert all(torch.equal(a, b) for a, b in zip(*outs))
    idx, val, r = outs[0]
    assert torch.equal(val, g[idx.long()].view(torch.int32)) and int((r == 0).sum()) >= k[0]
    assert float(g[idx.long()].abs().min()) >= float(r.view(torch.float32).abs().max())


@pytest.mark.parametrize("n", [150001])
def test_compress_adversarial(n):
    off = np.array([0, 1000, 70000, n], np.int64)
    for name, g, r in synth.adversarial_cases(n, seed=3):
        for k in ([10, 690, 800], [1000, 1, 80001], [500, 69000, 40000]):
            check_compress(g, r, off, np.array(k, np.int32), tag=f"{name} k={k}", large_groups=True)


@pytest.mark.parametrize("rho", [(2, 100), (3, 100), (5, 100), (75, 1000), (10, 100), (25, 100)])
def test_compress_density_range(rho):
    # Densities of the paper's Exp. 10 range and beyond: the candidate passes change shape with
    # the density (lanes per tile, slot size). Once with the workspace the binding sizes for
    # the call's seg_k, once with the minimum one (the tiles then overflow their slots).
    sizes = [300000, 70000, 1200000, 4097, 65536]
    off = synth.seg_offsets(sizes)
    k = synth.seg_topk(sizes, *rho)
    rs = np.random.RandomState(rho[0])
    n = int(off[-1])
    g = (rs.standard_t(3, n) * 1e-3).astype(np.float32)
    r = (rs.standard_t(3, n) * 3e-4).astype(np.float32)
    oi, ov, orr = check_compress(g, r, off, k, tag=f"rho={rho}", strategies=(ld.LD_COMPRESS_AUTO,), large_groups=True)
    assert ld.ld_compress_topk_workspace(off, k) >= ld.ld_compress_topk_workspace(off)
    small = torch.empty(ld.ld_compress_topk_workspace(off), dtype=torch.uint8, device=DEV)
    r_gpu = to_gpu(r)
    idx, val = ld.ld_compress_topk(to_gpu(g), r_gpu, off, k, workspace=small)
    torch.cuda.synchronize()
    path, _, over = compress_paths(small, off)
    assert np.all(path == ld.LD_PATH_CANDIDATES)
    if rho[0] * 100 >= 10 * rho[1]:  # 10 % and 25 %: far more candidates per tile than the minimum slot holds
        assert over[2] > 100, "the slots were expected to overflow"
    np.testing.assert_array_equal(idx.cpu().numpy(), oi)
    np.testing.assert_array_equal(bits(val.cpu().numpy()), bits(ov))
    np.testing.assert_array_equal(bits(r_gpu.cpu().numpy()), bits(orr))


@pytest.mark.parametrize("cluster", [1, 64, 65, 256, 257, 512, 513, 2049, 4090, 6000])
@pytest.mark.parametrize("distinct", [True, False])
def test_compress_selects_among_the_keys_of_one_bin(cluster, distinct):
    # the threshold bin holds about `cluster` keys around rank k, below magnitudes of twenty binades that make the bins wide: either side of what
    # one wave selects among in one, four and eight rows of registers, of what the workgroup does, and of what the list holds
    # (6000: several values redone in full, one value by index order); several groups, and ties on both sides of their borders
    n, k, above = 400_000, 3000, 3000 - min(cluster, 4000) // 2 - 1
    rs = np.random.RandomState(cluster + distinct)
    a = (rs.standard_normal(n) * 1e-6).astype(np.float32)
    where = rs.permutation(n)
    a[where[:above]] = np.exp2(rs.uniform(1.0, 20.0, above)).astype(np.float32)
    a[where[above:above + cluster]] = 1.0 + (rs.permutation(cluster) * 2.0 ** -23 if distinct else 0.0)
    a *= np.where(rs.rand(n) < 0.5, 1, -1).astype(np.float32)
    for off, kk in ((np.array([0, n], np.int64), [k]), (np.array([0, 50_000, 50_000 + n], np.int64), [500, k])):
        x = a if off.size == 2 else np.concatenate([(rs.standard_normal(50_000)).astype(np.float32), a])
        check_compress(x, np.zeros(x.size, np.float32), off, np.array(kk, np.int32), tag=f"{cluster} keys, distinct {distinct}", large_groups=True)


def test_compress_massive_ties_at_the_threshold():
    # More equal keys at the threshold than a segment's gather list holds (4096 + n_s / 4096).
    # One repeated value (zeros of a frozen layer, values on a grid): taken by index order without
    # leaving the candidate path. Two adjacent values sharing one overfull bin: the full-segment
    # path. Both must give the oracle's records, bit for bit.
    rs = np.random.RandomState(17)
    n = 1_000_000
    off = np.array([0, n], np.int64)
    k = np.array([10_000], np.int32)
    base = (rs.standard_normal(n) * 1e-3).astype(np.float32)
    order = np.argsort(-np.abs(base), kind="stable")
    cluster = order[7_000:13_000]                 # ranks around k
    lo_val = np.float32(np.abs(base[order[13_000]]))
    one = base.copy()
    one[cluster] = np.where(rs.rand(cluster.size) < 0.5, lo_val, -lo_val)
    # as drawn, a few other keys just below the repeated value share its fine bin: several values in an
    # overfull bin, so the segment is redone in full
    def redone(path, tied, over):
        assert path[0] == ld.LD_PATH_FULL
    check_compress(one, np.zeros(n, np.float32), off, k, tag="one repeated value and close neighbours", want=redone, large_groups=True)
    # with the next 300 ranks moved away the repeated value has its bin to itself: candidate path
    def stays(path, tied, over):
        assert path[0] == ld.LD_PATH_CANDIDATES and not tied[0]
    alone = one.copy()
    alone[order[13_000:13_300]] *= np.float32(0.25)
    check_compress(alone, np.zeros(n, np.float32), off, k, tag="one repeated value across the threshold", want=stays, large_groups=True)
    # values on a dyadic grid (exact in fp32, so equal magnitudes are equal keys): ~7000 copies of the
    # threshold value, more than the gather list's 4340 entries, one value per bin
    dyadic = (np.round(base * 4096) / 4096).astype(np.float32)
    check_compress(dyadic, np.zeros(n, np.float32), off, k, tag="dyadic grid", want=stays, large_groups=True)
    two = one.copy()
    up = np.nextafter(lo_val, np.float32(1.0))
    two[cluster[::2]] = up
    check_compress(two, np.zeros(n, np.float32), off, k, tag="two adjacent values across the threshold", want=redone, large_groups=True)
    # frozen layer next to a live one, and values on a coarse grid (heavy duplication everywhere)
    sizes = [600_000, 400_000]
    off2 = synth.seg_offsets(sizes)
    g = base.copy()
    g[:600_000] = 0.0
    g[123] = -0.0
    def frozen(path, tied, over):
        assert path[0] == ld.LD_PATH_TIES and tied[0], "the zeros of the frozen segment: ties by index"
        assert path[1] == ld.LD_PATH_CANDIDATES and not tied[1]
    check_compress(g, np.zeros(n, np.float32), off2, synth.seg_topk(sizes, 1, 100), tag="frozen segment", want=frozen, large_groups=True)
    grid = (np.round(base * 3e4) / 3e4).astype(np.float32)
    check_compress(grid, (np.round(base[::-1] * 1e4) / 3e4).astype(np.float32), off2,
                   synth.seg_topk(sizes, 1, 100), tag="values on a grid", large_groups=True)


@pytest.mark.parametrize("copies", [1, 250, 256, 257, 1000, 4300, 30_000])
@pytest.mark.parametrize("spread", [True, False])
def test_compress_keys_in_the_threshold_bin(copies, spread):
    # The keys of the threshold bin are placed one by one or a workgroup's at a time, by how many there are: copies of
    # one key at the threshold, all over the segment or in consecutive elements (whole tiles of them: more than a
    # tile's slots hold), up to more than the gather list takes. Two segments, so that one workgroup's waves
    # hold tiles of a second group.
    rs = np.random.RandomState(copies)
    n, k_s = 700_001, 7000
    off = np.array([0, n, n + 90_000], np.int64)
    g = rs.permutation(np.linspace(1e-4, 1.0, n)).astype(np.float32) ** 8
    order = np.argsort(-g, kind="stable")
    at = rs.choice(n - copies, copies, replace=False) if spread else n // 3 + np.arange(copies)
    x = g[order[k_s - 1]]
    g[at] = x                                    # some of the copies were above, most below: x stays near rank k
    g *= np.where(rs.rand(n) < 0.5, 1, -1).astype(np.float32)
    g = np.concatenate([g, rs.standard_normal(90_000).astype(np.float32)])
    for rank in (k_s - copies // 2, k_s + copies // 2):
        check_compress(g, np.zeros_like(g), off, np.array([max(rank, 1), 900], np.int32), tag=f"{copies} copies, k={rank}",
                       strategies=(ld.LD_COMPRESS_AUTO,))


def test_compress_tied_segment_with_and_without_enough_ties():
    # A segment is treated as "tied" when the 16 K-element sample holds the candidate threshold's
    # own key hundreds of times. White-box: the sample positions are rebuilt here (256 jittered runs
    # of 64 elements), so that the sample can be made to see a repeated key X at the threshold.
    # (a) the rest of the segment holds X often enough: X is the threshold, ties by index;
    # (b) it does not: the tied guess is wrong, the threshold lies below X, full-segment path.
    ns, k_s, X = 2_000_000, 20_000, np.float32(0.3)   # a key whose low mantissa bits are not zero
    stride = ns // 256
    pos = []
    for run in range(256):
        x = (run * 2654435761) & 0xFFFFFFFF
        x ^= x >> 16
        x = (x * 0x7FEB352D) & 0xFFFFFFFF
        x ^= x >> 15
        x = (x * 0x846CA68B) & 0xFFFFFFFF
        x ^= x >> 16
        pos.append(run * stride + ((x * (stride - 63)) >> 32) + np.arange(64))
    pos = np.concatenate(pos)
    rs = np.random.RandomState(23)
    sign = lambda m: np.where(rs.rand(m) < 0.5, 1.0, -1.0).astype(np.float32)
    base = (rs.uniform(0.0, 0.25, ns).astype(np.float32) * sign(ns))
    picked = rs.permutation(pos)
    base[picked[:200]] = rs.uniform(2.0, 3.0, 200).astype(np.float32) * sign(200)
    base[picked[200:800]] = X * sign(600)
    off = np.array([0, ns], np.int64)
    k = np.array([k_s], np.int32)
    z = np.zeros(ns, np.float32)
    few = base.copy()                                  # (b): 800 elements reach X, k is 20,000
    def wrong_guess(path, tied, over):
        assert tied[0], "the sample was built to show a massively repeated key at the threshold"
        assert path[0] == ld.LD_PATH_FULL, "too few ties: the segment must have been redone in full"
    check_compress(few, z, off, k, tag="tied guess, too few ties", strategies=(ld.LD_COMPRESS_AUTO,), want=wrong_guess,
                   large_groups=True)
    many = base.copy()                                 # (a): 25,000 more copies of +-X elsewhere
    rest = np.setdiff1d(np.arange(ns), pos)
    many[rs.choice(rest, 25_000, replace=False)] = X * sign(25_000)
    def right_guess(path, tied, over):
        assert tied[0] and path[0] == ld.LD_PATH_TIES
    oi, ov, _ = check_compress(many, z, off, k, tag="tied guess, enough ties", strategies=(ld.LD_COMPRESS_AUTO,),
                               want=right_guess, large_groups=True)
    assert np.count_nonzero(np.abs(ov) == X) == k_s - 200 and np.count_nonzero(np.abs(ov) > X) == 200


def test_compress_resnet50_shape():
    wl = synth.workload("resnet50")
    g = synth.gradient(wl, 0).numpy()
    r = (synth.gradient(wl, 1).numpy() * np.float32(0.5))
    check_compress(g, r, wl.seg_off, wl.seg_k, tag="resnet50")


def test_compress_is_deterministic_and_reads_only_grad():
    wl = synth.workload("flat1m")
    g = synth.gradient(wl, 5, device=DEV)
    g0 = g.clone()
    outs = []
    for _ in range(2):
        r = torch.zeros(wl.n, device=DEV)
        i, v = ld.ld_compress_topk(g, r, wl.seg_off, wl.seg_k)
        outs.append((i.clone(), v.clone(), r.clone()))
    torch.cuda.synchronize()
    assert torch.equal(g, g0)
    for a, b in zip(outs[0], outs[1]):
        assert torch.equal(a.view(torch.int32), b.view(torch.int32))


# -------------------------------------------------------------- sparse merge

def _diff_chain(wl, W, n=None):
    n = wl.n if n is None else n
    off = wl.seg_off
    k = wl.seg_k
    r = np.zeros(n, np.float32)
    idxs, vals = [], []
    for t in range(W):
        g = synth.gradient(wl, t).numpy()
        i, v, r = oracle.topk_ef(g, r, off, k, select=True)
        idxs.append(i)
        vals.append(v)
    return idxs, vals


@pytest.mark.parametrize("strategy", [ld.LD_MERGE_SWEEP, ld.LD_MERGE_SCATTER, ld.LD_MERGE_AUTO])
def test_merge_flat_window(strategy):
    wl = synth.workload("flat1m")
    idxs, vals = _diff_chain(wl, wl.window)
    w0 = synth.base_weights(wl.n).numpy()
    ref = oracle.merge_sparse(w0, idxs, vals, wl.lr)
    w = to_gpu(w0)
    ld.ld_merge_sparse(w, [to_gpu(i) for i in idxs], [to_gpu(v) for v in vals], wl.lr, strategy=strategy)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(bits(w.cpu().numpy()), bits(ref))
    # the window in one call == one call per diff == any prefix
    w2 = to_gpu(w0)
    for j in range(wl.window):
        ld.ld_merge_sparse(w2, [to_gpu(idxs[j])], [to_gpu(vals[j])], wl.lr, strategy=strategy)
        if j == 3:
            torch.cuda.synchronize()
            np.testing.assert_array_equal(bits(w2.cpu().numpy()),
                                          bits(oracle.merge_sparse(w0, idxs[:4], vals[:4], wl.lr)))
    torch.cuda.synchronize()
    np.testing.assert_array_equal(bits(w2.cpu().numpy()), bits(ref))


@pytest.mark.parametrize("n,W,dens", [(1, 1, 1.0), (4095, 3, 0.5), (4097, 5, 0.02), (1000003, 9, 0.03),
                                      (300000, 140, 0.004), (123457, 2, 1.0), (50000, 4, 0.0),
                                      (2000003, 40, 0.0005), (2000003, 100, 0.0004)])
def test_merge_ragged_and_dense_windows(n, W, dens):
    rs = np.random.RandomState(n % 1000 + W)
    w0 = (rs.standard_normal(n) * 0.02).astype(np.float32)
    idxs, vals = [], []
    for t in range(W):
        kk = int(round(n * dens)) if t != 1 else min(n, int(round(n * dens * 2)))
        i = np.sort(rs.choice(n, kk, replace=False)).astype(np.int32)
        idxs.append(i)
        vals.append(rs.standard_normal(kk).astype(np.float32))
    ref = oracle.merge_sparse(w0, idxs, vals, 0.1)
    for strategy in (ld.LD_MERGE_SWEEP, ld.LD_MERGE_SCATTER):
        w = to_gpu(w0)
        ld.ld_merge_sparse(w, [to_gpu(i) for i in idxs], [to_gpu(v) for v in vals], 0.1, strategy=strategy)
        torch.cuda.synchronize()
        np.testing.assert_array_equal(bits(w.cpu().numpy()), bits(ref), err_msg=f"strategy {strategy}")


@pytest.mark.parametrize("n", [2047, 2049, 49152, 100003])
@pytest.mark.parametrize("per8192", [2, 99, 101, 201, 900])
@pytest.mark.parametrize("W", [3, 66])
def test_merge_sweep_shapes(n, per8192, W):
    # the record windows that a sweep of sub-tiles of 2048 elements picks by its densest diff (8192 where at most 16
    # records per 8192 elements come from each of more than ten), at the edges of sub-tiles and chunks, with one
    # and two sets of diffs per lane and records bunched at one end in every other diff
    rs = np.random.RandomState(n + per8192 + W)
    K = max(1, n * per8192 // 8192)
    idxs = []
    for t in range(W):
        hi = n if t % 2 == 0 else max(K, n // 3)
        idxs.append(np.sort(rs.choice(hi, K, replace=False)).astype(np.int32))
    vals = [(rs.standard_normal(K) * 1e-2).astype(np.float32) for _ in range(W)]
    w0 = synth.base_weights(n).numpy()
    w = to_gpu(w0)
    ws = torch.empty(int(ld.load().ld_merge_sparse_workspace(n, W, None)), dtype=torch.uint8, device=DEV)
    ld.ld_merge_sparse(w, [to_gpu(i) for i in idxs], [to_gpu(v) for v in vals], 0.1, ws, strategy=ld.LD_MERGE_SWEEP)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(bits(w.cpu().numpy()), bits(oracle.merge_sparse(w0, idxs, vals, 0.1)))


@pytest.mark.parametrize("n", [79_999_999, 80_000_003])
@pytest.mark.parametrize("per8192", [82, 150, 300])
@pytest.mark.parametrize("W", [3, 66])
@pytest.mark.parametrize("kind", ["even", "bunched"])
def test_merge_sweep_shapes_of_large_arrays(n, per8192, W, kind):
    # From 80 M elements on the sub-tile follows the densest diff alone: 8192, 4096 or 2048 elements, with one and
    # two sets of diffs per lane. Bunched: the records of a chunk crowd at its beginning or its end (the guess of
    # where a sub-tile's records start comes too late, or the window ends before they do), and other
    # chunks have none. Against one torch operation per diff (product rounded, then the difference).
    gen = torch.Generator(device=DEV).manual_seed(n + per8192 + W)
    count = n * per8192 // 8192
    base = torch.randn(n, device=DEV, generator=gen)
    w, ref, lr = base.clone(), base, torch.tensor(0.1, device=DEV)
    diffs = 3 if W == 3 else 6
    idxs = []
    for t in range(diffs):
        if kind == "even":
            i = torch.randint(0, n, (count,), device=DEV, generator=gen)
        else:
            chunk = torch.randint(0, n // 49152 + 1, (count,), device=DEV, generator=gen)
            if t % 3 == 2:
                chunk = chunk // 3
            x = (torch.rand(count, device=DEV, generator=gen) ** 4 * 49152).long().clamp_(max=49151)
            i = chunk * 49152 + (x if t % 2 == 0 else 49151 - x)
            i = i[i < n]
        i = torch.unique(i)
        assert kind == "bunched" or i.numel() > count * 0.95
        idxs.append(i.int())
    # the last diff has exactly the density; the others may fall short of it by their duplicates
    step = max(1, n // count)
    idxs[-1] = torch.arange(count, device=DEV, dtype=torch.int32) * step
    vals = [torch.randn(i.numel(), device=DEV, generator=gen) * 1e-2 for i in idxs]
    idx, val = [idxs[t % diffs] for t in range(W)], [vals[t % diffs] for t in range(W)]
    ws = torch.empty(int(ld.load().ld_merge_sparse_workspace(n, W, None)), dtype=torch.uint8, device=DEV)
    ld.ld_merge_sparse(w, idx, val, 0.1, ws, strategy=ld.LD_MERGE_SWEEP)
    for i, v in zip(idx, val):
        at = i.long()
        ref[at] = ref[at] - lr * v
    torch.cuda.synchronize()
    assert torch.equal(w.view(torch.int32), ref.view(torch.int32))


def table_of(n, W, sub):
    """Bytes of the table of records per sub-tile that a window asks for: the sub-tile tells which kernel merges it (4096: a
    lane per record, 2048: a window of records per diff)."""
    return -(-(W * (-(-n // sub) + 1) * 4) // 256) * 256


@pytest.mark.parametrize("n", [100, 4095, 4097, 100003])
@pytest.mark.parametrize("per8192", [3, 47, 49])
@pytest.mark.parametrize("W", [11, 64, 65, 128, 131])
def test_merge_lane_per_record_edges(n, per8192, W):
    # the window rule's edge, ragged last sub-tiles, one and two diffs per lane, a second group of diffs, empty
    # diffs among them, and the same elements in neighbouring diffs
    rs = np.random.RandomState(n + per8192 + W)
    K = max(1, n * per8192 // 8192)
    idxs = [np.sort(rs.choice(n, 0 if t % 7 == 3 else K, replace=False)).astype(np.int32) for t in range(W)]
    for t in range(5, W, 9):
        idxs[t] = idxs[t - 1].copy()
    vals = [(rs.standard_normal(i.size) * 1e-2).astype(np.float32) for i in idxs]
    w0 = synth.base_weights(n).numpy()
    w = to_gpu(w0)
    ws = torch.empty(ld.ld_merge_sparse_workspace(n, [i.size for i in idxs]), dtype=torch.uint8, device=DEV)
    ld.ld_merge_sparse(w, [to_gpu(i) for i in idxs], [to_gpu(v) for v in vals], 0.1, ws, strategy=ld.LD_MERGE_SWEEP)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(bits(w.cpu().numpy()), bits(oracle.merge_sparse(w0, idxs, vals, 0.1)))


@pytest.mark.parametrize("n", [999_937, 999_424 + 5])
@pytest.mark.parametrize("W", [11, 64, 65, 131])
@pytest.mark.parametrize("case", ["line", "rows", "full", "column", "columns"])
def test_merge_lane_per_record_dense_sub_tiles_and_columns(n, W, case):
    # Windows that the rule takes for sparse (at most 48 records per 8192 elements of all, with 11 diffs 20: the last two cases
    # go by windows of records there) and that are not evenly so:
    #   line     every sub-tile a few records either side of where it goes through diff after diff
    #   rows     runs of 768 elements in the first, a middle and the ragged last sub-tile, the same in every diff
    #   full     whole sub-tiles, four trips of records and more
    #   column   the same elements 256 apart in every diff
    #   columns  another column in each diff, 1024 apart
    rs = np.random.RandomState(W)
    limit = 48 * n // 8192
    idxs = []
    for t in range(W):
        if case == "line":
            at = [s * 4096 + rs.choice(min(4096, n - s * 4096), min(126 + t % 4, n - s * 4096), replace=False)
                  for s in (0, 1, 17, 200, (n - 1) // 4096)]
        elif case == "rows":
            at = [np.arange(s, s + 768) for s in (0, 4096 * 100 - 300, n - 768)]
        elif case == "full":
            at = [np.arange(4096 * 7 - t, 4096 * 8 + t), np.arange(n - 700, n)]
        elif case == "column":
            at = [np.arange(5, n, 256)]
        else:
            at = [np.arange(37 * t % 1024, n, 1024)]
        idxs.append(np.sort(np.concatenate(at)).astype(np.int32))
        assert idxs[-1].size <= limit
    vals = [(rs.standard_normal(i.size) * 1e-2).astype(np.float32) for i in idxs]
    w0 = synth.base_weights(n).numpy()
    w = to_gpu(w0)
    ws = torch.empty(ld.ld_merge_sparse_workspace(n, [i.size for i in idxs]), dtype=torch.uint8, device=DEV)
    ld.ld_merge_sparse(w, [to_gpu(i) for i in idxs], [to_gpu(v) for v in vals], 0.1, ws, strategy=ld.LD_MERGE_SWEEP)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(bits(w.cpu().numpy()), bits(oracle.merge_sparse(w0, idxs, vals, 0.1)))


@pytest.mark.parametrize("W,per8192,case", [(11, 19, "even"), (11, 20, "even"), (11, 21, "even"), (17, 20, "even"), (18, 20, "even"),
                                            (18, 48, "even"), (18, 49, "even"), (11, 16, "column"), (18, 32, "column"), (131, 32, "column")])
def test_merge_lane_per_record_where_its_line_lies(W, per8192, case):
    # either side of the line of small arrays, 20 records per 8192 elements up to 17 diffs and 48 with more, and the same column of
    # elements 512 or 256 apart in every diff (all on one slot of the owner table, were it not for the hash)
    n = 8192 * 41
    rs = np.random.RandomState(W + per8192)
    K = n * per8192 // 8192
    idxs = [np.arange(5, n, 8192 // per8192) if case == "column" else np.sort(rs.choice(n, K, replace=False)) for _ in range(W)]
    idxs = [i.astype(np.int32) for i in idxs]
    assert max(i.size for i in idxs) == K
    nbytes = ld.ld_merge_sparse_workspace(n, [i.size for i in idxs])
    lanes = per8192 <= (48 if W > 17 else 20)
    assert nbytes == max(table_of(n, min(W, 128), 4096 if lanes else 2048), table_of(n, W - 128, 2048) if W > 128 else 0)
    vals = [(rs.standard_normal(i.size) * 1e-2).astype(np.float32) for i in idxs]
    w0 = synth.base_weights(n).numpy()
    w = to_gpu(w0)
    ws = torch.empty(nbytes, dtype=torch.uint8, device=DEV)
    ld.ld_merge_sparse(w, [to_gpu(i) for i in idxs], [to_gpu(v) for v in vals], 0.1, ws, strategy=ld.LD_MERGE_SWEEP)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(bits(w.cpu().numpy()), bits(oracle.merge_sparse(w0, idxs, vals, 0.1)))


@pytest.mark.parametrize("n", [100, 2047, 2049, 8192 * 3, 300_007])
@pytest.mark.parametrize("per8192", [21, 100, 168, 169, 900])
@pytest.mark.parametrize("W", [1, 17, 18, 65, 130])
def test_merge_rows_edges(n, per8192, W):
    # small arrays with the workspace their window asks for: records looked up per 2048 elements, one or two windows of 64
    # per diff, 17 or 10 diffs a batch, one and two diffs per lane, a second group. Every third diff is crowded into
    # a quarter of the array (more records in a sub-tile than its windows hold), every seventh has none, some share positions.
    rs = np.random.RandomState(n + per8192 + W)
    K = max(1, n * per8192 // 8192)
    idxs = []
    for t in range(W):
        hi = n if t % 3 else max(K, n // 4)
        idxs.append(np.sort(rs.choice(hi, 0 if t % 7 == 3 else K, replace=False)).astype(np.int32))
    for t in range(5, W, 9):
        idxs[t] = idxs[t - 1].copy()
    vals = [(rs.standard_normal(i.size) * 1e-2).astype(np.float32) for i in idxs]
    w0 = synth.base_weights(n).numpy()
    ref = oracle.merge_sparse(w0, idxs, vals, 0.1)
    gi, gv = [to_gpu(i) for i in idxs], [to_gpu(v) for v in vals]
    for strategy in (ld.LD_MERGE_SWEEP, ld.LD_MERGE_AUTO):
        w = to_gpu(w0)
        ws = torch.full((ld.ld_merge_sparse_workspace(n, [i.size for i in idxs]),), 0xA5, dtype=torch.uint8, device=DEV)
        ld.ld_merge_sparse(w, gi, gv, 0.1, ws, strategy=strategy)
        torch.cuda.synchronize()
        np.testing.assert_array_equal(bits(w.cpu().numpy()), bits(ref), err_msg=f"strategy {strategy}")


@pytest.mark.parametrize("n,sub", [(3_000_001, 2048), (14_000_003, 4096)])
@pytest.mark.parametrize("K", [78_100, 78_150])
def test_merge_tables_of_few_and_of_many_records(n, sub, K):
    # either side of 10 M records, from which a thread of the table's pass looks at eight of them instead of four
    W = 128
    gen = torch.Generator(device=DEV).manual_seed(K + n)
    idx = [torch.randperm(n, device=DEV, generator=gen)[:K - t % 2].sort().values.int() for t in range(4)]
    idx = [idx[t % 4] for t in range(W)]
    val = [torch.randn(i.numel(), generator=gen, device=DEV) for i in idx]
    counts = [i.numel() for i in idx]
    assert ld.ld_merge_sparse_workspace(n, counts) == table_of(n, W, sub)
    w = torch.randn(n, generator=gen, device=DEV)
    ref = w.clone()
    ws = torch.full((table_of(n, W, sub),), 0xA5, dtype=torch.uint8, device=DEV)
    ld.ld_merge_sparse(w, idx, val, 0.1, ws)
    lr = torch.tensor(0.1, device=DEV)
    for i, v in zip(idx, val):
        at = i.long()
        ref[at] = ref[at] - lr * v
    assert torch.equal(w.view(torch.int32), ref.view(torch.int32))


@pytest.mark.parametrize("W", [2, 10, 40])
@pytest.mark.parametrize("way", ["full", "minimum", "misaligned", "static"])
def test_merge_of_sparse_windows_with_and_without_tables(W, way):
    # windows that touch little of w: with the workspace that the query gives they run from a table where that is faster,
    # else, and with index arrays that are not 16-byte aligned, as scatters
    n, K = 1_000_003, 1000
    rs = np.random.RandomState(W)
    idxs = [np.sort(rs.choice(n, K, replace=False)).astype(np.int32) for _ in range(W)]
    idxs[-1] = idxs[0].copy()
    vals = [rs.standard_normal(K).astype(np.float32) for _ in range(W)]
    w0 = synth.base_weights(n).numpy()
    gi, gv = [to_gpu(i) for i in idxs], [to_gpu(v) for v in vals]
    if way == "misaligned":
        buf = torch.empty(K + 1, dtype=torch.int32, device=DEV)
        buf[1:].copy_(gi[1])
        gi[1] = buf[1:]
    w = to_gpu(w0)
    if way == "static":
        ld.ld_merge_sparse_static(w, gi, gv, 0.1)
    else:
        least = int(ld.load().ld_merge_sparse_workspace(n, W, None))
        ws = torch.empty(least if way == "minimum" else ld.ld_merge_sparse_workspace(n, [K] * W), dtype=torch.uint8, device=DEV)
        ld.ld_merge_sparse(w, gi, gv, 0.1, ws)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(bits(w.cpu().numpy()), bits(oracle.merge_sparse(w0, idxs, vals, 0.1)))


@pytest.mark.parametrize("W", [11, 65])
def test_merge_lane_per_record_whole_sub_tiles(W):
    # sub-tiles of 4096 that a diff records whole, four trips of 16 rows, in a window that is sparse all in all; the workspace
    # holds the table of sub-tiles of 4096 and no larger one, and so has both windows run a lane per record
    n = 2_000_003
    idxs = [np.concatenate([np.arange(4096 * 7 - t, 4096 * 8 + t), np.arange(n - 60, n)]).astype(np.int32) for t in range(W)]
    K = [i.size for i in idxs]
    nbytes = table_of(n, W, 4096)
    assert max(K) * 8192 <= 20 * n and int(ld.load().ld_merge_sparse_workspace(n, W, None)) < nbytes <= ld.ld_merge_sparse_workspace(n, K)
    rs = np.random.RandomState(W)
    vals = [(rs.standard_normal(i.size) * 1e-2).astype(np.float32) for i in idxs]
    w0 = synth.base_weights(n).numpy()
    w = to_gpu(w0)
    ld.ld_merge_sparse(w, [to_gpu(i) for i in idxs], [to_gpu(v) for v in vals], 0.1,
                       workspace=torch.empty(nbytes, dtype=torch.uint8, device=DEV), strategy=ld.LD_MERGE_SWEEP)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(bits(w.cpu().numpy()), bits(oracle.merge_sparse(w0, idxs, vals, 0.1)))


@pytest.mark.parametrize("case", ["random", "identical", "pairs", "clustered", "short_then_long"])
def test_merge_thin_long_windows(case):
    # Long windows of sparse diffs run a lane per record: the records of a sub-tile go through in rows of
    # 64, elements touched by several diffs of a row are applied in diff order.
    #   random          a few elements shared by two or three diffs
    #   identical       every diff records the same positions: a row holds each element of its diffs once per diff
    #   pairs           diffs 2j and 2j+1 share all positions, values far apart in magnitude
    #   clustered       one diff puts 300 records into two sub-tiles that have a few from the others
    #   short_then_long 70 diffs (two sets of lanes), the first ones empty or tiny
    # Each also with the minimum workspace (no per-sub-tile table: the ordinary sweep) - same bits.
    n = 3_000_017
    rs = np.random.RandomState({"random": 1, "identical": 2, "pairs": 3, "clustered": 4, "short_then_long": 5}[case])
    w0 = (rs.standard_normal(n) * 0.02).astype(np.float32)
    W, k = 100, 3000
    idxs, vals = [], []
    if case == "random":
        for t in range(W):
            idxs.append(np.sort(rs.choice(n, k, replace=False)).astype(np.int32))
    elif case == "identical":
        same = np.sort(rs.choice(n, k, replace=False)).astype(np.int32)
        idxs = [same.copy() for _ in range(W)]
    elif case == "pairs":
        for t in range(0, W, 2):
            i = np.sort(rs.choice(n, k, replace=False)).astype(np.int32)
            idxs += [i, i.copy()]
    elif case == "clustered":
        for t in range(W):
            i = rs.choice(n, k, replace=False)
            if t == 37:
                i[:300] = 16_384 + rs.choice(8192, 300, replace=False)   # sub-tile 2
            idxs.append(np.unique(i).astype(np.int32))
    else:
        W = 70
        for t in range(W):
            kk = [0, 1, 2][t] if t < 3 else k
            idxs.append(np.sort(rs.choice(n, kk, replace=False)).astype(np.int32))
    for t, i in enumerate(idxs):
        scale = 1.0 if case != "pairs" else (1e-4 if t % 2 else 10.0)
        vals.append((rs.standard_normal(i.size) * scale).astype(np.float32))
    ref = oracle.merge_sparse(w0, idxs, vals, 0.1)
    gi, gv = [to_gpu(i) for i in idxs], [to_gpu(v) for v in vals]
    K = [i.size for i in idxs]
    full_ws = ld.ld_merge_sparse_workspace(n, K)
    min_ws = int(ld.load().ld_merge_sparse_workspace(n, len(K), None))
    assert full_ws == table_of(n, len(K), 4096) > min_ws, "this window was meant to run a lane per record"
    for nbytes in (full_ws, min_ws):
        w = to_gpu(w0)
        ws = torch.empty(nbytes, dtype=torch.uint8, device=DEV)
        ld.ld_merge_sparse(w, gi, gv, 0.1, workspace=ws, strategy=ld.LD_MERGE_SWEEP)
        torch.cuda.synchronize()
        np.testing.assert_array_equal(bits(w.cpu().numpy()), bits(ref), err_msg=f"{case}, workspace {nbytes}")


@pytest.mark.parametrize("W", [11, 40, 65, 128])
def test_merge_lane_per_record_blocks(W):
    # Lists of a sub-tile around the 512 records of a block, the 128 of its end and the 64 that wait their turn together, over element pools from the
    # whole sub-tile (few wait) to 16 elements (rows take turns), within the ragged last sub-tile too. With the table
    # of sub-tiles of 4096 all of them run a lane per record.
    n = 4096 * 900 + 1234
    rs = np.random.RandomState(W)
    recs = [set() for _ in range(W)]
    totals = [1, 2, 63, 64, 65, 127, 128, 129, 511, 512, 513, 575, 1023, 1024, 1025, 1400, 640, 641]
    for s, (total, pool) in enumerate([(t, p) for t in totals for p in (4096, 1000, 300, 60, 16)] + [(300, 1234)]):
        base, span = (4096 * 900, 1234) if pool == 1234 else (4096 * (9 * s + 3), 4096)
        where = base + rs.choice(span, min(pool, span), replace=False)
        owner = rs.randint(0, W, min(total, W * where.size))
        for t, count in zip(*np.unique(owner, return_counts=True)):
            recs[t].update(rs.choice(where, min(count, where.size), replace=False).tolist())
    idxs = [np.array(sorted(r), np.int32) for r in recs]
    vals = [(rs.standard_normal(i.size) * 10.0 ** rs.uniform(-4, 1, i.size)).astype(np.float32) for i in idxs]
    K = [i.size for i in idxs]
    nbytes = table_of(n, W, 4096)
    assert max(K) * 8192 <= 48 * n and ld.ld_merge_sparse_workspace(n, K) >= nbytes
    w0 = synth.base_weights(n).numpy()
    w = to_gpu(w0)
    ld.ld_merge_sparse(w, [to_gpu(i) for i in idxs], [to_gpu(v) for v in vals], 0.1,
                       workspace=torch.empty(nbytes, dtype=torch.uint8, device=DEV), strategy=ld.LD_MERGE_SWEEP)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(bits(w.cpu().numpy()), bits(oracle.merge_sparse(w0, idxs, vals, 0.1)))


def test_merge_uneven_diffs_across_many_chunks():
    # Record positions are looked up per 49152-element chunk from guesses that assume evenly
    # spread records; these diffs are anything but (dense runs between long gaps, everything
    # in the last percent, only the first half, one record), the window spans several
    # workgroups of the lookup kernel, and two index arrays start at addresses that are
    # only 4-byte aligned.
    n = 60_000_003
    rs = np.random.RandomState(7)
    w0 = (rs.standard_normal(n) * 0.02).astype(np.float32)
    starts = np.sort(rs.choice(n - 6000, 120, replace=False)).astype(np.int64)
    runs = np.unique(np.concatenate([np.arange(s0, s0 + 5000) for s0 in starts]))
    idxs = [runs.astype(np.int32),
            (n - 600_000 + np.sort(rs.choice(600_000, 400_000, replace=False))).astype(np.int32),
            np.sort(rs.choice(n, 600_000, replace=False)).astype(np.int32),
            np.arange(0, n // 2, 64, dtype=np.int32),
            np.array([n - 1], np.int32),
            np.unique(np.concatenate([np.arange(0, 40_000), np.arange(n - 40_000, n)])).astype(np.int32)]
    vals = [rs.standard_normal(i.size).astype(np.float32) for i in idxs]
    ref = oracle.merge_sparse(w0, idxs, vals, 0.1)

    def shifted(a, shift):  # device copy whose first element sits `shift` elements into an allocation
        buf = torch.empty(a.size + shift, dtype=torch.from_numpy(a[:1]).dtype, device=DEV)
        buf[shift:].copy_(torch.from_numpy(a))
        return buf[shift:]

    gi = [shifted(i, (1, 0, 3, 0, 0, 2)[t]) for t, i in enumerate(idxs)]
    gv = [shifted(v, (0, 0, 1, 0, 0, 3)[t]) for t, v in enumerate(vals)]
    w = to_gpu(w0)
    ld.ld_merge_sparse(w, gi, gv, 0.1, strategy=ld.LD_MERGE_SWEEP)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(bits(w.cpu().numpy()), bits(ref))


def test_merge_order_and_zero_diff():
    # order sensitivity: swapping two diffs changes the fp32 result; the GPU follows list order
    n = 8192
    w0 = np.ones(n, np.float32)
    i = np.arange(n, dtype=np.int32)
    v1 = np.full(n, -(2.0 ** -24 + 2.0 ** -30), np.float32)
    v2 = np.ones(n, np.float32)
    for order in ((v1, v2), (v2, v1)):
        ref = oracle.merge_sparse(w0, [i, i], list(order), 1.0)
        w = to_gpu(w0)
        ld.ld_merge_sparse(w, [to_gpu(i), to_gpu(i)], [to_gpu(order[0]), to_gpu(order[1])], 1.0,
                           strategy=ld.LD_MERGE_SWEEP)
        torch.cuda.synchronize()
        np.testing.assert_array_equal(bits(w.cpu().numpy()), bits(ref))
    # a zero diff leaves w bit-identical, -0.0 weights included
    w0 = np.random.RandomState(0).standard_normal(n).astype(np.float32)
    w0[:100] = -0.0
    w = to_gpu(w0)
    ld.ld_merge_sparse(w, [to_gpu(i)], [to_gpu(np.zeros(n, np.float32))], 0.1, strategy=ld.LD_MERGE_SWEEP)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(bits(w.cpu().numpy()), bits(w0))


@pytest.mark.timeout(600)
def test_compress_then_merge_end_to_end_resnet_window():
    """Config 2 whole: ResNet-50-shaped, 161 segments, 1 %, the configuration's 50-diff window built by
    50 chained compress calls and merged in one call; every record, residual and weight against the oracle."""
    wl = synth.workload("resnet50")
    W = wl.window
    assert W == 50
    r_cpu = np.zeros(wl.n, np.float32)
    r_gpu = torch.zeros(wl.n, device=DEV)
    ws = torch.empty(ld.ld_compress_topk_workspace(wl.seg_off), dtype=torch.uint8, device=DEV)
    gi, gv, oi, ov = [], [], [], []
    for t in range(W):
        if t % 10 == 0:
            print(f"[resnet50 window] diff {t}", flush=True)
        g = synth.gradient(wl, t).numpy()
        a, b = ld.ld_compress_topk(to_gpu(g), r_gpu, wl.seg_off, wl.seg_k, workspace=ws)
        gi.append(a)
        gv.append(b)
        i, v, r_cpu = oracle.topk_ef(g, r_cpu, wl.seg_off, wl.seg_k, select=True)
        oi.append(i)
        ov.append(v)
    w0 = synth.base_weights(wl.n).numpy()
    w = to_gpu(w0)
    ld.ld_merge_sparse(w, gi, gv, wl.lr)
    torch.cuda.synchronize()
    for t in range(W):
        np.testing.assert_array_equal(gi[t].cpu().numpy(), oi[t], err_msg=f"idx t={t}")
        np.testing.assert_array_equal(bits(gv[t].cpu().numpy()), bits(ov[t]), err_msg=f"val t={t}")
    np.testing.assert_array_equal(bits(r_gpu.cpu().numpy()), bits(r_cpu))
    np.testing.assert_array_equal(bits(w.cpu().numpy()), bits(oracle.merge_sparse(w0, oi, ov, wl.lr)))


# ------------------------------------------------------------------ snapshot

@pytest.mark.parametrize("n", [0, 1, 7, 8191, 8192, 1 << 20, (1 << 20) + 3, 11008 * 4096])
def test_snapshot_bit_exact(n):
    src = torch.randint(-32768, 32767, (n + 9,), dtype=torch.int16, device=DEV).view(torch.bfloat16)
    for shift in (0, 1):  # 16-byte aligned and 2-byte aligned views
        s = src[shift:shift + n]
        d = torch.zeros(n + 2, dtype=torch.bfloat16, device=DEV)
        ld.ld_snapshot_layer(s, d[1:1 + n] if shift else d[:n])
        torch.cuda.synchronize()
        got = (d[1:1 + n] if shift else d[:n]).view(torch.int16).cpu().numpy().view(np.uint16)
        ref = oracle.snapshot(s.view(torch.int16).cpu().numpy().view(np.uint16))
        np.testing.assert_array_equal(got, ref)
        rest = d[:1] if shift else d[n:]
        assert torch.all(rest.view(torch.int16) == 0)  # nothing written outside


@pytest.mark.parametrize("n", [1, 2, 7, 8, 9, 15, 17, 2047, 8185, 8191, 8192, 8193, 16391, 30001])
@pytest.mark.parametrize("a,b", [(0, 0), (1, 1), (1, 0), (0, 3), (7, 2)])
def test_snapshot_at_any_two_byte_alignment(n, a, b):
    # source and destination start a and b elements past a 16-byte boundary; nothing around is written
    bits16 = torch.randint(-32768, 32767, (n + 16,), dtype=torch.int16, device=DEV)
    src = bits16.view(torch.bfloat16)
    for many in (False, True):
        out = torch.full((n + 16,), 77, dtype=torch.int16, device=DEV)
        dst = out.view(torch.bfloat16)
        if many:
            ld.ld_snapshot_layers([src[a:a + n], src[:0]], [dst[b:b + n], dst[:0]])
        else:
            ld.ld_snapshot_layer(src[a:a + n], dst[b:b + n])
        torch.cuda.synchronize()
        want = torch.full((n + 16,), 77, dtype=torch.int16)
        want[b:b + n] = bits16.cpu()[a:a + n]
        assert torch.equal(out.cpu(), want)


def test_snapshot_many_layers_one_launch():
    wl = synth.workload("llama7b")
    sizes = [s // 64 for s in wl.sizes[:40]] + [0, 1, 17]
    srcs = [torch.randint(-32768, 32767, (s,), dtype=torch.int16, device=DEV).view(torch.bfloat16) for s in sizes]
    dsts = [torch.zeros_like(s) for s in srcs]
    ld.ld_snapshot_layers(srcs, dsts)
    torch.cuda.synchronize()
    for a, b in zip(srcs, dsts):
        assert torch.equal(a.view(torch.int16), b.view(torch.int16))


@pytest.mark.parametrize("count", [1, 2, 3, 8, 15, 16, 17, 18, 175, 176, 177, 353])
def test_snapshot_layers_around_a_launch(count):
    # a launch takes 176 layers, found in groups of 16, up to 16 by a binary search; more are shared out evenly;
    # whole blocks of 8192 elements, one element less and more, empty layers, sources and destinations an element apart in alignment, nothing
    # around them written
    rs = np.random.RandomState(count)
    sizes = [int(rs.choice([1, 7, 64, 8191, 8192, 8193, 16384, 30_001, 0])) for _ in range(count)]
    sizes[-1] = 8193
    src = torch.randint(-32768, 32767, (sum(sizes) + 3 * count,), dtype=torch.int16, device=DEV)
    dst, want = torch.full_like(src, 77), torch.full_like(src, 77)
    at, srcs, dsts = 0, [], []
    for s in sizes:
        srcs.append(src[at + 1:at + 1 + s].view(torch.bfloat16))
        dsts.append(dst[at + 2:at + 2 + s].view(torch.bfloat16))
        want[at + 2:at + 2 + s] = src[at + 1:at + 1 + s]
        at += s + 3
    ld.ld_snapshot_layers(srcs, dsts)
    torch.cuda.synchronize()
    assert torch.equal(dst, want)


# ---------------------------------------------------------------------- Adam

def _bf16_bits_t(t):
    return t.view(torch.int16).cpu().numpy().view(np.uint16)


def check_adam_close(got, ref, tag):
    for name, a, b in zip("wmv", got, ref):
        a = a.cpu().numpy().astype(np.float64)
        b = b.astype(np.float64)
        err = np.abs(a - b)
        assert np.all(err <= 1e-7 + 1e-6 * np.abs(b)), f"{tag} {name}: max err {err.max()}"
    # v is a sum of non-negative terms: hold it to the relative bound alone
    a, b = got[2].cpu().numpy().astype(np.float64), ref[2].astype(np.float64)
    assert np.all(np.abs(a - b) <= 1e-6 * np.abs(b)), f"{tag} v relative"


@pytest.mark.parametrize("n", [1, 7, 8, 1000003])
@pytest.mark.parametrize("W,step0", [(1, 0), (4, 0), (3, 1000)])
def test_adam_replay_parity(n, W, step0):
    rs = np.random.RandomState(n % 97 + W)
    w0 = (rs.standard_normal(n) * 0.02).astype(np.float32)
    m0 = np.zeros(n, np.float32) if step0 == 0 else (rs.standard_normal(n) * 1e-4).astype(np.float32)
    v0 = np.zeros(n, np.float32) if step0 == 0 else (rs.standard_normal(n) ** 2 * 1e-7).astype(np.float32)
    grads = [to_gpu((rs.standard_normal(n) * 1e-3).astype(np.float32)).to(torch.bfloat16) for _ in range(W)]
    hp = dict(lr=1e-4, **synth.ADAM)
    ref = oracle.adam_replay(w0, m0, v0, [_bf16_bits_t(g) for g in grads], step0, **hp)
    w, m, v = to_gpu(w0), to_gpu(m0), to_gpu(v0)
    ld.ld_merge_dense_adam(w, m, v, grads, step0, **hp)
    torch.cuda.synchronize()
    check_adam_close((w, m, v), ref, f"n={n} W={W} step0={step0}")
    # fused window == chain of single-step calls, bit for bit
    w2, m2, v2 = to_gpu(w0), to_gpu(m0), to_gpu(v0)
    for t in range(W):
        ld.ld_merge_dense_adam(w2, m2, v2, [grads[t]], step0 + t, **hp)
    torch.cuda.synchronize()
    for a, b in ((w, w2), (m, m2), (v, v2)):
        assert torch.equal(a.view(torch.int32), b.view(torch.int32))


@pytest.mark.parametrize("eps", [0.0, 1e-20])
def test_adam_with_no_eps_and_denormal_second_moments(eps):
    # With eps = 0 (or far below the root of a denormal) the denominator is sqrt(v / bc2) alone, and for
    # gradients below 1e-19 that argument is a denormal fp32 number: a square root that takes denormals
    # for zero would divide by zero. Gradients from 1e-3 down to 3e-20, no zeros (0 / 0 has no value to
    # compare); dense replay and sparse replay of the same gradients.
    n, W = 40_003, 3
    rs = np.random.RandomState(71)
    w0 = (rs.standard_normal(n) * 0.02).astype(np.float32)
    z = np.zeros(n, np.float32)
    grads = []
    for _ in range(W):
        mag = 10.0 ** rs.uniform(-19.5, -3.0, n)
        g = (mag * np.where(rs.rand(n) < 0.5, 1.0, -1.0)).astype(np.float32)
        grads.append(to_gpu(g).to(torch.bfloat16))
    assert all(bool((g.float().abs() > 1e-20).all()) for g in grads)
    hp = dict(lr=1e-4, beta1=0.9, beta2=0.999, eps=eps)
    gb = [_bf16_bits_t(g) for g in grads]
    ref = oracle.adam_replay(w0, z, z, gb, 0, **hp)
    assert np.all(np.isfinite(ref[0]))
    assert int((grads[0].float().abs() < 1.0e-19).sum()) > 500   # first step: v / bc2 = g^2 is a denormal for these
    w, m, v = to_gpu(w0), to_gpu(z), to_gpu(z)
    ld.ld_merge_dense_adam(w, m, v, grads, 0, **hp)
    # the same gradients as sparse diffs that record every position
    ws, ms_, vs = to_gpu(w0), to_gpu(z), to_gpu(z)
    allpos = torch.arange(n, dtype=torch.int32, device=DEV)
    ld.ld_merge_sparse_adam(ws, ms_, vs, [allpos] * W, [g.float() for g in grads], 0, **hp)
    torch.cuda.synchronize()
    for got in ((w, m, v), (ws, ms_, vs)):
        for name, a, b in zip("wmv", got, ref):
            a = a.cpu().numpy().astype(np.float64)
            err = np.abs(a - b.astype(np.float64))
            assert np.all(err <= 1e-7 + 1e-6 * np.abs(b)), f"eps={eps} {name}: max err {err.max()}"
        a, b = got[2].cpu().numpy().astype(np.float64), ref[2].astype(np.float64)
        normal = b >= 1.1755e-38   # a denormal v has few bits: the relative bound is for the normal ones
        assert np.all(np.abs(a - b)[normal] <= 1e-6 * b[normal])
        assert np.all(np.abs(a - b)[~normal] <= 3e-45)   # and at most two steps of the denormal grid elsewhere
    for a, b in ((w, ws), (m, ms_), (v, vs)):
        assert torch.equal(a.view(torch.int32), b.view(torch.int32))


def test_adam_zero_gradient_and_closed_form():
    n = 4096
    hp = dict(lr=1e-2, **synth.ADAM)
    w0 = np.random.RandomState(2).standard_normal(n).astype(np.float32)
    v0 = (np.random.RandomState(3).standard_normal(n) ** 2 * 1e-6).astype(np.float32)
    w, m, v = to_gpu(w0), torch.zeros(n, device=DEV), to_gpu(v0)
    ld.ld_merge_dense_adam(w, m, v, [torch.zeros(n, dtype=torch.bfloat16, device=DEV)], 5, **hp)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(bits(w.cpu().numpy()), bits(w0))
    assert torch.all(m == 0)
    np.testing.assert_allclose(v.cpu().numpy(), np.float64(np.float32(0.999)) * v0, rtol=1e-6)
    # constant gradient from zero state: every step moves w by lr*c/(|c|+eps)
    c = torch.linspace(-2, 2, n, device=DEV).to(torch.bfloat16)
    T = 20
    w, m, v = torch.ones(n, device=DEV), torch.zeros(n, device=DEV), torch.zeros(n, device=DEV)
    ld.ld_merge_dense_adam(w, m, v, [c] * T, 0, **hp)
    torch.cuda.synchronize()
    cd = c.float().cpu().numpy().astype(np.float64)
    want = 1.0 - T * hp["lr"] * cd / (np.abs(cd) + hp["eps"])
    want[cd == 0] = 1.0
    np.testing.assert_allclose(w.cpu().numpy(), want, rtol=3e-6)


# ------------------------------------------------- sparse diffs through Adam

@pytest.mark.parametrize("n,W,dens,step0", [(1, 1, 1.0, 0), (7, 3, 0.5, 0), (2047, 4, 0.05, 3), (2049, 5, 0.01, 0),
                                            (1000003, 6, 0.01, 1000), (300000, 70, 0.004, 2),
                                            (123457, 3, 1.0, 0), (50000, 4, 0.0, 5)])
def test_sparse_adam_replay_parity(n, W, dens, step0):
    rs = np.random.RandomState(n % 1000 + W)
    w0 = (rs.standard_normal(n) * 0.02).astype(np.float32)
    m0 = np.zeros(n, np.float32) if step0 == 0 else (rs.standard_normal(n) * 1e-4).astype(np.float32)
    v0 = np.zeros(n, np.float32) if step0 == 0 else (rs.standard_normal(n) ** 2 * 1e-7).astype(np.float32)
    idxs, vals = [], []
    for t in range(W):
        kk = int(round(n * dens)) if t != 1 else min(n, int(round(n * dens * 2)))
        idxs.append(np.sort(rs.choice(n, kk, replace=False)).astype(np.int32))
        vals.append((rs.standard_normal(kk) * 1e-3).astype(np.float32))
    hp = dict(lr=1e-4, **synth.ADAM)
    print(f"[sparse_adam] n={n} W={W} dens={dens} step0={step0}", flush=True)
    ref = oracle.sparse_adam_replay(w0, m0, v0, idxs, vals, step0, **hp)
    gi, gv = [to_gpu(i) for i in idxs], [to_gpu(v) for v in vals]
    w, m, v = to_gpu(w0), to_gpu(m0), to_gpu(v0)
    ld.ld_merge_sparse_adam(w, m, v, gi, gv, step0, **hp)
    torch.cuda.synchronize()
    for name, a, b in zip("wmv", (w, m, v), ref):
        a = a.cpu().numpy().astype(np.float64)
        err = np.abs(a - b.astype(np.float64))
        assert np.all(err <= 1e-7 + 1e-6 * np.abs(b)), f"{name}: max err {err.max()}"
    # v never cancels: hold it to a relative bound alone (W roundings of 2^-24 each)
    a, b = v.cpu().numpy().astype(np.float64), ref[2].astype(np.float64)
    assert np.all(np.abs(a - b) <= max(1e-6, W * 1.2e-7) * np.abs(b)), "v relative"
    # the window in one call == one call per diff, bit for bit
    w2, m2, v2 = to_gpu(w0), to_gpu(m0), to_gpu(v0)
    for t in range(W):
        ld.ld_merge_sparse_adam(w2, m2, v2, [gi[t]], [gv[t]], step0 + t, **hp)
    torch.cuda.synchronize()
    for a, b in ((w, w2), (m, m2), (v, v2)):
        assert torch.equal(a.view(torch.int32), b.view(torch.int32))


@pytest.mark.parametrize("n,W,dens", [(1023, 3, 0.02), (1025, 2, 0.024), (49153, 5, 0.0234), (1 << 18, 3, 0.0235),
                                      ((1 << 18) + 5, 65, 0.003), (300000, 4, 0.2)])
@pytest.mark.parametrize("lr,eps", [(1e-4, 1e-8), (-1e-3, 1e-8), (1e-11, 1e-8), (2e3, 1e-8), (1e-3, 1e-12)])
def test_sparse_adam_windows_and_forms(n, W, dens, lr, eps):
    # either side of the densities where one record window per diff becomes two, sub-tile edges, more
    # than one group of diffs, and learning rates / eps on either side of the folded form's range (what small
    # learning rates do to w: the next test)
    rs = np.random.RandomState(n + W)
    w0 = synth.base_weights(n).numpy()
    m0 = (rs.standard_normal(n) * 1e-4).astype(np.float32)
    v0 = (rs.standard_normal(n) ** 2 * 1e-6).astype(np.float32)
    K = max(1, int(n * dens))
    idxs = [np.sort(rs.choice(n, K, replace=False)).astype(np.int32) for _ in range(W)]
    vals = [(rs.standard_normal(K) * 1e-2).astype(np.float32) for _ in range(W)]
    w, m, v = to_gpu(w0), to_gpu(m0), to_gpu(v0)
    hp = dict(lr=lr, beta1=0.9, beta2=0.999, eps=eps)
    ld.ld_merge_sparse_adam(w, m, v, [to_gpu(i) for i in idxs], [to_gpu(x) for x in vals], 2, **hp)
    torch.cuda.synchronize()
    ref = oracle.sparse_adam_replay(w0, m0, v0, idxs, vals, 2, **hp)
    # a step moves an element by at most about lr: each is a few ulp of its own size off
    scale = max(1.0, abs(lr) * W * 10)
    np.testing.assert_allclose(w.cpu().numpy(), ref[0], rtol=1e-6, atol=1e-7 * scale)
    np.testing.assert_allclose(m.cpu().numpy(), ref[1], rtol=1e-6, atol=1e-7)
    np.testing.assert_allclose(v.cpu().numpy(), ref[2], rtol=1e-6, atol=0)


@pytest.mark.parametrize("n", [49152 * 3, 49152 * 2 + 1027])
def test_sparse_adam_record_windows_that_miss(n):
    # where the records of a chunk of 49152 elements lie is guessed from its ends: lists shorter than a window of 64,
    # empty ones, lists that end inside a window, records crowded at a chunk's begin (the window comes too early and
    # ends too early) or end (too late), and on a few sub-tiles of 1024 alone, all in one window
    rs = np.random.RandomState(n)
    chunk = 49152

    def some(lo, hi, k):
        return lo + rs.choice(hi - lo, k, replace=False)

    idxs = [some(0, n, 63), np.zeros(0, np.int64), some(0, n, 64), some(chunk - 900, chunk, 700), some(chunk, chunk + 1500, 900),
            np.concatenate([some(0, 1024, 65), some(2 * chunk - 1024, 2 * chunk, 100)]), some(n - 1000, n, 300), some(0, n, 1),
            np.concatenate([some(chunk, chunk + 1024, 400), some(chunk + 40 * 1024, chunk + 41 * 1024, 20), some(n - 3, n, 3)]),
            some(0, n, n // 60)]
    idxs = [np.sort(np.unique(i)).astype(np.int32) for i in idxs]
    vals = [(rs.standard_normal(i.size) * 1e-2).astype(np.float32) for i in idxs]
    w0 = synth.base_weights(n).numpy()
    m0 = (rs.standard_normal(n) * 1e-4).astype(np.float32)
    v0 = (rs.standard_normal(n) ** 2 * 1e-6).astype(np.float32)
    hp = dict(lr=1e-4, **synth.ADAM)
    w, m, v = to_gpu(w0), to_gpu(m0), to_gpu(v0)
    ld.ld_merge_sparse_adam(w, m, v, [to_gpu(i) for i in idxs], [to_gpu(x) for x in vals], 2, **hp)
    torch.cuda.synchronize()
    ref = oracle.sparse_adam_replay(w0, m0, v0, idxs, vals, 2, **hp)
    # as above: a few roundings of 6e-8 per step; a record put wrong moves v by 1e-7 of its 1e-6
    np.testing.assert_allclose(w.cpu().numpy(), ref[0], rtol=1e-6, atol=1e-7)
    np.testing.assert_allclose(m.cpu().numpy(), ref[1], rtol=2e-6, atol=1e-9)
    np.testing.assert_allclose(v.cpu().numpy(), ref[2], rtol=2e-6, atol=0)


@pytest.mark.parametrize("lr,eps", [(0.99e-10, 1e-8), (1.01e-10, 1e-8), (1e-11, 1e-8), (-1e-20, 1e-8), (999.0, 1e-8),
                                    (1001.0, 1e-8), (1e-3, 3.1e-11), (1e-3, 3.3e-11), (1e-3, 999.0), (1e-3, 1001.0)])
@pytest.mark.parametrize("W", [1, 3])
def test_adam_updates_either_side_of_the_folded_form(lr, eps, W):
    # From w = 0, with moments that keep their sign, w is the sum of steps of one sign: it is as exact, relative to
    # itself, as a step. A step has some ten roundings (two of each moment, root and reciprocal of one unit,
    # scalars, denominator, product) and w one more per step: below 14 of 6e-8 each, 1e-6 with the scalars' own.
    n = 5003
    rs = np.random.RandomState(W)
    sign = np.where(rs.rand(n) < 0.5, 1, -1)
    m0 = (sign * rs.uniform(0.5e-4, 2e-4, n)).astype(np.float32)
    v0 = rs.uniform(1e-9, 1e-6, n).astype(np.float32)
    z = np.zeros(n, np.float32)
    idxs = [np.sort(rs.choice(n, 50, replace=False)).astype(np.int32) for _ in range(W)]
    vals = [rs.uniform(-1e-5, 1e-5, 50).astype(np.float32) for _ in range(W)]
    hp = dict(lr=lr, beta1=0.9, beta2=0.999, eps=eps)
    w, m, v = to_gpu(z), to_gpu(m0), to_gpu(v0)
    ld.ld_merge_sparse_adam(w, m, v, [to_gpu(i) for i in idxs], [to_gpu(x) for x in vals], 4, **hp)
    ref = oracle.sparse_adam_replay(z, m0, v0, idxs, vals, 4, **hp)
    torch.cuda.synchronize()
    assert np.all(np.abs(ref[0]) > 0)
    np.testing.assert_allclose(w.cpu().numpy(), ref[0], rtol=1e-6, atol=0)
    # the dense replay runs the same step
    gb = [to_gpu(rs.uniform(-1e-5, 1e-5, n).astype(np.float32)).bfloat16() for _ in range(W)]
    w, m, v = to_gpu(z), to_gpu(m0), to_gpu(v0)
    ld.ld_merge_dense_adam(w, m, v, gb, 4, **hp)
    every = [np.arange(n, dtype=np.int32)] * W
    ref = oracle.sparse_adam_replay(z, m0, v0, every, [b.float().cpu().numpy() for b in gb], 4, **hp)
    np.testing.assert_allclose(w.cpu().numpy(), ref[0], rtol=1e-6, atol=0)


def test_sparse_adam_equals_dense_adam_on_full_diffs():
    # diffs that record every position with bf16-representable values are dense gradients:
    # both entry points must then agree bit for bit (they share the per-element step)
    n, W = 70001, 3
    rs = np.random.RandomState(9)
    w0 = (rs.standard_normal(n) * 0.02).astype(np.float32)
    gb = [to_gpu((rs.standard_normal(n) * 1e-3).astype(np.float32)).to(torch.bfloat16) for _ in range(W)]
    hp = dict(lr=1e-4, **synth.ADAM)
    w, m, v = to_gpu(w0), torch.zeros(n, device=DEV), torch.zeros(n, device=DEV)
    ld.ld_merge_dense_adam(w, m, v, gb, 0, **hp)
    allidx = torch.arange(n, dtype=torch.int32, device=DEV)
    w2, m2, v2 = to_gpu(w0), torch.zeros(n, device=DEV), torch.zeros(n, device=DEV)
    ld.ld_merge_sparse_adam(w2, m2, v2, [allidx] * W, [g.float() for g in gb], 0, **hp)
    torch.cuda.synchronize()
    for a, b in ((w, w2), (m, m2), (v, v2)):
        assert torch.equal(a.view(torch.int32), b.view(torch.int32))


def test_sparse_adam_after_compress_resnet_window():
    # diffs as ld_compress_topk emits them (161 segments of very different sizes)
    wl = synth.workload("resnet50")
    W = 4
    r_gpu = torch.zeros(wl.n, device=DEV)
    gi, gv = [], []
    for t in range(W):
        a, b = ld.ld_compress_topk(to_gpu(synth.gradient(wl, t).numpy()), r_gpu, wl.seg_off, wl.seg_k)
        gi.append(a)
        gv.append(b)
    rs = np.random.RandomState(4)
    w0 = synth.base_weights(wl.n).numpy()
    m0 = (rs.standard_normal(wl.n) * 1e-4).astype(np.float32)
    v0 = (rs.standard_normal(wl.n) ** 2 * 1e-7).astype(np.float32)
    hp = dict(lr=1e-4, **synth.ADAM)
    w, m, v = to_gpu(w0), to_gpu(m0), to_gpu(v0)
    ld.ld_merge_sparse_adam(w, m, v, gi, gv, 10, **hp)
    torch.cuda.synchronize()
    ref = oracle.sparse_adam_replay(w0, m0, v0, [i.cpu().numpy() for i in gi], [x.cpu().numpy() for x in gv], 10, **hp)
    check_adam_close((w, m, v), ref, "resnet50 window")


# ------------------------------------------------- combine of per-worker lists

def check_combine(idxs, vals, n, scale=1.0, tag=""):
    print(f"[combine] {tag} n={n} N={len(idxs)} K={[len(i) for i in idxs][:8]}", flush=True)
    oi, ov = oracle.combine_sparse(idxs, vals, n, scale)
    gi, gv, cnt = ld.ld_combine_sparse([to_gpu(i) for i in idxs], [to_gpu(v) for v in vals], n, scale)
    torch.cuda.synchronize()
    c = int(cnt.item())
    assert c == len(oi), f"{tag}: count {c} != {len(oi)}"
    np.testing.assert_array_equal(gi[:c].cpu().numpy(), oi, err_msg=f"idx {tag}")
    np.testing.assert_array_equal(bits(gv[:c].cpu().numpy()), bits(ov), err_msg=f"val {tag}")


@pytest.mark.parametrize("n,N,dens", [(1, 1, 1.0), (100, 3, 0.3), (8191, 4, 0.05), (8193, 5, 0.5),
                                      (1000003, 8, 0.01), (3000000, 64, 0.002), (200000, 2, 1.0),
                                      (50000, 4, 0.0)])
def test_combine_parity(n, N, dens):
    rs = np.random.RandomState(n % 997 + N)
    idxs, vals = [], []
    for r in range(N):
        kk = int(round(n * dens)) if r != 1 else min(n, int(round(n * dens * 1.5)))
        idxs.append(np.sort(rs.choice(n, kk, replace=False)).astype(np.int32))
        vals.append(rs.standard_normal(kk).astype(np.float32))
    check_combine(idxs, vals, n, tag="sum")
    check_combine(idxs, vals, n, scale=1.0 / N, tag="mean")


def test_combine_worker_order_cancellation_and_clusters():
    n = 100000
    one = np.array([77777], np.int32)
    a, b, c = np.float32(1.0), np.float32(2.0 ** -24), np.float32(2.0 ** -24)
    check_combine([one, one, one], [np.array([a]), np.array([b]), np.array([c])], n, tag="order abc")
    check_combine([one, one, one], [np.array([b]), np.array([c]), np.array([a])], n, tag="order bca")
    i = np.arange(100, 5000, 7, dtype=np.int32)
    v = np.random.RandomState(0).standard_normal(len(i)).astype(np.float32)
    check_combine([i, i], [v, -v], n, tag="cancel")  # zeros stay in the list
    # all records of every worker packed into one corner, the rest of the index space empty
    rs = np.random.RandomState(1)
    idxs = [np.sort(rs.choice(9000, 3000, replace=False)).astype(np.int32) + 40000 for _ in range(5)]
    vals = [rs.standard_normal(3000).astype(np.float32) for _ in range(5)]
    check_combine(idxs, vals, n, tag="clustered")
    # nothing at all, and a single empty worker among full ones
    e = np.zeros(0, np.int32)
    check_combine([e, e], [e.astype(np.float32)] * 2, n, tag="empty")
    check_combine([idxs[0], e, idxs[1]], [vals[0], e.astype(np.float32), vals[1]], n, tag="one empty")


def test_combine_of_compressed_diffs_and_truncated_output():
    # lists as ld_compress_topk emits them for 4 "workers" (different gradients, same segments)
    wl = synth.workload("resnet50")
    gi, gv = [], []
    for t in range(4):
        r = torch.zeros(wl.n, device=DEV)
        a, b = ld.ld_compress_topk(to_gpu(synth.gradient(wl, t).numpy()), r, wl.seg_off, wl.seg_k)
        gi.append(a)
        gv.append(b)
    torch.cuda.synchronize()
    idxs, vals = [x.cpu().numpy() for x in gi], [x.cpu().numpy() for x in gv]
    check_combine(idxs, vals, wl.n, scale=0.25, tag="resnet50 x4")
    # an output buffer that is too small: the count still tells the full size, nothing is written past the end
    oi, ov = oracle.combine_sparse(idxs, vals, wl.n, 0.25)
    cap = len(oi) // 2
    out_i = torch.full((cap + 64,), -1, dtype=torch.int32, device=DEV)
    out_v = torch.zeros(cap + 64, device=DEV)
    _, _, cnt = ld.ld_combine_sparse(gi, gv, wl.n, 0.25, out_idx=out_i[:cap], out_val=out_v[:cap])
    torch.cuda.synchronize()
    assert int(cnt.item()) == len(oi)
    np.testing.assert_array_equal(out_i[:cap].cpu().numpy(), oi[:cap])
    assert bool((out_i[cap:] == -1).all())


def test_snapshot_into_pinned_host_memory():
    # the paper's snapshot leaves the GPU: the same entry points with a page-locked host destination
    n = (1 << 22) + 5
    src = torch.randint(-32768, 32767, (n,), dtype=torch.int16, device=DEV).view(torch.bfloat16)
    dst = torch.zeros(n, dtype=torch.bfloat16).pin_memory()
    ld.ld_snapshot_layer(src, dst)
    torch.cuda.synchronize()
    assert torch.equal(dst.view(torch.int16), src.cpu().view(torch.int16))
    sizes = [1, 4096, 70001, 1 << 20]
    srcs = [torch.randint(-32768, 32767, (k,), dtype=torch.int16, device=DEV).view(torch.bfloat16) for k in sizes]
    dsts = [torch.zeros(k, dtype=torch.bfloat16).pin_memory() for k in sizes]
    ld.ld_snapshot_layers(srcs, dsts)
    torch.cuda.synchronize()
    for a, b in zip(srcs, dsts):
        assert torch.equal(b.view(torch.int16), a.cpu().view(torch.int16))


# ------------------------------------------------------------ pipelined recovery

@pytest.mark.parametrize("least", [True, False])
def test_merge_from_pinned_host_with_the_least_workspace(least):
    # a group of sparse diffs runs a lane per record where the workspace holds its table, as a sweep otherwise
    n, W = 500_003, 24
    rs = np.random.RandomState(7)
    w0 = (rs.standard_normal(n) * 0.02).astype(np.float32)
    idxs = [np.sort(rs.choice(n, n * 30 // 8192, replace=False)).astype(np.int32) for _ in range(W)]
    vals = [rs.standard_normal(i.size).astype(np.float32) for i in idxs]
    need = [int(ld.load().ld_merge_sparse_workspace(n, 12, None)), ld.ld_merge_sparse_workspace(n, [i.size for i in idxs[:12]])]
    assert need[0] < need[1]
    w = to_gpu(w0)
    ld.ld_merge_sparse_from_host(w, [torch.from_numpy(i).pin_memory() for i in idxs],
                                 [torch.from_numpy(v).pin_memory() for v in vals], 0.1, group=12,
                                 workspace=torch.empty(need[0 if least else 1], dtype=torch.uint8, device=DEV))
    torch.cuda.synchronize()
    np.testing.assert_array_equal(bits(w.cpu().numpy()), bits(oracle.merge_sparse(w0, idxs, vals, 0.1)))


@pytest.mark.parametrize("group", [1, 2, 3, 64])
def test_merge_from_pinned_host_equals_the_window_merge(group):
    # diffs in page-locked host memory, copied group by group on one stream while the previous
    # group is merged on another: same bits as the one-call merge and as the oracle
    n, W = 3_000_001, 7
    rs = np.random.RandomState(41 + group)
    w0 = (rs.standard_normal(n) * 0.02).astype(np.float32)
    idxs, vals = [], []
    for t in range(W):
        kk = [30_000, 0, 45_000, 1, 30_000, 60_000, 29_999][t]
        idxs.append(np.sort(rs.choice(n, kk, replace=False)).astype(np.int32))
        vals.append(rs.standard_normal(kk).astype(np.float32))
    ref = oracle.merge_sparse(w0, idxs, vals, 0.1)
    hi = [torch.from_numpy(i).pin_memory() for i in idxs]
    hv = [torch.from_numpy(v).pin_memory() for v in vals]
    copy_s, merge_s = torch.cuda.Stream(), torch.cuda.Stream()
    w = to_gpu(w0)
    torch.cuda.synchronize()
    ld.ld_merge_sparse_from_host(w, hi, hv, 0.1, group=group, copy_stream=copy_s, merge_stream=merge_s)
    merge_s.synchronize()
    copy_s.synchronize()
    np.testing.assert_array_equal(bits(w.cpu().numpy()), bits(ref))
    # both roles on the current stream, twice in a row with the same staging buffers
    w2 = to_gpu(w0)
    K = [i.numel() for i in hi]
    staging = torch.empty(max(256, ld.load().ld_merge_sparse_from_host_staging(
        np.array(K, np.int64).ctypes.data_as(__import__("ctypes").c_void_p), W, min(group, W))), dtype=torch.uint8, device=DEV)
    for _ in range(2):
        w2.copy_(to_gpu(w0))
        ld.ld_merge_sparse_from_host(w2, hi, hv, 0.1, group=group, staging=staging)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(bits(w2.cpu().numpy()), bits(ref))
    # with four events of the caller's the call creates none of its own; the same events serve call after call
    import ctypes
    hip = ctypes.CDLL("libamdhip64.so")
    events = []
    for _ in range(4):
        e = ctypes.c_void_p()
        assert hip.hipEventCreateWithFlags(ctypes.byref(e), 2) == 0     # hipEventDisableTiming
        events.append(e.value)
    for _ in range(2):
        w3 = to_gpu(w0)
        torch.cuda.synchronize()
        ld.ld_merge_sparse_from_host(w3, hi, hv, 0.1, group=group, copy_stream=copy_s, merge_stream=merge_s, events=events)
        merge_s.synchronize()
        copy_s.synchronize()
        np.testing.assert_array_equal(bits(w3.cpu().numpy()), bits(ref))
    for e in events:
        assert hip.hipEventDestroy(ctypes.c_void_p(e)) == 0


# ------------------------------------------------- workspaces hold anything on entry

@pytest.mark.parametrize("fill", [0x00, 0xFF, 0x5A, "random"])
def test_workspace_and_output_contents_on_entry_are_irrelevant(fill):
    def dirty(nbytes):
        if fill == "random":
            return torch.randint(0, 256, (nbytes,), dtype=torch.uint8, device=DEV)
        return torch.full((nbytes,), fill, dtype=torch.uint8, device=DEV)

    sizes = [70001, 64, 300000, 0, 4097, 200000]
    off = synth.seg_offsets(sizes)
    k = synth.seg_topk(sizes, 1, 100) * (np.array(sizes) > 0)
    n, K = int(off[-1]), int(k.sum())
    rs = np.random.RandomState(9)
    g = rs.standard_normal(n).astype(np.float32)
    g[70065:370065][rs.rand(300000) < 0.7] = np.float32(0.25)     # massive ties in the large segment
    r0 = (rs.standard_normal(n) * 0.1).astype(np.float32)
    r0[70065:370065] = 0
    oi, ov, orr = oracle.topk_ef(g, r0, off, k, select=True)
    for strategy in (ld.LD_COMPRESS_AUTO, ld.LD_COMPRESS_FULL):
        ws = dirty(ld.ld_compress_topk_workspace(off, k))
        out_i = dirty(4 * K).view(torch.int32)
        out_v = dirty(4 * K).view(torch.float32)
        r = to_gpu(r0)
        ld.ld_compress_topk(to_gpu(g), r, off, k, out_i, out_v, ws, strategy=strategy)
        ld.ld_compress_topk(to_gpu(g), to_gpu(r0), off, k, out_i, out_v, ws, strategy=strategy)  # reused as left
        torch.cuda.synchronize()
        np.testing.assert_array_equal(out_i.cpu().numpy(), oi)
        np.testing.assert_array_equal(bits(out_v.cpu().numpy()), bits(ov))
        np.testing.assert_array_equal(bits(r.cpu().numpy()), bits(orr))
    # the replays and the combine on two diffs
    g2 = rs.standard_normal(n).astype(np.float32)
    oi2, ov2, _ = oracle.topk_ef(g2, orr, off, k, select=True)
    idxs, vals = [oi, oi2], [ov, ov2]
    w0 = (rs.standard_normal(n) * 0.02).astype(np.float32)
    w = to_gpu(w0)
    ld.ld_merge_sparse(w, [to_gpu(i) for i in idxs], [to_gpu(v) for v in vals], 0.1,
                       dirty(ld.ld_merge_sparse_workspace(n, [K, K])), strategy=ld.LD_MERGE_SWEEP)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(bits(w.cpu().numpy()), bits(oracle.merge_sparse(w0, idxs, vals, 0.1)))
    z = np.zeros(n, np.float32)
    wa, ma, va = to_gpu(w0), to_gpu(z), to_gpu(z)
    ld.ld_merge_sparse_adam(wa, ma, va, [to_gpu(i) for i in idxs], [to_gpu(v) for v in vals], 0, 1e-4, **synth.ADAM,
                            workspace=dirty(ld.ld_merge_sparse_adam_workspace(n, [K, K])))
    torch.cuda.synchronize()
    check_adam_close((wa, ma, va), oracle.sparse_adam_replay(w0, z, z, idxs, vals, 0, 1e-4, **synth.ADAM), "sparse adam")
    c_i, c_v, c_n = ld.ld_combine_sparse([to_gpu(i) for i in idxs], [to_gpu(v) for v in vals], n, 1.0,
                                         dirty(8 * K).view(torch.int32), dirty(8 * K).view(torch.float32),
                                         dirty(8).view(torch.int64), dirty(ld.ld_combine_sparse_workspace(n, 2)))
    torch.cuda.synchronize()
    e_i, e_v = oracle.combine_sparse(idxs, vals, n, 1.0)
    cnt = int(c_n.item())
    assert cnt == e_i.size
    np.testing.assert_array_equal(c_i[:cnt].cpu().numpy(), e_i)
    np.testing.assert_array_equal(bits(c_v[:cnt].cpu().numpy()), bits(e_v))


# ------------------------------------------------------ checking a loaded diff

def test_check_diff_counts_match_oracle():
    n = 5_000_000
    rs = np.random.RandomState(3)
    good = np.sort(rs.choice(n, 300_001, replace=False)).astype(np.int32)
    vals = rs.standard_normal(good.size).astype(np.float32)
    cases = {"good": (good, vals), "no values": (good, None), "empty": (good[:0], vals[:0]), "one": (good[:1], vals[:1])}
    bad = good.copy()
    bv = vals.copy()
    # damage at the start, at workgroup boundaries (2048 records each), in the ragged tail
    for j in (0, 1, 2047, 2048, 2049, 4096, 100_000, 299_999, 300_000):
        bad[j] = bad[j - 1] if j and j % 2 else (-7 if j % 3 == 0 else n + j)
    bv[[0, 2048, 123_456, 300_000]] = np.nan
    bv[5] = np.inf
    cases["damaged"] = (bad, bv)
    cases["descending"] = (good[::-1].copy(), vals)
    cases["all equal"] = (np.full(10_000, 17, np.int32), np.zeros(10_000, np.float32))
    counts = torch.empty(3, dtype=torch.int64, device=DEV)
    for name, (i, v) in cases.items():
        got = ld.ld_check_diff(to_gpu(i), None if v is None else to_gpu(v), n, counts)
        torch.cuda.synchronize()
        assert tuple(got.cpu().tolist()) == oracle.check_diff(i, v, n), name
    assert tuple(ld.ld_check_diff(to_gpu(good), to_gpu(vals), int(good[-1])).cpu().tolist()) == (1, 0, 0)


@pytest.mark.parametrize("K", [1, 4095, 4096, 4097, 8192, 20481])
@pytest.mark.parametrize("skip", [0, 1])
def test_check_diff_at_workgroup_edges(K, skip):
    # whole workgroups read 16 bytes at a time, the last one and misaligned arrays element by element
    rs = np.random.RandomState(K)
    n = 1 << 20
    i = np.sort(rs.choice(n, K + skip, replace=False)).astype(np.int32)
    v = rs.standard_normal(K + skip).astype(np.float32)
    for j in {0, 3, 4, 255, 256, 1023, 1024, 4095, 4096, K - 1}:
        if j < K:
            i[skip + j] = [i[skip + j - 1], -1, n, 5][j % 4] if skip + j else -1
            v[skip + j] = np.nan if j % 3 == 0 else v[skip + j]
    gi, gv = to_gpu(i)[skip:], to_gpu(v)[skip:]
    got = ld.ld_check_diff(gi, gv, n)
    torch.cuda.synchronize()
    assert tuple(got.cpu().tolist()) == oracle.check_diff(i[skip:], v[skip:], n)


@pytest.mark.parametrize("K", [4098, 16381, 16383, 16384, 16385, 20_480, 33_000])
def test_check_diff_in_one_workgroup_and_beyond(K):
    # up to 16384 records one workgroup writes the counts itself, whatever they held before; damage in the last, broken vectors too
    rs = np.random.RandomState(K)
    n = 1 << 20
    i = np.sort(rs.choice(n, K, replace=False)).astype(np.int32)
    v = rs.standard_normal(K).astype(np.float32)
    for j in (0, 63, 255, 256, 1024, 4096, K - 5, K - 2, K - 1):
        i[j] = [-3, n + 9, i[j - 1]][j % 3] if j else i[j]
        v[j] = np.nan
    counts = torch.full((3,), -1, dtype=torch.int64, device=DEV)
    for _ in range(2):
        ld.ld_check_diff(to_gpu(i), to_gpu(v), n, counts)
        torch.cuda.synchronize()
        assert tuple(counts.cpu().tolist()) == oracle.check_diff(i, v, n)


# ------------------------------------------------------------ graph capture

def test_calls_can_be_captured_in_a_graph_and_replayed():
    # The entry points only enqueue kernels on the caller's stream (no allocation, no copy, no
    # memset, no synchronisation), so a compress + merge + Adam sequence can be captured once and
    # replayed. Every replay, with fresh inputs and eager work in between, must give what
    # the oracle gives.
    wl = synth.workload("flat1m")
    off, k = wl.seg_off, wl.seg_k
    K = int(k.sum())
    n = wl.n
    g = torch.zeros(n, device=DEV)
    r = torch.zeros(n, device=DEV)
    w = torch.zeros(n, device=DEV)
    m = torch.zeros(n, device=DEV)
    v = torch.zeros(n, device=DEV)
    gb = torch.zeros(n, dtype=torch.bfloat16, device=DEV)
    snap = torch.zeros(n, dtype=torch.bfloat16, device=DEV)
    oi = torch.empty(K, dtype=torch.int32, device=DEV)
    ov = torch.empty(K, dtype=torch.float32, device=DEV)
    ws_c = torch.empty(ld.ld_compress_topk_workspace(off, k), dtype=torch.uint8, device=DEV)
    ws_m = torch.empty(ld.ld_merge_sparse_workspace(n, [K]), dtype=torch.uint8, device=DEV)

    def sequence():
        ld.ld_compress_topk(g, r, off, k, oi, ov, ws_c)
        ld.ld_merge_sparse(w, [oi], [ov], wl.lr, ws_m, strategy=ld.LD_MERGE_SWEEP)
        ld.ld_snapshot_layer(gb, snap)
        ld.ld_merge_dense_adam(w, m, v, [snap], 0, 1e-4, **synth.ADAM)

    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        sequence()  # warm-up outside the capture
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        sequence()

    r_host = np.zeros(n, np.float32)
    for rep in range(3):
        g_host = synth.gradient(wl, 10 + rep).numpy()
        w_host = synth.base_weights(n).numpy() * np.float32(1 + rep)
        gb_t = (synth.gradient(wl, 20 + rep) * 1e-3).to(torch.bfloat16)
        g.copy_(torch.from_numpy(g_host))
        r.copy_(torch.from_numpy(r_host))
        w.copy_(torch.from_numpy(w_host))
        m.zero_()
        v.zero_()
        gb.copy_(gb_t)
        graph.replay()
        torch.cuda.synchronize()
        ei, ev, er = oracle.topk_ef(g_host, r_host, off, k, select=True)
        np.testing.assert_array_equal(oi.cpu().numpy(), ei, err_msg=f"replay {rep}")
        np.testing.assert_array_equal(bits(ov.cpu().numpy()), bits(ev), err_msg=f"replay {rep}")
        np.testing.assert_array_equal(bits(r.cpu().numpy()), bits(er), err_msg=f"replay {rep}")
        w_merged = oracle.merge_sparse(w_host, [ei], [ev], wl.lr)
        gbits = gb_t.view(torch.int16).numpy().view(np.uint16)
        np.testing.assert_array_equal(snap.cpu().view(torch.int16).numpy().view(np.uint16), gbits)
        zeros = np.zeros(n, np.float32)
        rw, rm, rv = oracle.adam_replay(w_merged, zeros, zeros, [gbits], 0, 1e-4, **synth.ADAM)
        check_adam_close((w, m, v), (rw, rm, rv), f"replay {rep}")
        r_host = er
        # eager work between the replays, on the same buffers' neighbours
        torch.randn(1 << 20, device=DEV).sum().item()


# ------------------------------------------------------------ two streams

def test_independent_calls_on_two_streams_do_not_interfere():
    # The library keeps no state between calls and works only in the buffers it is handed: two
    # pipelines (chained compress calls, then the window merge), each with buffers and workspaces of
    # its own, enqueued alternately on two streams so that their kernels overlap on the GPU, must
    # each give what the oracle gives for it alone.
    T = 3
    cases = []
    for seed, sizes, rho in ((5, [1_500_000, 70_001, 2_300_000, 4096, 900_000, 3], (1, 100)),
                             (6, [65_537, 3_100_000, 0, 1_000_000, 131_072], (3, 100))):
        rs = np.random.RandomState(seed)
        off = synth.seg_offsets(sizes)
        k = synth.seg_topk(sizes, *rho) * (np.array(sizes) > 0)
        n, K = int(off[-1]), int(k.sum())
        case = dict(
            off=off, k=k, n=n, K=K, lr=0.1 * (seed - 4),
            g=[(rs.standard_t(3, n) * 1e-3).astype(np.float32) for _ in range(T)],
            r0=(rs.standard_normal(n) * 1e-4).astype(np.float32),
            w0=synth.base_weights(n).numpy() * np.float32(seed),
            stream=torch.cuda.Stream())
        case["g_gpu"] = [to_gpu(x) for x in case["g"]]
        case["r_gpu"] = to_gpu(case["r0"])
        case["w_gpu"] = to_gpu(case["w0"])
        case["idx"] = [torch.empty(K, dtype=torch.int32, device=DEV) for _ in range(T)]
        case["val"] = [torch.empty(K, dtype=torch.float32, device=DEV) for _ in range(T)]
        case["ws_c"] = torch.empty(ld.ld_compress_topk_workspace(off, k), dtype=torch.uint8, device=DEV)
        case["ws_m"] = torch.empty(ld.ld_merge_sparse_workspace(n, [K] * T), dtype=torch.uint8, device=DEV)
        cases.append(case)
    torch.cuda.synchronize()
    for t in range(T):
        for c in cases:
            ld.ld_compress_topk(c["g_gpu"][t], c["r_gpu"], c["off"], c["k"], c["idx"][t], c["val"][t], c["ws_c"],
                                stream=c["stream"])
    for c in cases:
        ld.ld_merge_sparse(c["w_gpu"], c["idx"], c["val"], c["lr"], c["ws_m"], stream=c["stream"])
    torch.cuda.synchronize()
    for j, c in enumerate(cases):
        r = c["r0"]
        idxs, vals = [], []
        for t in range(T):
            oi, ov, r = oracle.topk_ef(c["g"][t], r, c["off"], c["k"], select=True)
            np.testing.assert_array_equal(c["idx"][t].cpu().numpy(), oi, err_msg=f"pipeline {j} idx t={t}")
            np.testing.assert_array_equal(bits(c["val"][t].cpu().numpy()), bits(ov), err_msg=f"pipeline {j} val t={t}")
            idxs.append(oi)
            vals.append(ov)
        np.testing.assert_array_equal(bits(c["r_gpu"].cpu().numpy()), bits(r), err_msg=f"pipeline {j} residual")
        w = oracle.merge_sparse(c["w0"], idxs, vals, c["lr"])
        np.testing.assert_array_equal(bits(c["w_gpu"].cpu().numpy()), bits(w), err_msg=f"pipeline {j} w")


# ------------------------------------------------------------ randomised shapes

def _random_case(seed):
    """Segment table, k per segment, gradient and residual drawn from a mixture of shapes and value laws
    (tiny to 2.5 M-element segments; k from 0 to n_s; normal, heavy-tailed, quantised, mostly-zero,
    constant and fp16-rounded values; zero, random or cancelling residual)."""
    rs = np.random.RandomState(seed)
    sizes = []
    for _ in range(int(rs.choice([1, 2, 3, 8, 25]))):
        u = rs.rand()
        sizes.append(int(rs.randint(0, 200) if u < 0.25 else rs.randint(200, 70000) if u < 0.6
                         else rs.randint(70000, 600000) if u < 0.9 else rs.randint(600000, 2500000)))
    off = synth.seg_offsets(sizes)
    n = int(off[-1])
    ks = []
    for s_ in sizes:
        u = rs.rand()
        k_ = (0 if s_ == 0 else max(1, int(np.ceil(s_ * rs.choice([0.001, 0.01, 0.03, 0.1])))) if u < 0.5
              else int(rs.randint(0, s_ + 1)) if u < 0.7 else s_ if u < 0.8 else 1 if u < 0.9 else 0)
        ks.append(min(s_, k_))
    u = rs.rand()
    if u < 0.35:
        g = rs.standard_normal(n).astype(np.float32)
    elif u < 0.5:
        g = (rs.standard_t(3, n) * 1e-3).astype(np.float32)
    elif u < 0.65:
        g = (np.round(rs.standard_normal(n) * rs.choice([2, 8, 64])) / 8).astype(np.float32)
    elif u < 0.8:
        g = rs.standard_normal(n).astype(np.float32)
        g[rs.rand(n) < rs.choice([0.5, 0.9, 0.995])] = 0
    elif u < 0.9:
        g = np.full(n, rs.choice([0.0, 1.5, -2.0]), np.float32)
    else:
        g = rs.standard_normal(n).astype(np.float32).astype(np.float16).astype(np.float32)
    r = np.zeros(n, np.float32) if rs.rand() < 0.4 else (rs.standard_normal(n) * 0.3).astype(np.float32)
    if rs.rand() < 0.2:
        r = (-g).astype(np.float32)
    return rs, off, np.array(ks, np.int32), g, r


def test_configuration_model_fed_with_measured_costs():
    # Sec. V-C closed loop, as bench.py runs it: R_B(b) and C_B(b) measured with this library (window merge
    # fed from page-locked host memory; diffs copied out to it), handed to ld_config_select over the 24
    # candidates of the paper's Example; every T_w and the selection must be what the oracle's Eq. (10) gives
    # for the same measured inputs.
    import bench
    leg = bench.SparseLeg(synth.workload("resnet50"), torch.device(DEV), pool=4)
    leg.step(bench.Timer())            # fills the window's 50 diffs
    torch.cuda.synchronize()
    row = bench.config_model_row(leg)
    st, ms = row["stated"], row["measured_s"]
    fs, bs = (10, 30, 50, 100), row["b_values"]
    assert list(bs) == [1, 2, 3, 4, 5, 6]
    tw = {}
    for f in fs:
        for b in bs:
            tw[(f, b)] = oracle.wasted_time(st["N"], st["T_s"], st["M_s"], st["tau_s"], f, b, ms["R_F"], ms["R_B"][str(b)],
                                            ms["C_F"], ms["C_B"][str(b)])
    best = min(tw, key=tw.get)
    assert (row["selected"]["f"], row["selected"]["b"]) == best
    assert abs(row["selected"]["T_w_s"] - tw[best]) <= 1e-12 * tw[best]
    for f in fs:
        for j, b in enumerate(bs):
            assert abs(row["T_w_normalised"][f"f={f}"][j] - tw[(f, b)] / tw[best]) <= 1e-12 * tw[(f, b)] / tw[best]
    for b in bs:
        want = oracle.critical_interval(st["M_s"], st["tau_s"], b, ms["R_B"][str(b)], ms["C_F"], ms["C_B"][str(b)])
        assert abs(row["f_c"][str(b)] - want) <= 1e-12 * want
        assert 0 < ms["C_replay"][str(b)] <= ms["R_B"][str(b)]      # replay is part of the recovery of a batch
    assert all(ms["R_B"][str(b)] > 0 and ms["C_B"][str(b)] > 0 for b in bs) and ms["C_F"] > 0 and ms["R_F"] > 0


def test_binding_temporaries_outlive_work_on_a_side_stream():
    # The binding allocates a workspace itself when none is given and drops it when the call
    # returns. With the kernels enqueued on a side stream that is still busy, torch's allocator
    # must not hand that block to the next allocation on the default stream: the block is marked as
    # in use on the side stream. Here the default stream grabs and zeroes same-sized blocks right
    # after the call (an all-zero chunk table would make the merge skip every record).
    n, W = 6_000_000, 12
    rs = np.random.RandomState(5)
    w0 = (rs.standard_normal(n) * 0.02).astype(np.float32)
    idxs, vals = [], []
    for t in range(W):
        i = np.sort(rs.choice(n, n // 100, replace=False)).astype(np.int32)
        idxs.append(i)
        vals.append(rs.standard_normal(i.size).astype(np.float32))
    ref = oracle.merge_sparse(w0, idxs, vals, 0.1)
    gi, gv = [to_gpu(i) for i in idxs], [to_gpu(v) for v in vals]
    ws_bytes = ld.ld_merge_sparse_workspace(n, [i.size for i in idxs])
    side = torch.cuda.Stream()
    ballast = torch.empty(1 << 28, dtype=torch.float32, device=DEV)  # 1 GiB: each fill keeps the side stream busy
    w = to_gpu(w0)
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        for _ in range(12):
            ballast.fill_(1.0)
    ld.ld_merge_sparse(w, gi, gv, 0.1, stream=side, strategy=ld.LD_MERGE_SWEEP)   # workspace allocated inside
    grabbed = [torch.zeros(ws_bytes, dtype=torch.uint8, device=DEV) for _ in range(4)]  # default stream, at once
    torch.cuda.synchronize()
    np.testing.assert_array_equal(bits(w.cpu().numpy()), bits(ref))
    del grabbed, ballast


@pytest.mark.parametrize("block", range(4))
def test_randomised_shapes_against_the_oracle(block):
    for seed in range(100 * block, 100 * block + 12):
        rs, off, k, g, r = _random_case(seed)
        n = int(off[-1])
        print(f"[random] seed={seed} n={n} n_seg={len(k)} K={int(k.sum())}", flush=True)
        W = int(rs.choice([1, 2, 5]))
        idxs, vals, r_ref = [], [], r
        r_gpu = to_gpu(r)
        for t in range(W):
            gt = g if t == 0 else (rs.standard_normal(n) * 0.5).astype(np.float32)
            oi, ov, r_ref = oracle.topk_ef(gt, r_ref, off, k, select=True)
            nbytes = ld.ld_compress_topk_workspace(off) if rs.rand() < 0.3 else ld.ld_compress_topk_workspace(off, k)
            gi, gv = ld.ld_compress_topk(to_gpu(gt), r_gpu, off, k,
                                         workspace=torch.empty(nbytes, dtype=torch.uint8, device=DEV))
            torch.cuda.synchronize()
            np.testing.assert_array_equal(gi.cpu().numpy(), oi, err_msg=f"idx seed {seed} t {t}")
            np.testing.assert_array_equal(bits(gv.cpu().numpy()), bits(ov), err_msg=f"val seed {seed} t {t}")
            np.testing.assert_array_equal(bits(r_gpu.cpu().numpy()), bits(r_ref), err_msg=f"residual seed {seed} t {t}")
            idxs.append(oi)
            vals.append(ov)
        if n == 0:
            continue
        w0 = (rs.standard_normal(n) * 0.02).astype(np.float32)
        ref = oracle.merge_sparse(w0, idxs, vals, 0.1)
        for strategy in (ld.LD_MERGE_SWEEP, ld.LD_MERGE_SCATTER):
            w = to_gpu(w0)
            ld.ld_merge_sparse(w, [to_gpu(i) for i in idxs], [to_gpu(v) for v in vals], 0.1, strategy=strategy)
            torch.cuda.synchronize()
            np.testing.assert_array_equal(bits(w.cpu().numpy()), bits(ref), err_msg=f"merge seed {seed}")
        z = np.zeros(n, np.float32)
        wa, ma, va = to_gpu(w0), to_gpu(z), to_gpu(z)
        ld.ld_merge_sparse_adam(wa, ma, va, [to_gpu(i) for i in idxs], [to_gpu(v) for v in vals], 3, 1e-3, **synth.ADAM)
        torch.cuda.synchronize()
        check_adam_close((wa, ma, va), oracle.sparse_adam_replay(w0, z, z, idxs, vals, 3, 1e-3, **synth.ADAM),
                         f"sparse adam seed {seed}")
        ci, cv, cn = ld.ld_combine_sparse([to_gpu(i) for i in idxs], [to_gpu(v) for v in vals], n, 1.0)
        torch.cuda.synchronize()
        ei, ev = oracle.combine_sparse(idxs, vals, n, 1.0)
        cnt = int(cn.item())
        assert cnt == ei.size, f"combine count seed {seed}"
        np.testing.assert_array_equal(ci[:cnt].cpu().numpy(), ei, err_msg=f"combine idx seed {seed}")
        np.testing.assert_array_equal(bits(cv[:cnt].cpu().numpy()), bits(ev), err_msg=f"combine val seed {seed}")


def test_randomised_dense_replays_against_the_oracle():
    rs = np.random.RandomState(77)
    for case in range(16):
        n = int(rs.choice([1, 3, 4095, 4096, 4097, 65537, 300001, 1500000]))
        W = int(rs.randint(1, 10))
        step0 = int(rs.choice([0, 1, 7, 1000, 123456]))
        hp = dict(lr=float(10.0 ** rs.uniform(-5, -2)), beta1=float(rs.choice([0.0, 0.8, 0.9])),
                  beta2=float(rs.choice([0.9, 0.99, 0.999])), eps=float(rs.choice([1e-8, 1e-6])))
        print(f"[random dense] case={case} n={n} W={W} step0={step0} {hp}", flush=True)
        w0 = (rs.standard_normal(n) * 0.02).astype(np.float32)
        m0 = (rs.standard_normal(n) * 1e-3).astype(np.float32)
        v0 = (rs.standard_normal(n) ** 2 * 1e-6).astype(np.float32)
        scale = float(10.0 ** rs.uniform(-4, 0))
        grads = [torch.from_numpy((rs.standard_normal(n) * scale).astype(np.float32)).to(torch.bfloat16) for _ in range(W)]
        gbits = [g.view(torch.int16).numpy().view(np.uint16) for g in grads]
        src = [g.to(DEV) for g in grads]
        snaps = [torch.empty_like(s) for s in src]
        if case % 2:
            ld.ld_snapshot_layers(src, snaps)
        else:
            for a, b in zip(src, snaps):
                ld.ld_snapshot_layer(a, b)
        w, m, v = to_gpu(w0), to_gpu(m0), to_gpu(v0)
        ld.ld_merge_dense_adam(w, m, v, snaps, step0, **hp)
        torch.cuda.synchronize()
        for s_, b_ in zip(snaps, gbits):
            np.testing.assert_array_equal(s_.cpu().view(torch.int16).numpy().view(np.uint16), b_)
        check_adam_close((w, m, v), oracle.adam_replay(w0, m0, v0, gbits, step0, **hp), f"case {case}")


@pytest.mark.parametrize("n,K", [(5_000_000, 5_000_000), (5_400_013, 5_000_003), (90_000_001, 5_000_064),
                                 (310_000_007, 6_000_001)])
@pytest.mark.parametrize("shift", [0, 4])  # floats: 4 leaves w off its granules, word by word
def test_scatter_by_granules(n, K, shift):
    """Diffs of 5 M records and more: every element, neighbours within a granule and across waves, an array that ends
    inside a granule, denormals, infinities and NaNs beside the records. The definition in torch, bit for bit."""
    print(f"[scatter] granules n={n} K={K} shift={shift}", flush=True)
    gen = torch.Generator(device=DEV).manual_seed(n + K)
    gaps = torch.randint(0, 2 * (n - K) // K + 1, (K,), generator=gen, device=DEV)
    idx = torch.cumsum(gaps + 1, 0) - 1
    idx = torch.minimum(idx, n - K + torch.arange(K, device=DEV)).to(torch.int32)
    idx[-1] = n - 1
    val = torch.randn(K, generator=gen, device=DEV)
    w = torch.randn(n + shift, generator=gen, device=DEV)[shift:]
    odd = torch.randint(0, n, (1000,), generator=gen, device=DEV)
    w[odd] = torch.tensor([float("inf"), 1e-42, -0.0, float("nan")], device=DEV).repeat(250)
    val[::997] = 1e-41
    want = w.clone()
    for lr in (0.1, -1.0):  # the second pass on updated elements
        at = idx.long()
        want[at] = want[at] - torch.tensor(lr, device=DEV) * val
        ld.ld_merge_sparse(w, [idx], [val], lr, strategy=ld.LD_MERGE_SCATTER)
        assert torch.equal(w.view(torch.int32), want.view(torch.int32))


def combine_by(strategy, idxs, vals, n, scale, cap=None):
    """ld_combine_sparse_strategy on numpy lists: (idx, val, count) with what lies past the count or cap cut off."""
    lib = ld.load()
    gi, gv = [to_gpu(i) for i in idxs], [to_gpu(v) for v in vals]
    N, total = len(idxs), sum(len(i) for i in idxs)
    cap = total if cap is None else cap
    oi = torch.full((cap + 64,), -1, dtype=torch.int32, device=DEV)
    ov = torch.full((cap + 64,), 7.0, device=DEV)
    cnt = torch.full((1,), -1, dtype=torch.int64, device=DEV)
    ws = torch.full((ld.ld_combine_sparse_workspace(n, N),), 0xA5, dtype=torch.uint8, device=DEV)
    V = ctypes.c_void_p
    ip, vp = (V * N)(*[t.data_ptr() for t in gi]), (V * N)(*[t.data_ptr() for t in gv])
    K = (ctypes.c_int64 * N)(*[len(i) for i in idxs])
    st = lib.ld_combine_sparse_strategy(ip, vp, K, N, n, ctypes.c_float(scale), V(oi.data_ptr()), V(ov.data_ptr()), cap,
                                        V(cnt.data_ptr()), V(ws.data_ptr()), ws.numel(), V(0), strategy)
    assert st == 0
    torch.cuda.synchronize()
    count = int(cnt.item())
    kept = min(count, cap)
    assert bool((oi[kept:] == -1).all()) and bool((ov[kept:] == 7.0).all())
    return oi[:kept].cpu().numpy(), ov[:kept].cpu().numpy(), count


@pytest.mark.parametrize("name", list(COMBINE_LISTS))
@pytest.mark.parametrize("strategy", [1, 2, 3])
def test_combine_strategies(name, strategy):
    """Two passes, one pass, and one pass whose workgroups wait for nobody, on a dirty workspace: the oracle bit for bit."""
    n, counts, span = COMBINE_LISTS[name][:3]
    print(f"[combine] strategy {strategy} {name} n={n}", flush=True)
    rs = np.random.RandomState(len(name))
    a, b = span or (0, n)
    idxs = [np.sort(rs.choice(b - a, k, replace=False)).astype(np.int32) + a for k in counts]
    vals = [rs.standard_normal(k).astype(np.float32) for k in counts]
    ei, ev = oracle.combine_sparse(idxs, vals, n, 0.125)
    gi, gv, count = combine_by(strategy, idxs, vals, n, 0.125)
    assert count == ei.size
    np.testing.assert_array_equal(gi, ei)
    np.testing.assert_array_equal(bits(gv), bits(ev))
    cap = ei.size // 2
    gi, gv, count = combine_by(strategy, idxs, vals, n, 0.125, cap)
    assert count == ei.size
    np.testing.assert_array_equal(gi, ei[:cap])
    np.testing.assert_array_equal(bits(gv), bits(ev[:cap]))


def lowest_times(calls, reps=5, turns=5):
    """Milliseconds per call of each of `calls`, the lowest of several turns in which they take turns."""
    best = [float("inf")] * len(calls)
    for f in calls:
        f()
    for _ in range(turns):
        for j, f in enumerate(calls):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(reps):
                f()
            b.record()
            b.synchronize()
            best[j] = min(best[j], a.elapsed_time(b) / reps)
    return best


def combine_times(strategies, idxs, n):
    """Milliseconds per combine by each of the strategies; their outputs agree."""
    lib, N = ld.load(), len(idxs)
    gen = torch.Generator(device=DEV).manual_seed(n)
    vals = [torch.randn(i.numel(), device=DEV, generator=gen) for i in idxs]
    cap = sum(i.numel() for i in idxs)
    ws = torch.empty(ld.ld_combine_sparse_workspace(n, N), dtype=torch.uint8, device=DEV)
    V = ctypes.c_void_p
    ip, vp = (V * N)(*[t.data_ptr() for t in idxs]), (V * N)(*[t.data_ptr() for t in vals])
    K = (ctypes.c_int64 * N)(*[i.numel() for i in idxs])
    outs = [(torch.full((cap,), -1, dtype=torch.int32, device=DEV), torch.zeros(cap, device=DEV),
             torch.zeros(1, dtype=torch.int64, device=DEV)) for _ in strategies]

    def call(strategy, out):
        assert lib.ld_combine_sparse_strategy(ip, vp, K, N, n, ctypes.c_float(0.125), V(out[0].data_ptr()),
                                              V(out[1].data_ptr()), cap, V(out[2].data_ptr()), V(ws.data_ptr()), ws.numel(),
                                              V(0), strategy) == 0

    times = lowest_times([lambda s=s, o=o: call(s, o) for s, o in zip(strategies, outs)])
    for o in outs[1:]:
        assert torch.equal(o[0], outs[0][0]) and torch.equal(o[1].view(torch.int32), outs[0][1].view(torch.int32))
        assert torch.equal(o[2], outs[0][2])
    return times


@pytest.mark.parametrize("n,N,K,part", [(5_000_000, 8, 13_000, 50), (20_000_000, 16, 28_000, 50), (3_200_000, 24, 4_800, 50),
                                        (400_000_000, 8, 1_600_000, 50)])
def test_combine_of_crowded_lists_takes_no_longer_in_one_pass(n, N, K, part):
    """All records in the first fiftieth: a round reads its pieces of the lists, not all of them again. Reading them
    all took two to six times as long as two passes that did the same, which those now take two to three times less than."""
    print(f"[combine] crowded n={n} N={N} K={K}", flush=True)
    gen = torch.Generator(device=DEV).manual_seed(K)
    idxs = [torch.randperm(n // part, device=DEV, generator=gen)[:K].sort().values.int() for _ in range(N)]
    one, two = combine_times((0, 1), idxs, n)
    print(f"[combine] {one * 1e3:.0f} us, two passes {two * 1e3:.0f}", flush=True)
    assert one <= 2.2 * two, f"{one * 1e3:.0f} us, two passes {two * 1e3:.0f}"


@pytest.mark.parametrize("n,N,K,part", [(119_000_000, 64, 357_000, 10), (100_000_000, 16, 300_000, 50)])
def test_combine_of_crowded_lists_in_two_passes(n, N, K, part):
    """The emission of a crowded sub-tile takes pieces of the lists too. With all of them read in every round the first took
    7.1 times the one pass's time, now 2.1."""
    print(f"[combine] crowded, two passes n={n} N={N} K={K}", flush=True)
    gen = torch.Generator(device=DEV).manual_seed(K)
    idxs = [torch.randperm(n // part, device=DEV, generator=gen)[:K].sort().values.int() for _ in range(N)]
    two, one = combine_times((1, 2), idxs, n)
    print(f"[combine] {two * 1e3:.0f} us, one pass {one * 1e3:.0f}", flush=True)
    assert two <= 3.5 * one, f"{two * 1e3:.0f} us, one pass {one * 1e3:.0f}"


@pytest.mark.parametrize("n,N,K", [(119_177_435, 64, 380_000), (329_999_869, 12, 2_558_000), (76_868_857, 16, 512_000),
                                   (31_779_675, 64, 108_000), (300_000_001, 16, 300_000), (1_000_000_007, 8, 4_000_000)])
def test_combine_takes_the_faster_way_for_even_lists(n, N, K):
    """More than 8 lists, thousands of chunks, arrays above 100 M elements: what the library picks is no slower than two
    passes, with the same output. The first four took 1.35 to 1.75 times as long in one pass."""
    print(f"[combine] even n={n} N={N} K={K}", flush=True)
    gen = torch.Generator(device=DEV).manual_seed(K)
    idxs = []
    for _ in range(N):
        at = torch.randint(1, 2 * n // K, (K,), device=DEV, generator=gen).cumsum(0) - 1
        idxs.append(torch.minimum(at, n - K + torch.arange(K, device=DEV)).int())
    auto, two = combine_times((0, 1), idxs, n)
    assert auto <= 1.15 * two, f"{auto * 1e3:.0f} us, two passes {two * 1e3:.0f}"


def test_combine_asks_again_what_it_waited_for_in_vain():
    """Workgroups that wait for nobody: a chunk that has been told meanwhile is not counted from its records again. Without
    asking again a workgroup counts up to 64 chunks one after another here, 28 times the time with waiting; asking, 1.8 times."""
    n, N, K = 1_500_000_000, 8, 15_000_000
    print(f"[combine] asking again n={n}", flush=True)
    gen = torch.Generator(device=DEV).manual_seed(K)
    idxs = []
    for _ in range(N):
        at = torch.randint(1, 2 * n // K - 1, (K,), device=DEV, generator=gen).cumsum(0) - 1
        idxs.append(torch.minimum(at, n - K + torch.arange(K, device=DEV)).int())
    waiting, alone = combine_times((2, 3), idxs, n)
    assert alone <= 6 * waiting, f"{alone * 1e3:.0f} us, waiting {waiting * 1e3:.0f}"


def records_of(kind, n, K, gen):
    """About K ascending positions of [0, n): rows of 768, all in the first fiftieth, one in nine, or runs and gaps in turn."""
    if kind == "rows":
        rows = torch.randperm(n // 768, device=DEV, generator=gen)[:K // 768].sort().values
        at = (rows[:, None] * 768 + torch.arange(768, device=DEV)).reshape(-1)
    elif kind == "first fiftieth":
        at = torch.arange(max(K, n // 50), device=DEV)[:K]
    elif kind == "one in nine":  # about half of the waves are crowded
        at = torch.arange(n, device=DEV)[torch.rand(n, device=DEV, generator=gen) < K / n]
    else:  # 40 records in a run, then 40 some way apart, with ends at every place of a granule and of a wave
        gaps = torch.randint(1, 60, (K,), device=DEV, generator=gen)
        gaps[(torch.arange(K, device=DEV) // 40) % 2 == 0] = 1
        at = gaps.cumsum(0)
        at = at[at < n]
    return at.int()


@pytest.mark.parametrize("kind,n,K", [("one in nine", 50_000_003, 5_600_000), ("runs and gaps", 200_000_001, 9_500_000),
                                      ("rows", 700_000_000, 9_600_000), ("first fiftieth", 700_000_017, 14_000_000)])
def test_scatter_of_crowded_and_sparse_waves(kind, n, K):
    """Waves that go by granules beside waves that go word by word, granules that both have records of. Bit for bit, and where
    the records crowd no slower than all of it word by word (w off its granules): as chains of one granule's records ten times."""
    print(f"[scatter] {kind} n={n} K={K}", flush=True)
    gen = torch.Generator(device=DEV).manual_seed(K)
    idx = records_of(kind, n, K, gen)
    assert idx.numel() >= 9_000_000 or (idx.numel() >= 5_000_000 and idx.numel() * 80 >= n)
    val = torch.randn(idx.numel(), generator=gen, device=DEV)
    w = torch.randn(n, generator=gen, device=DEV)
    want = w.clone()
    want[idx.long()] -= torch.tensor(0.1, device=DEV) * val
    ld.ld_merge_sparse(w, [idx], [val], 0.1, strategy=ld.LD_MERGE_SCATTER)
    assert torch.equal(w.view(torch.int32), want.view(torch.int32))
    if kind in ("rows", "first fiftieth"):
        del want
        off = torch.zeros(n + 4, device=DEV)[4:]
        here, words = lowest_times([lambda x=x: ld.ld_merge_sparse(x, [idx], [val], 0.1, strategy=ld.LD_MERGE_SCATTER) for x in (w, off)])
        assert here <= 1.25 * words, f"{here * 1e3:.0f} us, word by word {words * 1e3:.0f}"


@pytest.mark.parametrize("n,W,K,kind", [(52_583_779, 8, 142_000, "first fiftieth"), (35_059_415, 4, 252_000, "rows"),
                                        (81_993_579, 3, 811_000, "first fiftieth"), (300_176_903, 13, 622_000, "rows")])
def test_merge_of_crowded_sparse_windows_is_scattered(n, W, K, kind):
    """Windows that touch little of w, all of it in one place: with the workspace that the query gives they take no longer than
    with the least, with which they are scattered. Priced as if every record cost a line of its own they went through a table
    of all of w: three to nine times as long."""
    print(f"[merge] {kind} n={n} W={W} K={K}", flush=True)
    gen = torch.Generator(device=DEV).manual_seed(K)
    idx = [records_of(kind, n, K, gen) for _ in range(W)]
    val = [torch.randn(i.numel(), generator=gen, device=DEV) for i in idx]
    w = [torch.zeros(n, device=DEV) for _ in range(2)]
    nbytes = (ld.ld_merge_sparse_workspace(n, [i.numel() for i in idx]), int(ld.load().ld_merge_sparse_workspace(n, W, None)))
    assert nbytes[0] > nbytes[1]
    ws = [torch.empty(b, dtype=torch.uint8, device=DEV) for b in nbytes]
    asked, least = lowest_times([lambda j=j: ld.ld_merge_sparse(w[j], idx, val, 0.1, ws[j]) for j in range(2)])
    assert torch.equal(w[0].view(torch.int32), w[1].view(torch.int32))
    assert asked <= 1.25 * least, f"{asked * 1e3:.0f} us, with the least workspace {least * 1e3:.0f}"


@pytest.mark.parametrize("part", [7453, 10559, 14391])
def test_sparse_adam_finds_the_records_of_a_short_last_chunk(part):
    """An array that ends early in a chunk of the range table is not slower than one that fills it: the last sub-tiles' windows lie
    where the records do. Guessed as if the chunk were whole, they missed, and the call took a third longer."""
    W, rho = 37, 197
    calls = []
    for n in (49152 * 9 + part, 49152 * 10):
        gen = torch.Generator(device=DEV).manual_seed(n)
        idx = [torch.randperm(n, device=DEV, generator=gen)[:n // rho].sort().values.int() for _ in range(W)]
        val = [torch.randn(i.numel(), device=DEV, generator=gen) * 1e-2 for i in idx]
        w, m, v = (torch.randn(n, device=DEV, generator=gen), torch.zeros(n, device=DEV), torch.ones(n, device=DEV) * 1e-6)
        ws = torch.empty(ld.ld_merge_sparse_adam_workspace(n, [i.numel() for i in idx]), dtype=torch.uint8, device=DEV)
        calls.append(lambda w=w, m=m, v=v, idx=idx, val=val, ws=ws: ld.ld_merge_sparse_adam(
            w, m, v, idx, val, 2, workspace=ws, lr=1e-4, **synth.ADAM))
    short, whole = lowest_times(calls, reps=20)
    assert short <= 1.12 * whole, f"{short * 1e3:.1f} us, {whole * 1e3:.1f}"
