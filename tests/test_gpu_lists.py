"""Tile lists where the binning kernels change their way of working: list lengths at the borders between the sorts of
k_tile_depth_sort, which depend on how many tiles there are; blocks of 256 points whose rectangle of tiles is larger than the
counting table, which go past it; point counts at which a block gets another number of threads. Bit-exact against the oracle, which sorts by
(tile, depth bits, point index)."""
import numpy as np
import pytest

import oracle
from paper_2512_20017_amd import binding as B

from gpu_pipeline import GpuView
from test_gpu_edge import _cam, _rand_state

pytestmark = pytest.mark.gpu


def _check(st, depth, w, h):
    st = dict(st, depth=np.asarray(depth, dtype=np.float32))
    n = len(st["opacity"])
    ref = oracle.bin_sort(np.asarray(st["mean2d"], dtype=np.float32).astype(np.float64), np.asarray(st["radius"], dtype=np.int32), st["depth"], w, h)
    view = GpuView(n, _cam(w, h), max(ref["P"], 1))
    view.splats = B.Splats.from_numpy(st)
    for _ in range(2):      # the lists' order before the sort varies from run to run, the result does not
        B.pbdr_bin_sort(view.splats, view.cam, view.cap, view.ws)
        got = view.lists()
        assert got["P_raw"] == ref["P"]
        assert np.array_equal(got["ranges"], ref["ranges"])
        assert np.array_equal(got["keys"], ref["keys"])
        assert np.array_equal(got["vals"], ref["vals"])
    return ref


LENGTHS = [1, 2, 63, 64, 65, 126, 127, 128, 129, 192, 193, 254, 255, 256, 257, 384, 385, 511, 512, 513, 765, 766, 767, 768, 1024, 1025,
           1536, 1537, 2048, 2049, 3072, 3073, 4096, 4097, 5632, 5633, 8192, 8193]


@pytest.mark.parametrize("w,h", [(320, 320), (1280, 720), (1936, 1040)])      # 400, 3,600 and 7,865 tiles
@pytest.mark.parametrize("kind", ["uniform", "octaves", "pairs", "twos", "runs", "walls", "one_depth"])
def test_list_lengths_at_the_borders_of_the_sorts(w, h, kind):
    """One tile per length, its points scattered over the point order. Depths: spread evenly; over seven octaves on both sides of 2.0; each value twice, as copied points
    leave them; in twos that differ in the last place, at even or at odd places of the list, so that in half of the lists such a two lies
    across every border between rounds of 64 entries; in runs of a hundred equal ones and, in every tenth list, in the top bits alone; in walls of 1 to 257 points at
    nearly one depth, on both sides of the lengths up to which equal ones are put right by counting; one for all."""
    rng = np.random.default_rng(w + len(kind))
    tx = (w + 15) // 16
    tile = np.repeat(np.arange(len(LENGTHS)) * 7 + tx + 3, LENGTHS)
    n = len(tile)
    centre = np.stack([(tile % tx) * 16 + rng.uniform(3, 13, n), (tile // tx) * 16 + rng.uniform(3, 13, n)], 1).astype(np.float32)
    if kind == "uniform":
        depth = rng.uniform(8, 20, n)
    elif kind == "octaves":
        depth = np.exp2(rng.uniform(-1.5, 5.5, n))
    elif kind == "pairs":
        depth = rng.uniform(8, 20, n)
        depth[1::2] = depth[:-1:2][:len(depth[1::2])]
    elif kind == "twos":
        depth = np.empty(n, dtype=np.float32)
        for t in np.unique(tile):
            at = np.flatnonzero(tile == t)
            i = np.arange(len(at)) + (t // 7) % 2
            depth[at] = ((8 + 12 * (i // 2) / len(at)).astype(np.float32).view(np.uint32) + (i % 2).astype(np.uint32)).view(np.float32)
    elif kind == "runs":
        depth = 3 + (rng.permutation(n) // 100) * 0.01
        steep = tile % 10 == 0
        depth[steep] = 2.0 + rng.integers(0, 5, steep.sum()) * 2.0 ** -22 + (rng.random(steep.sum()) < 0.01) * 1e6
    elif kind == "walls":
        depth = np.empty(n, dtype=np.float32)
        for t in np.unique(tile):
            at = np.flatnonzero(tile == t)
            walls = rng.permutation([1, 2, 15, 16, 17, 18, 63, 64, 65, 255, 256, 257] if t % 3 else [1, 2, 3, 15, 16])
            wall = np.repeat(np.arange(len(at)), np.resize(walls, len(at)))[:len(at)]
            depth[at] = 8 + 0.25 * (wall % 4000)
        near = rng.random(n) < 0.3      # a few last places away
        depth[near] = (depth[near].view(np.uint32) + rng.integers(1, 4, near.sum(), dtype=np.uint32)).view(np.float32)
    else:
        depth = np.full(n, 4.25)
    order = rng.permutation(n)
    st = dict(mean2d=centre[order], conic=np.tile([0.1, 0, 0.1], (n, 1)), opacity=np.full(n, 0.01), color=np.zeros((n, 3)),
              radius=np.full(n, 1, dtype=np.int32))
    ref = _check(st, depth[order], w, h)
    lengths = ref["ranges"][:, 1].astype(int) - ref["ranges"][:, 0]
    assert sorted(lengths[lengths > 0]) == LENGTHS      # the case is what it claims


@pytest.mark.parametrize("w,h", [(65536, 100), (3840, 2160), (48, 65536)])
@pytest.mark.parametrize("n", [255, 600])
def test_blocks_of_points_all_over_a_large_grid(w, h, n):
    """Points in no spatial order: a block's rectangle of tiles is the whole grid, and its pairs are counted in memory. Also with room
    for less than half of the pairs: the first in point order, row by row, are kept."""
    rng = np.random.default_rng(w + n)
    st = _rand_state(rng, n, w, h, rmax=70)
    st["radius"][rng.integers(0, n, 12)] = rng.integers(500, 5000, 12)      # points on hundreds of tiles
    depth = rng.uniform(0.3, 50, n)
    ref = _check(st, depth, w, h)
    cap = int(0.45 * ref["P"])
    view = GpuView(n, _cam(w, h), cap)
    view.splats = B.Splats.from_numpy(dict(st, depth=depth.astype(np.float32)))
    B.pbdr_bin_sort(view.splats, view.cam, cap, view.ws)
    got = view.lists()
    assert B.pbdr_query_lists(view.ws, n, w, h, cap) == (ref["P"], True)
    kept = np.sort(np.lexsort((ref["keys"] >> np.uint64(32), ref["vals"]))[:cap])
    assert np.array_equal(got["keys"][:cap], ref["keys"][kept])
    assert np.array_equal(got["vals"][:cap], ref["vals"][kept])


@pytest.mark.parametrize("n", [1, 255, 256, 257, 4096, 4097, 262144 + 1, 300000])
def test_dense_blocks_on_few_tiles(n):
    """All points of a block on the same few tiles (its counters of pairs reach 256), on both sides of the point count from which a
    block gets 256 instead of 1,024 threads."""
    rng = np.random.default_rng(n)
    w, h = 80, 64
    m = min(n, 4097)
    st = dict(mean2d=rng.uniform(20, 60, (n, 2)).astype(np.float32), conic=np.tile([0.1, 0, 0.1], (n, 1)), opacity=np.full(n, 0.01),
              color=np.zeros((n, 3)), radius=np.zeros(n, dtype=np.int32))
    st["radius"][n - m:] = rng.integers(1, 40, m)
    _check(st, rng.uniform(0.3, 50, n), w, h)


@pytest.mark.parametrize("length", [700, 5600, 5700])
def test_many_depths_and_one_wall_far_apart_in_the_point_order(length):
    """A wall of 40 points among points of their own depths, 2^24 points from the first to the last: the number of a run of equal
    depths and the distance in the point order together take more than a word, and the list is sorted by point index and depth."""
    rng = np.random.default_rng(length)
    n, w, h = (1 << 24) + 1, 32, 32
    at = np.concatenate([[0], np.sort(rng.choice(n - 2, length - 2, replace=False) + 1), [n - 1]])
    st = dict(mean2d=np.full((n, 2), 8.0, dtype=np.float32), conic=np.tile(np.float32([0.1, 0, 0.1]), (n, 1)), opacity=np.full(n, 0.01, dtype=np.float32),
              color=np.zeros((n, 3), dtype=np.float32), radius=np.zeros(n, dtype=np.int32))
    st["radius"][at] = 1
    depth = np.ones(n, dtype=np.float32)
    depth[at] = 1 + rng.permutation(length) / 64
    depth[rng.choice(at, 40, replace=False)] = 3.0
    _check(st, depth, w, h)


@pytest.mark.parametrize("n", [1 << 24, (1 << 24) + 1, (1 << 24) + 3 * 32768 + 257])
def test_sums_over_many_blocks(n):
    """On both sides of the point count from which the sums that a block adds up are those of 128 blocks, not of 16: listed points in the
    blocks on both sides of such parts, in the first and last block, and in every block of one part."""
    rng = np.random.default_rng(n)
    w, h = 320, 200
    parts = rng.choice(n // 32768 - 1, 60, replace=False) * 32768
    at = np.unique(np.concatenate([[0, n - 1], parts, parts + 32767, parts + 32768, parts[0] + np.arange(0, 32768, 100), rng.choice(n, 500, replace=False)]))
    st = dict(mean2d=np.full((n, 2), 8.0, dtype=np.float32), conic=np.tile(np.float32([0.1, 0, 0.1]), (n, 1)), opacity=np.full(n, 0.01, dtype=np.float32),
              color=np.zeros((n, 3), dtype=np.float32), radius=np.zeros(n, dtype=np.int32))
    st["mean2d"][at] = np.stack([rng.uniform(0, w, len(at)), rng.uniform(0, h, len(at))], 1)
    st["radius"][at] = rng.integers(1, 30, len(at))
    depth = np.ones(n, dtype=np.float32)
    depth[at] = rng.uniform(0.3, 50, len(at))
    _check(st, depth, w, h)
