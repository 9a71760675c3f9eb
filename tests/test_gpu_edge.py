"""GPU edge cases through the C ABI: empty and degenerate inputs, adversarial sort keys, capacity overflow."""
import numpy as np
import pytest
import torch

import oracle
from gpu_pipeline import GpuView
from helpers import grad_close
from paper_2512_20017_amd import binding as B
from paper_2512_20017_amd import synth

pytestmark = pytest.mark.gpu


def _cam(w, h):
    return synth.pinhole(w, h, 60.0, np.eye(3), [0.0, 0.0, 3.0])


def _lists_case(st, depth, w, h, cap=None):
    """st: host splat dict (mean2d[n,2], conic, opacity, color, radius); returns (gpu lists, oracle lists, view)."""
    st = dict(st); st["depth"] = np.asarray(depth, dtype=np.float32)
    n = len(st["opacity"])
    ref = oracle.bin_sort(np.asarray(st["mean2d"], dtype=np.float32).astype(np.float64), np.asarray(st["radius"], dtype=np.int32),
                          st["depth"], w, h)
    view = GpuView(n, _cam(w, h), cap if cap is not None else max(ref["P"], 1))
    view.splats = B.Splats.from_numpy(st)
    B.pbdr_bin_sort(view.splats, view.cam, view.cap, view.ws)
    return view.lists(), ref, view


def _rand_state(rng, n, w, h, rmax=60):
    return dict(mean2d=np.stack([rng.uniform(-20, w + 20, n), rng.uniform(-20, h + 20, n)], 1).astype(np.float32),
                conic=np.tile([0.02, 0.0, 0.02], (n, 1)).astype(np.float32), opacity=rng.uniform(0.05, 0.9, n).astype(np.float32),
                color=rng.uniform(0, 1, (n, 3)).astype(np.float32), radius=rng.integers(0, rmax, n).astype(np.int32))


@pytest.mark.parametrize("w,h,n,seed", [(64, 64, 500, 0), (200, 120, 3000, 1), (33, 17, 100, 2), (1920, 1080, 20000, 3)])
def test_lists_random_states_with_ties(w, h, n, seed):
    rng = np.random.default_rng(seed)
    st = _rand_state(rng, n, w, h)
    depth = rng.uniform(0.3, 50, n).astype(np.float32)
    depth[rng.integers(0, n, n // 3)] = depth[0]         # many exact ties -> order must fall back to the index
    got, ref, _ = _lists_case(st, depth, w, h)
    assert got["P_raw"] == ref["P"]
    assert np.array_equal(got["keys"], ref["keys"])
    assert np.array_equal(got["vals"], ref["vals"])
    assert np.array_equal(got["ranges"], ref["ranges"])


@pytest.mark.parametrize("n", [262144, 262145, 263000, 1048577 + 256, 2097152 + 300])
def test_lists_point_counts_around_a_scan_chunk(n):
    """The block scan and the packing order are made by one workgroup per 1,024 blocks of 256 points, each adding up what
    precedes its chunk by itself: point counts of exactly one chunk, one point more, a short second chunk, and a fifth
    chunk of two blocks, and just past two million points (from where a workgroup takes 4,096 blocks), with heavy and
    light blocks mixed (a few splats of large radius)."""
    rng = np.random.default_rng(n % 1000)
    w, h = 640, 360
    st = _rand_state(rng, n, w, h, rmax=3)
    big = rng.integers(0, n, 40)
    st["radius"][big] = rng.integers(100, 400, 40)
    st["radius"][rng.integers(0, n, n // 2)] = 0
    depth = rng.uniform(0.3, 50, n).astype(np.float32)
    got, ref, _ = _lists_case(st, depth, w, h)
    assert got["P_raw"] == ref["P"]
    assert np.array_equal(got["vals"], ref["vals"])
    assert np.array_equal(got["keys"], ref["keys"])
    assert np.array_equal(got["ranges"], ref["ranges"])


def test_lists_all_equal_depth_one_tile():
    n = 5000                                               # one tile, one depth: pure index order, several sort blocks
    st = dict(mean2d=np.full((n, 2), 8.0, dtype=np.float32), conic=np.tile([0.1, 0, 0.1], (n, 1)), opacity=np.full(n, 0.01),
              color=np.zeros((n, 3)), radius=np.full(n, 3, dtype=np.int32))
    got, ref, _ = _lists_case(st, np.full(n, 2.5), 16, 16)
    assert got["vals"].tolist() == list(range(n))
    assert got["ranges"].tolist() == [[0, n]]
    assert np.array_equal(got["keys"], ref["keys"])


@pytest.mark.parametrize("n", [2, 3, 63, 64, 65, 257, 511, 600, 1021, 1022, 1023, 2048, 2049, 4097, 6400, 6401, 9000, 70001])
@pytest.mark.parametrize("kind", ["narrow", "wide", "two_values", "wide_short_runs"])
def test_one_crowded_tile_depth_order(n, kind):
    """Every splat in one tile: the list's depth order is made by one workgroup - by counting up to 256 entries, in LDS up
    to 2048, through the global scratch arrays beyond - over the bit positions in which the depths differ: depths from a
    narrow band (few differing bits), from many octaves (all exponent bits differ), and only two distinct values; a
    third of the entries tied in each of these, so that the order among equals (point index) is exercised too; and depths over
    many octaves with short runs of near-equal values out of point order."""
    rng = np.random.default_rng(n * 7 + len(kind))
    st = dict(mean2d=rng.uniform(17.0, 30.0, (n, 2)).astype(np.float32), conic=np.tile([0.1, 0, 0.1], (n, 1)),
              opacity=np.full(n, 0.01), color=np.zeros((n, 3)), radius=np.full(n, 1, dtype=np.int32))
    if kind == "narrow":
        depth = rng.uniform(7.0, 7.01, n).astype(np.float32)
    elif kind == "wide":
        depth = np.exp(rng.uniform(np.log(1e-3), np.log(1e9), n)).astype(np.float32)
    elif kind == "wide_short_runs":
        # many bit positions differ, and entries that agree in the top 16 of them come in runs of two to eight: exact
        # ties, and neighbours a few units in the last place apart, out of order by point index
        depth = np.exp(rng.uniform(np.log(0.5), np.log(300.0), n)).astype(np.float32)
        for start in rng.integers(0, max(n - 8, 1), max(n // 6, 1)):
            run = int(rng.integers(2, 9))
            bits = depth[start:start + 1].view(np.uint32)[0] + rng.integers(0, 40, run).astype(np.uint32)
            where = rng.integers(0, n, run)
            depth[where] = bits.view(np.float32)
    else:
        depth = rng.choice(np.array([2.5, 2.5000002], dtype=np.float32), n)
    if kind != "wide_short_runs":
        depth[rng.integers(0, n, n // 3)] = depth[0]
    got, ref, _ = _lists_case(st, depth, 48, 48)
    assert ref["ranges"][4].tolist() == [0, n]             # tile (1, 1) of the 3 x 3 grid holds them all
    assert np.array_equal(got["vals"], ref["vals"])
    assert np.array_equal(got["keys"], ref["keys"])
    assert np.array_equal(got["ranges"], ref["ranges"])


def test_lists_empty_single_and_adversarial_bits():
    # nothing visible
    st = dict(mean2d=np.zeros((7, 2)), conic=np.zeros((7, 3)), opacity=np.zeros(7), color=np.zeros((7, 3)), radius=np.zeros(7, dtype=np.int32))
    got, ref, view = _lists_case(st, np.ones(7), 48, 32)
    assert got["P_raw"] == 0 and (got["ranges"] == 0).all()
    out = view.render_fwd([0.25, 0.5, 0.75])
    assert (out["image"] == np.array([0.25, 0.5, 0.75], dtype=np.float32)).all() and (out["final_T"] == 1).all()
    assert (out["last_idx"] == 0).all()
    # a single pair
    st = dict(mean2d=[[40.0, 20.0]], conic=[[0.1, 0, 0.1]], opacity=[0.5], color=[[1, 1, 1]], radius=[2])
    got, ref, _ = _lists_case(st, [1.0], 48, 32)
    assert got["P_raw"] == 1 and got["vals"].tolist() == [0] and got["ranges"][2 + 3 * 1].tolist() == [0, 1]
    # depth bit patterns that differ only in one byte each, plus denormal-small and huge values
    depths = np.array([1.0, np.nextafter(np.float32(1.0), np.float32(2)), 256.0, 65536.0, 1.6e7, 1e-30, 3.4e38, 0.5, 0.5], dtype=np.float32)
    n = len(depths)
    st = dict(mean2d=np.full((n, 2), 20.0), conic=np.tile([0.1, 0, 0.1], (n, 1)), opacity=np.full(n, 0.5), color=np.zeros((n, 3)),
              radius=np.full(n, 30, dtype=np.int32))
    got, ref, _ = _lists_case(st, depths, 48, 32)
    assert np.array_equal(got["keys"], ref["keys"]) and np.array_equal(got["vals"], ref["vals"])


def test_zero_points():
    cam = _cam(32, 32)
    view = GpuView(0, cam, 16)
    scene = B.Scene.from_numpy(dict(mean=np.zeros((0, 3)), log_scale=np.zeros((0, 3)), quat=np.zeros((0, 4)), logit=np.zeros(0),
                                    sh=np.zeros((0, 1, 3)), sh_degree=0))
    B.pbdr_preprocess(scene, cam, view.splats)
    out = view.render_fwd([1.0, 0.0, 0.5])
    assert (out["image"][..., 0] == 1).all() and (out["image"][..., 2] == 0.5).all()
    grads = scene.zeros_like()
    view.render_bwd([1.0, 0.0, 0.5], np.ones((32, 32, 3), dtype=np.float32), scene=scene, grads=grads)
    # the same without a splat-state gradient output, and the batched calls on an empty cloud
    G = torch.ones((3, 32, 32), device="cuda")
    B.pbdr_render_bwd(scene, view.splats, cam, [1.0, 0.0, 0.5], view.cap, view.final_T, view.last_idx, G, None, grads, view.ws,
                      first_view=True)
    torch.cuda.synchronize()


def _untouched(st, w, h):
    """Points with radius > 0 whose tile rectangle misses the image (binning does not list them)."""
    r = np.asarray(st["radius"], dtype=np.int64)
    ix = np.floor(np.asarray(st["mean2d"], dtype=np.float32)[:, 0]).astype(np.int64)
    iy = np.floor(np.asarray(st["mean2d"], dtype=np.float32)[:, 1]).astype(np.int64)
    tx, ty = (w + 15) // 16, (h + 15) // 16
    x0, x1 = np.clip((ix - r) >> 4, 0, tx), np.clip((ix + r + 15) >> 4, 0, tx)
    y0, y1 = np.clip((iy - r) >> 4, 0, ty), np.clip((iy + r + 15) >> 4, 0, ty)
    return int(((r > 0) & ((x1 - x0) * (y1 - y0) == 0)).sum())


def test_capacity_overflow_is_reported_and_in_bounds():
    rng = np.random.default_rng(5)
    n, w, h = 2000, 128, 96
    st = _rand_state(rng, n, w, h)
    depth = rng.uniform(0.3, 50, n).astype(np.float32)
    full, ref, roomy = _lists_case(st, depth, w, h)
    assert np.array_equal(full["vals"], ref["vals"])
    cap = ref["P"] // 3
    got, _, view = _lists_case(st, depth, w, h, cap=cap)
    n_dup, over = B.pbdr_query_lists(view.ws, n, w, h, cap)
    assert over and n_dup == ref["P"]
    assert got["P"] == cap
    # the same through the status words a caller can poll without a synchronising call: {pairs found, overflow, listed}
    words = B.pbdr_status_view(view.ws, n, w, h, cap).cpu().numpy()
    assert words.tolist() == [ref["P"], 1, int((np.asarray(st["radius"]) > 0).sum() - _untouched(st, w, h))]
    words_ok = B.pbdr_status_view(roomy.ws, n, w, h, roomy.cap).cpu().numpy()      # the run with room for every pair
    assert words_ok[0] == ref["P"] and words_ok[1] == 0
    # what was kept is a sorted subset of the true pairs, and ranges stay inside the capacity
    assert (np.diff(got["keys"].astype(np.uint64).astype(object)) >= 0).all()
    assert got["ranges"].max() <= cap
    true_pairs = set(zip(ref["keys"].tolist(), ref["vals"].tolist()))
    assert set(zip(got["keys"].tolist(), got["vals"].tolist())) <= true_pairs
    # rendering from truncated lists must still run and stay finite
    out = view.render_fwd([0, 0, 0])
    assert np.isfinite(out["image"]).all()


@pytest.mark.parametrize("w,h", [(640, 480), (5000, 40), (40, 5000)])
@pytest.mark.parametrize("share", [1.0, 0.37])
def test_lists_with_points_on_hundreds_of_tiles(w, h, share):
    """Pairs of a point on 256 tiles or more are written by its whole workgroup, those of the others by their wavefront, which
    steps over the former: rectangles on both sides of that size and over the whole image, alone, next to each other, at the
    ends of a wavefront and of a block, in rows longer and shorter than the workgroup - and with room for all pairs and for a
    part of them only, which is the first ones in point order."""
    rng = np.random.default_rng(w)
    n = 900
    st = _rand_state(rng, n, w, h, rmax=40)
    r256 = 120 if min(w, h) > 300 else 680      # about 256 tiles: 16 x 16, or three rows of 85
    sizes = [r256 - 8, r256 - 2, r256 - 1, r256, r256 + 1, r256 + 2, r256 + 7, r256 + 8, 2 * r256, 2000, 100000]
    at = np.array([0, 1, 2, 63, 64, 200, 255, 256, 300, 383, 384, 385, 386, 387, 511, 512, 640, 899])
    st["radius"][at] = [sizes[k % len(sizes)] for k in range(len(at))]
    st["radius"][700:770] = r256 + 4 + np.arange(70) % 9
    st["mean2d"][700:770] = [w / 2, h / 2] + rng.uniform(-16, 16, (70, 2))
    depth = rng.uniform(0.3, 50, n).astype(np.float32)
    ref = oracle.bin_sort(st["mean2d"].astype(np.float64), st["radius"], depth, w, h)
    count = np.bincount(ref["vals"], minlength=n)
    assert (count >= 256).sum() > 10 and (count[count > 0] < 256).sum() > 100      # the case is what it claims
    cap = int(ref["P"] * share)
    got, _, view = _lists_case(st, depth, w, h, cap=cap)
    if share == 1.0:
        assert np.array_equal(got["keys"], ref["keys"]) and np.array_equal(got["vals"], ref["vals"])
        assert np.array_equal(got["ranges"], ref["ranges"])
        return
    assert B.pbdr_query_lists(view.ws, n, w, h, cap) == (ref["P"], True)
    kept = np.sort(np.lexsort((ref["keys"] >> np.uint64(32), ref["vals"]))[:cap])      # by point, then row by row
    assert np.array_equal(got["keys"], ref["keys"][kept]) and np.array_equal(got["vals"], ref["vals"][kept])


def test_large_radius_covers_whole_image():
    w, h = 200, 120
    st = dict(mean2d=[[100.0, 60.0], [10.0, 10.0]], conic=[[1e-4, 0, 1e-4], [0.05, 0, 0.05]], opacity=[0.6, 0.9],
              color=[[1, 0, 0], [0, 1, 0]], radius=[100000, 9])
    got, ref, view = _lists_case(st, [2.0, 1.0], w, h)
    assert np.array_equal(got["keys"], ref["keys"]) and np.array_equal(got["ranges"], ref["ranges"])
    out = view.render_fwd([0, 0, 0])
    sp64 = {k: np.asarray(st[k], dtype=np.float32).astype(np.float64) for k in ("mean2d", "conic", "opacity", "color")}
    r = oracle.render_fwd(sp64, ref, w, h, [0, 0, 0])
    assert np.abs(out["image"] - r["image"]).max() < 1e-5


def test_caller_supplied_conics_that_are_not_positive_definite():
    """pbdr_render_fwd / pbdr_render_bwd accept any splat state. A conic that is not positive definite makes the
    quadratic form negative on part of the image, where the rule is "skip" (no blend); the compositing kernels leave that
    test out only for batches whose conics are all safely positive definite, so a scene that mixes indefinite,
    near-degenerate and ordinary conics over several staging batches exercises both loops, forward and backward."""
    rng = np.random.default_rng(17)
    w, h, n = 96, 80, 900                                   # ~40 splats per tile on average, several batches of 256 in the busy ones
    st = dict(mean2d=np.stack([rng.uniform(0, w, n), rng.uniform(0, h, n)], 1).astype(np.float32),
              conic=np.zeros((n, 3), dtype=np.float32), opacity=rng.uniform(0.05, 0.6, n).astype(np.float32),
              color=rng.uniform(0, 1, (n, 3)).astype(np.float32), radius=rng.integers(4, 40, n).astype(np.int32))
    a = rng.uniform(0.01, 0.08, n); c = rng.uniform(0.01, 0.08, n)
    b = rng.uniform(-0.9, 0.9, n) * np.sqrt(a * c)          # positive definite ...
    kind = rng.integers(0, 4, n)
    b[kind == 1] = (1.5 * np.sqrt(a * c) * rng.choice([-1, 1], n))[kind == 1]                  # ... indefinite ...
    b[kind == 2] = (np.sqrt(a * c) * (1 - 1e-7) * rng.choice([-1, 1], n))[kind == 2]            # ... within rounding of degenerate
    st["conic"] = np.stack([a, b, c], 1).astype(np.float32)
    st["mean2d"][:300] = rng.uniform(30, 50, (300, 2)).astype(np.float32)                     # a crowd, so that lists exceed one batch
    depth = rng.uniform(0.5, 20, n).astype(np.float32)
    got_l, ref_l, view = _lists_case(st, depth, w, h)
    assert np.array_equal(got_l["vals"], ref_l["vals"])
    assert (ref_l["ranges"][:, 1] - ref_l["ranges"][:, 0]).max() > 256
    bg = [0.1, 0.2, 0.3]
    got = view.render_fwd(bg)
    st64 = {k: np.asarray(v, dtype=np.float32).astype(np.float64) for k, v in st.items() if k != "radius"} | {"radius": st["radius"]}
    ref = oracle.render_fwd(st64, ref_l, w, h, bg)
    ok = ref["fragile"] == 0
    assert ok.mean() > 0.95
    assert np.abs(got["image"] - ref["image"])[ok].max() <= 1e-4
    assert np.array_equal(got["last_idx"][ok], ref["last_idx"][ok])
    G = rng.normal(size=(h, w, 3)).astype(np.float32)
    G[~ok] = 0.0
    G[got["last_idx"] != ref["last_idx"]] = 0.0
    g = view.render_bwd(bg, G)
    rg = oracle.render_bwd(st64, ref_l, w, h, bg, G.astype(np.float64))
    for k in ("mean2d", "conic", "opacity", "color"):
        # a pixel that sits within rounding of sigma = 0 of an indefinite splat is flagged fragile and carries no loss;
        # what is left must agree
        grad_close("indefinite conics " + k, g[k], rg[k])


@pytest.mark.parametrize("count", [1, 2, 3, 4, 5, 63, 64, 65, 127, 128, 130, 259])
@pytest.mark.parametrize("opacity", [0.03, 0.5])
def test_walk_of_lists_around_the_batch_and_reduction_sizes(count, opacity):
    """The compositing walks take splats from a 64-bit mask per batch of 64, two at a time forward, and reduce four at a
    time backward: list lengths on both sides of each of these, with pixels that stay open (opacity 0.03) and pixels that
    end at different places within the list (0.5)."""
    rng = np.random.default_rng(count)
    w, h = 16, 16
    st = dict(mean2d=rng.uniform(4, 12, (count, 2)).astype(np.float32),
              conic=np.tile([0.02, 0.003, 0.03], (count, 1)).astype(np.float32), opacity=np.full(count, opacity, dtype=np.float32),
              color=rng.uniform(0, 1, (count, 3)).astype(np.float32), radius=np.full(count, 12, dtype=np.int32))
    got_l, ref_l, view = _lists_case(st, rng.uniform(0.5, 20, count).astype(np.float32), w, h)
    assert np.array_equal(got_l["vals"], ref_l["vals"])
    bg = [0.1, 0.2, 0.3]
    got = view.render_fwd(bg)
    st64 = {k: np.asarray(v).astype(np.float64) for k, v in st.items() if k != "radius"} | {"radius": st["radius"]}
    ref = oracle.render_fwd(st64, ref_l, w, h, bg)
    ok = ref["fragile"] == 0
    assert ok.mean() > 0.95
    assert np.abs(got["image"] - ref["image"])[ok].max() <= 1e-4
    assert np.abs(got["final_T"] - ref["final_T"])[ok].max() <= 1e-4
    assert np.array_equal(got["last_idx"][ok], ref["last_idx"][ok])
    G = rng.normal(size=(h, w, 3)).astype(np.float32)
    G[~ok] = 0.0
    g = view.render_bwd(bg, G)
    rg = oracle.render_bwd(st64, ref_l, w, h, bg, G.astype(np.float64))
    for k in ("mean2d", "conic", "opacity", "color"):
        grad_close(f"walk of {count} " + k, g[k], rg[k])


def _forward_backward_against_oracle(label, st, depth, w, h, seed):
    """Render and its backward on a caller-made state against the oracle: image, last index, and every splat gradient."""
    got_l, ref_l, view = _lists_case(st, depth, w, h)
    assert np.array_equal(got_l["vals"], ref_l["vals"])
    bg = [0.1, 0.2, 0.3]
    got = view.render_fwd(bg)
    st64 = {k: np.asarray(v).astype(np.float64) for k, v in st.items() if k != "radius"} | {"radius": st["radius"]}
    ref = oracle.render_fwd(st64, ref_l, w, h, bg)
    ok = ref["fragile"] == 0
    assert ok.mean() > 0.9
    assert np.abs(got["image"] - ref["image"])[ok].max() <= 1e-4
    assert np.array_equal(got["last_idx"][ok], ref["last_idx"][ok])
    G = np.random.default_rng(seed).normal(size=(h, w, 3)).astype(np.float32)
    G[~ok] = 0.0
    G[got["last_idx"] != ref["last_idx"]] = 0.0
    g = view.render_bwd(bg, G)
    rg = oracle.render_bwd(st64, ref_l, w, h, bg, G.astype(np.float64))
    listed = np.zeros(len(depth), dtype=bool)      # the gradients of the others are not written
    listed[ref_l["vals"]] = True
    for k in ("mean2d", "conic", "opacity", "color"):
        grad_close(f"{label} {k}", g[k][listed], rg[k][listed])


@pytest.mark.parametrize("count", [23, 24, 25, 48, 49, 191, 193, 255, 256, 257, 321, 513])
def test_lists_around_the_chunk_and_run_sizes(count):
    """The forward kernel finds the cells of 256 list positions at a time and stages 64 splats, the backward kernel searches
    256 positions and keeps the sums of 24 visits: lists on both sides of each, every splat on every cell of the tile, and
    faint, so that no pixel ends early."""
    rng = np.random.default_rng(count)
    st = dict(mean2d=rng.uniform(2, 14, (count, 2)).astype(np.float32), conic=np.tile([0.004, 0.001, 0.005], (count, 1)).astype(np.float32),
              opacity=np.full(count, 0.012, dtype=np.float32), color=rng.uniform(0, 1, (count, 3)).astype(np.float32),
              radius=np.full(count, 16, dtype=np.int32))
    _forward_backward_against_oracle(f"{count} splats", st, rng.uniform(0.5, 20, count).astype(np.float32), 16, 16, count)


@pytest.mark.parametrize("kind", ["thin", "sub-pixel", "large", "faint", "opaque", "far"])
def test_cells_that_a_splat_reaches(kind):
    """The compositing kernels visit only the 4x4 cells that the ellipse alpha >= 1/255 of a splat can reach. Shapes at the
    limits of that test - long and thin in every direction, smaller than a pixel, larger than the image, an ellipse that all
    but vanishes (opacity near 1/255), opacities above the clamp, centres far off the image - against the oracle, which
    tests every pixel of the splat's rectangle."""
    rng = np.random.default_rng(len(kind))
    # opaque: a pair leaves 1 - alpha = 0.01 with alpha's 1e-6 on it, 1e-4 of the transmittance recovered from it, so few of them
    # may lie on top of each other
    w, h, n = 72, 56, 40 if kind == "opaque" else 400
    mean = np.stack([rng.uniform(-4, w + 4, n), rng.uniform(-4, h + 4, n)], 1)
    opacity = rng.uniform(0.05, 0.9, n)
    # thin: alpha carries three roundings of terms up to log2(e)/2 a dx^2, 530 at the far end of a diagonal ellipse of 9 by
    # 0.55 px: 1e-4 of itself, which leaves a sum over pixels with cancelling signs within 1e-3
    long, short = dict(thin=((4, 9), (0.55, 0.7)), large=((40, 300), (30, 200))).get(kind, ((0.55, 4.0), (0.55, 3.0)))
    if kind == "sub-pixel":
        long = short = (0.12, 0.4)
    if kind == "faint":
        opacity = rng.uniform(1 / 255, 1.2 / 255, n)
    if kind == "opaque":
        opacity = rng.uniform(0.96, 1.0, n)
    s1, s2, a = rng.uniform(*long, n), rng.uniform(*short, n), rng.uniform(0, np.pi, n)
    if kind == "far":       # a rim of large splats around the image
        t = rng.uniform(0, 2 * np.pi, n)
        s1, s2 = rng.uniform(20, 80, n), rng.uniform(15, 60, n)
        mean = np.stack([w / 2 + 150 * np.cos(t), h / 2 + 150 * np.sin(t)], 1)
    c, s = np.cos(a), np.sin(a)
    conic = np.stack([(c / s1) ** 2 + (s / s2) ** 2, c * s * (1 / s1 ** 2 - 1 / s2 ** 2), (s / s1) ** 2 + (c / s2) ** 2], 1)
    st = dict(mean2d=mean.astype(np.float32), conic=conic.astype(np.float32), opacity=opacity.astype(np.float32),
              color=rng.uniform(0, 1, (n, 3)).astype(np.float32), radius=np.ceil(3.4 * np.maximum(s1, s2)).astype(np.int32))
    _forward_backward_against_oracle(kind, st, rng.uniform(0.5, 20, n).astype(np.float32), w, h, n)


@pytest.mark.parametrize("value", [np.nan, np.inf, -np.inf])
@pytest.mark.parametrize("opacity", [(0.02, 0.3), (0.985, 1.0)])
def test_a_pixel_gradient_that_is_not_finite_stays_with_the_splats_it_blended(value, opacity):
    """One pixel of the image gradient is NaN or infinite, in one colour. The gradients of the splats which that pixel blended
    are lost; those of every other splat are what they are with a zero in its place: of splats that only come near the pixel,
    that reach its cell without blending, or that lie behind its last blended one, in lists of several batches."""
    rng = np.random.default_rng(7)
    w, h, n = 40, 24, 700
    # small and mostly faint, so that pixels stay open; the second range adds splats above the 0.99 clamp, few on a pixel
    o = rng.uniform(0.02, 0.3, n)
    pick = rng.uniform(size=n) < 0.02
    o[pick] = rng.uniform(*opacity, n)[pick]
    s = rng.uniform(0.6, 2.5, n)
    st = dict(mean2d=np.stack([rng.uniform(0, w, n), rng.uniform(0, h, n)], 1).astype(np.float32),
              conic=np.stack([1 / s ** 2, 0.2 / s ** 2, 1.3 / s ** 2], 1).astype(np.float32), opacity=o.astype(np.float32),
              color=rng.uniform(0, 1, (n, 3)).astype(np.float32), radius=np.ceil(3.4 * s).astype(np.int32))
    lists, ref_l, view = _lists_case(st, rng.uniform(0.5, 20, n), w, h)
    assert np.array_equal(lists["vals"], ref_l["vals"])
    assert (ref_l["ranges"][:, 1] - ref_l["ranges"][:, 0]).max() > 128
    bg = [0.1, 0.2, 0.3]
    got = view.render_fwd(bg)
    st64 = {k: np.asarray(v).astype(np.float64) for k, v in st.items() if k != "radius"} | {"radius": st["radius"]}
    ref = oracle.render_fwd(st64, ref_l, w, h, bg)
    ok = (ref["fragile"] == 0) & (got["last_idx"] == ref["last_idx"])
    assert ok.mean() > 0.9
    listed = np.zeros(n, dtype=bool)
    listed[ref_l["vals"]] = True
    for y, x in [(3, 5), (11, 17), (18, 30), (23, 39)]:
        y, x = next((a, b) for a, b in [(y, x), (y - 1, x), (y, x - 1), (y - 1, x - 1)] if ok[a, b] and ref["last_idx"][a, b])
        one = np.zeros((h, w, 3))
        one[y, x] = 1.0
        blended = oracle.render_bwd(st64, ref_l, w, h, bg, one)["color"].any(axis=1)
        assert blended.any()
        G = rng.normal(size=(h, w, 3)).astype(np.float32)
        G[~ok] = 0.0
        G[y, x] = 0.0
        rg = oracle.render_bwd(st64, ref_l, w, h, bg, G.astype(np.float64))
        G[y, x, 1] = value
        g = view.render_bwd(bg, G)
        assert not np.isfinite(g["color"][blended, 1]).any()
        for k in ("mean2d", "conic", "opacity", "color"):
            assert np.isfinite(g[k][listed & ~blended]).all(), k
            grad_close(f"{value} at ({x}, {y}) {k}", g[k][listed & ~blended], rg[k][listed & ~blended])


def test_opacities_and_forms_outside_the_usual_range():
    """Caller-supplied states: an opacity that is NaN or infinite blends with the alpha of the clamp, one below zero nowhere, and
    a quadratic form below zero nowhere however little it is below. Among ordinary splats, in lists of several batches."""
    rng = np.random.default_rng(3)
    w, h, n = 64, 48, 600
    s = rng.uniform(0.6, 3.0, n)
    st = dict(mean2d=np.stack([rng.uniform(0, w, n), rng.uniform(0, h, n)], 1).astype(np.float32),
              conic=np.stack([1 / s ** 2, 0.2 / s ** 2, 1.3 / s ** 2], 1).astype(np.float32), opacity=rng.uniform(0.02, 0.3, n).astype(np.float32),
              color=rng.uniform(0, 1, (n, 3)).astype(np.float32), radius=np.ceil(3.4 * s).astype(np.int32))
    special = np.arange(5, n, 40)
    st["mean2d"][special] = [(x, y) for y in (8, 24, 40) for x in (6, 19, 32, 45, 58)]      # apart: T behind 0.01 is the last to compare
    st["conic"][special] = [0.3, 0.0, 0.3]
    st["opacity"][special] = [np.nan, -0.5, np.inf] * 5
    st["radius"][special] = 4
    depth = rng.uniform(0.5, 20, n).astype(np.float32)
    bg = [0.1, 0.2, 0.3]
    got_l, ref_l, view = _lists_case(st, depth, w, h)
    got = view.render_fwd(bg)
    st64 = {k: np.asarray(v).astype(np.float64) for k, v in st.items() if k != "radius"} | {"radius": st["radius"]}
    ref = oracle.render_fwd(st64, ref_l, w, h, bg)
    ok = (ref["fragile"] == 0) & (got["last_idx"] == ref["last_idx"])
    assert ok.mean() > 0.9 and np.array_equal(got["last_idx"][ref["fragile"] == 0], ref["last_idx"][ref["fragile"] == 0])
    assert np.abs(got["image"] - ref["image"])[ok].max() <= 1e-4
    blended = B.pbdr_render_stats(view.cam, n, view.cap, view.ws)[1]
    assert abs(blended - ref["n_blend"]) <= 1e-3 * ref["n_blend"]
    G = rng.normal(size=(h, w, 3)).astype(np.float32)
    G[~ok] = 0.0
    g = view.render_bwd(bg, G)
    rg = oracle.render_bwd(st64, ref_l, w, h, bg, G.astype(np.float64))
    ordinary = np.ones(n, dtype=bool)
    ordinary[special] = False
    for k in ("mean2d", "conic", "opacity", "color"):
        keep = ordinary if k != "color" else np.ones(n, dtype=bool)
        grad_close("unusual opacities " + k, g[k][keep], rg[k][keep])
    assert np.abs(rg["color"][special[st["opacity"][special] < 0]]).max() == 0.0      # the case is what it claims
    for shown in (np.isnan(st["opacity"]), np.isinf(st["opacity"])):      # (one of them may lie behind two others)
        assert rg["color"][shown].any(axis=1).sum() >= 4

    # forms below zero by 1e-9 of a square pixel and less: as if those splats were not there
    below = 100
    more = {k: np.concatenate([np.asarray(v), np.asarray(v)[:below]]) for k, v in st.items()}
    more["mean2d"][n:] = np.floor(more["mean2d"][n:]) + np.float32(0.25)      # off the lines through the pixel centres, where a form is zero
    more["conic"][n:] = np.array([[0.0, 0.0, -1e-9], [-1e-9, 0.0, 0.0]], dtype=np.float32)[np.arange(below) % 2]
    more["opacity"][n:], more["radius"][n:] = 0.4, 12
    _, ref_l, view = _lists_case(more, np.concatenate([depth, depth[:below]]), w, h)
    got_m = view.render_fwd(bg)
    assert np.abs(got_m["image"] - got["image"]).max() <= 1e-6
    gm = view.render_bwd(bg, G)
    listed = np.unique(ref_l["vals"])
    for k in ("mean2d", "conic", "opacity", "color"):
        assert not gm[k][listed[listed >= n]].any(), k
        grad_close("beside forms below zero " + k, gm[k][:n][ordinary], g[k][ordinary])


def _mixed_list(count, kind):
    """count splats on one 16 x 16 tile, every one on every cell and faint there. kind: opacities above the alpha clamp on all of
    them or on one in 40, seen from afar, and a few on a pixel where the clamp fires; or an indefinite conic on one in 40."""
    rng = np.random.default_rng(count)
    a = rng.uniform(0, 2 * np.pi, count)
    near = rng.uniform(2, 14, (count, 2))
    far = 8 + 47 * np.stack([np.cos(a), np.sin(a)], 1)
    some = np.arange(count) % 40 == 3
    opaque = np.ones(count, dtype=bool) if kind == "opaque" else some & (kind == "mixed")
    st = dict(mean2d=np.where(opaque[:, None], far, near), conic=np.where(opaque[:, None], [0.004, 0.0, 0.004], [0.004, 0.001, 0.005]),
              opacity=np.where(opaque, rng.choice([0.981, 0.985, 0.995, 1.0], count), 0.012), color=rng.uniform(0, 1, (count, 3)))
    clamped = np.array([0, count // 2, count - 1]) if kind != "indefinite" else np.zeros(0, dtype=int)
    st["mean2d"][clamped] = np.array([[3.55, 4.55], [11.55, 2.45], [7.45, 12.55]])[:len(clamped)]
    st["conic"][clamped] = [3.0, 0.0, 3.0]
    st["opacity"][clamped] = 1.0
    if kind == "indefinite":
        st["conic"][some] = [0.004, 0.006, 0.005]
    return {k: v.astype(np.float32) for k, v in st.items()} | dict(radius=np.full(count, 64, dtype=np.int32)), rng.uniform(0.5, 20, count).astype(np.float32)


@pytest.mark.parametrize("count", [3, 24, 25, 63, 64, 65, 129, 255, 256, 257, 321, 513])
@pytest.mark.parametrize("kind", ["mixed", "opaque", "indefinite"])
def test_lists_of_each_kind_of_walk_around_the_chunk_and_run_sizes(count, kind):
    """Windows and batches take a walk without the alpha clamp and the sign test, with the clamp, or with both, by what their
    splats can do: lists around the staging sizes whose batches take the second and the third, some next to the first."""
    st, depth = _mixed_list(count, kind)
    _forward_backward_against_oracle(f"{count} splats, {kind}", st, depth, 16, 16, count)


@pytest.mark.parametrize("aspect", [1, 30, 300, 1000, 1400, 3000, "indefinite"])
def test_the_cull_keeps_every_pixel_that_a_needle_blends(aspect):
    """One splat alone in an image of several hundred cells, at any angle, needles up to 3000 : 1: on both sides of the determinant
    below which the cull takes everything as reached (about 1400 : 1), and forms that are negative in places. Which pixels it
    blends is the oracle's answer, which tests every pixel, wherever rounding does not decide."""
    rng = np.random.default_rng(len(str(aspect)) + (aspect if isinstance(aspect, int) else 0))
    w, h = 112, 96
    st = dict(depth=np.ones(1, dtype=np.float32), color=np.ones((1, 3), dtype=np.float32), radius=np.array([400], dtype=np.int32))
    view = GpuView(1, _cam(w, h), 64)
    shown = decided = 0
    for k in range(40):
        r = aspect if isinstance(aspect, int) else 5
        s2 = np.exp(rng.uniform(np.log(0.3), np.log(3.0)))
        s1 = s2 * r
        a = np.pi / 4 * rng.integers(0, 4) + rng.choice([0.0, 1e-3, 0.3]) if k % 2 else rng.uniform(0, np.pi)
        c, s = np.cos(a), np.sin(a)
        conic = [(c / s1) ** 2 + (s / s2) ** 2, c * s * (1 / s1 ** 2 - 1 / s2 ** 2), (s / s1) ** 2 + (c / s2) ** 2]
        if aspect == "indefinite":
            conic[1] *= 1.0 + rng.uniform(0.0, 0.5) if conic[0] * conic[2] < 1.2 * conic[1] ** 2 else 3.0
        o = rng.choice([1.02 / 255, 1.5 / 255, 0.05, 0.4, 0.97, 1.0])
        st.update(mean2d=np.array([[rng.uniform(-10, w + 10), rng.uniform(-10, h + 10)]], dtype=np.float32),
                  conic=np.array([conic], dtype=np.float32), opacity=np.array([o], dtype=np.float32))
        st64 = {q: v.astype(np.float64) for q, v in st.items() if q != "radius"} | {"radius": st["radius"]}
        lists = oracle.bin_sort(st64["mean2d"], st["radius"], st["depth"], w, h)
        assert lists["P"] == 42
        view.splats = B.Splats.from_numpy(st)
        got = view.render_fwd([0, 0, 0])
        ref = oracle.render_fwd(st64, lists, w, h, [0, 0, 0])
        ok = ref["fragile"] == 0
        bad = ok & (got["last_idx"] != ref["last_idx"])
        assert not bad.any(), (k, np.degrees(a), s2, o, int(bad.sum()), np.argwhere(bad)[:4].tolist())
        shown += int((ok & (ref["last_idx"] == 1)).sum())
        decided += int(ok.sum())
    assert decided > 0.5 * 40 * w * h and shown > 500      # the case is what it claims


@pytest.mark.parametrize("n", [5 * 256, 5 * 256 - 100])
def test_lists_of_blocks_around_the_size_from_which_a_workgroup_writes_a_point(n):
    """A block of 256 points has its workgroup write those on 256 tiles or more if one of them is on 320 or more: blocks whose
    points are all on 255, on 258, on 318 and on 321 tiles, and one of the first two with a single point of the last."""
    w, h = 5000, 40                                          # three rows of 313 tiles
    rng = np.random.default_rng(n)
    cols = np.repeat([85, 86, 106, 107, 0], 256)[:n]
    cols[4 * 256:] = rng.choice([85, 86], n - 4 * 256)
    cols[4 * 256 + 77] = 107
    st = _rand_state(rng, n, w, h)
    st["mean2d"] = np.stack([16.0 * rng.integers(60, 250, n) + 8 * (cols % 2), np.full(n, 20.0)], 1).astype(np.float32)
    st["radius"] = (8 * cols - 8).astype(np.int32)
    depth = rng.uniform(0.3, 50, n).astype(np.float32)
    got, ref, _ = _lists_case(st, depth, w, h)
    assert np.array_equal(np.bincount(ref["vals"], minlength=n), 3 * cols)      # the case is what it claims
    assert np.array_equal(got["keys"], ref["keys"]) and np.array_equal(got["vals"], ref["vals"])
    assert np.array_equal(got["ranges"], ref["ranges"])
