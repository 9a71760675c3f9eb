"""The sums over a point's pairs (pair_reduce.h) where they are cut: a wavefront adds up 64 pairs, or 256 in steps of 64 if there are
more than 2^20, and a point cut by such a border is put together by the kernel that reads the point's record. Points with pair
counts on both sides of every border, among points of one pair that move the borders about; both models, with and without the
splat-state gradient; room for fewer pairs than there are. Against the oracle."""
import numpy as np
import pytest
import torch

import oracle
from gpu_pipeline import GpuView
from helpers import grad_close
from paper_2512_20017_amd import binding as B
from paper_2512_20017_amd import synth
from test_gpu_surfels import SurfelView

pytestmark = pytest.mark.gpu

TILES = 640
W, H = 16 * TILES, 16
BG = [0.1, 0.3, 0.2]
SIZES = [1, 2, 63, 64, 65, 127, 128, 129, 191, 192, 193, 255, 256, 257, 319, 320, 321, 511, 512, 513, 640]
KEYS = dict(gauss=("mean2d", "conic", "opacity", "color"), surfel=("mean2d", "T", "opacity", "color"))


def _strip(model, seed):
    """One row of tiles; every point of SIZES lies on that many of them, and 300 more on one each. Returns camera and state."""
    rng = np.random.default_rng(seed)
    size = rng.permutation(np.concatenate([SIZES, np.ones(300, dtype=np.int64)]))
    n = len(size)
    first = (rng.random(n) * (TILES + 1 - size)).astype(np.int64)
    centre = np.stack([16.0 * first + 8 * size, np.full(n, 8.0)], 1)
    cam = synth.pinhole(W, H, 60.0, np.eye(3), [0.0, 0.0, 3.0])
    depth = rng.uniform(0.5, 20, n)
    st = dict(mean2d=centre.astype(np.float32), opacity=rng.uniform(0.05, 0.3, n).astype(np.float32),
              color=rng.uniform(0, 1, (n, 3)).astype(np.float32), radius=(8 * size - 1).astype(np.int32), depth=depth.astype(np.float32))
    sx = 3.0 * size
    if model == "gauss":
        st["conic"] = np.stack([1 / sx ** 2, np.zeros(n), np.full(n, 1 / 25.0)], 1).astype(np.float32)
    else:
        f, mid = cam["fx"], (centre - [cam["cx"], cam["cy"]]) / cam["fx"]
        H3 = np.zeros((n, 3, 3))      # columns: half axes and centre, in camera space
        H3[:, 0, 0] = sx * depth / f
        H3[:, 1, 1] = 5.0 * depth / f
        H3[:, :2, 2], H3[:, 2, 2] = mid * depth[:, None], depth
        K = np.array([[f, 0, cam["cx"]], [0, f, cam["cy"]], [0, 0, 1]])
        st["T"] = (K @ H3).reshape(n, 9).astype(np.float32)
    return cam, st, int(size.sum())


def _view(model, cam, st, cap):
    view = (GpuView if model == "gauss" else SurfelView)(len(st["opacity"]), cam, cap)
    view.splats = (B.Splats if model == "gauss" else B.Splats2D).from_numpy(st)
    return view


def _state64(model, st):
    return {k: st[k].astype(np.float64) for k in KEYS[model]} | {"radius": st["radius"]}


def _loss_gradient(model, st, lists, seed):
    """dL/dimage, zero at the pixels whose blending rounding may decide either way."""
    ref = (oracle.render_fwd if model == "gauss" else oracle.render_fwd2d)(_state64(model, st), lists, W, H, BG)
    G = np.random.default_rng(seed).normal(size=(H, W, 3)).astype(np.float32)
    G[ref["fragile"] != 0] = 0.0
    return G


def _reference(model, st, lists, G):
    return (oracle.render_bwd if model == "gauss" else oracle.render_bwd2d)(_state64(model, st), lists, W, H, BG, G.astype(np.float64))


@pytest.mark.parametrize("model", ["gauss", "surfel"])
@pytest.mark.parametrize("seed", [0, 1, 2])
def test_room_for_fewer_pairs_than_there_are(model, seed):
    """The pairs beyond the capacity are dropped, the first in point order stay: the gradient is that of the lists that are left,
    and a point none of whose pairs was kept gets zeros, whatever an earlier call on the workspace left there."""
    cam, st, P = _strip(model, seed)
    cap = P // 2 + seed
    other = dict(st, radius=np.full_like(st["radius"], 7))      # one pair a point: fills the records of those that the second call drops
    view = _view(model, cam, other, cap)
    view.render_fwd(BG)
    view.render_bwd(BG, np.ones((H, W, 3), dtype=np.float32))
    view.splats = _view(model, cam, st, 1).splats
    view.render_fwd(BG)
    lists = view.lists()
    assert lists["P_raw"] == P and len(lists["vals"]) == cap
    G = _loss_gradient(model, st, lists, seed)
    got, ref = view.render_bwd(BG, G), _reference(model, st, lists, G)
    dropped = np.ones(len(st["opacity"]), dtype=bool)
    dropped[lists["vals"]] = False
    assert dropped.sum() > 50
    for k in KEYS[model]:
        grad_close(f"{model} cut {k}", got[k], ref[k])
        assert not got[k][dropped].any()


@pytest.mark.parametrize("model", ["gauss", "surfel"])
@pytest.mark.parametrize("seed", [0, 1])
def test_borders_of_the_sums(model, seed):
    """Every point against the oracle; and the same bits whatever the room, on both sides of 2^20 pairs of it."""
    cam, st, P = _strip(model, seed)
    lists = oracle.bin_sort(st["mean2d"].astype(np.float64), st["radius"], st["depth"], W, H)
    assert lists["P"] == P
    G = _loss_gradient(model, st, lists, seed)
    ref, got = _reference(model, st, lists, G), []
    for cap in (P, 1 << 20, (1 << 20) + 1):
        view = _view(model, cam, st, cap)
        view.render_fwd(BG)
        got.append(view.render_bwd(BG, G))
    for k in KEYS[model]:
        grad_close(f"{model} {k}", got[0][k], ref[k])
        for g in got[1:]:
            assert np.array_equal(g[k], got[0][k]), k


@pytest.mark.parametrize("model", ["gauss", "surfel"])
def test_borders_of_the_long_chunks(model):
    """More than 2^20 pairs, in points of 1 to 640 of them: 256 pairs a wavefront, a segment open from one step of 64 to the next.
    Three of four points are too faint to blend: the lists are 1,640 splats deep, and 410 blended ones keep the rounding of the
    walk over them, which is not the subject, as small as in a usual scene."""
    cam, st, P = _strip(model, 5)
    copies = (1 << 20) // P + 2
    n1 = len(st["opacity"])
    big = {k: np.concatenate([v] * copies) for k, v in st.items()}
    big["opacity"] = np.where(np.arange(n1 * copies) // n1 % 4 == 0, 0.02, 0.003).astype(np.float32)
    lists = oracle.bin_sort(big["mean2d"].astype(np.float64), big["radius"], big["depth"], W, H)
    assert lists["P"] == P * copies > 1 << 20
    G = _loss_gradient(model, big, lists, 5)
    view = _view(model, cam, big, lists["P"])
    view.render_fwd(BG)
    got, ref = view.render_bwd(BG, G), _reference(model, big, lists, G)
    for k in KEYS[model]:
        grad_close(f"{model} long {k}", got[k], ref[k])
