"""GPU parity for 2D Gaussian surfels: the HIP path (through the C ABI) against the CPU oracle, element by element.

Staged like the 3D-Gaussian tests:
  A. preprocess: fp32 vs fp64 with tolerances; visibility and extent exact except where the oracle flags the decision
     as within 2e-5 of flipping (or the extent as ill-conditioned).
  B. tile lists bit-exact, oracle binning fed with the GPU's own fp32 (mean2d, radius, depth).
  C. compositing forward / backward: oracle fed with the GPU's fp32 state and the identical lists; image within 1e-4
     absolute, gradients within 1e-3 relative + floor; pixels the oracle flags as fragile carry no loss gradient.
  D. splatting backward: oracle fed with the GPU's splat-state gradient.
  E. a full-size view of the 1M-surfel configuration.
"""
import numpy as np
import pytest
import torch

import oracle
from gpu_pipeline import to_chw_dev, to_hwc
from helpers import grad_close, to_f64
from paper_2512_20017_amd import binding as B
from paper_2512_20017_amd import synth

pytestmark = pytest.mark.gpu

BG = [0.1, 0.3, 0.2]
IMG_ATOL = 1e-4
GRAD_RTOL = 1e-3
STATE_KEYS = ("mean2d", "T", "opacity", "color")
PARAM_KEYS = ("mean", "tan_u", "tan_v", "log_scale", "logit", "sh")


class SurfelView:
    def __init__(self, n, cam, cap):
        self.n, self.cam, self.cap = n, cam, int(cap)
        self.W, self.H = cam["width"], cam["height"]
        self.splats = B.Splats2D.empty(n)
        self.ws = B.alloc_workspace2d(n, self.W, self.H, self.cap)
        self.image = torch.empty((3, self.H, self.W), dtype=torch.float32, device="cuda")
        self.final_T = torch.empty((self.H, self.W), dtype=torch.float32, device="cuda")
        self.last_idx = torch.empty((self.H, self.W), dtype=torch.int32, device="cuda")
        self.g_splats = B.SplatGrads2D.empty(n)

    def preprocess(self, scene):
        B.pbdr2d_preprocess(scene, self.cam, self.splats)
        torch.cuda.synchronize()
        return self.splats.to_numpy()

    def render_fwd(self, bg):
        B.pbdr2d_render_fwd(self.splats, self.cam, bg, self.cap, self.image, self.final_T, self.last_idx, self.ws)
        torch.cuda.synchronize()
        return dict(image=to_hwc(self.image), final_T=self.final_T.cpu().numpy(),
                    last_idx=self.last_idx.cpu().numpy().astype(np.uint32))

    def lists(self):
        return B.pbdr2d_lists_view(self.ws, self.n, self.W, self.H, self.cap)

    def render_bwd(self, bg, G_hwc, scene=None, grads=None):
        B.pbdr2d_render_bwd(scene, self.splats, self.cam, bg, self.cap, self.final_T, self.last_idx, to_chw_dev(G_hwc),
                            self.g_splats, grads, self.ws)
        torch.cuda.synchronize()
        return self.g_splats.to_numpy()


def _state64(sp):
    return {k: sp[k].astype(np.float64) for k in STATE_KEYS} | {"radius": sp["radius"]}


def _grad_close(name, got, ref):
    grad_close("surfels " + name, got, ref)


def _check_preprocess(sp, ref, cam, sc, max_tie=0.01):
    # S: magnitude of the world coordinates entering p = R x + t (fp32 leaves ~4e-7 S absolute error in p)
    S = float(np.abs(sc["mean"]).max() + np.abs(cam["t"]).max())
    tie = ref["near_tie"] != 0
    assert tie.mean() < max_tie
    assert np.array_equal(sp["radius"][~tie], ref["radius"][~tie])
    vis = (sp["radius"] > 0) & (ref["radius"] > 0)
    if vis.any():
        f = max(cam["fx"], cam["fy"])
        z = ref["depth"][vis]
        # the centre comes through p = R x + t and a perspective divide, the transform through products with f and c
        slope = np.abs(ref["mean2d"][vis] - np.array([cam["cx"], cam["cy"]])) / f
        m_tol = 1e-4 + 3e-7 * np.abs(ref["mean2d"][vis]) + 4e-7 * S * f * (1.0 + slope) / z[:, None]
        m_err = np.abs(sp["mean2d"][vis] - ref["mean2d"][vis])
        assert (m_err <= m_tol).all(), (int((m_err > m_tol).sum()), float(m_err.max()))
        # rows of T are sums of products of size (f + c) x |p|; compare against the row's size and that floor
        scale = np.abs(ref["T"][vis]).reshape(-1, 3, 3).max(axis=2, keepdims=True)
        t_tol = (3e-6 * scale + 6e-7 * (f + max(cam["cx"], cam["cy"])) * S) * np.ones((1, 1, 3))
        t_tol[:, 2, :] = 3e-6 * scale[:, 2, :] + 6e-7 * S
        t_err = np.abs(sp["T"][vis].reshape(-1, 3, 3) - ref["T"][vis].reshape(-1, 3, 3))
        assert (t_err <= t_tol).all(), (int((t_err > t_tol).sum()), float(t_err.max()))
        np.testing.assert_allclose(sp["opacity"][vis], ref["opacity"][vis], rtol=2e-6, atol=1e-7)
        np.testing.assert_allclose(sp["color"][vis], ref["color"][vis], rtol=2e-5, atol=4e-6)
        np.testing.assert_allclose(sp["depth"][vis], ref["depth"][vis], rtol=2e-6, atol=2e-6 + 6e-7 * S)
        # Gram-Schmidt loses accuracy as the raw tangents approach parallel: error ~ eps / sin(angle between them)
        a, b = np.asarray(sc["tan_u"], dtype=np.float64)[vis], np.asarray(sc["tan_v"], dtype=np.float64)[vis]
        sin = np.linalg.norm(np.cross(a, b), axis=1) / (np.linalg.norm(a, axis=1) * np.linalg.norm(b, axis=1))
        n_err = np.abs(sp["normal"][vis] - ref["normal"][vis]).max(axis=1)
        assert (n_err <= 2e-6 / sin).all(), float((n_err * sin).max())
    return tie, vis


CASES = [
    ("deg3_ragged", lambda: (synth.random_small_surfels(21, 500, 3, spread=1.2, ls_mu=-2.4),
                             synth.pinhole(200, 120, 60.0, *synth.look_at([0.4, 0.3, -3.0], [0, 0, 0], [0, 1, 0])))),
    ("deg2_ragged", lambda: (synth.random_small_surfels(22, 300, 2, spread=0.9),
                             synth.pinhole(75, 51, 50.0, np.eye(3), [0.0, 0.1, 2.6]))),
    ("deg1_dense", lambda: (synth.random_small_surfels(23, 2000, 1, spread=0.5, ls_mu=-2.0),
                            synth.pinhole(64, 64, 50.0, np.eye(3), [0.0, 0.0, 2.0]))),
    ("deg0_small_disks", lambda: (synth.random_small_surfels(24, 3000, 0, spread=1.0, ls_mu=-4.5),     # low-pass dominated
                                  synth.pinhole(160, 96, 55.0, np.eye(3), [0.0, 0.0, 2.5]))),
]


@pytest.fixture(scope="module", params=CASES, ids=[c[0] for c in CASES])
def case(request):
    sc, cam = request.param[1]()
    n = sc["mean"].shape[0]
    scene = B.Scene2D.from_numpy(sc)
    ref = oracle.preprocess2d(to_f64(sc), cam)
    probe = SurfelView(n, cam, 1)
    sp = probe.preprocess(scene)
    lists = oracle.bin_sort(sp["mean2d"].astype(np.float64), sp["radius"], sp["depth"], cam["width"], cam["height"])
    view = SurfelView(n, cam, lists["P"] + 17)
    sp2 = view.preprocess(scene)
    for k in sp:
        assert np.array_equal(sp[k][sp["radius"] > 0], sp2[k][sp["radius"] > 0])
    return dict(sc=sc, cam=cam, n=n, scene=scene, ref=ref, view=view, sp=sp, lists=lists)


def test_a_preprocess(case):
    _check_preprocess(case["sp"], case["ref"], case["cam"], case["sc"], max_tie=0.02)
    assert (case["sp"]["radius"] > 0).sum() > 0.3 * case["n"]


def test_b_lists_bit_exact(case):
    view, lists = case["view"], case["lists"]
    view.render_fwd(BG)
    gl = view.lists()
    assert gl["P_raw"] == lists["P"]
    assert np.array_equal(gl["keys"], lists["keys"])
    assert np.array_equal(gl["vals"], lists["vals"])
    assert np.array_equal(gl["ranges"], lists["ranges"])


def test_c_compositing(case):
    view, lists, cam, sp = case["view"], case["lists"], case["cam"], case["sp"]
    W, H = cam["width"], cam["height"]
    got = view.render_fwd(BG)
    st = _state64(sp)
    ref = oracle.render_fwd2d(st, lists, W, H, BG)
    ok = ref["fragile"] == 0
    assert (~ok).mean() < 0.02
    assert np.abs(got["image"] - ref["image"])[ok].max() <= IMG_ATOL
    assert np.abs(got["final_T"] - ref["final_T"])[ok].max() <= IMG_ATOL
    assert np.array_equal(got["last_idx"][ok], ref["last_idx"][ok])
    assert ref["n_blend"] > 10 * W * H / 256
    G = np.random.default_rng(5).normal(size=(H, W, 3)).astype(np.float32)
    G[~ok] = 0.0
    gs = view.render_bwd(BG, G)
    ref_b = oracle.render_bwd2d(st, lists, W, H, BG, G.astype(np.float64))
    v = sp["radius"] > 0
    assert np.abs(ref_b["T"]).max() > 0 and np.abs(ref_b["mean2d"]).max() > 0
    # the transform's gradient is judged row by row against that row's own magnitude (rows differ by the focal length)
    for r in range(3):
        _grad_close(f"T{r}", gs["T"][v][:, 3 * r:3 * r + 3], ref_b["T"][v][:, 3 * r:3 * r + 3])
    for k in ("mean2d", "opacity", "color"):
        _grad_close(k, gs[k][v], ref_b[k][v])


def test_d_splatting_backward(case):
    view, cam, sp, sc, scene = case["view"], case["cam"], case["sp"], case["sc"], case["scene"]
    W, H = cam["width"], cam["height"]
    view.render_fwd(BG)
    G = np.random.default_rng(6).normal(size=(H, W, 3)).astype(np.float32)
    grads = scene.zeros_like()
    gs = view.render_bwd(BG, G, scene=scene, grads=grads)
    got = grads.to_numpy()
    ref = oracle.preprocess_bwd2d(to_f64(sc), cam, {k: gs[k].astype(np.float64) for k in STATE_KEYS})
    both = (sp["radius"] > 0) & (case["ref"]["radius"] > 0) & (case["ref"]["near_tie"] == 0)
    for k in PARAM_KEYS:
        _grad_close(k, got[k][both], ref[k][both])
    # accumulation: a second backward doubles the parameter gradient (up to the order of the in-tile float sums)
    view.render_bwd(BG, G, scene=scene, grads=grads)
    got2 = grads.to_numpy()
    for k in PARAM_KEYS:
        np.testing.assert_allclose(got2[k], 2.0 * got[k], rtol=1e-4, atol=1e-5 * np.abs(got[k]).max())


def test_edge_empty_and_all_culled():
    cam = synth.pinhole(48, 40, 50.0, np.eye(3), [0.0, 0.0, 2.0])
    # no points at all
    view = SurfelView(0, cam, 1)
    scene = B.Scene2D.from_numpy(dict(mean=np.zeros((0, 3)), tan_u=np.zeros((0, 3)), tan_v=np.zeros((0, 3)),
                                      log_scale=np.zeros((0, 2)), logit=np.zeros(0), sh=np.zeros((0, 1, 3)), sh_degree=0))
    view.preprocess(scene)
    out = view.render_fwd(BG)
    assert np.allclose(out["image"], np.asarray(BG, dtype=np.float32)[None, None, :])
    assert (out["final_T"] == 1).all() and (out["last_idx"] == 0).all()
    # every point behind the camera
    sc = synth.random_small_surfels(31, 100, 1)
    sc["mean"][:, 2] -= 10.0
    scene = B.Scene2D.from_numpy(sc)
    view = SurfelView(100, cam, 64)
    sp = view.preprocess(scene)
    assert (sp["radius"] == 0).all()
    out = view.render_fwd(BG)
    assert np.allclose(out["image"], np.asarray(BG, dtype=np.float32)[None, None, :])
    assert view.lists()["P_raw"] == 0
    grads = scene.zeros_like()
    view.render_bwd(BG, np.ones((40, 48, 3), dtype=np.float32), scene=scene, grads=grads)
    assert all(not v.any() for k, v in grads.to_numpy().items() if k != "sh_degree")


def test_edge_capacity_overflow_is_contained():
    sc = synth.random_small_surfels(23, 2000, 1, spread=0.5, ls_mu=-2.0)
    cam = synth.pinhole(64, 64, 50.0, np.eye(3), [0.0, 0.0, 2.0])
    scene = B.Scene2D.from_numpy(sc)
    view = SurfelView(2000, cam, 500)
    view.preprocess(scene)
    out = view.render_fwd(BG)
    gl = view.lists()
    assert gl["P_raw"] > 500 and gl["P"] == 500
    assert np.isfinite(out["image"]).all()
    gs = view.render_bwd(BG, np.ones((64, 64, 3), dtype=np.float32))
    v = view.splats.radius.cpu().numpy() > 0
    assert all(np.isfinite(gs[k][v]).all() for k in STATE_KEYS)


@pytest.mark.timeout(600)
def test_e_full_size_view():
    """1M surfels, SH3, 1920x1080 (the surfel benchmark configuration), every stage over the whole image."""
    sc = synth.scene_surfels(0)
    cam = synth.cameras_sphere()[0]
    n = sc["mean"].shape[0]
    W, H = cam["width"], cam["height"]
    scene = B.Scene2D.from_numpy(sc)
    cap = 8_000_000
    view = SurfelView(n, cam, cap)
    sp = view.preprocess(scene)
    sc64 = to_f64(sc)
    ref = oracle.preprocess2d(sc64, cam)
    tie, vis = _check_preprocess(sp, ref, cam, sc)
    lists = oracle.bin_sort(sp["mean2d"].astype(np.float64), sp["radius"], sp["depth"], W, H)
    assert lists["P"] <= cap
    got = view.render_fwd([0.0, 0.0, 0.0])
    gl = view.lists()
    assert gl["P_raw"] == lists["P"]
    assert np.array_equal(gl["keys"], lists["keys"])
    assert np.array_equal(gl["vals"], lists["vals"])
    assert np.array_equal(gl["ranges"], lists["ranges"])
    st = _state64(sp)
    ref_f = oracle.render_fwd2d(st, lists, W, H, [0.0, 0.0, 0.0])
    ok = ref_f["fragile"] == 0
    assert (~ok).mean() < 0.02
    assert np.abs(got["image"] - ref_f["image"])[ok].max() <= IMG_ATOL
    assert np.abs(got["final_T"] - ref_f["final_T"])[ok].max() <= IMG_ATOL
    assert np.array_equal(got["last_idx"][ok], ref_f["last_idx"][ok])
    G = np.random.default_rng(0).normal(size=(H, W, 3)).astype(np.float32)
    G[~ok] = 0.0
    grads = scene.zeros_like()
    gs = view.render_bwd([0.0, 0.0, 0.0], G, scene=scene, grads=grads)
    ref_b = oracle.render_bwd2d(st, lists, W, H, [0.0, 0.0, 0.0], G.astype(np.float64))
    v = sp["radius"] > 0
    for r in range(3):
        _grad_close(f"T{r}", gs["T"][v][:, 3 * r:3 * r + 3], ref_b["T"][v][:, 3 * r:3 * r + 3])
    for k in ("mean2d", "opacity", "color"):
        _grad_close(k, gs[k][v], ref_b[k][v])
    ref_g = oracle.preprocess_bwd2d(sc64, cam, {k: gs[k].astype(np.float64) for k in STATE_KEYS})
    got_g = grads.to_numpy()
    both = vis & ~tie
    for k in PARAM_KEYS:
        _grad_close(k, got_g[k][both], ref_g[k][both])


def test_first_view_writes_what_zero_then_accumulate_leaves():
    """Surfel twin of the 3D test: first_view stores instead of accumulating and zeroes the points the view skips."""
    sc = synth.random_small_surfels(41, 400, 2, spread=1.2)
    cam = synth.pinhole(96, 64, 45.0, *synth.look_at([0.3, 0.1, -2.5], [0, 0, 0], [0, 1, 0]))
    scene = B.Scene2D.from_numpy(sc)
    view = SurfelView(400, cam, 200000)
    sp = view.preprocess(scene)
    assert 0 < (sp["radius"] > 0).sum() < 400
    view.render_fwd(BG)
    G = np.random.default_rng(2).normal(size=(64, 96, 3)).astype(np.float32)
    ref = scene.zeros_like()
    view.render_bwd(BG, G, scene=scene, grads=ref)
    got = scene.zeros_like()
    for t in (got.mean, got.tan_u, got.tan_v, got.log_scale, got.logit, got.sh):
        t.fill_(float("nan"))
    B.pbdr2d_render_bwd(scene, view.splats, cam, BG, view.cap, view.final_T, view.last_idx, to_chw_dev(G), view.g_splats, got,
                        view.ws, first_view=True)
    torch.cuda.synchronize()
    a, b = got.to_numpy(), ref.to_numpy()
    unused = sp["radius"] <= 0
    for k in PARAM_KEYS:
        assert np.isfinite(a[k]).all(), k
        np.testing.assert_allclose(a[k], b[k], rtol=4e-6, atol=1e-6 * np.abs(b[k]).max())
        assert not a[k][unused].any(), k


def test_backward_without_splat_gradient_output():
    """g_splats = NULL with a scene: the splatting backward reads the per-point records in the workspace instead of the
    planes; the parameter gradient is the one the two-step path gives (same values and formulas; the two compositing runs
    differ by the rounding of their LDS adds and the two kernel variants by the compiler's choice of fused multiply-adds:
    4e-6 relative, as between the store and accumulate variants), as a store and as an accumulation, for the whole image
    and for a patch."""
    sc = synth.random_small_surfels(43, 3000, 2, spread=1.2)
    cam = synth.pinhole(160, 96, 50.0, *synth.look_at([0.3, 0.1, -2.5], [0, 0, 0], [0, 1, 0]))
    scene = B.Scene2D.from_numpy(sc)
    view = SurfelView(3000, cam, 400000)
    sp = view.preprocess(scene)
    assert 0 < (sp["radius"] > 0).sum() < 3000
    view.render_fwd(BG)
    G = to_chw_dev(np.random.default_rng(3).normal(size=(96, 160, 3)).astype(np.float32))
    for first in (True, False):
        ref, got = scene.zeros_like(), scene.zeros_like()
        if not first:
            for t in (ref, got):
                t.mean.fill_(0.25); t.sh.fill_(-0.5)
        B.pbdr2d_render_bwd(scene, view.splats, cam, BG, view.cap, view.final_T, view.last_idx, G, view.g_splats, ref, view.ws,
                            first_view=first)
        B.pbdr2d_render_bwd(scene, view.splats, cam, BG, view.cap, view.final_T, view.last_idx, G, None, got, view.ws,
                            first_view=first)
        torch.cuda.synchronize()
        a, b = got.to_numpy(), ref.to_numpy()
        for k in PARAM_KEYS:
            np.testing.assert_allclose(a[k], b[k], rtol=4e-6, atol=1e-6 * np.abs(b[k]).max(), err_msg=f"{k} {first}")
            assert np.array_equal(a[k] == 0, b[k] == 0) or first is False, k      # the same points get exact zeros
        assert np.abs(b["mean"]).max() > 0
    # a patch
    patch = (37, 10, 140, 81)
    w, h = patch[2] - patch[0], patch[3] - patch[1]
    splats = B.Splats2D.empty(3000)
    B.pbdr2d_preprocess_patch(scene, cam, patch, splats)
    image = torch.empty((3, h, w), device="cuda"); T = torch.empty((h, w), device="cuda")
    last = torch.empty((h, w), dtype=torch.int32, device="cuda")
    B.pbdr2d_render_fwd_patch(splats, cam, patch, BG, view.cap, image, T, last, view.ws)
    Gp = G[:, patch[1]:patch[3], patch[0]:patch[2]].contiguous()
    ref, got = scene.zeros_like(), scene.zeros_like()
    B.pbdr2d_render_bwd_patch(scene, splats, cam, patch, BG, view.cap, T, last, Gp, view.g_splats, ref, view.ws, first_view=True)
    B.pbdr2d_render_bwd_patch(scene, splats, cam, patch, BG, view.cap, T, last, Gp, None, got, view.ws, first_view=True)
    torch.cuda.synchronize()
    a, b = got.to_numpy(), ref.to_numpy()
    for k in PARAM_KEYS:
        np.testing.assert_allclose(a[k], b[k], rtol=4e-6, atol=1e-6 * np.abs(b[k]).max(), err_msg=k)
    # no output at all is still an error
    with pytest.raises(B.PbdrError):
        B.pbdr2d_render_bwd(None, view.splats, cam, BG, view.cap, view.final_T, view.last_idx, G, None, None, view.ws)


def test_backward_writes_every_per_pair_record_itself():
    """The backward pass needs no cleared workspace: records of pairs that lie behind the last splat their tile blended are
    written as zeros by the compositing kernel. A dense scene (most lists end early on transmittance) is rendered with
    the whole workspace poisoned with NaN bit patterns before the forward pass; the gradient equals that of a clean run."""
    sc = synth.random_small_surfels(47, 6000, 1, spread=0.5, ls_mu=-1.6)     # large, overlapping disks
    sc["logit"] = np.full(6000, 4.0, dtype=np.float32)                       # nearly opaque: pixels saturate early
    cam = synth.pinhole(160, 96, 50.0, *synth.look_at([0.2, 0.1, -2.5], [0, 0, 0], [0, 1, 0]))
    scene = B.Scene2D.from_numpy(sc)
    G = np.random.default_rng(9).normal(size=(96, 160, 3)).astype(np.float32)
    out = []
    for poison in (False, True):
        view = SurfelView(6000, cam, 600000)
        view.ws.fill_(0xFF if poison else 0)
        vis = view.preprocess(scene)["radius"] > 0
        fw = view.render_fwd(BG)
        lists = view.lists()
        grads = scene.zeros_like()
        g2 = view.render_bwd(BG, G, scene=scene, grads=grads)
        out.append((g2, grads.to_numpy(), fw, lists))
    (g2a, ga, fwa, la), (g2b, gb, fwb, lb) = out
    # the case is what it claims: many pairs lie behind the last blended splat of their tile
    tiles = la["ranges"]
    walked = 0
    last = fwa["last_idx"]
    for t in range(tiles.shape[0]):
        ty, tx = divmod(t, 10)
        walked += int(last[ty * 16:(ty + 1) * 16, tx * 16:(tx + 1) * 16].max())
    assert walked < 0.8 * la["P"], (walked, la["P"])
    assert np.array_equal(fwa["image"], fwb["image"])
    for k in g2a:      # the splat-state gradient is written for the listed points only
        assert np.isfinite(g2b[k][vis]).all(), k
        np.testing.assert_allclose(g2b[k][vis], g2a[k][vis], rtol=1e-5, atol=1e-6 * np.abs(g2a[k][vis]).max(), err_msg=k)
    for k in PARAM_KEYS:
        assert np.isfinite(gb[k]).all(), k
        np.testing.assert_allclose(gb[k], ga[k], rtol=1e-5, atol=1e-6 * np.abs(ga[k]).max(), err_msg=k)


def _image_space_state(rng, centre, sigma, depth, tilt, opacity, cam):
    """Splat state of disks of `sigma` pixels around `centre`, tilted out of the image plane by up to `tilt` radians."""
    n = len(centre)
    f, c = cam["fx"], np.array([cam["cx"], cam["cy"]])
    mid = np.concatenate([(centre - c) / f, np.ones((n, 1))], 1) * depth[:, None]
    ang, lean = rng.uniform(0, 2 * np.pi, n), rng.uniform(0, tilt, n)
    tu = np.stack([np.cos(ang) * np.cos(lean), np.sin(ang) * np.cos(lean), np.sin(lean)], 1)
    tv = np.stack([-np.sin(ang), np.cos(ang), np.zeros(n)], 1)
    H = np.stack([tu * (sigma * depth / f)[:, None], tv * (sigma * depth / f)[:, None], mid], 2)      # columns u, v, centre
    K = np.array([[f, 0, c[0]], [0, f, c[1]], [0, 0, 1]])
    T = (K @ H).reshape(n, 9).astype(np.float32)
    return dict(mean2d=(T[:, [2, 5]] / T[:, 8:9]).astype(np.float32), T=T, opacity=np.broadcast_to(opacity, n).astype(np.float32),
                color=rng.uniform(0, 1, (n, 3)).astype(np.float32), radius=np.full(n, 12, dtype=np.int32),
                depth=depth.astype(np.float32))


def _one_tile_walk_case(count, opacity):
    """`count` disks over one 16 x 16 tile, every third of them so small that the low-pass is what shows."""
    rng = np.random.default_rng(count)
    cam = synth.pinhole(16, 16, 30.0, np.eye(3), [0.0, 0.0, 0.0])
    sigma = np.where(np.arange(count) % 3 == 2, rng.uniform(0.05, 0.3, count), rng.uniform(1.0, 3.0, count))
    return cam, _image_space_state(rng, rng.uniform(1, 15, (count, 2)), sigma, rng.uniform(0.5, 20, count), 0.9, opacity, cam)


@pytest.mark.parametrize("count", [1, 2, 3, 4, 5, 7, 63, 64, 65, 129, 255, 256, 257, 321, 515])
@pytest.mark.parametrize("opacity", [0.03, 0.5])
def test_walk_of_lists_around_the_batch_and_reduction_sizes(count, opacity):
    """The surfel walks stage 256 (forward) and 64 (backward) splats at a time, take them from 64-bit masks two at a time
    forward, note which of them a quadrant blended, and reduce the pixels' sums four visits at a time backward: list
    lengths on both sides of each of these, with pixels that stay open (opacity 0.03) and pixels that end at different
    places within the list (0.5)."""
    cam, st = _one_tile_walk_case(count, opacity)
    view = SurfelView(count, cam, count)
    view.splats = B.Splats2D.from_numpy(st)
    lists = oracle.bin_sort(st["mean2d"].astype(np.float64), st["radius"], st["depth"], 16, 16)
    assert lists["P"] == count
    got = view.render_fwd(BG)
    ref = oracle.render_fwd2d(_state64(st), lists, 16, 16, BG)
    ok = ref["fragile"] == 0
    assert ok.mean() > 0.95
    assert np.abs(got["image"] - ref["image"])[ok].max() <= IMG_ATOL
    assert np.abs(got["final_T"] - ref["final_T"])[ok].max() <= IMG_ATOL
    assert np.array_equal(got["last_idx"][ok], ref["last_idx"][ok])
    G = np.random.default_rng(7).normal(size=(16, 16, 3)).astype(np.float32)
    G[~ok] = 0.0
    gs = view.render_bwd(BG, G)
    ref_b = oracle.render_bwd2d(_state64(st), lists, 16, 16, BG, G.astype(np.float64))
    for r in range(3):
        _grad_close(f"walk of {count} T{r}", gs["T"][:, 3 * r:3 * r + 3], ref_b["T"][:, 3 * r:3 * r + 3])
    for k in ("mean2d", "opacity", "color"):
        _grad_close(f"walk of {count} {k}", gs[k], ref_b[k])


@pytest.mark.parametrize("count, blended", [
    (300, [0]), (300, [255]), (300, [256]), (257, [0, 255, 256]), (513, [0, 511, 512]),
    (600, list(range(1, 600, 9))), (512, list(range(0, 512, 8))), (520, list(range(0, 520, 8))),      # 67, 64 and 65 of them
    (700, list(range(190, 320)) + [512, 699]), (256, list(range(256))),
    (66000, [3, 40000, 65279, 65280, 65534, 65535, 65536, 65537, 65791, 65792, 65999] + list(range(64700, 65500, 10)))])
def test_backward_finds_the_blended_entries_of_a_list(count, blended):
    """The surfel backward kernel searches a tile's list 256 positions at a time for the entries that some quadrant blended
    and stages 64 of those at a time; positions are kept in 16 bits with their upper half apart. Blended splats on both
    sides of each of these limits among others that reach no pixel or only the gaps between pixel centres: the gradient is
    the oracle's and, since a splat's sums do not depend on its place, bit for bit that of a list of the blended ones
    alone, and zero for the others whatever the workspace held."""
    rng = np.random.default_rng(count)
    cam = synth.pinhole(16, 16, 30.0, np.eye(3), [0.0, 0.0, 0.0])
    shown = np.zeros(count, dtype=bool)
    shown[blended] = True
    gap = rng.uniform(size=count) < 0.5      # o exp(-1/2) < 1/255 at the four pixel centres around a corner, o > 1/255
    centre = np.where(shown[:, None], rng.uniform(1, 15, (count, 2)), rng.integers(2, 15, (count, 2)))
    st = _image_space_state(rng, centre, np.where(shown, rng.uniform(1.0, 3.0, count), 0.2), 1.0 + 0.001 * np.arange(count), 0.6,
                            np.where(shown, 0.03, np.where(gap, 0.005, 0.002)), cam)
    lists = oracle.bin_sort(st["mean2d"].astype(np.float64), st["radius"], st["depth"], 16, 16)
    assert np.array_equal(lists["vals"], np.arange(count))
    G = rng.normal(size=(16, 16, 3)).astype(np.float32)
    G[oracle.render_fwd2d(_state64(st), lists, 16, 16, BG)["fragile"] != 0] = 0.0
    ref = oracle.render_bwd2d(_state64(st), lists, 16, 16, BG, G.astype(np.float64))
    out = []
    for keep in (np.ones(count, dtype=bool), shown):
        part = {k: v[keep] for k, v in st.items()}
        view = SurfelView(int(keep.sum()), cam, int(keep.sum()))
        view.ws.fill_(0xFF)
        view.splats = B.Splats2D.from_numpy(part)
        fw = view.render_fwd(BG)
        out.append((fw, view.render_bwd(BG, G)))
    (fwa, ga), (fwb, gb) = out
    assert np.array_equal(fwa["image"], fwb["image"])
    for k in STATE_KEYS:
        assert np.array_equal(ga[k][shown], gb[k]), k
        assert not ga[k][~shown].any(), k
    for r in range(3):
        _grad_close(f"{len(blended)} of {count} T{r}", ga["T"][:, 3 * r:3 * r + 3], ref["T"][:, 3 * r:3 * r + 3])
    for k in ("mean2d", "opacity", "color"):
        _grad_close(f"{len(blended)} of {count} {k}", ga[k], ref[k])


def _ended_quadrant_case():
    """One 16 x 16 tile. 40 disks around (3, 3) end every pixel of the first quadrant and leave the far corner of the last
    one open; behind them come faint disks around (13, 13), from the 65th splat on (the first quadrant's wavefront has left
    the list by then) in turn with disks that reach into the first quadrant only."""
    rng = np.random.default_rng(3)
    n = 240
    cam = synth.pinhole(16, 16, 30.0, np.eye(3), [0.0, 0.0, 0.0])
    far = np.arange(n) >= 40
    behind = (np.arange(n) >= 64) & (np.arange(n) % 2 == 1)
    centre = np.where((far & ~behind)[:, None], 13.0, 3.0) + rng.uniform(-0.3, 0.3, (n, 2))
    sigma = np.where(behind, 1.0, np.where(far, 1.5, 5.0))
    opacity = np.where(behind, 0.5, np.where(far, 0.05, 0.95))
    return cam, behind, _image_space_state(rng, centre, sigma, 1.0 + 0.01 * np.arange(n), 0.3, opacity, cam)


@pytest.mark.parametrize("poison", [0x00, 0xFF])
def test_backward_does_not_visit_splats_behind_a_quadrants_last_blended_one(poison):
    """A splat that no pixel of a quadrant blended must not enter that quadrant's backward walk, whatever the workspace held
    before the forward pass: with a colour that is not finite, one visit turns the quadrant's running sums into NaN
    (0 * inf). The gradient is that of the same splats with finite colours behind, element for element."""
    cam, behind, st = _ended_quadrant_case()
    lists = oracle.bin_sort(st["mean2d"].astype(np.float64), st["radius"], st["depth"], 16, 16)
    assert lists["P"] == 240 and np.array_equal(lists["vals"], np.arange(240))
    ref = oracle.render_fwd2d(_state64(st), lists, 16, 16, BG)
    assert ref["last_idx"][:8, :8].max() <= 40 and ref["last_idx"].max() > 200      # the case is what it claims
    G = np.random.default_rng(8).normal(size=(16, 16, 3)).astype(np.float32)
    out = []
    for value in (0.5, np.inf):
        view = SurfelView(240, cam, 240)
        view.ws.fill_(poison)
        colour = st["color"].copy()
        colour[behind] = value
        view.splats = B.Splats2D.from_numpy(dict(st, color=colour))
        fw = view.render_fwd(BG)
        assert np.isfinite(fw["image"]).all() and np.array_equal(fw["last_idx"], ref["last_idx"])
        out.append((fw, view.render_bwd(BG, G)))
    (fwa, ga), (fwb, gb) = out
    assert np.array_equal(fwa["image"], fwb["image"])
    for k in STATE_KEYS:
        assert np.isfinite(gb[k]).all(), k
        assert np.array_equal(ga[k], gb[k]), k
        assert not gb[k][behind].any(), k


def test_backward_after_other_views_on_the_same_workspace():
    """The words the forward pass leaves per list position belong to its own view: a view that ends early, a sparse one and a
    dense one in turn on one workspace give each the gradient that it gives on a fresh workspace."""
    sc = synth.random_small_surfels(51, 4000, 1, spread=0.6, ls_mu=-2.0)
    sc["logit"] = np.full(4000, 2.0, dtype=np.float32)
    cams = [synth.pinhole(160, 96, fov, *synth.look_at(eye, [0, 0, 0], [0, 1, 0]))
            for fov, eye in ((25.0, [0.2, 0.1, -2.5]), (80.0, [0.0, 0.4, -4.0]), (50.0, [1.5, 0.1, -2.0]))]
    scene = B.Scene2D.from_numpy(sc)
    G = np.random.default_rng(10).normal(size=(96, 160, 3)).astype(np.float32)
    shared = SurfelView(4000, cams[0], 400000)
    for cam in cams + cams[:1]:
        fresh = SurfelView(4000, cam, 400000)
        shared.cam = cam
        got = []
        for view in (shared, fresh):
            vis = view.preprocess(scene)["radius"] > 0
            view.render_fwd(BG)
            got.append(view.render_bwd(BG, G))
        assert vis.any()
        for k in STATE_KEYS:
            assert np.array_equal(got[0][k][vis], got[1][k][vis]), k


def _spread_disks(rng, centre, sigma, tilt, opacity):
    """One disk per tile of a 640 x 640 image, away from its neighbours, its surroundings empty."""
    cam = synth.pinhole(640, 640, 50.0, np.eye(3), [0.0, 0.0, 0.0])
    corner = np.stack(np.meshgrid(np.arange(40), np.arange(40)), 2).reshape(-1, 2) * 16.0
    st = _image_space_state(rng, corner + centre, sigma, rng.uniform(0.5, 20, 1600), tilt, opacity, cam)
    st["radius"][:] = 6
    return cam, st


def _gradient_and_reference(cam, st, G):
    lists = oracle.bin_sort(st["mean2d"].astype(np.float64), st["radius"], st["depth"], 640, 640)
    view = SurfelView(1600, cam, lists["P"])
    view.splats = B.Splats2D.from_numpy(st)
    black = [0.0, 0.0, 0.0]
    view.render_fwd(black)
    G[oracle.render_fwd2d(_state64(st), lists, 640, 640, black)["fragile"] != 0] = 0.0
    return view.render_bwd(black, G), oracle.render_bwd2d(_state64(st), lists, 640, 640, black, G.astype(np.float64))


@pytest.mark.parametrize("off", [0.02, 0.005])
def test_low_pass_centre_gradient_keeps_its_precision_beside_the_centre(off):
    """Sub-pixel disks `off` pixels from a pixel's centre, with a loss on that pixel only: the gradient of the projected
    centre is one product with that offset. Eight roundings of half a unit in the last place (offset, two exponentials
    of one unit each, transmittance, weight, products) are 5e-7; a sum about a point three pixels away rounds at three
    pixels instead of at `off` (1e-5 and 4e-5)."""
    rng = np.random.default_rng(5)
    cam, st = _spread_disks(rng, rng.integers(4, 12, (1600, 2)) + 0.5 + rng.choice([-1, 1], (1600, 2)) * off,
                            np.full(1600, 0.1), 0.3, 0.5)
    px = np.floor(st["mean2d"]).astype(int)
    G = np.zeros((640, 640, 3), dtype=np.float32)
    G[px[:, 1], px[:, 0]] = rng.uniform(0.5, 1.5, (1600, 3))
    got, ref = _gradient_and_reference(cam, st, G)
    ok = np.abs(ref["mean2d"]) > 0
    assert ok.mean() > 0.99
    assert (np.abs(got["mean2d"] - ref["mean2d"])[ok] / np.abs(ref["mean2d"])[ok]).max() <= 1e-6


def test_opacity_gradient_of_faint_disks_keeps_its_precision():
    """Disks of opacity 0.008 to 0.06, far from each other. The gradient is a sum of G^ dL/dalpha over the pixels; four
    roundings a term (exponential, weight, their product, dL/dalpha), each half a unit at most and 0.29 of 2^-23 in the
    mean square, are 7e-8 before the sum averages them. Formed as (o G^) / o the terms share the rounding of
    log2(o) + ex, of size 5: 2e-7 in the mean square."""
    rng = np.random.default_rng(5)
    cam, st = _spread_disks(rng, 8 + rng.uniform(-1, 1, (1600, 2)), rng.uniform(1.0, 2.0, 1600), 0.5, rng.uniform(0.008, 0.06, 1600))
    got, ref = _gradient_and_reference(cam, st, rng.uniform(0.5, 1.5, (640, 640, 3)).astype(np.float32))
    err = (got["opacity"] - ref["opacity"]) / ref["opacity"]
    assert np.sqrt((err ** 2).mean()) <= 1e-7
    # an opacity that is not finite is clamped everywhere: no gradient reaches it
    st["opacity"][::7] = np.inf
    view = SurfelView(1600, cam, 160000)
    view.splats = B.Splats2D.from_numpy(st)
    view.render_fwd(BG)
    assert not view.render_bwd(BG, np.ones((640, 640, 3), dtype=np.float32))["opacity"][::7].any()
