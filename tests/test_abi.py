"""Host-side checks of the C-ABI library that need no GPU: it loads, exports every declared symbol, sizes
workspaces sensibly and rejects bad arguments before touching the device."""
import ctypes as C
import os
import re

import pytest

from paper_2512_20017_amd import binding as B
from paper_2512_20017_amd import synth

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _declared():
    text = open(os.path.join(ROOT, "include", "pbdr.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(pbdr(?:2d)?_[a-z0-9_]+)\s*\(", text)))


def test_library_exports_every_declared_symbol():
    names = _declared()
    assert set(names) == set(B.EXPORTS)
    L = C.CDLL(B.LIB_PATH)
    for n in names:
        assert getattr(L, n) is not None
    assert B.pbdr_version() == 100


def test_workspace_bytes():
    small = B.pbdr_workspace_bytes(4096, 128, 128, 20000)
    big = B.pbdr_workspace_bytes(1_000_000, 1920, 1080, 8_000_000)
    assert 0 < small < big
    assert big % 256 == 0
    # 132 B/point (64-byte raster record, depth bits, tile count, offset, slot base, rank -> point, 48-byte gradient record) + 70 B/pair
    # (point index, the unsorted {depth bits, point index} or inspection keys, 8 B that the sort and the gather use in turn, 48 B of
    # partial gradient sums, two bytes of cell bits; chunk owners are four bytes per 256 pairs) + 12 B/tile
    for n, cap in ((1_000_000, 8_000_000), (3_000_000, 2_500_000)):
        big = B.pbdr_workspace_bytes(n, 1920, 1080, cap)
        assert abs(big - (132 * n + (70 + 4 / 256) * cap + 12 * 8160)) < 1e5
        # surfels: 16 B more per point (64-byte gradient records) and 16 B more per pair (64 B of partial sums)
        big2 = B.pbdr2d_workspace_bytes(n, 1920, 1080, cap)
        assert abs((big2 - big) - (16 * n + 16 * cap)) < 1e4
    with pytest.raises(B.PbdrError):
        B.pbdr_workspace_bytes(-1, 128, 128, 10)
    with pytest.raises(B.PbdrError):
        B.pbdr_workspace_bytes(10, 0, 128, 10)
    with pytest.raises(B.PbdrError):
        B.pbdr_workspace_bytes(10, 128, 128, 1 << 40)


@pytest.mark.parametrize("size", [B.pbdr_workspace_bytes, B.pbdr2d_workspace_bytes])
def test_workspace_of_a_large_grid(size):
    """Twelve bytes a tile: where its list starts and ends, and its place in the order."""
    one_tile = size(1000, 16, 16, 400_000)
    for w, h in ((65536, 65536), (65536, 100), (3840, 2160)):
        tiles = (w + 15) // 16 * ((h + 15) // 16)
        assert size(1000, w, h, 400_000) - one_tile <= 12 * tiles + 1024


# (points, width, height, pairs): bytes of the 3D and of the surfel workspace that calls of these sizes have been served with
SERVED = {(30_011, 1031, 517, 400_000): (34_024_192, 41_704_192), (1000, 65536, 65536, 400_000): (231_494_144, 238_710_016),
          (100_000, 1280, 720, 1 << 20): (91_980_288, 112_454_656), (4096, 128, 128, 20_000): (2_047_232, 2_472_704),
          (1, 1, 1, 1): (8448, 8448), (7_722_898, 4772, 16, 28_794): (1_022_196_480, 1_146_281_216),
          (1_000_000, 1920, 1080, 8_000_000): (732_805_376, 892_805_376)}


@pytest.mark.parametrize("args", SERVED)
def test_a_workspace_that_served_a_call_still_does(args):
    assert B.pbdr_workspace_bytes(*args) <= SERVED[args][0]
    assert B.pbdr2d_workspace_bytes(*args) <= SERVED[args][1]


@pytest.mark.parametrize("size", [B.pbdr_workspace_bytes, B.pbdr2d_workspace_bytes])
def test_a_workspace_serves_every_smaller_capacity(size):
    """Also around 2^20 pairs, where the sums over a point's pairs change their way of working."""
    for n, w, h in ((100_000, 1280, 720), (1, 16, 16)):
        caps = [0, 1, 2, 63, 64, 65, 255, 256, 257, 1_040_000, (1 << 20) - 1, 1 << 20, (1 << 20) + 1, 1_050_000, 1 << 21, (1 << 22) - 1, 1 << 22, (1 << 22) + 1, 1 << 24]
        sizes = [size(n, w, h, c) for c in caps]
        assert sizes == sorted(sizes)


def test_invalid_arguments_are_rejected_on_the_host():
    L = B.lib()
    cam = B.camera_struct(dict(width=64, height=64, fx=50, fy=50, cx=32, cy=32, R=[1, 0, 0, 0, 1, 0, 0, 0, 1], t=[0, 0, 3]))
    sc = B.CScene(-5, 0, None, None, None, None, None)
    sp = B.CSplats(-5, None, None, None, None, None, None)
    assert L.pbdr_preprocess(C.byref(sc), C.byref(cam), C.byref(sp), None) == B.PBDR_ERR_INVALID_ARG
    sc = B.CScene(8, 7, None, None, None, None, None)      # bad SH degree
    sp = B.CSplats(8, None, None, None, None, None, None)
    assert L.pbdr_preprocess(C.byref(sc), C.byref(cam), C.byref(sp), None) == B.PBDR_ERR_INVALID_ARG
    sc = B.CScene(8, 0, 16, 16, 16, 16, 16)                  # null splat outputs
    assert L.pbdr_preprocess(C.byref(sc), C.byref(cam), C.byref(sp), None) == B.PBDR_ERR_INVALID_ARG
    sc = B.CScene(8, 0, 20, 16, 16, 16, 16)                  # misaligned pointer
    sp = B.CSplats(8, 16, 16, 16, 16, 16, 16)
    assert L.pbdr_preprocess(C.byref(sc), C.byref(cam), C.byref(sp), None) == B.PBDR_ERR_INVALID_ARG
    bad = B.camera_struct(dict(width=64, height=64, fx=50, fy=50, cx=32, cy=32, R=[1, 0, 0, 0, 1, 0, 0, 0, 1], t=[0, 0, 3], near=0.0))
    sc = B.CScene(8, 0, 16, 16, 16, 16, 16)
    assert L.pbdr_preprocess(C.byref(sc), C.byref(bad), C.byref(sp), None) == B.PBDR_ERR_INVALID_ARG
    # workspace too small / misaligned
    bg = (C.c_float * 3)(0, 0, 0)
    assert L.pbdr_render_fwd(C.byref(sp), C.byref(cam), bg, C.c_uint64(100), C.c_void_p(16), C.c_void_p(16), C.c_void_p(16),
                             C.c_void_p(256), C.c_size_t(64), None) == B.PBDR_ERR_WORKSPACE_TOO_SMALL
    assert L.pbdr_render_fwd(C.byref(sp), C.byref(cam), bg, C.c_uint64(100), C.c_void_p(16), C.c_void_p(16), C.c_void_p(16),
                             C.c_void_p(272), C.c_size_t(1 << 30), None) == B.PBDR_ERR_INVALID_ARG
    assert B.lib().pbdr_status_string(C.c_int(-2)).decode() == "workspace too small"


def test_batch_calls_reject_bad_arguments_on_the_host():
    L = B.lib()
    cam = dict(width=64, height=64, fx=50, fy=50, cx=32, cy=32, R=[1, 0, 0, 0, 1, 0, 0, 0, 1], t=[0, 0, 3])
    sc = B.CScene(8, 0, 16, 16, 16, 16, 16)
    grads = B.CScene(8, 0, 16, 16, 16, 16, 16, 0)

    def arrays(count, n=8):
        cams = (B.CCamera * count)(*[B.camera_struct(cam) for _ in range(count)])
        sps = (B.CSplats * count)(*[B.CSplats(n, 16, 16, 16, 16, 16, 16) for _ in range(count)])
        g2s = (B.CSplatGrads * count)(*[B.CSplatGrads(n, 16, 16, 16, 16) for _ in range(count)])
        return cams, sps, g2s

    cams, sps, g2s = arrays(17)
    for count in (0, -1, 17):          # 1 .. PBDR_MAX_BATCH_VIEWS views
        assert L.pbdr_preprocess_batch(C.byref(sc), C.c_int32(count), cams, sps, C.c_int32(0), None, None, None) == B.PBDR_ERR_INVALID_ARG
        assert L.pbdr_preprocess_bwd_batch(C.byref(sc), C.c_int32(count), cams, sps, g2s, C.byref(grads), None) == B.PBDR_ERR_INVALID_ARG
    cams, sps, g2s = arrays(2)
    assert L.pbdr_preprocess_batch(C.byref(sc), C.c_int32(2), None, sps, C.c_int32(0), None, None, None) == B.PBDR_ERR_INVALID_ARG
    assert L.pbdr_preprocess_batch(C.byref(sc), C.c_int32(2), cams, sps, C.c_int32(300), None, None, None) == B.PBDR_ERR_INVALID_ARG
    # group test asked for, but no bounds / keep
    assert L.pbdr_preprocess_batch(C.byref(sc), C.c_int32(2), cams, sps, C.c_int32(256), None, None, None) == B.PBDR_ERR_INVALID_ARG
    _, odd, _ = arrays(2, n=9)         # a view whose arrays are sized for another cloud
    assert L.pbdr_preprocess_batch(C.byref(sc), C.c_int32(2), cams, odd, C.c_int32(0), None, None, None) == B.PBDR_ERR_INVALID_ARG
    assert L.pbdr_preprocess_bwd_batch(C.byref(sc), C.c_int32(2), cams, sps, g2s, None, None) == B.PBDR_ERR_INVALID_ARG
    # pbdr_render_bwd: no splat-state gradient output only together with a scene
    bg = (C.c_float * 3)(0, 0, 0)
    sp = B.CSplats(8, 16, 16, 16, 16, 16, 16)
    c1 = B.camera_struct(cam)
    assert L.pbdr_render_bwd(None, C.byref(sp), C.byref(c1), bg, C.c_uint64(100), C.c_void_p(16), C.c_void_p(16), C.c_void_p(16),
                             None, None, C.c_void_p(256), C.c_size_t(1 << 30), None) == B.PBDR_ERR_INVALID_ARG


def _table3():
    """{'3dgs': [(name, elems), ...], '2dgs': [...]} from the fixture that restates the paper's Table 3."""
    out, cur = {}, None
    for line in open(os.path.join(os.path.dirname(__file__), "golden", "table3_state_layout.txt")):
        line = line.strip()
        if not line or line.startswith("#"):
            continue
        if line.startswith("["):
            cur = line.strip("[]")
            out[cur] = []
        else:
            name, k = line.split()
            out[cur].append((name, int(k)))
    return out


def _struct_fields(header_text, struct):
    """[(field, elements per point)] of a state struct of the header, from its '[k][n]' / '[n]' layout comments."""
    body = re.search(r"typedef struct %s \{(.*?)\} %s;" % (struct, struct), header_text, re.S).group(1)
    fields = []
    for m in re.finditer(r"\*\s*(\w+);\s*/\*\s*\[(\d+)\]\[n\]|\*\s*(\w+);\s*/\*\s*\[n\]", body):
        fields.append((m.group(1), int(m.group(2))) if m.group(1) else (m.group(3), 1))
    return fields


def test_state_layout_is_table_3():
    """The per-view state that crosses the boundary is the paper's Table 3, field by field: same order, same element
    counts, 11 and 20 elements per point; the oracle's arrays have the same widths."""
    t3 = _table3()
    text = open(os.path.join(ROOT, "include", "pbdr.h")).read()
    for key, struct in (("3dgs", "pbdr_splats"), ("2dgs", "pbdr2d_splats")):
        rows = t3[key]
        assert rows[-1][0] == "total" and rows[-1][1] == sum(k for _, k in rows[:-1])
        fields = _struct_fields(text, struct)
        assert [k for _, k in fields] == [k for _, k in rows[:-1]], (struct, fields)
        # names agree up to the plural and the underscore style
        for (f, _), (r, _) in zip(fields, rows[:-1]):
            assert f.replace("_", "")[:4] == r.replace("_", "")[:4], (f, r)
    assert t3["3dgs"][-1][1] * 4 == 44 and t3["2dgs"][-1][1] * 4 == 80

    import numpy as np
    import oracle
    from paper_2512_20017_amd import synth
    sc, cam = synth.scene_tiny(0), synth.camera_tiny()
    sp = oracle.preprocess({k: (v.astype(np.float64) if isinstance(v, np.ndarray) else v) for k, v in sc.items()}, cam)
    widths = dict(mean2d=2, conic=3, opacity=1, color=3, radius=1, depth=1)
    for (name, k), (field, w) in zip(t3["3dgs"][:-1], widths.items()):
        assert k == w
        arr = np.asarray(sp[field])
        assert (arr.shape[1] if arr.ndim == 2 else 1) == k, field


def test_static_scratch_limits_and_arguments():
    L = B.lib()
    cam_ok = B.camera_struct(synth.camera_tiny(64, 64))
    cam_big = B.camera_struct(synth.camera_tiny(B.PBDR_STATIC_MAX_SIDE + 16, 64))
    bg = (C.c_float * 3)(0, 0, 0)
    sp_big = B.CSplats(B.PBDR_STATIC_MAX_POINTS + 1, 16, 16, 16, 16, 16, 16)
    sp_ok = B.CSplats(8, 16, 16, 16, 16, 16, 16)
    args = (C.c_void_p(16), C.c_void_p(16), C.c_void_p(16), None, None)
    assert L.pbdr_render_fwd_static(C.byref(sp_big), C.byref(cam_ok), bg, *args) == B.PBDR_ERR_STATIC_LIMIT
    assert L.pbdr_render_fwd_static(C.byref(sp_ok), C.byref(cam_big), bg, *args) == B.PBDR_ERR_STATIC_LIMIT
    assert L.pbdr_render_fwd_static(C.byref(sp_ok), C.byref(cam_ok), bg, C.c_void_p(0), C.c_void_p(16), C.c_void_p(16), None,
                                    None) == B.PBDR_ERR_INVALID_ARG
    assert "static scratch" in L.pbdr_status_string(C.c_int(B.PBDR_ERR_STATIC_LIMIT)).decode()
    # the largest admitted sizes fit the array
    assert B.pbdr_workspace_bytes(B.PBDR_STATIC_MAX_POINTS, B.PBDR_STATIC_MAX_SIDE, B.PBDR_STATIC_MAX_SIDE,
                                  B.PBDR_STATIC_MAX_PAIRS) <= B.PBDR_STATIC_SCRATCH_BYTES
