"""The C ABI library loads, exports what include/sne.h declares, and rejects
bad arguments with status codes before touching the GPU."""
import ctypes
import os

import pytest

from paper_2005_08165_amd import sne


def test_exports_every_declared_function():
    L = sne.lib()
    names = sne.header_functions()
    assert len(names) >= 13
    for n in names:
        assert hasattr(L, n), n
    assert set(sne._SIGS) <= set(names)


def test_header_constants_match_binding():
    import re
    text = open(sne.HEADER).read()
    m = re.search(r"#define SNE_NOALLOC_MAX_FRAMES (\d+)", text)
    assert m and int(m.group(1)) == sne.SNE_NOALLOC_MAX_FRAMES
    m = re.search(r"#define SNE_LENIENT (0x[0-9a-f]+)", text)
    assert m and int(m.group(1), 16) == sne.SNE_LENIENT
    for name in ("SNE_ERR_ARG", "SNE_ERR_BUDGET", "SNE_ERR_STATE"):
        m = re.search(r"#define %s \((-\d+)\)" % name, text)
        assert m and int(m.group(1)) == getattr(sne, name), name


def test_noalloc_rejects_bad_arguments_before_the_gpu():
    L = sne.lib()
    # a NULL context is refused first, whatever else is passed
    assert L.sne_estimate_batched_noalloc(None, None, 1, 1, 0, 0, 1, None) == sne.SNE_ERR_ARG


def test_version_and_status_strings():
    assert sne.version() == 10500
    assert sne.status_string(0) == "ok"
    assert sne.status_string(-1) == "invalid argument"
    assert sne.status_string(12345) == "unknown status"


def _K(fx=500.0, fy=500.0, u0=10.0, v0=10.0):
    return sne.Intrinsics(fx, fy, u0, v0)


FAKE = 0x10000  # never dereferenced: every call below fails validation first


@pytest.mark.parametrize("case", [
    dict(inp=None), dict(normals=None), dict(H=0), dict(W=0), dict(in_pitch=5),
    dict(out_pitch=5), dict(mask_pitch=5), dict(kind=7), dict(grad=-1), dict(agg=2),
    dict(out=2), dict(K=_K(fx=0.0)), dict(K=_K(fy=-1.0)), dict(K=_K(u0=float("nan"))),
    dict(K=_K(fx=float("inf"))), dict(kind=3, K=_K(fx=500.0, fy=501.0)), dict(Knull=True),
    dict(kind=0x200), dict(kind=0x104), dict(kind=0x103, K=_K(fx=500.0, fy=501.0)),
])
def test_estimate_argument_errors(case):
    L = sne.lib()
    a = dict(inp=FAKE, H=10, W=10, in_pitch=10, kind=0, grad=0, agg=0, out=0, normals=FAKE,
             out_pitch=10, mask=FAKE, mask_pitch=10, K=_K())
    a.update(case)
    K = None if case.get("Knull") else ctypes.byref(a["K"])
    rc = L.sne_estimate(None, a["inp"], a["H"], a["W"], a["in_pitch"], K, a["kind"], a["grad"],
                        a["agg"], a["out"], a["normals"], a["out_pitch"], a["mask"],
                        a["mask_pitch"], None)
    assert rc == -1


def test_uniform_argument_errors():
    L = sne.lib()
    K = _K()
    # frame strides too small for B > 1
    assert L.sne_estimate_uniform(None, FAKE, 4, 10, 10, 10, 50, ctypes.byref(K), 0, 0, 0, 0,
                                  FAKE, 10, 300, FAKE, 10, 100, None) == -1
    assert L.sne_estimate_uniform(None, FAKE, 4, 10, 10, 10, 100, ctypes.byref(K), 0, 0, 0, 0,
                                  FAKE, 10, 299, FAKE, 10, 100, None) == -1
    assert L.sne_estimate_uniform(None, FAKE, -1, 10, 10, 10, 100, ctypes.byref(K), 0, 0, 0, 0,
                                  FAKE, 10, 300, FAKE, 10, 100, None) == -1
    # B = 0 is a valid empty batch: nothing is launched, NULL pointers allowed
    assert L.sne_estimate_uniform(None, FAKE, 0, 10, 10, 10, 100, ctypes.byref(K), 0, 0, 0, 0,
                                  FAKE, 10, 300, FAKE, 10, 100, None) == 0
    assert L.sne_estimate_uniform(None, None, 0, 10, 10, 10, 0, ctypes.byref(K), 0, 0, 0, 0,
                                  None, 10, 0, None, 10, 0, None) == 0
    # ... but not NULL pointers for a real frame
    assert L.sne_estimate_uniform(None, None, 1, 10, 10, 10, 0, ctypes.byref(K), 0, 0, 0, 0,
                                  FAKE, 10, 0, None, 10, 0, None) == -1


def test_null_context_errors():
    L = sne.lib()
    t = sne.Tile(2, 8)
    assert L.sne_set_tile(None, ctypes.byref(t)) == -1
    assert L.sne_estimate_batched(None, None, 1, 0, 0, 0, 0, None) == -1
    assert L.sne_set_intrinsics_table(None, None, 1) == -1
    assert L.sne_autotune(None, 10, 10, 1, 0, 0, 0, 0, None) == -1
    assert L.sne_autotune_batched(None, None, 1, 0, 0, 0, 0, None) == -1
    assert L.sne_accuracy(None, None, 0, None, None, 0, 0, None, 0, None, None) == -1
    assert L.sne_autotune_save(None, b"/tmp/x") == -1
    assert L.sne_ctx_destroy(None) == 0
    assert L.sne_ctx_create(None, 0) == -1
    assert L.sne_get_tile(None, 0, 10, 1, 0, 0, 0, 0, ctypes.byref(t)) == -1
    assert L.sne_get_tile(None, 10, 10, 0, 0, 0, 0, 0, ctypes.byref(t)) == -1
    kx = (ctypes.c_float * 49)()
    assert L.sne_set_gradient_kernel(None, kx) == -1
    assert L.sne_set_gradient_kernel_n(None, 5, kx) == -1
    assert L.sne_autotune_pitched(None, 10, 10, 1, 16, 16, 0, 0, 0, 0, None) == -1
    assert L.sne_get_tile_pitched(None, 10, 10, 1, 16, 16, 0, 0, 0, 0, None) == -1
    assert L.sne_get_tile_pitched(None, 10, 10, 1, 8, 16, 0, 0, 0, 0, ctypes.byref(t)) == -1


def test_row_pitch():
    """The smallest pitch >= W whose rows are 256-byte multiples."""
    L = sne.lib()
    assert L.sne_row_pitch(1242, 4) == 1280 and L.sne_row_pitch(640, 4) == 640
    assert L.sne_row_pitch(1, 4) == 64 and L.sne_row_pitch(64, 4) == 64
    assert L.sne_row_pitch(65, 4) == 128 and L.sne_row_pitch(320, 2) == 384
    assert L.sne_row_pitch(1920, 2) == 1920 and L.sne_row_pitch(1242, 1) == 1280
    assert L.sne_row_pitch(0, 4) < 0 and L.sne_row_pitch(10, 8) < 0 and L.sne_row_pitch(10, 3) < 0
    import torch
    assert sne.row_pitch(1242, torch.float32) == 1280
    assert sne.row_pitch(1242, torch.uint8) == 1280 and sne.row_pitch(1242, torch.float16) == 1280
    # without a context the heuristic applies to both layouts alike
    t1, t2 = sne.Tile(), sne.Tile()
    assert L.sne_get_tile_pitched(None, 375, 1242, 128, 1280, 1280, 3, 2, 1, 0,
                                  ctypes.byref(t1)) == 0
    assert L.sne_get_tile(None, 375, 1242, 128, 3, 2, 1, 0, ctypes.byref(t2)) == 0
    assert (t1.cols_per_lane, t1.rows, t1.lanes) == (t2.cols_per_lane, t2.rows, t2.lanes)


def test_default_tile_shape_without_context():
    L = sne.lib()
    t = sne.Tile()
    assert L.sne_get_tile(None, 480, 640, 64, 0, 0, 0, 0, ctypes.byref(t)) == 0
    assert t.cols_per_lane in (1, 2, 4) and 1 <= t.rows <= 1024 and t.lanes in (32, 64)
    # 640 = 5 x 128: the chosen strip width leaves no idle lane
    assert 640 % (t.cols_per_lane * t.lanes) == 0


def test_binding_fails_loudly_without_library(monkeypatch, tmp_path):
    monkeypatch.setattr(sne, "_lib", None)
    monkeypatch.setattr(sne, "LIB_PATH", str(tmp_path / "missing.so"))
    with pytest.raises(RuntimeError, match="not built"):
        sne.lib()


def test_shipped_tuning_table_is_well_formed():
    """Every line of the shipped tile table parses as sne_autotune_save
    writes it, with shapes the library accepts; the batched 480x640
    Sobel-median workload has an entry."""
    from paper_2005_08165_amd import tune
    assert os.path.exists(sne.TUNING_TABLE) and sne.TUNING_TABLE == tune.TABLE
    keys = set()
    for line in open(sne.TUNING_TABLE):
        if line.startswith("#") or not line.strip():
            continue
        f = line.split()
        assert len(f) == 14, line
        arch, ver, H, W, bc, kind, grad, agg, out, layout, px, rows, remap, half = (
            [f[0]] + [int(x) for x in f[1:]])
        assert ver == sne.TILE_CACHE_VERSION and H >= 1 and W >= 1 and bc in (0, 1, 2, 3)
        assert kind in sne.KIND.values() and grad in sne.GRAD.values()
        assert agg in sne.AGG.values() and out in (0, 1) and layout in (0, 1)
        assert px in (1, 2, 4) and 1 <= rows <= 1024 and 0 <= remap <= 1024 and half in (0, 1)
        # the row-layout class of a dense frame follows from its width; the
        # uneven-batch class is always tuned and looked up as unaligned
        if bc == 3:
            assert layout == 0
        keys.add((H, W, bc, kind, grad, agg, out, layout))
    assert (480, 640, 2, 0, 1, 1, 0, 1) in keys          # headline, 2560-byte rows
    assert (375, 1242, 2, 3, 2, 1, 0, 0) in keys         # stereo, dense
    assert (375, 1242, 2, 3, 2, 1, 0, 1) in keys         # stereo, rows padded to 1280
    src = open(os.path.join(os.path.dirname(sne.LIB_PATH), "csrc", "sne_host.h")).read()
    assert "kTileCacheVersion = %d;" % sne.TILE_CACHE_VERSION in src


def test_frames_past_the_32bit_offset_limits_are_rejected():
    """The kernels address a frame with 32-bit byte offsets: the input (with
    a row of margin above and below) must stay below 2^31 bytes, each output
    plane and the mask below 4 GiB.  Larger frames return
    SNE_ERR_UNSUPPORTED before anything is launched (fake pointers here)."""
    L = sne.lib()
    K = _K()

    def est(H, W, in_pitch, kind, out, out_pitch, mask_pitch):
        return L.sne_estimate(None, FAKE, H, W, in_pitch, ctypes.byref(K), kind, 1, 1, out, FAKE,
                              out_pitch, FAKE, mask_pitch, None)

    W = 32760
    assert (16386 + 2) * W * 4 < 2 ** 31 - 1 < (16387 + 2) * W * 4
    assert est(16387, W, W, 0, 0, W, W) == -2          # FP32 input one row too tall
    assert est(2 * 16387 + 1, W, W, 1, 1, W, W) == -2  # u16 input: twice the rows + 1
    assert est(1024, 1000, 1000, 0, 0, 1 << 20, 1000) == -2   # output plane = 4 GiB
    assert est(1024, 1000, 1000, 0, 0, 1000, 1 << 22) == -2   # mask = 4 GiB


def test_c_client_builds(tmp_path):
    """The C ABI client compiles against include/sne.h and links libsne and
    the oracle with a plain C++ compiler (it runs in the GPU tests)."""
    import shutil
    import sys
    sys.path.insert(0, os.path.dirname(os.path.abspath(__file__)))
    import c_client_build
    if shutil.which("g++") is None:
        pytest.skip("no g++")
    import oracle
    oracle.build(force=False)
    assert os.path.exists(c_client_build.build())


def test_header_compiles_as_c99(tmp_path):
    """include/sne.h is a C header: plain C99 with -Wall -Wextra -pedantic."""
    import shutil
    import subprocess
    gcc = shutil.which("gcc")
    if gcc is None:
        pytest.skip("no gcc")
    src = tmp_path / "t.c"
    src.write_text('#include "sne.h"\nint main(void) { return sne_version() > 0 ? 0 : 1; }\n')
    inc = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "include")
    r = subprocess.run([gcc, "-std=c99", "-Wall", "-Wextra", "-pedantic", "-Werror",
                        "-fsyntax-only", "-I" + inc, str(src)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr


def test_binding_rejects_host_tensors():
    """A host tensor's pointer handed to a kernel would fault the GPU: the
    binding refuses host tensors before calling the library."""
    import torch
    raw = torch.ones((8, 8))
    with pytest.raises(ValueError, match="on the GPU"):
        sne.estimate(raw, (8.0, 8.0, 3.5, 3.5), "depth_f32")
    with pytest.raises(ValueError, match="on the GPU"):
        sne.estimate_uniform(raw[None], (8.0, 8.0, 3.5, 3.5), "depth_f32")


@pytest.mark.parametrize("mode,n,src,dst,mask", [
    (9, 16, FAKE, FAKE, FAKE), (-1, 16, FAKE, FAKE, FAKE), (2, 6, FAKE, FAKE, FAKE),
    (2, -4, FAKE, FAKE, FAKE), (2, 16, None, FAKE, None), (1, 16, None, None, None),
    (2, 16, FAKE + 4, FAKE, None), (3, 16, FAKE, FAKE, None), (3, 16, FAKE, FAKE, FAKE + 1),
])
def test_bandwidth_probe_argument_errors(mode, n, src, dst, mask):
    assert sne.lib().sne_bandwidth_probe(mode, src, dst, mask, n, None) == sne.SNE_ERR_ARG


def test_lenient_kind_suffix():
    assert sne._kind("depth_u16+lenient") == 1 | sne.SNE_LENIENT
    assert sne._kind("disparity_f32") == 3
    with pytest.raises(ValueError):
        sne._kind("depth_u16+loose")


def test_rgbn_argument_errors():
    L = sne.lib()
    K = _K()
    good = dict(ctx=None, inp=FAKE, B=1, H=8, W=8, in_pitch=8, in_fs=0, K=ctypes.byref(K), kind=0,
                grad=0, agg=0, rgb=None, rgb_pitch=0, rgb_fs=0, out=FAKE, out_pitch=8, out_fs=0,
                mask=None, mask_pitch=0, mask_fs=0, stream=None)
    for bad in [dict(out=FAKE + 8), dict(rgb=FAKE, rgb_pitch=16), dict(rgb=FAKE, rgb_pitch=34),
                dict(rgb=FAKE + 2, rgb_pitch=32), dict(out_pitch=4), dict(kind=9), dict(inp=None),
                dict(B=2, out_fs=63)]:
        a = dict(good, **bad)
        assert L.sne_estimate_rgbn(*a.values()) == sne.SNE_ERR_ARG, bad


@pytest.mark.parametrize("B,H,W", [(1, 101, 103), (1, 240, 320), (1, 375, 1242), (1, 427, 561),
                                   (1, 480, 640), (1, 720, 1280), (4, 480, 640), (8, 480, 640),
                                   (1, 1080, 1920)])
@pytest.mark.parametrize("kind", ["depth_f32", "depth_u16", "disparity_f32", "depth_f32+lenient"])
def test_default_tile_spreads_small_launches(B, H, W, kind):
    """A launch that does not fill the GPU (256 CUs, 4 SIMDs each) takes as long
    as one of its wavefronts, which walks its rows one after the other: without
    a tuned entry it makes at least one wavefront per SIMD, or one per 64
    pixels of a row where the image has no more."""
    t = sne.Tile()
    assert sne.lib().sne_get_tile(None, H, W, B, sne._kind(kind), sne.GRAD["fd"],
                                  sne.AGG["mean"], sne.OUT["f32"], ctypes.byref(t)) == 0
    strips = -(-W // (t.lanes * t.cols_per_lane))
    bands = -(-H // t.rows)
    waves = B * strips * (-(-bands // 2) if t.lanes == 32 else bands)
    assert waves >= min(1024, B * H * -(-W // 64)), (t.cols_per_lane, t.rows, t.lanes, waves)


def test_tile_cache_version_is_newer_than_the_narrow_kernels():
    """Tables saved when rows of odd width or alignment took one or two columns
    per lane, and lenient ones four, carry version 10200; their entries would
    override shapes that are faster now."""
    assert sne.TILE_CACHE_VERSION > 10200
