"""GPU parity of the row-streaming kernels' column layout (marked gpu; run on
an MI355X): crop widths around a lane's columns, whole-line stores and their
remainders, walks of many rows over many images, column strips of wide crops
and of long source spans, RGB and I420, every output type and layout.

Exact arithmetic is selected, so every output equals the oracle's bit for bit.
"""
from __future__ import annotations

import numpy as np
import pytest

from paper_2007_13005_amd import smol, synthetic
from tests.gpu_util import run_gpu, run_oracle

pytestmark = pytest.mark.gpu

F32, F16, U8 = synthetic.OUT_F32, synthetic.OUT_F16, synthetic.OUT_U8
NCHW, NHWC = smol.LAYOUT_NCHW, smol.LAYOUT_NHWC


@pytest.fixture(autouse=True)
def _reset_tuning():
    smol.reset_tuning()
    yield
    smol.reset_tuning()


def _exact(wl, **tuning):
    smol.set_tuning(exact=1, **tuning)
    got, ref = run_gpu(wl), run_oracle(wl)
    bits = {F32: np.uint32, F16: np.uint16, U8: np.uint8}[wl.out_dtype]
    np.testing.assert_array_equal(got.view(bits), ref.view(bits))
    return smol.last_plan()


def _direct(wl, layout):
    wl.resize_mode, wl.layout = smol.RESIZE_DIRECT, layout
    return wl


def _rgb(sizes, crop, dtype, layout, seed=3):
    rng = np.random.default_rng(seed)
    imgs = [rng.integers(0, 256, size=(h, w, 3), dtype=np.uint8) for w, h in sizes]
    # a pad image keeps the last one's 16-byte chunks inside src
    wl = synthetic.rgb_workload("columns", imgs, 1, crop, dtype)
    wl.src = np.concatenate([wl.src, rng.integers(0, 256, 64, dtype=np.uint8)])
    return _direct(wl, layout)


def _yuv(sizes, crop, dtype, layout, siting, seed=4):
    rng = np.random.default_rng(seed)
    planes = [tuple(rng.integers(0, 256, size=s, dtype=np.uint8)
                    for s in ((h, w), ((h + 1) // 2, (w + 1) // 2), ((h + 1) // 2, (w + 1) // 2)))
              for w, h in sizes]
    wl = synthetic.yuv420_workload("columns", planes, 1, crop, dtype)
    wl.src = np.concatenate([wl.src, rng.integers(0, 256, 64, dtype=np.uint8)])
    wl.siting = siting
    return _direct(wl, layout)


WIDTHS = [1, 2, 3, 4, 5, 63, 64, 72, 112, 127, 128, 129, 130, 131, 136, 223, 224, 255, 256]


@pytest.mark.parametrize("width", WIDTHS)
@pytest.mark.parametrize("layout", [NCHW, NHWC])
@pytest.mark.parametrize("dtype", [F32, F16, U8])
def test_crop_widths(width, layout, dtype):
    """64 rows: an fp16 plane is whole 128-byte lines at every even width."""
    sizes = [(300, 90), (301, 200), (64, 33)]
    assert _exact(_rgb(sizes, (64, width), dtype, layout))["path"] == smol.PATH_ROWS


@pytest.mark.parametrize("crop", [(64, 72), (64, 224), (130, 72), (3, 128), (1, 96), (37, 224)])
@pytest.mark.parametrize("dtype", [F32, F16])
def test_long_walks(crop, dtype):
    """256 waves, each walking many rows (past 64, the rows prepared at once)
    over several images of different sizes."""
    n = 20000 // crop[0] if crop[1] < 200 else 3000 // crop[0]
    sizes = [(40, 30), (41, 30), (90, 64), (23, 90)]
    wl = _rgb([sizes[i % 4 if i % 7 else 0] for i in range(n)], crop, dtype, NCHW)
    assert _exact(wl, workgroups_per_cu=1)["path"] == smol.PATH_ROWS


@pytest.mark.parametrize("width", [257, 300, 352, 384, 385, 513, 600, 640, 701, 704, 833])
@pytest.mark.parametrize("layout", [NCHW, NHWC])
@pytest.mark.parametrize("dtype", [F32, F16, U8])
def test_wide_crops(width, layout, dtype):
    sizes = [(700, 50), (333, 70)]
    plan = _exact(_rgb(sizes, (48, width), dtype, layout))
    assert plan["path"] == smol.PATH_ROWS


@pytest.mark.parametrize("order", [1, 2])
@pytest.mark.parametrize("width,crop_w", [(3840, 224), (3001, 160), (5800, 224), (5000, 640)])
def test_long_spans(width, crop_w, order):
    """Source spans past 4 KiB, in both row orders."""
    wl = _rgb([(width, 60)] * 3, (40, crop_w), F16, NCHW)
    assert _exact(wl, row_order=order)["path"] == smol.PATH_ROWS


@pytest.mark.parametrize("siting", [smol.CHROMA_CENTER, smol.CHROMA_LEFT])
@pytest.mark.parametrize("width,crop_w", [(300, 1), (300, 131), (2100, 224), (3840, 224),
                                          (700, 257), (1500, 640), (4097, 301)])
@pytest.mark.parametrize("dtype,layout", [(F32, NCHW), (F16, NCHW), (F16, NHWC)])
def test_yuv_columns(width, crop_w, siting, dtype, layout):
    """I420 crops and luma spans of one or more strips, a ragged batch."""
    wl = _yuv([(width, 50), (width - 3, 41)], (40, crop_w), dtype, layout, siting)
    assert _exact(wl)["path"] == smol.PATH_ROWS


def test_yuv_uniform_strips():
    """A uniform batch: the waves of a workgroup share their strip's column
    table."""
    wl = _yuv([(2600, 60)] * 6, (64, 250), F16, NCHW, smol.CHROMA_LEFT)
    assert _exact(wl)["path"] == smol.PATH_ROWS


def _pick(sizes, n):
    return [sizes[i % len(sizes) if i % 7 else 0] for i in range(n)]


@pytest.mark.parametrize("siting", [smol.CHROMA_CENTER, smol.CHROMA_LEFT])
@pytest.mark.parametrize("layout", [NCHW, NHWC])
@pytest.mark.parametrize("crop,sizes", [((64, 72), [(40, 30), (41, 30), (90, 65), (23, 91)]),
                                        ((3, 131), [(300, 9), (301, 8), (299, 20)]),
                                        ((40, 224), [(2101, 20), (2100, 21)])],
                         ids=["many-rows", "many-images", "strips"])
def test_yuv_long_walks(crop, sizes, layout, siting):
    """256 waves, each walking many rows (past 64, the rows prepared at once)
    over several frames of different sizes."""
    wl = _yuv(_pick(sizes, 17000 // crop[0]), crop, F16, layout, siting)
    plan = _exact(wl, workgroups_per_cu=1)
    assert plan["path"] == smol.PATH_ROWS and plan["work_items"] > 64 * plan["grid"]


@pytest.mark.parametrize("siting", [smol.CHROMA_CENTER, smol.CHROMA_LEFT])
@pytest.mark.parametrize("crop", [(16, 72), (16, 200)])
def test_yuv_equal_rois_walk(crop, siting):
    """Regions of one size at any place of frames of two widths, many rows per
    wave: the chroma columns a luma column reads depend on the region's place
    in its frame and on the frame's width, not on the region's size alone."""
    rng = np.random.default_rng(8)
    n = 400
    sizes = [(97, 40) if i % 3 else (64, 40) for i in range(n)]
    wl = _yuv(sizes, crop, F32, NCHW, siting)
    x = [int(rng.integers(0, w - 33 + 1)) if i % 5 else w - 33 for i, (w, _) in enumerate(sizes)]
    wl.rois = np.array([(x[i], int(rng.integers(0, 20)), 33, 20) for i in range(n)], np.int32)
    plan = _exact(wl, workgroups_per_cu=1)
    assert plan["path"] == smol.PATH_ROWS and plan["work_items"] > 8 * plan["grid"]


@pytest.mark.parametrize("dtype", [F32, F16])
@pytest.mark.parametrize("layout", [NCHW, NHWC])
@pytest.mark.parametrize("kind,width,crop_w", [("rgb", 700, 600), ("rgb", 300, 513),
                                               ("rgb", 3840, 224), ("rgb", 1300, 1024),
                                               ("yuv", 700, 600), ("yuv", 2600, 224)])
def test_past_the_row_limits_exact_by_default(kind, width, crop_w, layout, dtype):
    """Crops past 512 columns and spans past one staged row are the oracle's
    bit for bit without the exact knob, on whichever kernel they run."""
    sizes, crop = [(width, 40), (width - 1, 33)], (48, crop_w)
    wl = (_rgb(sizes, crop, dtype, layout) if kind == "rgb" else
          _yuv(sizes, crop, dtype, layout, smol.CHROMA_CENTER))
    bits = {F32: np.uint32, F16: np.uint16}[dtype]
    np.testing.assert_array_equal(run_gpu(wl).view(bits), run_oracle(wl).view(bits))


@pytest.mark.parametrize("crop_w,path", [(100, smol.PATH_GATHER), (112, smol.PATH_GATHER),
                                         (128, smol.PATH_GATHER), (160, smol.PATH_ROWS),
                                         (224, smol.PATH_ROWS)])
def test_no_strip_below_the_narrowest(crop_w, path):
    """Spans of 3840 columns need three strips or more: fewer than 48 columns
    each below a crop of 144."""
    assert _exact(_rgb([(3840, 24)] * 2, (8, crop_w), F16, NCHW))["path"] == path


@pytest.mark.parametrize("wide,path", [(1, smol.PATH_GATHER), (3, smol.PATH_GATHER),
                                       (4, smol.PATH_ROWS), (7, smol.PATH_ROWS)])
def test_few_long_spans(wide, path):
    """Images of long spans among images that fit their crop's own strips: strips
    for all only where at least half of them need it."""
    wl = _rgb([(3000, 20)] * wide + [(400, 30)] * (8 - wide), (16, 224), F16, NCHW)
    assert _exact(wl)["path"] == path


@pytest.mark.parametrize("width", [1, 3, 128, 130, 131, 224, 256])
@pytest.mark.parametrize("layout", [NCHW, NHWC])
@pytest.mark.parametrize("dtype", [F32, F16, U8])
def test_long_rows_in_ranges(width, layout, dtype):
    """Ragged batches of long staged rows (past 2 KiB), one row and many per
    wave: pairs of columns per lane instead of four side by side."""
    sizes = [(1300, 40), (1299, 33), (900, 70)]
    wl = _rgb(sizes, (64, width), dtype, layout)
    assert _exact(wl)["path"] == smol.PATH_ROWS
    assert _exact(_rgb(sizes * 30, (64, width), dtype, layout), workgroups_per_cu=1)["grid"] == 256


@pytest.mark.parametrize("crop_w,strips", [(300, 2), (384, 2), (448, 2), (512, 2), (600, 3),
                                           (640, 5), (768, 3), (896, 7), (1024, 4)])
def test_rgb_strip_counts(crop_w, strips):
    """RGB crops run in the fewest strips of up to 256 columns, or in strips of
    128 where only those are whole fp16 lines."""
    wl = _rgb([(640, 40), (633, 41)], (16, crop_w), F16, NCHW)
    assert _exact(wl)["work_items"] == 2 * 16 * strips


# Crops past one strip of 256 columns: one strip of four column pairs per lane
# for uniform batches and uint8 output of long rows, interleaved float rows and
# float I420.
@pytest.mark.parametrize("crop_w", [257, 258, 300, 385, 511, 512])
@pytest.mark.parametrize("kind,dtype,layout,strips", [
    ("long", F32, NCHW, 1), ("long", F16, NCHW, 1), ("long", F32, NHWC, 1), ("long", F16, NHWC, 1),
    ("long", U8, NCHW, 1), ("ragged", U8, NCHW, 1), ("ragged", U8, NHWC, 1),
    ("short", U8, NHWC, 2), ("ragged", F16, NCHW, 2), ("ragged", F32, NHWC, 2),
    ("short", F32, NHWC, 1), ("short", F32, NCHW, 2), ("short", F16, NHWC, 2),
    ("yuv", F32, NCHW, 1), ("yuv", F32, NHWC, 1), ("yuv", F16, NHWC, None)])
def test_wide_crops(kind, dtype, layout, strips, crop_w):
    sizes = {"long": [(1200, 30)] * 3, "ragged": [(1200, 30), (1100, 31), (1200, 29)],
             "short": [(600, 30), (601, 20)], "yuv": [(1280, 30), (1281, 31)]}[kind]
    wl = (_yuv(sizes, (24, crop_w), dtype, layout, smol.CHROMA_LEFT) if kind == "yuv" else
          _rgb(sizes, (24, crop_w), dtype, layout))
    plan = _exact(wl)
    assert plan["path"] == smol.PATH_ROWS
    if strips is not None:
        assert plan["work_items"] == len(sizes) * 24 * strips


@pytest.mark.parametrize("order", [1, 2])
@pytest.mark.parametrize("dtype,layout", [(F32, NCHW), (F16, NCHW), (F32, NHWC), (F16, NHWC)])
@pytest.mark.parametrize("width", [1200, 600])
def test_wide_crops_in_either_order(width, dtype, layout, order):
    """Either row walk of wide crops, uniform and ragged, with both prefetch depths."""
    for sizes in ([(width, 30)] * 3, [(width, 30), (width - 1, 31)]):
        for band in (0, 1, 2):
            _exact(_rgb(sizes, (24, 300), dtype, layout), row_order=order, band_rows=band)


# The default arithmetic: one unit in the last place of the result (fp32: the
# product with RN(1/std) against the quotient; fp16: one rounding instead of two).
@pytest.mark.parametrize("crop", [(64, 72), (64, 131), (64, 224), (64, 300), (40, 513), (24, 640)])
@pytest.mark.parametrize("layout", [NCHW, NHWC])
@pytest.mark.parametrize("dtype", [F32, F16, U8])
@pytest.mark.parametrize("kind", ["rgb", "long", "yuv"])
def test_default_arithmetic(kind, dtype, layout, crop):
    sizes = [(300, 90), (301, 200), (64, 33)] if kind != "long" else [(1300, 70), (1299, 64)]
    wl = (_yuv(sizes, crop, dtype, layout, smol.CHROMA_CENTER) if kind == "yuv" else
          _rgb(sizes, crop, dtype, layout))
    got, ref = run_gpu(wl), run_oracle(wl)
    if dtype == U8:
        np.testing.assert_array_equal(got, ref)
        return
    ulp = np.maximum(np.spacing(np.abs(ref)), np.spacing(np.abs(got))).astype(np.float64)
    assert (np.abs(got.astype(np.float64) - ref.astype(np.float64)) <= ulp).all()


@pytest.mark.parametrize("budget,lds", [(4096, 4096), (7167, 4096), (7168, 7168), (0, 7168)])
def test_line_rings_within_the_lds_budget(budget, lds):
    wl = _rgb([(500, 40), (501, 33)], (64, 224), F16, NCHW)
    assert _exact(wl, path=smol.PATH_ROWS, lds_budget=budget)["lds_bytes"] == lds
