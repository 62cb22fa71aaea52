"""GPU parity of the row-streaming kernels' column layout (marked gpu; run on
an MI355X): crop widths around a lane's columns, whole-line stores and their
remainders, walks of many rows over many images, every output type and layout.

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
