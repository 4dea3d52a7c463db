"""The blend adjoint of strokes far thinner than a pixel: Gaussians that reach
no pixel centre (1 / sigma^3 and log2(e) / (2 sigma^2) above the FP32 range) and
ones that reach exactly one, at a small fraction of their sigma."""
from __future__ import annotations

import numpy as np
import pytest

from helpers import PARAM_NAMES, gpu_run, gpu_vs_oracle
from paper_2606_31764_amd import synth
from paper_2606_31764_amd.render import Params

pytestmark = pytest.mark.gpu


def _line(p0, p1, width, scene_hw=(15, 21), opacity=0.6):
    part = dict(scene=0, degree=1, flags=0, key_xy=np.array([p0, p1], np.float64), key_w=np.ones(2),
                key_s=np.full(2, width), tau=[1.0], color=[0.2, 0.5, 0.9], opacity=opacity)
    return synth._assemble([part], [list(scene_hw)], [[1.0, 1.0, 1.0]], 3)


@pytest.mark.parametrize("tile", [8, 16, 32])
@pytest.mark.parametrize("width", [1e-5, 1e-12, 1e-14, 1e-20, 1e-30])
def test_reaching_no_pixel(width, tile):
    """The image is the background and every gradient is exactly 0."""
    b = _line([3.25, 4.2], [9.75, 8.3], width)   # off the pixel centres (x + 1/2, y + 1/2)
    up = np.random.default_rng(3).normal(size=3 * 15 * 21)
    out = gpu_run(b, Params(delta_c=3.0, tile=tile), upstream=up)
    assert len(out["idx"]) > 0
    assert (out["image"] == 1.0).all()
    for n in PARAM_NAMES:
        assert (out["grads"][n] == 0.0).all(), n


@pytest.mark.parametrize("tile", [8, 16, 32])
@pytest.mark.parametrize("width", [1e-5, 3e-5, 1e-4, 1e-3, 1e-2, 0.1, 0.2, 0.5])
def test_reaching_one_pixel(width, tile):
    """A line along a row of pixel centres at a fifth of its sigma from them,
    17 samples at a spacing of 1: up to a width of 0.2 each reaches one pixel."""
    d = 0.1 * width
    y = float(np.float32(2.5 + d))
    b = _line([1.5, y], [17.5, y], width, opacity=0.3)
    target = np.random.default_rng(4).uniform(0.0, 1.0, 3 * 15 * 21)
    gpu_vs_oracle(b, Params(delta_c=1.05, tile=tile, kappa=0), target)


@pytest.mark.parametrize("tile", [8, 16, 32])
@pytest.mark.parametrize("width", [1e-8, 1e-7, 1e-6, 1e-3])
def test_along_the_first_row_of_pixel_centres(width, tile):
    """Offsets from 0 to 6e-8 px, exact in tile-local FP32 there: far below the
    rounding of a sum over the block's pixels."""
    y1 = float(np.nextafter(np.float32(0.5), np.float32(1.0)))
    b = _line([1.5, 0.5], [17.5, y1], width, opacity=0.3)
    target = np.random.default_rng(5).uniform(0.0, 1.0, 3 * 15 * 21)
    gpu_vs_oracle(b, Params(delta_c=1.05, tile=tile, kappa=0), target)
