"""The forward of long lists (a block per quadrant, an eighth of each 512
positions per wavefront): list lengths around the first long length, a window
and a chunk, with pixels that stop and with opacities below zero, against the
oracle; and against the wavefront-per-quadrant form, which a given chunk
length selects."""
from __future__ import annotations

import numpy as np
import pytest

from helpers import EPS32, IMG_TOL, gpu_run, gpu_vs_oracle, grad_check, oracle_params, oracle_reference
from paper_2606_31764_amd import synth
from paper_2606_31764_amd.render import Params

pytestmark = pytest.mark.gpu


def _scene(count, opacity, seed, flags=0, C=3):
    """A stroke per opacity through one 8 x 8 block and beyond it."""
    rng = np.random.default_rng(seed)
    parts = []
    for o in opacity:
        xy = np.stack([rng.uniform(1.0, 10.0, 4), rng.uniform(1.0, 10.0, 4)], 1)
        parts.append(dict(scene=0, degree=3, flags=flags, key_xy=xy, key_w=np.ones(4), key_s=rng.uniform(1.0, 3.0, 4),
                          tau=[1.0], color=rng.uniform(0, 1, C), opacity=o))
    return synth._assemble(parts, [[15, 13]], [[1.0] * C], C)


def _params(b, count, tile, **kw):
    """Sampled densely enough for lists of roughly count positions."""
    length = sum(float(np.hypot(*np.diff(b.key_xy[4 * c:4 * c + 4], axis=0).T).sum()) for c in range(b.n_curves))
    return Params(delta_c=1.8 * count / length, kappa=0, tile=tile, **kw)


@pytest.mark.parametrize("tile", [8, 16])
@pytest.mark.parametrize("count", [110, 150, 500, 560, 1000, 1700])
@pytest.mark.parametrize("opacity", [(0.002, 0.004, 0.003), (0.02, 0.5, 0.1), (0.9, 0.9, 0.9), (0.05, -0.002, 0.03)])
def test_against_oracle(opacity, count, tile):
    b = _scene(count, opacity, seed=count + tile)
    p = _params(b, count, tile)
    target = np.random.default_rng(count).uniform(0.0, 1.0, 3 * 15 * 13)
    if min(opacity) >= 0:
        gpu_vs_oracle(b, p, target)
        return
    # the oracle's error scale sums |dL/dT| alpha T, which is signed where alpha
    # is: its magnitude
    img, up, ref, scale = oracle_reference(b, target, oracle_params(p))
    out = gpu_run(b, p, upstream=up)
    assert np.abs(out["image"] - img).max() <= IMG_TOL
    worst, rep = grad_check(out["grads"], ref, {n: np.abs(x) for n, x in scale.items()})
    assert worst <= 1.0, rep


@pytest.mark.parametrize("persistent", [False, True])
@pytest.mark.parametrize("C,flags", [(1, 0), (3, 0), (3, synth.ANISO)])
@pytest.mark.parametrize("count", [180, 512, 2500])
def test_against_one_wavefront(count, C, flags, persistent):
    """The same list in both forms: T is a product of at most n factors in
    another order (n relative roundings of 2^-24 on either side), and the
    colour a sum of alpha T of at most 1; where a pixel stops one entry
    earlier or later, eps_T more."""
    # (tangent-aligned strokes have two or three Gaussians each here)
    opacity = (0.02, 0.3, 0.6) if flags == 0 else (0.005, 0.02, 0.1) * (count // 6)
    b = _scene(count, opacity, seed=7 * count, flags=flags, C=C)
    up = np.random.default_rng(5).normal(size=C * 15 * 13)
    p = _params(b, count, 16)
    a = gpu_run(b, p, upstream=up, persistent=persistent)
    c = gpu_run(b, p.replace(chunk=512), upstream=up, persistent=persistent)
    n = int((a["ranges"][:, 1] - a["ranges"][:, 0]).max())
    assert n >= 128  # a long list
    np.testing.assert_array_equal(a["idx"], c["idx"])
    other = a["n_last"] != c["n_last"]
    assert other.sum() <= 2
    tol = 2 * n * EPS32 + np.where(np.tile(np.ravel(other), C), p.eps_T, 0.0)
    assert (np.abs(np.ravel(a["image"]) - np.ravel(c["image"])) <= tol).all()


@pytest.mark.parametrize("delta_c", [4.0, 12.0, 44.0])
@pytest.mark.parametrize("tile", [8, 16])
def test_chosen_chunk_against_a_given_one(tile, delta_c):
    """Left to choose, a launch of this size takes chunks of 128, 256 or 512
    positions, and the same lists give the same gradients up to the order of
    the sums (as batched against plain)."""
    from helpers import PARAM_NAMES, grad_close
    b = synth.config2(seed=31, n_curves=24, size=160)
    p = Params(delta_c=delta_c, tile=tile)
    up = np.random.default_rng(6).normal(size=3 * 160 * 160)
    a = gpu_run(b, p, upstream=up)
    c = gpu_run(b, p.replace(chunk=512), upstream=up)
    print("pairs", len(a["idx"]), flush=True)
    np.testing.assert_array_equal(a["idx"], c["idx"])
    n = int((c["ranges"][:, 1] - c["ranges"][:, 0]).max())
    assert (np.abs(np.ravel(a["image"]) - np.ravel(c["image"])) <= 2 * n * EPS32 + p.eps_T).all()
    assert all(np.isfinite(a["grads"][n]).all() for n in PARAM_NAMES)
    assert grad_close(a["grads"], c["grads"], rtol=1e-4, atol=1e-6) <= 1.0
