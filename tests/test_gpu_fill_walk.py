"""The forward's walk of a fill run by row number (no chunk boundary in the run,
nothing that alpha_max could cut beside the pixel's own lattice point) and the
general one, on both sides of what selects them: opacities around alpha_max and
around where a neighbour at distance 1 reaches it (2.4), and chunks shorter and
longer than a run."""
from __future__ import annotations

import numpy as np
import pytest

from helpers import gpu_vs_oracle
from paper_2606_31764_amd import synth
from paper_2606_31764_amd.render import Params

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tile", [8, 16, 32])
@pytest.mark.parametrize("chunk", [512, 8192])
@pytest.mark.parametrize("opacity", [0.02, 0.97, 1.0, 2.3, 2.6, 40.0])
def test_fill_runs_against_oracle(opacity, chunk, tile):
    """Three overlapping filled curves whose windows end inside and outside the tiles."""
    rng = np.random.default_rng(int(100 * opacity) + tile)
    parts = []
    for k in range(3):
        a = 2 * np.pi * np.arange(7) / 7 + rng.uniform(0, 1)
        r = rng.uniform(6.0, 14.0, 7)
        xy = np.stack([18.0 + 5 * k + r * np.cos(a), 17.0 - 3 * k + r * np.sin(a)], 1)
        parts.append(dict(scene=0, degree=3, flags=3, key_xy=xy, key_w=np.ones(7), key_s=np.ones(7), tau=np.ones(7),
                          color=rng.uniform(0, 1, 3), opacity=opacity if k else 0.05))
    b = synth._assemble(parts, [[37, 43]], [[1.0, 1.0, 1.0]], 3)
    gpu_vs_oracle(b, Params(h=1.0, tile=tile, chunk=chunk), rng.uniform(0.0, 1.0, 3 * 37 * 43))
