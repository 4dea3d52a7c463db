"""A launch whose thread count, bounded from the pair capacity, passes 2^32."""
from __future__ import annotations

import numpy as np
import pytest

from helpers import grad_close, gpu_run
from paper_2606_31764_amd import synth
from paper_2606_31764_amd.render import Params

pytestmark = pytest.mark.gpu
PAIRS_MAX = 0x7fffffff


@pytest.mark.parametrize("tile", [16, 32])
def test_largest_pair_capacity(tile):
    """The largest capacity that is taken (about 110 GB of workspace), on a
    small scene: the same image as with a small one, and gradients up to the
    order of the atomics."""
    import torch
    if torch.cuda.mem_get_info()[0] < 160e9:
        pytest.skip("needs 160 GB of free device memory")
    b = synth.config2(seed=5, n_curves=6, size=96)
    up = np.random.default_rng(2).normal(size=3 * 96 * 96)
    p = Params(delta_c=3.0, tile=tile, chunk=512)
    small = gpu_run(b, p, upstream=up)
    large = gpu_run(b, p, upstream=up, caps=dict(gauss=4 * len(small["gauss"]["sigma"]), pairs=PAIRS_MAX, boundary=16))
    np.testing.assert_array_equal(large["image"], small["image"])
    assert grad_close(large["grads"], small["grads"], rtol=1e-5, atol=1e-6) <= 1.0
    del large
    torch.cuda.empty_cache()
