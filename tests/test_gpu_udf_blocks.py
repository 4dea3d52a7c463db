"""The distance-weighted loss by 8 x 8 pixel blocks: odd scene sizes, more
scenes than lanes, curves outside the canvas, a radius smaller and larger than
the scenes, against the oracle."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
from helpers import oracle_params
from paper_2606_31764_amd import synth
from paper_2606_31764_amd.render import Params, Renderer, param_tensors

pytestmark = pytest.mark.gpu


def _scene(seed, H, W, n):
    ps = synth.fills(seed, n_paths=n, size=max(H, W), radius=(2.0, 14.0))
    ps += synth.strokes(seed + 1, n_curves=1, size=max(H, W), nk_range=(5, 5), margin=0.0)
    return synth._assemble(ps, [[H, W]], [[1.0, 1.0, 1.0]], 3)


@pytest.mark.parametrize("tau", [0.6, 7.5, 200.0])
@pytest.mark.parametrize("sizes", [[(3, 2)], [(17, 9), (8, 8), (7, 65), (33, 40)], [(9 + k % 5, 8 + k % 7) for k in range(70)]])
def test_blocks_match_oracle(sizes, tau):
    import torch
    b = synth.concat([_scene(300 + 2 * k, H, W, 3) for k, (H, W) in enumerate(sizes)])
    p = Params(delta_c=2.0, h=2.0)
    r = Renderer(b, p)
    t = param_tensors(b)
    img = r.run_forward(t).clone()
    tgt = torch.as_tensor(np.random.default_rng(5).uniform(0, 1, img.numel()).astype(np.float32), device="cuda")
    loss = torch.zeros(1, device="cuda")
    # the weights depend on no tile side: not on the binning's either
    dL = r.udf_loss(t, img, tgt, tau=tau, loss=loss, params=p.replace(tile=32))
    op = oracle_params(p)
    plan, _, _ = oracle.plan(b, op)
    v, dref, _ = oracle.udf_loss(b, plan, img.cpu().numpy(), tgt.cpu().numpy(), tau, params=op)
    got = dL.cpu().numpy().astype(np.float64)
    # FP32 weights and gradients: a few roundings of the largest
    assert np.abs(got - dref).max() <= 1e-5 * np.abs(dref).max() + 1e-12
    assert abs(float(loss.item()) - v) <= 1e-5 * abs(v) + 1e-9
