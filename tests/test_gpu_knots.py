"""Knot vectors bit for bit against the running sum in FP64, for interval
counts around the block's shares and the LDS capacity, with intervals whose
sums are exact in FP64 (summed in parallel) and intervals whose sums are not,
and the Euler identity of the interval gradients of long curves."""
from __future__ import annotations

import numpy as np
import pytest

from paper_2606_31764_amd import synth
from paper_2606_31764_amd.render import Params, Renderer, param_tensors

pytestmark = pytest.mark.gpu
KNOT_PAD = 11


def _curve(nt, closed, p, wide, rng):
    nk = nt if closed else nt + p
    t = np.linspace(0.0, 2 * np.pi, nk, endpoint=False)
    xy = np.stack([16.0 + 9.0 * np.cos(t), 16.0 + 9.0 * np.sin(2 * t)], 1)
    tau = rng.uniform(0.5, 1.5, nt)
    if wide == "zeros":
        tau[rng.random(nt) < 0.3] = 0.0
        tau[0] = 1.0
    elif wide:
        tau *= 2.0 ** rng.integers(-40, 1, nt)
    return dict(scene=0, degree=p, flags=int(closed), key_xy=xy, key_w=np.ones(nk), key_s=np.full(nk, 1.5), tau=tau,
                color=[0.2, 0.4, 0.6], opacity=0.5)


def _knots(part):
    p, closed = part["degree"], part["flags"] & 1
    tau = np.asarray(part["tau"], np.float32).astype(np.float64)
    n = len(tau)
    iv = tau[(np.arange(n + 2 * p) - p) % n] if closed else np.concatenate([np.zeros(p), tau, np.zeros(p)])
    U = [0.0]
    for x in iv:
        U.append(U[-1] + x)
    return np.array(U)


@pytest.mark.parametrize("wide", [False, "zeros", True])
@pytest.mark.parametrize("closed", [False, True])
def test_knots_are_the_running_sum(closed, wide):
    rng = np.random.default_rng(7 + closed)
    parts = [_curve(nt, closed, p, wide, rng) for nt in (6, 63, 64, 65, 250, 1023, 1024, 1025, 2049, 4084, 4089, 4090, 4095,
                                                       4096, 9000) for p in (1, 3, 5)]
    b = synth._assemble(parts, [[32, 32]], [[1.0, 1.0, 1.0]], 3)
    r = Renderer(b, Params(delta_c=1.0))
    r.sample(param_tensors(b))
    off = r.ws_ptr - r.ws.data_ptr()
    n = int(b.tau_off[-1]) + KNOT_PAD * b.n_curves
    got = r.ws[off:off + 8 * n].cpu().numpy().view(np.float64)
    for c, part in enumerate(parts):
        want = _knots(part)
        o = int(b.tau_off[c]) + c * KNOT_PAD
        assert np.array_equal(got[o:o + len(want)], want), (c, part["degree"], len(part["tau"]))


@pytest.mark.parametrize("nt", [60, 130, 1023, 5000])
@pytest.mark.parametrize("closed", [False, True])
def test_interval_gradients_are_suffix_sums(nt, closed):
    """Euler identity of the interval gradients (the fold of the knot adjoints)."""
    import torch
    rng = np.random.default_rng(nt)
    part = _curve(nt, closed, 3, False, rng)
    b = synth._assemble([part], [[32, 32]], [[1.0, 1.0, 1.0]], 3)
    t = param_tensors(b)
    r = Renderer(b, Params(delta_c=2.0))
    img = r.run_forward(t)
    dL = torch.as_tensor(rng.normal(size=img.numel()).astype(np.float32), device="cuda")
    got = r.backward(t, dL)[3].cpu().numpy().astype(np.float64)
    # scaling every interval leaves the image unchanged: sum tau dL/dtau = 0, a
    # sum over the whole suffix chain, within the FP32 roundings of its terms
    tau = np.asarray(part["tau"], np.float32).astype(np.float64)
    assert np.abs(got).max() > 0.0
    assert abs((tau * got).sum()) <= 2e-4 * np.abs(tau * got).sum()
