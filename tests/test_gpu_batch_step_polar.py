"""The launch between two passes of a batch of fits in polar parameters.

Sizes at the edges of the weight layout, as in the Cartesian form: waves per k-step
(16, 32, 48; each k-step count is a kernel of its own) and vectors per column group and
per vector group (16, 32).  A fit's NLL is the split-3 value at its point, so it meets
the oracle there within 1e-6 of the terms' size, and so does the value after three
evaluations along the reference L-BFGS in the same parameters: its steps move V by a
hundredth at first, which takes the gradient's 1e-6 down with it.
"""
import math

import numpy as np
import pytest

import oracle
import synth
from oracle.lbfgs import LbfgsOracle
from tests.tolerance import TOL, errors, reference

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k,nv", [(1, 3), (2, 33), (15, 16), (16, 17), (17, 31), (32, 65), (33, 15), (47, 17), (48, 40)])
def test_polar_fit_value_and_steps(k, nv):
    from paper_1108_5882_amd import Context
    print(f"case polar k={k} nv={nv}", flush=True)
    g = np.random.default_rng(10 * k + nv)
    Ad, Am = synth.random_amplitudes(g, 1500, k), synth.random_amplitudes(g, 4100, k)
    w = g.uniform(0.5, 1.5, 4100).astype(np.float32)
    V0 = synth.draw_v(g, nv, k)
    rmin = 0.5 * float(np.min(np.abs(V0)))
    with Context(0, "f32") as c:
        c.set_amplitudes("data", Ad)
        c.set_amplitudes("mc", Am, w=w)
        first = c.batch_fit(V0, 1, polar=True, rmin=rmin)
        third = c.batch_fit(V0, 3, polar=True, rmin=rmin)
        later = c.batch_fit(V0, 12, polar=True, rmin=rmin)
    phase = np.exp(-1j * np.angle(V0[:, :1]))
    assert np.allclose(first[0], V0 * phase, rtol=1e-14, atol=0)
    for V, nll, _, _ in (first, third, later):
        assert np.all(V[:, 0].imag == 0.0) and np.all(np.abs(V) >= rmin * (1 - 1e-15 * 4))
        for b in (0, nv // 2, nv - 1):
            ref = reference(Ad, Am, V[b], w=w)
            assert errors(ref, nll[b], ref["grad"])[0] < TOL["f32"], (k, b)
    assert np.all(later[1] <= first[1])
    for b in (0, nv - 1):
        v0 = V0[b] * phase[b]
        p0 = np.empty(2 * k)
        p0[0::2], p0[1::2] = np.abs(v0), [0.0] + [math.atan2(z.imag, z.real) for z in v0[1:]]
        ref = LbfgsOracle(lambda x: oracle.nll_grad(Ad, Am, x[0::2] + 1j * x[1::2], w=w), p0, polar=True, rmin=rmin)
        for _ in range(3):
            ref.step()
        Vr = ref.x[0::2] * np.exp(1j * ref.x[1::2])
        assert abs(third[1][b] - ref.f) < TOL["f32"] * reference(Ad, Am, Vr, w=w)["s_nll"]
