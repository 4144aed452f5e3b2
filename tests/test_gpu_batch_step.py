"""The launch between two passes of a batch of fits: sums, L-BFGS update and the
weights of the next trial point.

A fit's NLL is the split-3 value at its point, evaluated with the weights that the
update left; pwa_nll_batch at the returned point lays out its weights in a kernel
of its own.  Both carry out the same operations, so the values are equal to the last
bit.  Sizes at the edges of the weight layout: waves per k-step (16, 32, 48) and
vectors per column group and per vector group (16, 32).
"""

import numpy as np
import pytest

from paper_1108_5882_amd import Context

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("gram", [False, True])
@pytest.mark.parametrize("k,nv", [(1, 1), (2, 33), (15, 16), (16, 17), (17, 31), (32, 65), (33, 15), (47, 17), (48, 257)])
def test_fit_value_is_the_batch_value_at_its_point(k, nv, gram):
    rng = np.random.default_rng(100 * k + nv)

    def rows(n):
        return (rng.normal(size=(n, k)) + 1j * rng.normal(size=(n, k))).astype(np.complex64)

    ctx = Context(0, "f32")
    ctx.set_amplitudes("data", rows(1500))
    ctx.set_amplitudes("mc", rows(4100), w=rng.uniform(0.5, 1.5, 4100).astype(np.float32))
    ctx.set_mc_mode("gram" if gram else "stream")
    V0 = rng.normal(size=(nv, k)) + 1j * rng.normal(size=(nv, k))
    V0 *= 10.0 ** rng.uniform(-3, 3, size=(nv, 1))
    for iters in (1, 2, 5):
        V, nll, _, _ = ctx.batch_fit(V0, iters)
        assert np.isfinite(nll).all()
        again = ctx.nll_batch(V, grad=False, split=3)
        assert np.array_equal(again[0] if isinstance(again, tuple) else again, nll)
    ctx.close()
