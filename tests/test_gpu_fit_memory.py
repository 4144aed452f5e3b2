"""A batch fit of very many starts gives its states back when it returns.

20000 states are 0.57 GB.  The batched pass's own workspaces, which a context keeps,
exist before the fit; half of the states' size is left for what the runtime holds on to.
"""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


def test_states_of_a_large_fit_are_freed():
    import torch

    from paper_1108_5882_amd import Context
    g = np.random.default_rng(6)
    k, nv = 4, 20_000
    with Context(0, "f32") as c:
        c.set_amplitudes("data", synth.random_amplitudes(g, 1000, k))
        c.set_amplitudes("mc", synth.random_amplitudes(g, 2000, k))
        V0 = synth.draw_v(g, nv, k)
        c.nll_batch(V0, split=3)
        small = c.batch_fit(V0[:50], 3)
        torch.cuda.synchronize()
        before = torch.cuda.mem_get_info()[0]
        large = c.batch_fit(V0, 3)
        torch.cuda.synchronize()
        assert before - torch.cuda.mem_get_info()[0] < nv * 28_600 / 2
        # the states kept for small fits are made again
        again = c.batch_fit(V0[:50], 3)
        assert np.array_equal(small[0], again[0]) and np.array_equal(small[1], again[1])
        assert np.isfinite(large[1]).all()
