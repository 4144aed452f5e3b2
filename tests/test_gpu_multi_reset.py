"""Many fits are started when the call that starts them returns.

20000 fits without rows have 0.6 GB of states and 30 MB of start records in host
memory, so a start that were still under way would be seen on the caller's stream.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def test_the_stream_is_idle_after_a_start():
    import torch

    from paper_1108_5882_amd import MultiFit
    fits = 20_000
    none = np.zeros((0, 1), dtype=np.complex64)
    g = np.random.default_rng(4)
    V0, V1 = (g.normal(size=(fits, 1)) + 1j * g.normal(size=(fits, 1)) for _ in range(2))
    st = torch.cuda.Stream()
    m = MultiFit([(none, none, None, None)] * fits, list(V0), stream=st)
    assert st.query()
    assert np.array_equal(np.array(m.get()[0]), V0)
    m.reset(list(V1))
    assert st.query()
    V, nll, status, iters = m.get()
    assert np.array_equal(np.array(V), V1) and np.isnan(nll).all() and not status.any() and not iters.any()
    m.close()
