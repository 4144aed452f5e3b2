"""Calls that build a context's inputs refuse a capturing stream.

A build that is only recorded into a graph has not run, so it must not count as
done: after the refusal the same call, made outside the capture, gives the bits of a
fresh context.  The MC sample is replaced first, so that a matrix, planes or row
norms left from the earlier one would show.
"""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

CALLS = {
    "nll": lambda c, V: c.nll(V[0]),
    "nll_grad": lambda c, V: np.append(*c.nll_grad(V[0])),
    "hessian": lambda c, V: c.hessian(V[0]),
    "batch2": lambda c, V: np.column_stack(c.nll_batch(V, split=2)),
    "batch3": lambda c, V: np.column_stack(c.nll_batch(V, split=3)),
    "batch_fit": lambda c, V: np.column_stack(c.batch_fit(V, 3)[:2]),
}


@pytest.mark.parametrize("mode", ["stream", "gram"])
@pytest.mark.parametrize("call", sorted(CALLS))
def test_inputs_are_not_built_into_a_graph(call, mode):
    import torch

    from paper_1108_5882_amd import Context, PwaError
    if mode == "stream" and call in ("nll", "nll_grad"):
        pytest.skip("builds nothing")
    g = np.random.default_rng(3)
    k, n = 8, 2000
    Ad, Am, Bm = (synth.random_amplitudes(g, m, k, np.complex64) for m in (n, 3 * n, 3 * n))
    V = synth.draw_v(g, 5, k)
    st = torch.cuda.Stream()
    with Context(0, "f32", stream=st) as c, Context(0, "f32") as fresh:
        c.set_mc_mode(mode)
        fresh.set_mc_mode(mode)
        c.set_amplitudes("data", Ad)
        c.set_amplitudes("mc", Am)
        CALLS[call](c, V)                       # every workspace has its size
        c.set_amplitudes("mc", Bm)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.stream(st):
            graph.capture_begin(capture_error_mode="relaxed")
            try:
                with pytest.raises(PwaError):
                    CALLS[call](c, V)
            finally:
                graph.capture_end()             # the refusal leaves the capture whole
        st.synchronize()
        fresh.set_amplitudes("data", Ad)
        fresh.set_amplitudes("mc", Bm)
        assert np.array_equal(CALLS[call](c, V), CALLS[call](fresh, V))
