"""A sample is replaced while another stream captures, in this thread or another.

The replacement is no part of that capture: it succeeds, the capture ends well and
replays, and the context gives the bits of a fresh one.
"""
import threading

import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("source", ["host", "device"])
@pytest.mark.parametrize("mode,own_thread", [("relaxed", True), ("relaxed", False), ("thread_local", False)])
def test_replacement_beside_a_capture(mode, own_thread, source):
    import torch

    from paper_1108_5882_amd import Context
    print(f"case replacement beside a capture {mode} own_thread={own_thread} {source}", flush=True)
    g = np.random.default_rng(8)
    k = 5
    Ad, Am, Bd = (synth.random_amplitudes(g, n, k) for n in (2000, 6000, 1900))
    V = synth.draw_v(g, 1, k)[0]
    new = torch.from_numpy(Bd).cuda() if source == "device" else Bd
    x = torch.zeros(1000, device="cuda")
    side, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    begun, replaced, failed = threading.Event(), threading.Event(), []

    def capture(middle):
        try:
            with torch.cuda.stream(side):
                graph.capture_begin(capture_error_mode=mode)
                try:
                    x.add_(1.0)
                    middle()
                finally:
                    graph.capture_end()
        except Exception as e:      # noqa: BLE001 - reported by the test's thread
            failed.append(e)
            begun.set()

    with Context(0, "f32") as c, Context(0, "f32") as fresh:
        c.set_amplitudes("data", Ad)
        c.set_amplitudes("mc", Am)
        c.nll_grad(V)
        torch.cuda.synchronize()
        if own_thread:
            capture(lambda: c.set_amplitudes("data", new))
        else:
            t = threading.Thread(target=capture, args=(lambda: (begun.set(), replaced.wait(20)),))
            t.start()
            begun.wait(20)
            try:
                c.set_amplitudes("data", new)
            finally:
                replaced.set()
                t.join()
        assert not failed, failed
        graph.replay()
        torch.cuda.synchronize()
        assert float(x.min()) == float(x.max()) == 1.0
        fresh.set_amplitudes("data", Bd)
        fresh.set_amplitudes("mc", Am)
        a, b = c.nll_grad(V), fresh.nll_grad(V)
        assert a[0] == b[0] and np.array_equal(a[1], b[1])
