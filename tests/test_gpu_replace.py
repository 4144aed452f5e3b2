"""Samples replaced in a context give the bits of a fresh context.

The memory of a sample is kept for the one that replaces it when it fits, so the
sizes here grow, shrink a little (kept), shrink a lot (not kept), change k with
its row padding, and lose and regain the weights; host and device sources, and a
borrowed sample in between.
"""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

STEPS = [  # (k, MC rows, weighted, source)
    (5, 3000, True, "host"), (5, 2900, False, "device"), (5, 2999, True, "device"), (5, 9001, True, "host"),
    (5, 700, True, "host"), (11, 700, False, "device"), (11, 690, True, "borrow"), (11, 700, True, "device"),
    (5, 1400, False, "host"), (5, 1300, False, "device")]


@pytest.mark.parametrize("prec", ["f32", "f64"])
def test_replaced_samples_equal_a_fresh_context(prec):
    import torch
    from paper_1108_5882_amd import Context
    dtype = np.complex64 if prec == "f32" else np.complex128
    g = np.random.default_rng(5)
    with Context(0, prec) as kept:
        for k, n, weighted, source in STEPS:
            print(f"case replace prec={prec} k={k} n={n} weighted={weighted} {source}", flush=True)
            Ad, Am = synth.random_amplitudes(g, n // 3, k, dtype), synth.random_amplitudes(g, n, k, dtype)
            w = g.uniform(0.5, 2.0, n).astype(Am.real.dtype) if weighted else None
            V = synth.draw_v(g, 1, k)[0]
            got = []
            for ctx in (kept, Context(0, prec)):
                if source == "host":
                    ctx.set_amplitudes("data", Ad)
                    ctx.set_amplitudes("mc", Am, w=w, n_gen=2.0 * n)
                else:
                    ld = ctx.layout_ld(k) if source == "borrow" else k
                    pad = np.zeros((n, ld), dtype=dtype)
                    pad[:, :k] = Am
                    dev = torch.from_numpy(pad).cuda()
                    wd = None if w is None else torch.from_numpy(w).cuda()
                    torch.cuda.synchronize()
                    ctx.set_amplitudes("data", Ad)
                    ctx.set_amplitudes("mc", dev, w=wd, n_gen=2.0 * n, borrow=source == "borrow", k=k)
                for mode in ("stream", "gram"):
                    ctx.set_mc_mode(mode)
                    nll, grad = ctx.nll_grad(V)
                    got.append(np.append(grad, nll))
                if ctx is not kept:
                    ctx.close()
            assert np.array_equal(got[0], got[2]) and np.array_equal(got[1], got[3])
