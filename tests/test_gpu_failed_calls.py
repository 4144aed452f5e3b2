"""A synchronous call that refuses V leaves nothing of it on the stream.

The MC matrix of 4x10^5 borrowed rows at K = 48 takes some 0.3 ms to build.  A call that
started the build before it looked at V would return while the build still reads the
caller's array.
"""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

CALLS = {"nll": lambda c, v: c.nll(v), "nll_grad": lambda c, v: c.nll_grad(v), "hessian": lambda c, v: c.hessian(v),
         "batch0": lambda c, v: c.nll_batch(v[None], split=0), "batch3": lambda c, v: c.nll_batch(v[None], split=3),
         "batch_fit": lambda c, v: c.batch_fit(v[None], 1)}


@pytest.mark.parametrize("call", sorted(CALLS))
def test_a_refused_vector_starts_nothing(call):
    import torch

    from paper_1108_5882_amd import Context, PwaError
    k, n = 48, 400_000
    g = torch.Generator(device="cuda")
    g.manual_seed(2)
    mc = torch.view_as_complex(torch.randn((n, k, 2), generator=g, device="cuda"))
    data = mc[:500].clone()
    v = synth.draw_v(np.random.default_rng(2), 1, k)[0]
    bad = v.copy()
    bad[k - 1] = complex(np.nan, 0.0)
    st = torch.cuda.Stream()
    torch.cuda.synchronize()
    with Context(0, "f32", stream=st) as c:
        c.set_mc_mode("gram")
        c.set_amplitudes("data", data, borrow=True)
        c.set_amplitudes("mc", mc, borrow=True)
        for _ in range(2):
            with pytest.raises(PwaError) as e:
                CALLS[call](c, bad)
            assert e.value.status == 1 and st.query()
        c.nll(v)
