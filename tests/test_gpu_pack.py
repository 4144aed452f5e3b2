"""Device samples that need re-striding: the same bits as from host memory.

Host samples are packed on the host; device samples of other strides are packed
by a kernel (layouts of an even number of 8-byte units) or a pitched copy.  The
cases: every kind of padding (none, one column, several), sources with a row
stride of their own (even and odd), one row, row counts around a block's share,
and a source at an odd multiple of 8 bytes.
"""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("k,ld,first,n", [(1, 2, 0, 700), (3, 3, 0, 901), (3, 5, 1, 900), (5, 5, 0, 1365),
                                          (5, 9, 3, 1366), (7, 7, 0, 1), (13, 14, 1, 513), (16, 17, 0, 2048),
                                          (37, 37, 0, 171), (37, 41, 4, 5000), (49, 64, 15, 129)])
def test_device_rows_of_any_stride(prec, k, ld, first, n):
    import torch
    from paper_1108_5882_amd import Context
    print(f"case pack prec={prec} k={k} ld={ld} first={first} n={n}", flush=True)
    dtype = np.complex64 if prec == "f32" else np.complex128
    g = np.random.default_rng([k, ld, n])
    wide = synth.random_amplitudes(g, n, ld, dtype)
    V = synth.draw_v(g, 1, k)[0]
    host = np.ascontiguousarray(wide[:, first:first + k])
    dev = torch.from_numpy(wide).cuda()[:, first:first + k]
    torch.cuda.synchronize()
    got = []
    for A in (host, dev):
        with Context(0, prec) as ctx:
            ctx.set_amplitudes("data", A)
            ctx.set_amplitudes("mc", A, n_gen=3.0 * n)
            nll, grad = ctx.nll_grad(V)
            got.append(np.append(grad, nll))
    assert np.array_equal(got[0], got[1])
