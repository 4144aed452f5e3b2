"""One-launch inference against the layer-by-layer kernels, bit for bit.

Both round the same operands to FP16 and add the same terms in the same order, so
the outputs have to be equal.  The layer-by-layer form runs at more than 64 inputs:
the same network with zero columns appended to W1 and to the rows adds exact zeros.
Input widths sit at the edges of the 32-wide steps and of the 16-byte row loads,
row counts at those of the 16-row tiles and of the grid, and one case reads rows
that are only 4-byte aligned.
"""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_in,n,shift", [(1, 17, 0), (2, 1, 0), (7, 1000, 0), (8, 15, 0), (30, 33, 0), (32, 16, 0),
                                          (32, 70_001, 0), (32, 4097, 1), (33, 513, 0), (48, 257, 0), (63, 99, 1),
                                          (64, 9000, 0)])
def test_equal_to_the_layer_by_layer_form(n_in, n, shift):
    import torch
    import paper_1108_5882_amd as pwa
    print(f"case predict in={n_in} n={n} shift={shift}", flush=True)
    hidden, wide = 256, 72
    P = synth.mlp_init(n_in, hidden, seed=n)
    g = np.random.default_rng([n_in, n])
    X = g.normal(size=(n, n_in)).astype(np.float32)
    X[0, 0] = np.inf if n % 2 else 1e5          # past FP16's range either way
    Pw = np.concatenate([np.pad(P[:hidden * n_in].reshape(hidden, n_in), ((0, 0), (0, wide - n_in))).ravel(),
                         P[hidden * n_in:]])
    Xw = np.pad(X, ((0, 0), (0, wide - n_in)))
    flat = torch.zeros(n * n_in + shift, dtype=torch.float32, device="cuda")
    flat[shift:] = torch.from_numpy(X.ravel()).cuda()
    with pwa.Mlp(n_in, hidden, max_batch=64) as m, pwa.Mlp(wide, hidden, max_batch=4096) as layers:
        m.set_params(P)
        layers.set_params(Pw)
        y = m.predict(flat[shift:].view(n, n_in)).cpu().numpy()
        ref = layers.predict(torch.from_numpy(Xw).cuda()).cpu().numpy()
    assert np.array_equal(y, ref, equal_nan=True)
