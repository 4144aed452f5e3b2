"""The end of the streaming launch on either side of its limits: up to so many blocks
per sample the last block adds the partials itself, above it groups of blocks are
added first; few rows take fewer blocks.

Reference: the same sums in 64-bit numpy.  Gradient terms are formed and added in
FP64 (per lane, then compensated), so the error is a few roundings per addition of a
lane, far below 1e-12 of the sum of the terms' sizes; ln I is taken in FP32, 2^-22 of
the sum of |ln I| covers its error.
"""

import numpy as np
import pytest

from paper_1108_5882_amd import Context

pytestmark = pytest.mark.gpu


# rows per block are 4 U 64 / L; blocks added directly: 48 per sample at 16 waves, 32 at 24, 16 at 48
@pytest.mark.parametrize("k,cfg,nb_data,nb_mc", [
    (16, (8, 2, 4), 10, 48), (16, (8, 2, 4), 10, 49), (16, (8, 2, 4), 1, 1), (15, (8, 2, 2), 49, 12),
    (23, (8, 3, 2), 20, 32), (23, (8, 3, 2), 20, 33), (24, (8, 3, 1), 33, 1),
    (48, (16, 3, 2), 16, 16), (48, (16, 3, 2), 16, 17), (47, (16, 3, 1), 30, 34),
    # on either side of the most rows that keep to these blocks (112 KB each)
    (16, (8, 2, 4), 10, 336), (16, (8, 2, 4), 10, 338), (23, (8, 3, 2), 20, 298), (23, (8, 3, 2), 20, 300),
    (48, (16, 3, 2), 16, 149), (48, (16, 3, 2), 16, 151)])
@pytest.mark.parametrize("ragged", [0, 1])
def test_totals_across_the_limit(k, cfg, nb_data, nb_mc, ragged):
    L, C, U = cfg
    rows = 4 * U * 64 // L
    n = [b * rows - ragged * (rows // 2 + 1) for b in (nb_data, nb_mc)]
    rng = np.random.default_rng(k * 1000 + nb_mc + ragged)
    A = [(rng.normal(size=(m, k)) + 1j * rng.normal(size=(m, k))).astype(np.complex64) for m in n]
    w = rng.uniform(0.5, 1.5, n[1]).astype(np.float32)
    V = rng.normal(size=k) + 1j * rng.normal(size=k)
    ctx = Context(0, "f32")
    ctx.set_amplitudes("data", A[0])
    ctx.set_amplitudes("mc", A[1], w=w)
    ctx.set_stream_cfg(L, C, U, 4)
    nll, grad = ctx.nll_grad(V)
    again = ctx.nll_grad(V)
    ctx.close()
    assert again[0] == nll and np.array_equal(again[1], grad)

    D, M = A[0].astype(np.complex128), A[1].astype(np.complex128)
    z, y = D @ V, M @ V
    I, S = np.abs(z) ** 2, np.sum(w * np.abs(y) ** 2)
    ref = -np.sum(np.log(I)) + n[0] * np.log(S / n[1])
    assert abs(nll - ref) <= 2.0 ** -22 * np.sum(np.abs(np.log(I))) + 1e-12 * abs(ref)
    G, H = np.conj(D) * (z / I)[:, None], np.conj(M) * (w * y)[:, None]
    g = 2 * (-G.sum(0) + n[0] / S * H.sum(0))
    tol = 1e-12 * 2 * (np.abs(G).sum(0) + n[0] / S * np.abs(H).sum(0))
    got = np.asarray(grad)
    got = got if np.iscomplexobj(got) else got[0::2] + 1j * got[1::2]
    assert (np.abs(got.real - g.real) <= tol).all() and (np.abs(got.imag - g.imag) <= tol).all()
