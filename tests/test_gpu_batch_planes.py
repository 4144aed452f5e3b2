"""Operand planes of the batched pass at the edges of its tiles: 32 events, 16 and 32
real columns, rows and columns past the sample.

Reference: 64-bit numpy.  Bound of an event's share: operands of 22 bits and FP32
accumulation put 2^-20 sum_a |V_a A_a| on its coherent sum z (events whose |z| is
below |V| |A| / 8 are formed exactly), the two-term BF16 adjoint 2^-15 on its part of
the gradient, an FP32 logarithm 2^-20 on ln I.  A value out of its place is an error of
the size of the terms.
"""

import numpy as np
import pytest

from paper_1108_5882_amd import Context

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k", [1, 2, 7, 8, 9, 15, 16, 17, 31, 32, 33, 47, 48, 49, 63, 64])
@pytest.mark.parametrize("nd,nm", [(1, 1), (31, 33), (32, 64), (65, 4097)])
def test_batched_sums_at_the_edges(k, nd, nm):
    rng = np.random.default_rng(1000 * k + nd)
    scale = 10.0 ** rng.uniform(-2, 2, k)          # a scale of its own per wave

    def rows(n):
        return ((rng.normal(size=(n, k)) + 1j * rng.normal(size=(n, k))) * scale).astype(np.complex64)

    A, B = rows(nd), rows(nm)
    w = rng.uniform(0.5, 1.5, nm).astype(np.float32)
    V = (rng.normal(size=(5, k)) + 1j * rng.normal(size=(5, k))) / scale
    ctx = Context(0, "f32")
    ctx.set_amplitudes("data", A)
    ctx.set_amplitudes("mc", B, w=w)
    nll, grad = ctx.nll_batch(V, split=3)
    ctx.close()
    D, M, u20, u15 = A.astype(np.complex128), B.astype(np.complex128), 2.0 ** -20, 2.0 ** -15
    for b in range(V.shape[0]):
        z, y = D @ V[b], M @ V[b]
        ez, ey = u20 * (np.abs(D) @ np.abs(V[b])), u20 * (np.abs(M) @ np.abs(V[b]))
        I, S = np.abs(z) ** 2, np.sum(w * np.abs(y) ** 2)
        dS = np.sum(w * 2 * np.abs(y) * ey) / S + u20
        # an exact event's bound is no larger than one at |z| = |V| |A| / 8
        zc = np.maximum(np.abs(z), np.linalg.norm(V[b]) * np.linalg.norm(D, axis=1) / 8)
        ref = -np.sum(np.log(I)) + nd * np.log(S / nm)
        assert abs(nll[b] - ref) <= np.sum(2 * ez / zc + u20 * (1 + np.abs(np.log(I)))) + 2 * nd * dS
        G, H = np.conj(D) * (z / I)[:, None], np.conj(M) * (w * y)[:, None]
        c = nd / S
        g = 2 * (-G.sum(0) + c * H.sum(0))
        tol = 2 * (np.sum(np.abs(D) * (2 * ez / zc ** 2 + u15 / np.abs(z))[:, None], 0)
                   + c * np.sum(np.abs(M) * (w * (2 * ey + u15 * np.abs(y)))[:, None], 0)
                   + 2 * c * dS * np.abs(H).sum(0))
        got = np.asarray(grad[b])
        got = got if np.iscomplexobj(got) else got[0::2] + 1j * got[1::2]
        assert (np.abs(got.real - g.real) <= tol).all() and (np.abs(got.imag - g.imag) <= tol).all()
