"""The MC matrix of Eq. 3 against its definition in 64-bit numpy.

With no data rows the Eq. 3 form is NLL = V^H M V with gradient 2 M V, so unit
vectors V give M column by column.  Sizes sit at the edges of the build: tile
shapes (K up to 8, up to 20, above), odd K, one and several waves per chunk, and row
counts at the remainders of a stage (16 rows), a chunk and the grid.

Tolerance: every entry is a sum of at most 2 n products, each rounded a few
times, added in some order: (2 n + 8) 2^-53 sum_j |w_j| |A_ja| |A_jb| bounds it.
"""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


def _matrix(ctx, k):
    M = np.empty((k, k), dtype=np.complex128)
    for b in range(k):
        v = np.zeros(k, dtype=np.complex128)
        v[b] = 1.0
        nll, g = ctx.nll_grad(v)
        M[:, b] = 0.5 * (g[0::2] + 1j * g[1::2])
        assert nll == M[b, b].real
    return M


@pytest.mark.parametrize("prec,k,n,weighted", [
    ("f32", 1, 1, False), ("f32", 3, 5, True), ("f32", 8, 31, False), ("f32", 8, 4097, True),
    ("f32", 9, 63, True), ("f32", 16, 1024, False), ("f32", 17, 65, True), ("f32", 20, 64, False), ("f32", 21, 130, True), ("f32", 24, 40_001, True),
    ("f32", 25, 17, False), ("f32", 32, 1003, True), ("f32", 33, 70_000, False), ("f32", 40, 3, True),
    ("f32", 48, 2_050, True), ("f32", 49, 515, False), ("f32", 56, 129, True), ("f32", 64, 9_999, False),
    ("f64", 4, 16_001, True), ("f64", 13, 66, False), ("f64", 24, 2, True), ("f64", 37, 4_099, True),
    ("f64", 48, 777, False), ("f64", 64, 1_030, True)])
def test_matrix_against_its_definition(prec, k, n, weighted):
    from paper_1108_5882_amd import Context
    print(f"case gram matrix prec={prec} k={k} n={n} weighted={weighted}", flush=True)
    g = np.random.default_rng([k, n])
    dtype = np.complex64 if prec == "f32" else np.complex128
    A = synth.random_amplitudes(g, n, k, dtype)
    w = g.uniform(-0.5, 2.0, n).astype(A.real.dtype) if weighted else None
    with Context(0, prec) as ctx:
        ctx.set_amplitudes("data", np.empty((0, k), dtype=dtype))
        ctx.set_amplitudes("mc", A, w=w, n_gen=1.5 * n)
        ctx.set_mc_mode("gram", extended=True)
        M = _matrix(ctx, k)
    Ad = A.astype(np.complex128)
    wd = np.ones(n) if w is None else w.astype(np.float64)
    ref = (Ad.conj().T * wd) @ Ad / (1.5 * n)
    scale = (np.abs(Ad).T * np.abs(wd)) @ np.abs(Ad) / (1.5 * n)
    assert np.all(np.abs(M - ref) <= 2.0 * (2 * n + 8) * 2.0 ** -53 * scale)
    if prec == "f32":
        assert np.array_equal(M, M.conj().T)


@pytest.mark.parametrize("k,n", [(4, 5_000), (13, 1_030), (24, 2_049), (37, 63)])
def test_sums_keep_their_order(k, n):
    """Chunks of consecutive rows summed in row order, chunks in order: bit for bit.

    Products of FP32 values are exact in FP64 and unit weights leave no other
    rounding than the sums themselves, so numpy repeats them exactly.
    """
    from paper_1108_5882_amd import Context
    print(f"case gram order k={k} n={n}", flush=True)
    A = synth.random_amplitudes(np.random.default_rng([k, n, 1]), n, k)
    with Context(0, "f32") as ctx:
        ctx.set_amplitudes("data", np.empty((0, k), dtype=np.complex64))
        ctx.set_amplitudes("mc", A, n_gen=float(n))
        ctx.set_mc_mode("gram", extended=True)
        M = _matrix(ctx, k)
    blocks = (n + 63) // 64                     # fewer than two per compute unit at these sizes
    chunk = (n + blocks - 1) // blocks
    re, im = A.real.astype(np.float64), A.imag.astype(np.float64)
    total = np.zeros((2, k, k))
    for r0 in range(0, n, chunk):
        part = np.zeros((2, k, k))
        for r in range(r0, min(r0 + chunk, n)):
            part[0] += np.outer(re[r], re[r]) + np.outer(im[r], im[r])
            part[1] += np.outer(re[r], im[r]) - np.outer(im[r], re[r])
        total += part
    total *= 1.0 / n
    # the evaluation forms 2 (1 M_ab + 0 M_ac + ...) per entry, exact; the matrix halves it
    assert np.array_equal(M.real, total[0]) and np.array_equal(M.imag, total[1])

