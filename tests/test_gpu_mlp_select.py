"""The k smallest keys at the edges of the merging form: lists of 256 (k up to 256)
and 512 (k up to 512) numbers, 4096 keys per block, 64 lists per block of a later
round, and the sorting form above; ties, signed zeros, infinities and NaN."""
import numpy as np
import pytest

import oracle.mlp as OM

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,k", [(1, 1), (255, 255), (256, 256), (257, 1), (4096, 256), (4097, 256), (5000, 257),
                                 (8191, 512), (262_144, 512), (266_241, 200), (600_001, 256), (4500, 513),
                                 (70_000, 2048)])
@pytest.mark.parametrize("kind", ["spread", "ties", "special", "descending"])
def test_select_equals_the_oracle(n, k, kind):
    import torch
    import paper_1108_5882_amd as pwa
    print(f"case select n={n} k={k} {kind}", flush=True)
    g = np.random.default_rng([n, k])
    keys = g.normal(size=n).astype(np.float32)
    if kind == "ties":
        keys = g.integers(-2, 3, n).astype(np.float32) * np.float32(0.5)
        keys[g.random(n) < 0.3] = -0.0
    elif kind == "special":
        keys[g.random(n) < 0.5] = np.nan
        keys[g.random(n) < 0.3] = np.inf
        keys[g.random(n) < 0.1] = -np.inf
        keys[g.random(n) < 0.1] = 1e-42
    elif kind == "descending":
        keys = np.sort(keys)[::-1].copy()
    with pwa.Mlp(4, 8, max_batch=4) as m:
        idx = m.select(torch.from_numpy(keys).cuda(), k).cpu().numpy()
    assert np.array_equal(idx, OM.topk(keys, k))


@pytest.mark.parametrize("k,n", [(1, 33), (5, 1), (16, 64), (64, 31), (64, 1000)])
def test_features_rows_at_block_edges(k, n):
    """Blocks of 32 rows; a zero vector and a zero first wave among them."""
    import torch
    import paper_1108_5882_amd as pwa
    print(f"case features k={k} n={n}", flush=True)
    g = np.random.default_rng([k, n])
    V = g.normal(size=(n, k)) + 1j * g.normal(size=(n, k))
    V[n // 2] = 0.0
    V[-1, 0] = 0.0
    flat = np.empty((n, 2 * k))
    flat[:, 0::2], flat[:, 1::2] = V.real, V.imag
    with pwa.Mlp(2 * k, 8, max_batch=4) as m:
        X = m.features(torch.from_numpy(flat).cuda()).cpu().numpy()
    # FP64 up to the last rounding to FP32 (2^-24 of at most 1, plus 1e-15)
    assert np.max(np.abs(X - OM.features(V))) <= 2.0 ** -24 + 1e-15
