"""The fused training pass at the edges of its pieces: one row, 16-row slices that
end inside and at a 32-row piece, weight-pass rounds of 1024 rows, and every padded
input width (32, 64, 96, 128), against the network oracle.

Median and 99th percentile of the scaled errors are held as in the other gradient
tests.  The largest error of a weight gradient is one or two FP16 rounding decisions
tipped the other way: each moves one operand of one row's term by at most one ulp,
2^-10 of the term, so an entry may be off by twice that of its largest term (in a
small batch one term can be a quarter of the sum) besides 2e-6 of the sum."""
import numpy as np
import pytest

import oracle.mlp as OM
import synth
from tests.test_gpu_mlp import _blocks, _scales

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,n_in", [(16, 32), (17, 64), (32, 2), (33, 96), (48, 128), (49, 34), (1025, 66),
                                    (1040, 32)])
def test_gradient_at_slice_and_piece_edges(B, n_in):
    import torch
    import paper_1108_5882_amd as pwa
    print(f"case slices B={B} in={n_in}", flush=True)
    hidden = 256
    P = synth.mlp_init(n_in, hidden, seed=B)
    g = np.random.default_rng([B, n_in])
    X = OM.features(synth.draw_v(g, B, n_in // 2)).astype(np.float32)
    t = g.uniform(0.0, 3.0, B).astype(np.float32)
    with pwa.Mlp(n_in, hidden, max_batch=2048) as m:
        m.set_params(P)
        loss, G = m.loss_grad(torch.from_numpy(X).cuda(), torch.from_numpy(t).cuda())
        G = G.cpu().numpy()
    a = OM.forward(P, X, n_in, hidden, rounding=True)
    l_or, G_or = OM.loss_grad(P, X, t, n_in, hidden, rounding=True)
    sy, S = _scales(P.astype(np.float64), X.astype(np.float64), t.astype(np.float64), n_in, hidden)
    assert abs(loss - l_or) <= 1e-4 * np.mean(2 * np.abs(a["y"] - t) * sy) + 1e-6 * l_or
    r = OM.f16
    dZ2 = np.outer(np.abs(2.0 * (a["y"] - t)), np.abs(r(OM.unpack(P, n_in, hidden)[4]))) * np.abs(OM.gelu_d(a["Z2"]))
    dZ1 = (dZ2 @ np.abs(r(OM.unpack(P, n_in, hidden)[2]))) * np.abs(OM.gelu_d(a["Z1"]))     # at least |dZ1|
    terms = {"W1": (dZ1, np.abs(X)), "W2": (dZ2, np.abs(a["H1"]))}
    for nm, sl in _blocks(n_in, hidden):
        err, scale = np.abs(G[sl] - G_or[sl]), S[sl] + 1e-30
        assert np.median(err / scale) < 2e-6 and np.percentile(err / scale, 99) < 5e-5, nm
        if nm in terms:
            left, right = terms[nm]
            largest = np.zeros((hidden, right.shape[1]))
            for b in range(B):
                np.maximum(largest, np.outer(left[b], right[b]), out=largest)
            assert np.all(err <= 2.0 * 2.0 ** -10 * largest.ravel() / B + 2e-6 * scale), nm
        else:
            assert np.max(err / scale) < 1e-4, nm


def test_two_adam_steps_of_a_ragged_batch():
    """Steps after the first use the refreshed FP16 weights and the corrections of their own step."""
    import torch
    import paper_1108_5882_amd as pwa
    n_in, hidden, B, lr = 40, 256, 77, 1e-3
    P = synth.mlp_init(n_in, hidden, seed=1)
    g = np.random.default_rng(4)
    X = OM.features(synth.draw_v(g, 200, n_in // 2)).astype(np.float32)
    t = g.uniform(0.0, 3.0, 200).astype(np.float32)
    perm = np.concatenate([g.permutation(200)[:B], g.permutation(200)[:B]]).astype(np.int32)
    with pwa.Mlp(n_in, hidden, max_batch=128) as m:
        m.set_params(P)
        m.train(torch.from_numpy(X).cuda(), torch.from_numpy(t).cuda(), torch.from_numpy(perm).cuda(), B, lr)
        got = m.get_params()
    ref, mo, ve = P.astype(np.float64), np.zeros(P.size), np.zeros(P.size)
    for s in range(2):
        rows = perm[s * B:(s + 1) * B]
        G = OM.loss_grad(ref, X[rows], t[rows], n_in, hidden, rounding=True)[1]
        ref, mo, ve = OM.adam(ref, G, mo, ve, s, lr)
    # an update is at most 2 lr per step; where a gradient is near zero Adam's ratio
    # amplifies its error, so the bound is on the bulk (lr times the gradient's 5e-5
    # 99th percentile, amplified a hundredfold) and on the mean
    d = np.abs(got - ref)
    assert np.percentile(d, 95) < lr * 5e-3 and d.mean() < lr * 5e-3 and d.max() <= 4 * lr
