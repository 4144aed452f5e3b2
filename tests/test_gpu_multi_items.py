"""Sums over a fit's work items, at the edges of what one round of loads takes.

Sixteen slices add the items of a sample, four items of a slice per round, two slices
per wave; the partials of up to 31 waves take one column per lane, wider ones two.  A
work item left out or added twice is an error of its share of the sums, against the
oracle's 1e-6.
"""
import numpy as np
import pytest

import synth
from tests.tolerance import TOL, errors, reference

pytestmark = pytest.mark.gpu

# rows per work item: whole tiles of a wave (rows x bytes per row) to 256 KB, a multiple of four
TILE = {4: 128, 6: 64, 8: 64, 12: 32, 16: 32, 24: 32, 32: 16, 48: 16}


def _item_rows(k):
    ld = min(w for w in TILE if w >= k)
    tiles = max(4, (256 << 10) // (TILE[ld] * 8 * ld))
    return TILE[ld] * ((tiles + 3) // 4 * 4)


@pytest.mark.parametrize("k", [4, 24, 25, 48])
@pytest.mark.parametrize("data,mc", [(0, 1), (1, 15), (2, 16), (15, 17), (16, 64), (17, 65), (33, 80)])
def test_every_item_is_added_once(k, data, mc):
    from paper_1108_5882_amd import MultiFit
    print(f"case items k={k} data={data} mc={mc}", flush=True)
    g = np.random.default_rng(100 * k + mc)
    per = _item_rows(k)
    nd, nm = max(0, data * per - 3), mc * per - 5
    Ad, Am = synth.random_amplitudes(g, nd, k), synth.random_amplitudes(g, nm, k)
    w = g.uniform(0.5, 1.5, nm).astype(np.float32)
    V = synth.draw_v(g, 1, k)[0]
    m = MultiFit([(Ad, Am, w, 2.0 * nm)], [V])
    nll, grad = m.eval([V])
    m.reset([V])
    m.step(1)
    stepped = m.get()[1]
    m.close()
    if nd == 0:
        assert nll[0] == 0.0 and not grad[0].any()
        return
    e_n, e_g = errors(reference(Ad, Am, V, w=w, n_gen=2.0 * nm), nll[0], grad[0])
    assert e_n < TOL["f32"] and e_g < TOL["f32"], (e_n, e_g)
    assert stepped[0] == nll[0]
