"""Leaves without an index cache: trees of up to 6 internal nodes take them
from a table by their decisions, larger ones from the decision masks.  Trees of
exactly 0 to 9 nodes, bushy, left-most or right-most (whose nodes reach the
last heap slots of D = 8), in lockstep with the oracle."""
from __future__ import annotations

import numpy as np
import pytest

from paper_2410_23244_amd.inputs import make_inputs
from tests import parity

pytestmark = pytest.mark.gpu


def _grow(inp, nodes, shape, rng):
    """One tree: at most `nodes` internal nodes, each with cuts left."""
    H = 1 << (inp.D - 1)
    axis, cut = np.zeros(H, np.uint16), np.zeros(H, np.uint8)
    open_ = [(1, np.zeros(inp.p, np.int64), inp.n_cuts.astype(np.int64))]
    while nodes and open_:
        k = dict(left=0, right=-1).get(shape, int(rng.integers(len(open_))))
        h, lo, hi = open_.pop(k)
        ok = np.flatnonzero(hi > lo)
        if h >= H or not ok.size:
            continue
        a = int(rng.choice(ok))
        c = int(rng.integers(lo[a] + 1, hi[a] + 1))
        axis[h], cut[h], nodes = a, c, nodes - 1
        hl, lr = hi.copy(), lo.copy()
        hl[a], lr[a] = c - 1, c
        kids = [(2 * h, lo, hl), (2 * h + 1, lr, hi)]
        open_ = kids + open_ if shape == "left" else open_ + kids
    return axis, cut


def _state(inp, shape, rng):
    m, H, n = inp.m, 1 << (inp.D - 1), inp.n
    axis, cut = np.zeros((m, H), np.uint16), np.zeros((m, H), np.uint8)
    leaf = rng.normal(0.0, inp.hyper.sigma_mu, (m, 2 * H)).astype(np.float32)
    idx, f = np.zeros((m, n), np.uint8), np.zeros(n)
    for j in range(m):
        axis[j], cut[j] = _grow(inp, j % 10, shape, rng)
        h = np.ones(n, np.int64)
        for _ in range(inp.D - 1):
            hh = np.minimum(h, H - 1)
            inner = (h < H) & (cut[j, hh] != 0)
            right = inp.X_b[axis[j, hh], np.arange(n)] >= cut[j, hh]
            h = np.where(inner, 2 * h + right, h)
        live = np.zeros(2 * H, bool)
        live[1] = True
        for q in range(1, H):
            if live[q] and cut[j, q]:
                live[q], live[2 * q], live[2 * q + 1] = False, True, True
        leaf[j, ~live] = 0.0
        idx[j] = h
        f += leaf[j, h].astype(np.float64)
    resid = (inp.y_c.astype(np.float64) - f).astype(np.float32)
    return dict(axis=axis, cut=cut, leaf=leaf, idx=idx, resid=resid,
                sigma2=inp.hyper.sigma2_init, sweep=0, next=0)


@pytest.mark.parametrize("shape", ["bushy", "left", "right"])
@pytest.mark.parametrize("D", [3, 6, 8])
def test_trees_of_exactly_k_nodes(D, shape):
    from paper_2410_23244_amd.bart import from_inputs

    inp = make_inputs(2, n=9001, p=14, m=20, D=D, idx_bytes=0)
    g = from_inputs(inp, grid=2)
    print(f"D={D} {shape}", flush=True)
    g.set_state(_state(inp, shape, np.random.default_rng(4)))
    rep = parity.lockstep(inp, g, seed=9, warm_sweeps=0, n_steps=3 * (inp.m + 1))
    assert rep.moves > 0 and g.status() == 0
