"""Proposals where axes have different numbers of cuts (cut counts and axis
ranks from tables, some axes without a cut) and where all have the same (no
tables), in lockstep with the oracle, over launches of one sweep and of
several (a launch makes its first sweep's proposals itself and leaves none
behind)."""
from __future__ import annotations

import numpy as np
import pytest

from paper_2410_23244_amd.inputs import make_inputs
from tests import parity

pytestmark = pytest.mark.gpu


def _inputs(kind, D):
    inp = make_inputs(2, n=6007, p=9, m=23, D=D)
    K = dict(mixed=np.array([255, 3, 0, 17, 1, 255, 0, 2, 90]), few=np.full(9, 2),
             one=np.array([0, 0, 0, 0, 5, 0, 0, 0, 0]), all=np.full(9, 255))[kind]
    inp.n_cuts[:] = K
    inp.X_b[:] = np.minimum(inp.X_b, K[:, None]).astype(np.uint8)
    return inp


@pytest.mark.parametrize("residency", [1, 2])
@pytest.mark.parametrize("D", [6, 8])
@pytest.mark.parametrize("kind", ["mixed", "few", "one", "all"])
def test_cut_counts(kind, D, residency):
    from paper_2410_23244_amd.bart import from_inputs

    inp = _inputs(kind, D)
    a = from_inputs(inp, residency=residency, grid=3)
    print(f"{kind} D={D} residency={residency}", flush=True)
    rep = parity.lockstep(inp, a, seed=3, warm_sweeps=3, n_steps=2 * (inp.m + 1))
    assert rep.moves > 0
    # five launches of one sweep, against one of five
    b, c = (from_inputs(inp, residency=residency, grid=3) for _ in range(2))
    b.step(5, 8)
    for _ in range(5):
        c.step(1, 8)
    sb, sc = b.get_state(), c.get_state()
    for k in ["axis", "cut", "leaf", "idx", "resid"]:
        np.testing.assert_array_equal(sb[k], sc[k], err_msg=k)
    assert sb["sigma2"] == sc["sigma2"] and b.status() == 0 and c.status() == 0
