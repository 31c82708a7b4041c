"""The register kernel's exchange and decision at the edges of their branches,
in lockstep with the oracle: words per tree at and around the powers of two
that set the lanes per workgroup (7, 8, 15, 16, 31, 32, 63 and 64 leaves, one
and two more with the right-counts), 128 leaves (more words than a wave has
lanes), and numbers of workgroups around those that set the polling waves;
runs of steps that start inside a sweep (the first tree of a run makes its own
constants) and end right before and at its last trees; and cuts on both sides
of 128, where the byte compare of the route changes form."""
from __future__ import annotations

import numpy as np
import pytest

from paper_2410_23244_amd.inputs import make_inputs
from tests import parity

pytestmark = pytest.mark.gpu


def _state(inp, leaves, rng):
    """Trees of `leaves` leaves each (the leftmost growable node splits first),
    with random axes and cuts, as a state for set_state."""
    m, H, n = inp.m, 1 << (inp.D - 1), inp.n
    axis, cut = np.zeros((m, H), np.uint16), np.zeros((m, H), np.uint8)
    leaf, idx = np.zeros((m, 2 * H), np.float32), np.zeros((m, n), np.uint8)
    f = np.zeros(n)
    for j in range(m):
        for h in range(1, leaves):  # heap order: nodes 1..leaves-1 are internal
            axis[j, h] = rng.integers(inp.p)
            cut[j, h] = rng.integers(1, inp.n_cuts[axis[j, h]] + 1)
        leaf[j] = rng.normal(0.0, inp.hyper.sigma_mu, 2 * H)
        hh = np.ones(n, np.int64)
        for _ in range(inp.D - 1):
            inner = (hh < H) & (cut[j, np.minimum(hh, H - 1)] > 0)
            q = np.where(inner, hh, 0)
            right = inp.X_b[axis[j, q], np.arange(n)] >= cut[j, q]
            hh = np.where(inner, 2 * hh + right, hh)
        idx[j] = hh
        f += leaf[j, hh].astype(np.float64)
    resid = (inp.y_c.astype(np.float64) - f).astype(np.float32)
    return dict(axis=axis, cut=cut, leaf=leaf, idx=idx, resid=resid,
                sigma2=inp.hyper.sigma2_init, sweep=0, next=0)


def _run(inp, grid, leaves, steps):
    from paper_2410_23244_amd.bart import BART_RESID_REGISTERS, from_inputs

    g = from_inputs(inp, grid=grid, residency=BART_RESID_REGISTERS)
    print(f"leaves={leaves} grid={g.launch_info().grid} V={g.launch_info().chunks_per_thread}",
          flush=True)
    g.set_state(_state(inp, leaves, np.random.default_rng(leaves)))
    done = 0
    for k in steps:
        rep = parity.lockstep(inp, g, seed=11, warm_sweeps=0, n_steps=k)
        done += rep.moves
    assert done > 0 and g.status() == 0


@pytest.mark.parametrize("leaves", [1, 6, 7, 8, 14, 15, 16, 30, 31, 32, 62, 63, 64, 127, 128])
def test_words_per_tree(leaves):
    inp = make_inputs(5, n=9001, p=30, m=5, D=8)
    _run(inp, 5, leaves, [2 * (inp.m + 1)])


@pytest.mark.parametrize("grid", [1, 2, 3, 8, 9, 16, 17, 64, 65, 129, 256])
def test_workgroups(grid):
    inp = make_inputs(2, n=2003, p=30, m=7, D=6)
    for leaves in (4, 12, 24):
        _run(inp, grid, leaves, [2 * (inp.m + 1)])


@pytest.mark.parametrize("m", [1, 2, 3, 4, 5, 6])
def test_runs_that_start_and_end_inside_a_sweep(m):
    inp = make_inputs(2, n=5003, p=20, m=m, D=6)
    _run(inp, 4, 5, [1, 1, 2, 3, 1, 4, m + 1, 5])


@pytest.mark.parametrize("grid", [9, 17, 64, 245])
def test_sums_do_not_depend_on_where_a_launch_starts(grid):
    """A launch that starts inside a sweep adds every tree's partial sums in
    the order of one that runs through: the same bits, for trees whose words
    (with the first tree's extra one) lie on both sides of a layout's edge.
    The residuals differ by up to 2^40 from workgroup to workgroup, and the
    leaves stay too small to level them: partial sums of like size add up
    exactly in fp64, in any order."""
    from paper_2410_23244_amd.bart import BART_RESID_REGISTERS, from_inputs

    per = 2048  # observations of a workgroup
    inp = make_inputs(2, n=per * grid - 77, p=12, m=6, D=8)
    inp.hyper.sigma_mu = 1e-12
    one = from_inputs(inp, grid=grid, residency=BART_RESID_REGISTERS)
    two = from_inputs(inp, grid=grid, residency=BART_RESID_REGISTERS)
    for leaves in (6, 7, 8, 15, 31, 62, 63, 64, 100):
        rng = np.random.default_rng(leaves)
        st = _state(inp, leaves, rng)
        scale = 2.0 ** rng.integers(0, 41, grid)
        st["resid"] *= np.repeat(scale, per)[:inp.n].astype(np.float32)
        one.set_state(st)
        a = one.debug_steps(inp.m + 1, 5)
        want = one.get_state()
        for first in range(1, inp.m):
            print(f"grid={grid} leaves={leaves} first={first}", flush=True)
            two.set_state(st)
            b = np.concatenate([two.debug_steps(first, 5), two.debug_steps(inp.m + 1 - first, 5)])
            for f in ("sum", "log_r", "leaf_new", "ssr", "sigma2"):
                np.testing.assert_array_equal(b[f], a[f], err_msg=f)
            got = two.get_state()
            for k in ("leaf", "resid", "idx", "cut"):
                np.testing.assert_array_equal(got[k], want[k], err_msg=k)
    assert one.status() == 0 and two.status() == 0


@pytest.mark.parametrize("grid,V", [(3, 1), (1, 8)])
@pytest.mark.parametrize("slot", [0, 255])
def test_bad_entries_stay_out_of_the_sums(slot, grid, V):
    """An observation whose index entry is no leaf (0, or a slot outside its
    tree) is reported and takes no part in any leaf's sum: the other points'
    sums and leaves do not depend on its residual.  Trees of few leaves come
    before trees of as many as a bin pass holds."""
    from paper_2410_23244_amd.bart import BART_RESID_REGISTERS, from_inputs

    inp = make_inputs(2, n={1: 4999, 8: 16001}[V], p=30, m=6, D=8)
    runs = []
    for resid in (0.0, 1000.0):
        g = from_inputs(inp, grid=grid, residency=BART_RESID_REGISTERS)
        assert g.launch_info().chunks_per_thread == V
        parts = [_state(inp, k, np.random.default_rng(k)) for k in (4, 16, 32)]
        st = dict(parts[0])
        for k in ("axis", "cut", "leaf", "idx"):
            st[k] = np.concatenate([q[k][:2] for q in parts])
        st["resid"] = parts[0]["resid"].copy()
        i = 1234
        st["idx"][:, i] = slot
        st["resid"][i] = resid
        print(f"slot={slot} V={V} resid={resid}", flush=True)
        g.set_state(st)
        runs.append((g.debug_steps(inp.m, 7), g.get_state(), g.status()))
    (a, sa, bits), (b, sb, _) = runs
    assert bits & 2
    for f in ("sum", "leaf_new", "accept", "count"):
        np.testing.assert_array_equal(a[f], b[f], err_msg=f)
    np.testing.assert_array_equal(np.delete(sa["resid"], i), np.delete(sb["resid"], i))
    assert sb["resid"][i] == 1000.0


@pytest.mark.parametrize("n,grid,V", [(40003, 20, 1), (140003, 35, 2), (300007, 41, 4),
                                      (39711, 20, 1), (140063, 35, 2), (295711, 41, 4),
                                      (295711, 20, 8)])
def test_chunks_per_thread(n, grid, V):
    # 1, 2, 4 and 8 chunks per thread; with the last four sizes the last
    # workgroup that has points has them in 4 of its 8 waves.  Leaves on both
    # sides of a bin pass (31 ranks, 15 with 8 chunks per thread)
    from paper_2410_23244_amd.bart import BART_RESID_REGISTERS, from_inputs

    inp = make_inputs(2, n=n, p=20, m=5, D=8)
    info = from_inputs(inp, grid=grid, residency=BART_RESID_REGISTERS).launch_info()
    assert (info.chunks_per_thread, info.grid) == (V, grid)
    for leaves in {1: [9], 2: [9, 30, 31, 32], 4: [9, 30, 31, 32], 8: [14, 15, 16, 33]}[V]:
        _run(inp, grid, leaves, [inp.m + 1])
