"""Prediction by the compiled trees against the oracle's Algorithm 1: trees of
every form of the program (no node, a decision table of up to 6 nodes, a leaf
mask of up to 31, Algorithm 1 beyond), nodes left over below a leaf, ragged
groups of 16 trees, point counts around the tile size, every split of the
trees over waves, and predictor rows of any alignment.

The sums are fp64 sums of f32 leaves; their order (tree by tree here, in
parts there) moves them by at most m 2^-53 of the sum of magnitudes, so an f32
result differs by one rounding at most, and only if f lies that close to the
middle between two f32 values: equality is asserted up to one f32 ulp and for
all but a vanishing share exactly."""
from __future__ import annotations

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _forest(rng, m, D, p, grow):
    """Random trees: a node is internal with probability grow; some slots below
    a leaf keep a cut that no point reaches."""
    H = 1 << (D - 1)
    axis = rng.integers(0, p, (m, H)).astype(np.uint16)
    cut = np.where(rng.random((m, H)) < np.asarray(grow)[:, None], rng.integers(1, 256, (m, H)), 0)
    cut[:, 0] = 0
    leaf = rng.standard_normal((m, 2 * H)).astype(np.float32)
    return axis, cut.astype(np.uint8), leaf


def _check(m, D, p, nt, nchain, grow, seed, shift=0):
    import torch

    import oracle
    from paper_2410_23244_amd import bart as B

    rng = np.random.default_rng(seed)
    few = 64
    X0 = np.zeros((p, few), np.uint8)
    g = B.Bart(X0, np.zeros(few, np.float32), np.full(p, 255, np.int32), ntree=m, max_depth=D,
               nchain=nchain)
    Xt = rng.integers(0, 256, (p, nt)).astype(np.uint8)
    stride = B.x_stride_for(nt)
    buf = torch.zeros(p * stride + 16, dtype=torch.uint8, device="cuda")
    Xd = buf[shift:shift + p * stride].view(p, stride)
    Xd[:, :nt] = torch.from_numpy(Xt).cuda()
    ref = []
    for c in range(nchain):
        axis, cut, leaf = _forest(rng, m, D, p, grow)
        ch = oracle.Chain(oracle.make_config(few, p, m, D), X0, np.full(p, 255, np.int32),
                          np.zeros(few, np.float32), 1.0)
        idx = np.empty((m, few), np.uint8)
        for j in range(m):
            h = 1
            while h < cut.shape[1] and cut[j, h]:
                h = 2 * h  # bin 0 is below every cut
            idx[j] = h
        g.set_state(dict(axis=axis, cut=cut, leaf=leaf, idx=idx, resid=np.zeros(few, np.float32),
                         sigma2=1.0, sweep=0), c)
        ch.load(axis, cut, leaf, idx, np.zeros(few, np.float32), 1.0, 0)
        ref.append(ch.predict(Xt, 0.25))
    want = np.stack(ref)
    out = torch.full((nchain, nt), np.nan, dtype=torch.float32, device="cuda")
    print(f"m={m} D={D} p={p} nt={nt} nchain={nchain} shift={shift}", flush=True)
    B.bart_predict(g.h, Xd.data_ptr(), stride, nt, 0.25, out.data_ptr())
    got = out.cpu().numpy()
    np.testing.assert_allclose(got, want, rtol=1.2e-7, atol=1e-12 * m)
    assert np.mean(got != want) < 1e-3
    s = torch.ones((nchain, nt), dtype=torch.float64, device="cuda")
    s2 = torch.zeros_like(s)
    B.bart_predict_accumulate(g.h, Xd.data_ptr(), stride, nt, 0.25, s.data_ptr(), s2.data_ptr())
    s, s2 = s.cpu().numpy() - 1.0, s2.cpu().numpy()
    scale = np.abs(want).max() + 1.0
    np.testing.assert_allclose(s, want, rtol=0, atol=6e-8 * scale)
    np.testing.assert_allclose(s2, s * s, rtol=0, atol=1e-13 * scale * scale)
    assert g.status() == 0


@pytest.mark.parametrize("D", [2, 3, 6, 7, 8])
def test_forms_of_trees(D):
    # from single leaves to complete trees, in one forest
    m = 37
    _check(m, D, 300, 1501, 2, np.linspace(0.0, 1.0, m), 10 + D)


@pytest.mark.parametrize("grow", [0.0, 1.0])
def test_groups_of_one_form(grow):
    # groups of trees without a node, and groups without a decision table
    _check(33, 8, 9, 700, 1, np.full(33, grow), 3)


@pytest.mark.parametrize("nt,nchain,m", [(1, 1, 1), (3, 3, 16), (255, 1, 17), (257, 1, 32),
                                         (1025, 2, 300), (20001, 1, 200), (262143, 1, 48),
                                         (1048577, 1, 20), (262145, 4, 20)])
def test_tiles_and_splits(nt, nchain, m):
    _check(m, 6, 11, nt, nchain, np.full(m, 0.6), nt)


@pytest.mark.parametrize("shift", [1, 2, 3])
def test_rows_of_any_alignment(shift):
    _check(20, 6, 7, 1003, 1, np.full(20, 0.6), 5, shift)


@pytest.mark.parametrize("m,D", [(5, 6), (17, 6), (40, 8), (64, 6), (100, 6), (130, 8), (300, 6),
                                 (1000, 6)])
def test_sums_do_not_depend_on_the_batch(m, D):
    """The fp64 sum of a point is added in one order, whatever the number of
    points, their place in the batch and the number of chains (and so the
    number of waves that share a tile's trees): the same bits.  The leaves
    differ by up to 2^40, as f32 values of like size add up exactly in fp64,
    in any order."""
    import torch

    from paper_2410_23244_amd import bart as B

    rng = np.random.default_rng(m)
    p, few, nt = 11, 64, 150001
    Xt = torch.from_numpy(rng.integers(0, 256, (p, B.x_stride_for(nt))).astype(np.uint8)).cuda()
    axis, cut, leaf = _forest(rng, m, D, p, np.full(m, 0.6))
    leaf *= (2.0 ** rng.integers(-20, 21, leaf.shape)).astype(np.float32)
    handles = []
    for nchain in (1, 4):
        g = B.Bart(np.zeros((p, few), np.uint8), np.zeros(few, np.float32),
                   np.full(p, 255, np.int32), ntree=m, max_depth=D, nchain=nchain)
        idx = np.empty((m, few), np.uint8)
        for j in range(m):
            h = 1
            while h < cut.shape[1] and cut[j, h]:
                h = 2 * h  # bin 0 is below every cut
            idx[j] = h
        for c in range(nchain):
            g.set_state(dict(axis=axis, cut=cut, leaf=leaf, idx=idx,
                             resid=np.zeros(few, np.float32), sigma2=1.0, sweep=0), c)
        handles.append(g)

    def f(g, first, n):
        s = torch.zeros((g.nchain, n), dtype=torch.float64, device="cuda")
        s2 = torch.zeros_like(s)
        print(f"m={m} D={D} nchain={g.nchain} first={first} n={n}", flush=True)
        B.bart_predict_accumulate(g.h, Xt.data_ptr() + first, Xt.shape[1], n, 0.1, s.data_ptr(),
                                  s2.data_ptr())
        return s.cpu().numpy()

    want = f(handles[0], 0, nt)[0]
    for g in handles:
        for first, n in ((0, 100), (0, 4001), (0, 60001), (0, 100003), (777, 3001)):
            got = f(g, first, n)
            for c in range(g.nchain):
                np.testing.assert_array_equal(got[c], want[first:first + n])


def test_predictions_beside_steps():
    """A thread that predicts while another steps the handle gets the trees of
    one state, never the tables of one and the large trees of the next."""
    import threading

    import torch

    from paper_2410_23244_amd import bart as B
    from paper_2410_23244_amd.inputs import make_inputs
    from tests.test_register_exchange import _state

    inp = make_inputs(2, n=600, p=12, m=24, D=8)
    sweeps, seed, nt = 200, 3, 4000
    parts = [_state(inp, k, np.random.default_rng(k)) for k in (4, 40)]
    st = dict(parts[0])
    for k in ("axis", "cut", "leaf", "idx"):
        st[k] = np.concatenate([q[k][:12] for q in parts])
    rng = np.random.default_rng(1)
    Xt = torch.from_numpy(rng.integers(0, 256, (inp.p, B.x_stride_for(nt))).astype(np.uint8)).cuda()

    def f(g):
        out = torch.empty(nt, dtype=torch.float32, device="cuda")
        B.bart_predict(g.h, Xt.data_ptr(), Xt.shape[1], nt, 0.0, out.data_ptr())
        return out

    a, b = B.from_inputs(inp), B.from_inputs(inp)
    a.set_state(st)
    b.set_state(st)
    states = [f(a).cpu().numpy()]
    for _ in range(sweeps):
        a.step(1, seed)
        states.append(f(a).cpu().numpy())
    outs, stop = [], threading.Event()

    def predict():
        while not stop.is_set() and len(outs) < 20000:
            outs.append(f(b))

    th = threading.Thread(target=predict)
    th.start()
    for _ in range(sweeps):
        b.step(1, seed)
    stop.set()
    th.join()
    torch.cuda.synchronize()
    known = {s.tobytes() for s in states}
    bad = sum(o.cpu().numpy().tobytes() not in known for o in outs)
    print(f"{len(outs)} predictions beside {sweeps} sweeps, {bad} of no state", flush=True)
    assert outs and bad == 0 and b.status() == 0
