"""The loop that runs many outer iterations to a launch (k_resident) on the GPU.

It takes dense problems whose whole kernel matrix the row cache holds, and
promises the bits of the two-launch loop: working sets, alpha, bias,
objective and iteration counts.  So the bar is equality with the same
training without the row cache, which the other tests tie to the oracle.
Sizes sit at its edges: two rows a thread, 1920 rows a block, one to several
blocks that exchange their candidates, the smallest problems, working sets
of 2 to 16, ties of every key (alpha = 0) past the candidate list, eps-SVR
with both copies of a sample in a working set.
"""
import os
import re
from types import SimpleNamespace

import numpy as np
import pytest

from paper_1706_05544_amd import native as nv
from paper_1706_05544_amd import workloads

pytestmark = pytest.mark.gpu

SAME = ("iters", "b", "dual_obj", "gap", "kernel_rows", "status", "n_bounded")


def _train(w, alpha0=None, **kw):
    k = dict(type=w.type, C=w.C, epsilon=w.eps, gamma=w.gamma, tol=w.tol)
    k.update(kw)
    m = nv.svm_train(w.X, w.y, alpha0=alpha0, **k)
    return m.info(), nv.svm_model_get(m, 0, with_alpha=True)[2]


@pytest.fixture
def loops(capfd, monkeypatch):
    """What the trainings since the last call ran as, one after another:
    (iterations in the resident loop, all iterations, blocks, launches called
    off) of each that had a resident launch."""
    monkeypatch.setenv("SVM_LOG", "1")

    def read():
        err = capfd.readouterr().err
        found = re.findall(r"resident loop: (\d+) of (\d+) iterations in \d+ "
                           r"launches of (\d+) blocks, (\d+) called off", err)
        return [tuple(map(int, f)) for f in found]
    return read


def _same(w, loops, blocks, **kw):
    i0, a0 = _train(w, cache_bytes=-1, **kw)
    assert loops() == []
    i1, a1 = _train(w, **kw)
    np.testing.assert_array_equal(a1, a0)
    for k in SAME:
        assert i1[k] == i0[k], k
    # the loop under test ran, from the first iteration to the last
    assert loops() == [(i1["iters"], i1["iters"], blocks, 0)]
    return i1


@pytest.mark.parametrize("name,n,kw", [
    ("C1", 2, {}), ("C1", 3, {}), ("C1", 31, {}), ("C2", 29, {}),
    ("C1", 600, {}), ("C1", 1919, {}), ("C1", 1920, {}), ("C1", 1921, {}),
    ("C2", 1921, {}), ("C1", 3841, {}), ("C2", 3000, {}),
    ("C3", 12345, {}),
    ("C1", 777, dict(working_set=2)), ("C2", 2500, dict(working_set=6)),
    ("C1", 2100, dict(working_set=14)),
    ("C1", 1000, dict(kernel=1, coef0=1.0)), ("C1", 1000, dict(kernel=3)),
    ("C2", 2001, dict(kernel=0, max_iter=300)),
    ("C1", 1500, dict(max_iter=7)), ("C1", 2000, dict(check_every=3)),
    ("C1", 900, dict(max_inner=1)), ("C1", 1500, dict(scale=1)),
])
def test_same_bits_as_the_two_launch_loop(name, n, kw, loops):
    _same(workloads.make(name, n=n, n_test=4), loops, -(-n // 1920), **kw)


def _rows(n, d, svr=False):
    rng = np.random.default_rng(n + d)
    X = rng.standard_normal((n, d), dtype=np.float32)
    if svr:
        y = np.sin(3 * X[:, 0]) + 0.1 * rng.standard_normal(n)
    else:
        y = np.where(rng.random(n) < 0.5, 1.0, -1.0)
        X += np.float32(2.25 / np.sqrt(d)) * y[:, None].astype(np.float32)
    return SimpleNamespace(X=X, y=y.astype(np.float32), type=int(svr),
                           C=10.0 if svr else 1.0, eps=0.1, gamma=0.0,
                           tol=1e-3)


@pytest.mark.parametrize("n,d,svr,kw", [
    (2000, 20, False, {}),             # two blocks
    (4100, 20, True, {}),              # three
    (15361, 7, False, dict(max_iter=400)),               # nine
    (23041, 5, True, dict(max_iter=300)),                # thirteen
    (24001, 6, False, dict(max_iter=300, working_set=12)),
])
def test_late_block(n, d, svr, kw, monkeypatch, loops):
    # Every block solves the subproblem of an iteration for itself.  One that
    # takes up the exchanged candidates 20 us late, when the others are past
    # their iteration's end, has to find alpha as it was before it.
    w = _rows(n, d, svr)
    i0, a0 = _train(w, cache_bytes=-1, **kw)
    for lag in ("2000", None):
        if lag:
            monkeypatch.setenv("SVM_RESIDENT_LAG", lag)
        else:
            monkeypatch.delenv("SVM_RESIDENT_LAG")
        i1, a1 = _train(w, **kw)
        np.testing.assert_array_equal(a1, a0)
        for k in SAME:
            assert i1[k] == i0[k], k
        assert loops() == [(i1["iters"], i1["iters"], -(-n // 1920), 0)]


@pytest.mark.parametrize("n,d,svr,lag", [
    (61440, 4, False, "2000"),  # 32 blocks, the most, of 128 and 8 of 256
    (61439, 4, True, "0"),
    (50001, 8, False, "0"),
])
def test_most_blocks(n, d, svr, lag, monkeypatch, loops):
    w = _rows(n, d, svr)
    kw = dict(k=4, type=w.type, C=w.C, epsilon=w.eps, max_iter=150)
    D0, s0 = nv.svm_cross_validate(w.X, w.y, cache_bytes=-1, **kw)
    monkeypatch.setenv("SVM_RESIDENT_LAG", lag)
    D1, s1 = nv.svm_cross_validate(w.X, w.y, **kw)
    np.testing.assert_array_equal(D1, D0)
    assert s1["iters"] == s0["iters"]
    assert loops() == [(150, 150, -(-n // 1920), 0)] * 4


def test_more_rows_than_blocks_hold(loops):
    # one row past 32 blocks: the two-launch loop
    w = _rows(61441, 4)
    kw = dict(k=4, max_iter=50)
    D0, _ = nv.svm_cross_validate(w.X, w.y, cache_bytes=-1, **kw)
    D1, _ = nv.svm_cross_validate(w.X, w.y, **kw)
    np.testing.assert_array_equal(D1, D0)
    assert loops() == []


@pytest.mark.parametrize("n,d,sep,kw,ran", [
    # K costs more than a short solve gains: the two-launch loop begins, and
    # ends a short one
    (30001, 61, 8.0, {}, 0),
    (42424, 12, 8.0, {}, 0),
    (30001, 61, 2.25, {}, 12),    # told after 12 iterations
    (42424, 12, 2.25, dict(check_every=5), 12),
    (24001, 64, 8.0, {}, None),   # K cheap enough
    (42428, 4, 2.25, dict(max_iter=100), 0),   # K too large for one training
    (20001, 120, 2.25, dict(max_iter=60), 0),  # too few iterations to gain
])
def test_whole_k_only_where_it_pays(n, d, sep, kw, ran, loops):
    w = _rows(n, d)
    w.X += np.float32((sep - 2.25) / np.sqrt(d)) * w.y[:, None]
    i0, a0 = _train(w, cache_bytes=-1, **kw)
    i1, a1 = _train(w, **kw)
    np.testing.assert_array_equal(a1, a0)
    for k in SAME:
        assert i1[k] == i0[k], k
    assert i1["cache_fills"] + i1["cache_hits"] > 0
    blocks = -(-n // 1920)
    if ran == 0:
        assert loops() == []
    else:
        assert loops() == [(i0["iters"] - (ran or 0), i0["iters"], blocks, 0)]


@pytest.mark.parametrize("svr,C", [(True, 10.0), (False, 0.1)])
def test_first_iterations(svr, C, loops):
    # the stages at which the first iterations tell a long solve: after 12 and
    # after 32 of them
    n, kw = 30001, dict(C=C, max_iter=600)
    w = _rows(n, 61, svr)
    if not svr:
        w.X += np.float32(1.75 / np.sqrt(61)) * w.y[:, None]
    gap = [_train(w, cache_bytes=-1, **{**kw, "max_iter": k})[0]["gap"]
           for k in (1, 12, 32)]
    i0, a0 = _train(w, cache_bytes=-1, **kw)
    i1, a1 = _train(w, **kw)
    np.testing.assert_array_equal(a1, a0)
    for k in SAME:
        assert i1[k] == i0[k], k
    ran = (12 if gap[1] > 0.87 * gap[0] else
           32 if gap[2] > 0.5 * gap[0] else 192)
    if ran >= i0["iters"]:
        assert loops() == []
    else:
        assert loops() == [(i0["iters"] - ran, i0["iters"], 16, 0)]


@pytest.mark.parametrize("svr", [False, True])
def test_accepted_warm_start_computes_no_k(svr, loops):
    w = _rows(9001, 24, svr)
    kw = dict(max_iter=2000)
    i1, a1 = _train(w, **kw)
    assert len(loops()) == 1
    _train(w, alpha0=a1, **{**kw, "tol": max(2 * i1["gap"], 1e-3)})
    assert loops() == []


def test_duplicate_rows(loops):
    # equal rows: zero curvature, equal keys all along
    w = workloads.make("C2", n=2200, n_test=4)
    w.X[1100:] = w.X[:1100]
    _same(w, loops, 2, max_iter=400)


def test_launch_called_off(loops):
    # no time to wait for a problem's blocks: launches are called off and the
    # two-launch loop takes over from the state they left
    w = workloads.make("C2", n=4100, n_test=4)
    i0, a0 = _train(w, cache_bytes=-1)
    os.environ["SVM_RESIDENT_WAIT"] = "0"
    try:
        for _ in range(3):
            i1, a1 = _train(w)
            np.testing.assert_array_equal(a1, a0)
            assert i1["iters"] == i0["iters"] and i1["b"] == i0["b"]
            (done, iters, blocks, off), = loops()
            assert off > 0 and done == 0 and blocks == 3
    finally:
        del os.environ["SVM_RESIDENT_WAIT"]


def test_launch_called_off_once(loops, monkeypatch):
    # the resident loop takes the solve up again
    w = workloads.make("C2", n=4100, n_test=4)
    i0, a0 = _train(w, cache_bytes=-1)
    for first in (1, 2):  # (two launches are queued, then one at a time)
        monkeypatch.setenv("SVM_RESIDENT_OFF", str(first))
        i1, a1 = _train(w)
        np.testing.assert_array_equal(a1, a0)
        assert loops() == [(i0["iters"], i0["iters"], 3, first)]


def test_called_off_in_lockstep(capfd, monkeypatch):
    # who asks for lockstep groups gets them when the resident loop does not
    # run: 5 trainings in groups of 2, the last one alone
    w = workloads.make("C1", n=4000, n_test=4)
    kw = dict(k=5, type=w.type, C=w.C, epsilon=w.eps, gamma=w.gamma,
              tol=w.tol, lockstep=2)
    D0, s0 = nv.svm_cross_validate(w.X, w.y, cache_bytes=-1, **kw)
    monkeypatch.setenv("SVM_RESIDENT_WAIT", "0")
    monkeypatch.setenv("SVM_LOG", "1")
    capfd.readouterr()
    D1, s1 = nv.svm_cross_validate(w.X, w.y, **kw)
    err = capfd.readouterr().err
    np.testing.assert_array_equal(D1, D0)
    assert s1["iters"] == s0["iters"] and s1["status"] == s0["status"]
    assert err.count("resident loop: 0 of") == 5
    assert err.count("lockstep: 2 problems") == 2


@pytest.mark.parametrize("name,n,k,lockstep", [
    ("C1", 501, 3, 0), ("C2", 700, 4, 4), ("C1", 4000, 5, 2)])
def test_cross_validation_side_by_side(name, n, k, lockstep, loops):
    w = workloads.make(name, n=n, n_test=4)
    kw = dict(k=k, type=w.type, C=w.C, epsilon=w.eps, gamma=w.gamma,
              tol=w.tol, lockstep=lockstep)
    D0, s0 = nv.svm_cross_validate(w.X, w.y, cache_bytes=-1, **kw)
    D1, s1 = nv.svm_cross_validate(w.X, w.y, **kw)
    np.testing.assert_array_equal(D1, D0)
    for key in ("iters", "kernel_rows", "accuracy", "mse", "status"):
        assert s1[key] == s0[key], key
    ran = loops()
    assert len(ran) == k and sum(r[0] for r in ran) == s1["iters"]


def test_ovr_and_tuning_side_by_side(loops):
    w = workloads.make("C4", n=2003, n_test=50)
    kw = dict(C=w.C, gamma=w.gamma, tol=w.tol)
    m0 = nv.svm_train_ovr(w.X, w.y, w.n_classes, cache_bytes=-1, **kw)
    m1 = nv.svm_train_ovr(w.X, w.y, w.n_classes, **kw)
    for c in range(w.n_classes):
        np.testing.assert_array_equal(
            nv.svm_model_get(m1, c, with_alpha=True)[2],
            nv.svm_model_get(m0, c, with_alpha=True)[2])
    assert [r[0] for r in loops()] == [m1.info(c)["iters"]
                                       for c in range(w.n_classes)]
    w = workloads.c1(n=900, n_test=4)
    kw = dict(k=3, C=np.array([0.1, 1.0, 10.0]),
              gamma=np.array([0.05, 0.05, 0.2]), tol=w.tol)
    e0, b0 = nv.svm_tune(w.X, w.y, cache_bytes=-1, **kw)
    e1, b1 = nv.svm_tune(w.X, w.y, **kw)
    np.testing.assert_array_equal(e1, e0)
    assert b0 == b1
    assert len(loops()) == 9  # three folds of each
