"""Rows computed ahead for the kernel-row cache, and candidate records by wave.

Where X is large (2^24 floats and more) the columns of a streaming launch
that belong to cached samples compute rows that later working sets are
likely to need, and the cached samples' rows are read.  K values are the
same bits either way, so a training must give the bits of the one without
the cache: with a cache that keeps everything, with one so small that it
replaces rows all along, C-SVC and eps-SVR, another kernel, working sets
below 16, features past one LDS slice of the selection (where no row is
computed ahead), and shapes whose row kernel runs few blocks (a record per
wave) or many.  Rows computed ahead end where they do not lead to working
sets served from the cache.
"""
import re

import numpy as np
import pytest

from paper_1706_05544_amd import native as nv

pytestmark = pytest.mark.gpu


def _data(n, d, svr=False):
    rng = np.random.default_rng(n + d)
    X = rng.standard_normal((n, d), dtype=np.float32)
    if svr:
        z = np.sin(3 * X[:, 0]) + 0.1 * rng.standard_normal(n)
        return X, z.astype(np.float32)
    y = np.where(rng.random(n) < 0.5, 1.0, -1.0).astype(np.float32)
    return X + np.float32(2.25 / np.sqrt(d)) * y[:, None], y


@pytest.mark.parametrize("n,d,rows,kw", [
    (40009, 420, 0, {}),                       # many blocks
    (40009, 420, 90, {}),                      # constant replacement
    (21001, 800, 0, {}),                       # a record per wave
    (21001, 800, 200, dict(working_set=10)),
    (21001, 801, 0, dict(kernel=1, coef0=1.0)),
    (40000, 421, 0, dict(type=1, C=10.0, max_iter=400)),
    (40000, 421, 70, dict(type=1, C=10.0, max_iter=400)),
    (11000, 1600, 0, {}),                      # two slices
])
def test_same_bits_with_rows_computed_ahead(n, d, rows, kw):
    X, y = _data(n, d, kw.get("type") == 1)
    cache = rows * ((n + 3) // 4 * 4) * 4  # 0: the default (the whole K)
    got = []
    for cb in (-1, cache):
        m = nv.svm_train(X, y, cache_bytes=cb, **kw)
        got.append((m.info(), nv.svm_model_get(m, 0, with_alpha=True)[2]))
    (i0, a0), (i1, a1) = got
    np.testing.assert_array_equal(a1, a0)
    for k in ("iters", "b", "dual_obj", "gap", "kernel_rows", "status"):
        assert i1[k] == i0[k], k
    assert i1["cache_fills"] > 0
    assert i1["cache_hits"] <= i1["kernel_rows"]


def _ahead(err):
    """(rows in working sets served entirely, rows computed ahead) of the
    trainings whose SVM_LOG lines err holds."""
    found = re.findall(r"(\d+) of them whole sets, filled \d+, "
                       r"(\d+) of them ahead", err)
    return [tuple(map(int, f)) for f in found]


@pytest.mark.parametrize("n,d,rows,kw,ahead", [
    (70009, 460, 0, {}, "on"),
    (70009, 460, 90, {}, 90),               # a cache filled at once
    (41001, 801, 0, dict(kernel=1, coef0=1.0), "on"),
    (41001, 800, 200, dict(working_set=10), 200),
    (70000, 461, 0, dict(type=1, C=10.0, max_iter=300), 64 * 16),
    (39009, 427, 0, {}, None),              # too small an X
])
def test_rows_ahead_only_where_they_serve(n, d, rows, kw, ahead, capfd,
                                          monkeypatch):
    # "on": to the end; a number: at most so many, then no more
    X, y = _data(n, d, kw.get("type") == 1)
    cache = rows * ((n + 3) // 4 * 4) * 4
    monkeypatch.setenv("SVM_LOG", "1")
    capfd.readouterr()
    got = []
    for cb in (-1, cache):
        m = nv.svm_train(X, y, cache_bytes=cb, **kw)
        got.append((m.info(), nv.svm_model_get(m, 0, with_alpha=True)[2],
                    _ahead(capfd.readouterr().err)))
    (i0, a0, _), (i1, a1, ((whole, done),)) = got
    np.testing.assert_array_equal(a1, a0)
    for k in ("iters", "b", "dual_obj", "gap", "kernel_rows", "status"):
        assert i1[k] == i0[k], k
    if ahead == "on":
        assert done > 0 and 4 * whole > i1["kernel_rows"]
    elif ahead is None:
        assert done == 0
    else:
        assert done <= ahead
        assert whole < i1["kernel_rows"] // 4


@pytest.mark.parametrize("n,d,order", [
    (29001, 784, "mixed"),   # fewer groups of records than entries of a list
    (40009, 421, "sorted"),  # the candidates of a side in half of them
    (64001, 421, "uneven"),  # ... in less than half
])
def test_few_groups_of_records(n, d, order, capfd, monkeypatch):
    # The longer lists of candidates are cut by a bound that so many groups
    # of records have to reach.  With fewer that hold candidates every
    # candidate stayed, and ranking them took 15 times what it takes without
    # rows computed ahead (with them elsewhere up to 4 times).
    X, y = _data(n, d)
    if order != "mixed":
        take = np.argsort(y, kind="stable")
        if order == "uneven":
            take = take[:int((y < 0).sum()) + n // 6]
        X, y = X[take], y[take]
    monkeypatch.setenv("SVM_LOG", "1")
    capfd.readouterr()
    got, rank = [], []
    for cb in (-1, 0):
        for _ in range(2):  # (the first one warms the clocks up)
            m = nv.svm_train(X, y, cache_bytes=cb)
        got.append((m.info(), nv.svm_model_get(m, 0, with_alpha=True)[2]))
        err = capfd.readouterr().err
        rank.append(float(re.findall(r" rank ([\d.]+) groups", err)[-1]))
        ahead = _ahead(err)
    (i0, a0), (i1, a1) = got
    np.testing.assert_array_equal(a1, a0)
    for k in ("iters", "b", "dual_obj", "gap", "kernel_rows", "status"):
        assert i1[k] == i0[k], k
    assert ahead[-1][1] > 0
    assert rank[1] < 8 * rank[0]
