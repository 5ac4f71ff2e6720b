"""Kernel values that overflow fp32, of samples that are in no working set.

A polynomial kernel of large rows overflows to infinity.  A slot that a
working set does not use (it has fewer than 16 samples) must not bring such
a value into the responses: its coefficient is 0, and 0 times infinity is not
a number.  One row here is so large that its kernel value with another,
ordinary row overflows (every other value of its row of K is 0: the two have
a feature to themselves); it is never in a working set, and the ordinary row
is.  The bar is equality with the training without the row cache, whose
unused slots hold rows of zeros.
"""
import numpy as np
import pytest

from paper_1706_05544_amd import native as nv

pytestmark = pytest.mark.gpu

POLY = dict(type=nv.SVM_EPS_SVR, kernel=nv.SVM_KERNEL_POLY, degree=3,
            coef0=0.0)


@pytest.mark.parametrize("n,q,huge", [(300, 8, 0), (1000, 2, 0),
                                      (2500, 12, 0)])
def test_all_of_k_at_hand(n, q, huge):
    # the huge row is held out of the fold's training, the other one trained
    rng = np.random.default_rng(n)
    X = rng.standard_normal((n, 7), dtype=np.float32)
    z = (X[:, 1] * X[:, 2] ** 2 + 0.1 * rng.standard_normal(n)).astype("f4")
    X[:, 0] = 0.0
    other = n // 2
    X[huge], X[other] = 0.0, 0.0
    X[huge, 0], X[other, 0] = 1e18, 1.0
    z[other] = 3.0
    fold = (np.arange(n) % 3 == 1).astype(np.int32)
    fold[[huge, other]] = 0, 1
    kw = dict(POLY, k=2, fold=fold, C=10.0, epsilon=0.1, working_set=q,
              max_iter=200)
    D0, _ = nv.svm_cross_validate(X, z, cache_bytes=-1, **kw)
    D1, _ = nv.svm_cross_validate(X, z, **kw)
    rows = np.flatnonzero(fold == 0)
    rows = rows[rows != huge]
    assert np.all(np.isfinite(D0[rows]))
    np.testing.assert_array_equal(D1[rows], D0[rows])


def test_rows_computed_ahead():
    # Two outer iterations on responses that hardly move (C is tiny): the
    # working sets are ranks 1 and 2 of each side, then 3 and 4.  The huge row
    # has rank 8 of its side, so the first launch computes its row ahead in a
    # column past the working set, and the ordinary one rank 3 of the other.
    n, d = 70009, 460
    rng = np.random.default_rng(1)
    X = rng.standard_normal((n, d), dtype=np.float32)
    X[:, 0] = 0.0
    z = rng.uniform(-1, 1, n).astype(np.float32)
    # (far apart: a block of rows reports its best two only)
    top = 100 + 2000 * np.arange(10)
    low = 35100 + 2000 * np.arange(10)
    z[top] = 100.0 - np.arange(10)
    z[low] = -100.0 + np.arange(10)
    huge, other = top[7], low[2]
    X[huge], X[other] = 0.0, 0.0
    X[huge, 0], X[other, 0] = 1e18, 1.0
    kw = dict(POLY, C=1e-3, epsilon=0.1, working_set=4, max_iter=2)
    got = []
    for cb in (-1, 64 * ((n + 3) // 4 * 4) * 4 + (1 << 26)):
        m = nv.svm_train(X, z, cache_bytes=cb, **kw)
        got.append((nv.svm_model_get(m, 0, with_alpha=True)[2], m.info()))
    (a0, _), (a1, i1) = got
    assert i1["cache_fills"] > 8  # more rows than the working sets'
    assert a0[n + other] > 0 or a0[other] > 0
    assert a0[huge] == 0 and a0[n + huge] == 0
    np.testing.assert_array_equal(a1, a0)
