"""Decision values of few query rows and of wide rows against large batches.

The batch a row comes in chooses the path (few rows: kernel values of all
tiles at once, then the sums; many: one kernel), never the bits: rows of a
small call must equal, bit for bit, the same rows inside a batch of the
one-kernel path, and both the oracle.  Sizes around the tiles of both paths
(16, 64 and 128 rows; 16-, 32- and 64-feature chunks; one and several ranges
of support rows, whole and ragged) and of their rules.  Sparse rows: the table
path over ranges of support rows and slabs of query rows.
"""
import numpy as np
import pytest
import scipy.sparse as sp
import torch

import oracle
from paper_1706_05544_amd import native as nv

RBF, SIG = nv.SVM_KERNEL_RBF, nv.SVM_KERNEL_SIGMOID
pytestmark = pytest.mark.gpu


def _model(nsv, d, kernel, n_out):
    rng = np.random.default_rng(nsv * 1009 + d)
    X = rng.standard_normal((nsv, d), dtype=np.float32)
    kw = dict(kernel=kernel, gamma=1.0 / d, C=1.0, tol=1e6)
    if n_out > 1:
        y = (np.arange(nsv) % n_out).astype(np.float32)
        return X, nv.svm_train_ovr(X, y, n_out, kernel=kernel, gamma=1.0 / d,
                                   max_iter=60)
    y = np.where(np.arange(nsv) % 2 == 0, 1.0, -1.0).astype(np.float32)
    alpha = np.full(nsv, 0.5)  # every row a support row, y^T alpha = 0
    if nsv % 2:
        alpha[[-3, -1]] = 0.25
    return X, nv.svm_train(X, y, alpha0=alpha, **kw)


@pytest.mark.parametrize("nsv,d,kernel,n_out", [
    (700, 20, RBF, 1),       # one range, just past the tile-work rule
    (1601, 128, RBF, 1),     # two ranges, the last tile one row
    (3007, 129, RBF, 1),     # wide rows, a ragged chunk
    (1000, 160, SIG, 1),     # another kernel
    (12801, 131, RBF, 1),    # eight ranges
    (257, 784, RBF, 1),      # odd half step of 128 support rows
    (900, 130, RBF, 3),
    (1700, 40, RBF, 10),
])
def test_batch_does_not_change_the_bits(nsv, d, kernel, n_out):
    X, model = _model(nsv, d, kernel, n_out)
    rng = np.random.default_rng(d)
    big = 128 * 64 + 77
    Xt = torch.from_numpy(rng.standard_normal((big, d), dtype=np.float32))
    Xd = Xt.to("cuda:0")
    D = nv.svm_predict(model, Xd).reshape(big, -1)
    for m in (1, 15, 17, 64, 65, 300, 1111, 2049):
        Dm = nv.svm_predict(model, Xd[:m].contiguous()).reshape(m, -1)
        assert torch.equal(Dm, D[:m]), m
        out = torch.full((m, n_out), float("nan"), dtype=torch.float64,
                         device="cuda:0")
        nv.svm_predict_noalloc(model, Xd[:m].contiguous(), out)
        assert torch.equal(out, D[:m]), m
    if n_out == 1 and kernel == RBF:
        idx, cf, _ = nv.svm_model_get(model, 0)
        ref = oracle.decision(X[idx], cf, model.info()["b"],
                              Xt[:200].numpy(), 1.0 / d)
        # fp32 kernel values (d products, one exponential) against fp64
        tol = np.abs(cf).sum() * (d + 40) * 2.0 ** -24
        np.testing.assert_allclose(D[:200, 0].cpu().numpy(), ref, rtol=0,
                                   atol=tol)


@pytest.mark.parametrize("nsv,d", [
    (200, 200),    # a short chain of tiles: one kernel from 2 MB of values on
    (700, 256),    # ... from 3.07 million values on
    (400, 132), (1000, 256), (1032, 256), (257, 784), (40, 140)])
def test_medium_batches_keep_the_bits(nsv, d):
    # the lines between the two kernels, the one kernel's tiles of 64 x 64
    # rows and those of 128 x 128
    X, model = _model(nsv, d, RBF, 1)
    rng = np.random.default_rng(d)
    big = 128 * 96 + 1
    Xt = torch.from_numpy(rng.standard_normal((big, d), dtype=np.float32))
    Xd = Xt.to("cuda:0")
    D = nv.svm_predict(model, Xd)
    for m in (1, 2520, 2622, 4360, 4370, 128 * 95, 128 * 95 + 1):
        Dm = nv.svm_predict(model, Xd[:m].contiguous())
        assert torch.equal(Dm, D[:m]), m
        out = torch.full((m, 1), float("nan"), dtype=torch.float64,
                         device="cuda:0")
        nv.svm_predict_noalloc(model, Xd[:m].contiguous(), out)
        assert torch.equal(out[:, 0], D[:m]), m
    idx, cf, _ = nv.svm_model_get(model, 0)
    ref = oracle.decision(X[idx], cf, model.info()["b"], Xt[:200].numpy(),
                          1.0 / d)
    tol = np.abs(cf).sum() * (d + 40) * 2.0 ** -24
    np.testing.assert_allclose(D[:200].cpu().numpy(), ref, rtol=0, atol=tol)


def _csr(n, d, nnz, seed):
    rng = np.random.default_rng(seed)
    cols = (np.arange(n)[:, None] * 7 + np.cumsum(
        rng.integers(1, d // nnz, (n, nnz)), axis=1)) % d
    cols.sort(axis=1)
    vals = rng.standard_normal((n, nnz), dtype=np.float32)
    return sp.csr_matrix((vals.ravel(), cols.ravel().astype(np.int32),
                          np.arange(n + 1) * nnz), shape=(n, d))


@pytest.mark.parametrize("nsv,n_out,m", [
    (1500, 1, 700),        # one range
    (1601, 1, 5001),       # two, the last chunk one row
    (13003, 1, 3000),      # eight
    (9000, 10, 300001),    # more rows than one slab of partial sums
])
def test_sparse_ranges(nsv, n_out, m):
    # 20 of 1000 columns a row: the table path in every batch size
    X = _csr(nsv, 1000, 20, 1)
    if n_out > 1:
        y = (np.arange(nsv) % n_out).astype(np.float32)
        model = nv.svm_train_ovr(X, y, n_out, gamma=0.05, max_iter=50)
    else:
        y = np.where(np.arange(nsv) % 2 == 0, 1.0, -1.0).astype(np.float32)
        alpha = np.full(nsv, 0.5)
        if nsv % 2:
            alpha[[-3, -1]] = 0.25
        model = nv.svm_train(X, y, gamma=0.05, alpha0=alpha, tol=1e6)
    Xt = _csr(m, 1000, 20, 2)
    D = nv.svm_predict(model, Xt).reshape(m, -1)
    for a, b in ((0, 1), (0, 257), (m - 300, m)):
        np.testing.assert_array_equal(
            nv.svm_predict(model, Xt[a:b]).reshape(b - a, -1), D[a:b])
    idx, cf, _ = nv.svm_model_get(model, 0)
    SV = oracle.Matrix(X).rows(idx)
    ref = oracle.decision(SV, cf, model.info(0)["b"], Xt[-300:], 0.05)
    # fp32 kernel values (20 products, one exponential) against fp64
    np.testing.assert_allclose(D[-300:, 0], ref, rtol=0,
                               atol=np.abs(cf).sum() * 60 * 2.0 ** -24)
