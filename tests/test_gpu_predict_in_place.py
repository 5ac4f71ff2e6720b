"""svm_predict on device rows that are used where they are.

The values are checked after the decision kernels there and before them
otherwise: the same rows from host memory (copied, checked first) must give
the same bits and labels, and a value that is not finite the same error.
Sizes: one and several ranges of support rows, the path for few rows, and
buffers on both sides of 2 MB, where the call takes one or two.
"""
import numpy as np
import pytest
import torch

from paper_1706_05544_amd import native as nv

pytestmark = pytest.mark.gpu


def _model(nsv, d, n_out):
    rng = np.random.default_rng(nsv + d)
    X = rng.standard_normal((nsv, d), dtype=np.float32)
    y = (np.arange(nsv) % max(n_out, 2)).astype(np.float32)
    if n_out > 1:
        return nv.svm_train_ovr(X, y, n_out, gamma=1.0 / d, max_iter=40)
    return nv.svm_train(X, 2.0 * y - 1.0, gamma=1.0 / d, tol=1e6,
                        alpha0=np.full(nsv, 0.5))


@pytest.mark.parametrize("nsv,d,n_out,m", [
    (700, 20, 1, 1),         # few rows, one buffer
    (3000, 128, 1, 300),     # few rows, kernel values past 2 MB
    (2000, 256, 3, 700),     # few wide rows, two buffers
    (3400, 64, 1, 20001),    # three ranges, one buffer
    (12800, 32, 1, 40003),   # eight ranges, two buffers
    (1200, 64, 3, 9000),     # one range: nothing between the kernels
])
def test_same_bits_as_copied_rows(nsv, d, n_out, m):
    model = _model(nsv, d, n_out)
    X = np.random.default_rng(m).standard_normal((m, d), dtype=np.float32)
    Xd = torch.from_numpy(X).to("cuda:0")
    D = nv.svm_predict(model, Xd)
    np.testing.assert_array_equal(D.cpu().numpy().reshape(m, -1),
                                  nv.svm_predict(model, X).reshape(m, -1))
    L = nv.svm_predict_labels(model, Xd)
    np.testing.assert_array_equal(torch.as_tensor(L).cpu().numpy(),
                                  nv.svm_predict_labels(model, X))
    for bad in (float("nan"), float("inf"), 1e30):  # (its square overflows)
        Xb = Xd.clone()
        Xb[m - 1, d - 1] = bad
        with pytest.raises(nv.SvmError, match="not finite"):
            nv.svm_predict(model, Xb)
        with pytest.raises(nv.SvmError, match="not finite"):
            nv.svm_predict_labels(model, Xb)
    assert torch.equal(nv.svm_predict(model, Xd), D)
