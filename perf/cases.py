"""The work that users of this library have it do, as measurable cases.

A case is a dict of plain values.  Its ``kind`` says which public calls one
pass makes:

  train    svm_train on a dense matrix to the default tolerance, the fitted
           model read back (alpha, bias, objective), and the test points
           predicted: what fitting a model is in practice
  csr      the same on a sparse matrix in CSR form
  ovr      svm_train_ovr (one-vs-rest) and svm_predict
  cv       svm_cross_validate
  predict  svm_predict with a model at hand, on a batch of dense rows
  serve    svm_predict_noalloc into a buffer that the caller keeps
  pcsr     svm_predict on a batch of CSR rows

Inputs are drawn on the GPU from the seed alone, with the distributions of
``paper_1706_05544_amd/workloads.py``: two isotropic Gaussians for C-SVC, a
smooth function of three of the features plus noise for eps-SVR, sparse class
prototypes for the ten classes, 20 of 1000 columns a row for CSR.  The models
of the predicting cases are given coefficients (a share of them at C, as a
trained model has) through a warm start that is accepted as it stands, which
is how a program loads a model fitted elsewhere; their exact decision values
can then be computed without a training.
"""
import math

import numpy as np
import torch

from paper_1706_05544_amd import native as nv

SVC, SVR = nv.SVM_C_SVC, nv.SVM_EPS_SVR
KERNELS = {"linear": nv.SVM_KERNEL_LINEAR, "poly": nv.SVM_KERNEL_POLY,
           "rbf": nv.SVM_KERNEL_RBF, "sigmoid": nv.SVM_KERNEL_SIGMOID}
DEV = "cuda" if torch.cuda.is_available() else "cpu"


def listed():
    return [
        # the smallest training: a table of 2000 x 20 in host memory, as an R
        # or NumPy session has it; launches and latency are all there is
        dict(name="svc_2000x20_host", kind="train", task="svc", n=2000, d=20,
             m=1000, kernel="rbf", host=True),
        # regression, the slowly converging kind: thousands of short outer
        # iterations (the 20000 x 50 recipe at a fifth of its rows)
        dict(name="svr_4000x50", kind="train", task="svr", n=4000, d=50,
             m=1000, kernel="rbf", host=False),
        # the benchmark of this repository: a mid-size dense classification
        dict(name="svc_100000x128", kind="train", task="svc", n=100000, d=128,
             m=20000, kernel="rbf", host=False),
        # the shape of the paper's classification data set (odd in n and d)
        dict(name="svc_68971x501", kind="train", task="svc", n=68971, d=501,
             m=6897, kernel="rbf", host=False),
        # another kernel function, ordinary size
        dict(name="svc_20000x64_poly", kind="train", task="svc", n=20000,
             d=64, m=5000, kernel="poly", host=False),
        # the largest training: ten classes on 500000 images of 784 pixels
        dict(name="ovr10_500000x784", kind="ovr", n=500000, d=784, m=50000),
        # sparse text-like rows, a tenth of the 2M-row problem
        dict(name="svc_csr_200000x1000", kind="csr", n=200000, d=1000, nnz=20,
             m=100000),
        # model selection: 10-fold cross-validation, four folds in lockstep
        dict(name="cv10_20000x128", kind="cv", n=20000, d=128, folds=10,
             lockstep=4),
        # one request of a serving loop: a few rows, the latency of a call
        dict(name="serve_16x128", kind="serve", m=16, d=128, nsv=3000,
             kernel="rbf"),
        # scoring the benchmark's test set
        dict(name="predict_20000x128", kind="predict", m=20000, d=128,
             nsv=6600, kernel="rbf"),
        # scoring a large batch of wide rows, odd sizes
        dict(name="predict_50001x783", kind="predict", m=50001, d=783,
             nsv=12002, kernel="rbf"),
        # scoring sparse rows
        dict(name="predict_csr_100000x1000", kind="pcsr", m=100000, d=1000,
             nnz=20, nsv=20000),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["train", "train", "train", "csr", "ovr", "cv", "serve",
                       "predict", "predict", "pcsr"])
    if kind == "train":
        if rng.random() < 0.3:
            return dict(kind=kind, task="svr", n=_log(rng, 500, 6000),
                        d=_log(rng, 5, 120), m=_log(rng, 100, 2000),
                        kernel="rbf", host=rng.random() < 0.5)
        n = _log(rng, 500, 110000)
        kern = rng.choice(["rbf", "rbf", "rbf", "poly"])
        return dict(kind=kind, task="svc", n=n if kern == "rbf" else
                    min(n, 30000), d=_log(rng, 8, 500),
                    m=_log(rng, 100, 20000), kernel=kern,
                    host=n < 5000 and rng.random() < 0.5)
    if kind == "csr":
        return dict(kind=kind, n=_log(rng, 5000, 200000),
                    d=_log(rng, 300, 3000), nnz=rng.randint(8, 24),
                    m=_log(rng, 1000, 100000))
    if kind == "ovr":
        return dict(kind=kind, n=_log(rng, 5000, 300000),
                    d=_log(rng, 300, 784), m=_log(rng, 500, 30000))
    if kind == "cv":
        return dict(kind=kind, n=_log(rng, 1000, 20000), d=_log(rng, 8, 128),
                    folds=rng.choice([3, 5, 10]),
                    lockstep=rng.choice([0, 2, 4]))
    kern = rng.choice(["rbf", "rbf", "poly", "sigmoid"])
    if kind == "serve":
        return dict(kind=kind, m=_log(rng, 1, 512), d=_log(rng, 8, 800),
                    nsv=2 * _log(rng, 100, 8000), kernel=kern)
    if kind == "predict":
        return dict(kind=kind, m=_log(rng, 200, 50000), d=_log(rng, 8, 800),
                    nsv=2 * _log(rng, 100, 6000), kernel=kern)
    return dict(kind=kind, m=_log(rng, 1000, 100000), d=_log(rng, 300, 3000),
                nnz=rng.randint(5, 28), nsv=2 * _log(rng, 500, 10000))


# ---------------------------------------------------------------- inputs

def _gen(seed, stream):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) * 16 + stream)
    return g


def _randn(g, *shape):
    return torch.randn(*shape, generator=g, device=DEV)


def _rand(g, *shape):
    return torch.rand(*shape, generator=g, device=DEV)


def _shift(d):
    # the class means at +-shift * 1: the distance 0.5 sqrt(20) = 0.2 sqrt(128)
    # of the small and the mid-size problem; the paper's shape has 0.2
    return 0.2 if d >= 400 else 2.25 / math.sqrt(d)


def _svc_rows(g, n, d):
    y = torch.where(_rand(g, n) < 0.5, 1.0, -1.0)
    y[0], y[1] = 1.0, -1.0
    return _randn(g, n, d) + y[:, None] * _shift(d), y


def _svr_rows(g, n, d):
    X = 2 * _rand(g, n, d) - 1
    z = (torch.sin(3 * X[:, 0]) + 0.5 * X[:, 1] * X[:, 2]
         + 0.1 * _randn(g, n))
    return X, z


def _proto_rows(g, n, sup, inten):
    # ten classes of images: each class has its own fifth of the pixels, one
    # in ten of them dark, and about 16 more pixels lit at random
    classes, d = sup.shape
    lab = torch.randint(0, classes, (n,), generator=g, device=DEV)
    lab[:classes] = torch.arange(classes, device=DEV)
    X = torch.empty(n, d, device=DEV)
    for i in range(0, n, 65536):
        s = lab[i:i + 65536]
        on = sup[s]
        v = (inten[s] + 0.1 * _randn(g, len(s), d)).clamp_(0, 1)
        v *= on * (_rand(g, len(s), d) >= 0.1)
        off = _rand(g, len(s), d) * (_rand(g, len(s), d) < 16.0 / d) * ~on
        X[i:i + 65536] = v + off
    return X, lab.to(torch.int32)


def _csr_rows(g, m, d, nnz, w):
    # nnz distinct sorted columns a row: one from each of nnz even ranges
    lo = torch.arange(nnz, device=DEV) * d // nnz
    hi = (torch.arange(nnz, device=DEV) + 1) * d // nnz
    cols = lo + (_rand(g, m, nnz) * (hi - lo)).to(torch.int64)
    cols = torch.minimum(cols, hi - 1)
    vals = _randn(g, m, nnz)
    score = (vals * w[cols]).sum(1) + 0.5 * _randn(g, m)
    y = torch.where(score >= 0, 1.0, -1.0)
    y[0], y[1] = 1.0, -1.0
    crow = torch.arange(0, m * nnz + 1, nnz, device=DEV)
    X = torch.sparse_csr_tensor(crow, cols.reshape(-1).to(torch.int64),
                                vals.reshape(-1), size=(m, d))
    return X, y


def _inputs(case, seed):
    k, d, m = case["kind"], case["d"], case.get("m", 0)
    if k == "train":
        rows = _svc_rows if case["task"] == "svc" else _svr_rows
        X, y = rows(_gen(seed, 1), case["n"], d)
        Xt, _ = rows(_gen(seed, 2), m, d)
        return X, y, Xt
    if k == "ovr":
        g = _gen(seed, 0)
        sup = _rand(g, 10, d).argsort(1) < d // 5
        inten = _rand(g, 10, d)
        X, y = _proto_rows(_gen(seed, 1), case["n"], sup, inten)
        Xt, _ = _proto_rows(_gen(seed, 2), max(m, 10), sup, inten)
        return X, y, Xt
    if k == "cv":
        X, y = _svc_rows(_gen(seed, 1), case["n"], d)
        return X, y, None
    if k in ("csr", "pcsr"):
        w = _randn(_gen(seed, 0), d)
        X, y = _csr_rows(_gen(seed, 1), case["n"] if k == "csr" else
                         case["nsv"], d, case["nnz"], w)
        Xt, _ = _csr_rows(_gen(seed, 2), m, d, case["nnz"], w)
        return X, y, Xt
    X, y = _svc_rows(_gen(seed, 1), case["nsv"], d)
    return X, y, _svc_rows(_gen(seed, 2), m, d)[0]


def _given_model(case, seed):
    # labels alternate, and a pair has the same coefficient, so y'a = 0;
    # three in ten pairs are at the bound C = 1
    nsv = case["nsv"]
    g = _gen(seed, 3)
    a = 0.05 + 0.9 * _rand(g, nsv // 2).double()
    a[_rand(g, nsv // 2) < 0.3] = 1.0
    a = a.repeat_interleave(2)
    y = torch.ones(nsv, device=DEV)
    y[1::2] = -1.0
    return a, y


def _params(case):
    kern = case.get("kernel", "rbf")
    p = dict(kernel=KERNELS[kern])
    if kern == "poly":
        p.update(coef0=1.0, degree=3)
    if kern == "sigmoid":
        p.update(gamma=0.25 / case["d"])
    if case["kind"] in ("csr", "pcsr"):
        p.update(gamma=0.05)
    if case["kind"] == "ovr":
        p.update(C=10.0, gamma=0.02)
    if case.get("task") == "svr":
        p.update(type=SVR, C=10.0, epsilon=0.1)
    return p


def prepare(case, seed):
    X, y, Xt = _inputs(case, seed)
    p = _params(case)
    k = case["kind"]
    if k in ("serve", "predict", "pcsr"):
        a, y = _given_model(case, seed)
        model = nv.svm_train(X, y, alpha0=a.cpu().numpy(), tol=1e6, C=1.0,
                             **p)
        out = None
        if k == "serve":
            out = torch.empty((case["m"], 1), dtype=torch.float64, device=DEV)
        return dict(case=case, model=model, Xt=Xt, out=out)
    if case.get("host"):
        X, y, Xt = X.cpu().numpy(), y.cpu().numpy(), Xt.cpu().numpy()
    if k == "cv":
        y = y.cpu().numpy()
    return dict(case=case, X=X, y=y, Xt=Xt, params=p)


def run(state):
    case = state["case"]
    k = case["kind"]
    if k == "serve":
        return nv.svm_predict_noalloc(state["model"], state["Xt"],
                                      out=state["out"])
    if k in ("predict", "pcsr"):
        return nv.svm_predict(state["model"], state["Xt"])
    p = state["params"]
    if k == "cv":
        D, st = nv.svm_cross_validate(state["X"], y=state["y"],
                                      k=case["folds"],
                                      lockstep=case["lockstep"], **p)
        return {"decision": D, "accuracy": st["accuracy"]}
    if k == "ovr":
        model = nv.svm_train_ovr(state["X"], state["y"], 10, **p)
    else:
        model = nv.svm_train(state["X"], state["y"], **p)
    n_out = 10 if k == "ovr" else 1
    alpha, scalars = [], []
    for c in range(n_out):
        info = model.info(c)
        scalars.append([info["b"], info["dual_obj"]])
        alpha.append(nv.svm_model_get(model, c, with_alpha=True)[2])
    return {"decision": nv.svm_predict(model, state["Xt"]),
            "alpha": np.stack(alpha), "b_obj": np.array(scalars)}


# ----------------------------------------------------------------- floors

def work(case):
    """Inputs read once, outputs written once; the kernel values that no
    method does without: a training needs the row of every support vector
    against all samples once (their share of n is the problem's, as measured:
    3 to 90 in 100), a prediction every support vector against every point."""
    k, d, m = case["kind"], case["d"], case.get("m", 0)
    per = 2.0 * (case["nnz"] if k in ("csr", "pcsr") else d)  # flops a value
    row = 8.0 * case["nnz"] + 8 if k in ("csr", "pcsr") else 4.0 * d
    if k in ("serve", "predict", "pcsr"):
        nsv = case["nsv"]
        return {"bytes": row * (m + nsv) + 8.0 * (nsv + m),
                "flops": per * m * nsv}
    n = case["n"]
    share = {"train": 0.06, "csr": 0.4, "ovr": 0.005, "cv": 0.08}[k]
    if case.get("task") == "svr":
        share = 0.6
    if k == "ovr":
        return {"bytes": row * (n + m) + 84.0 * n + 80.0 * m,
                "flops": per * 10 * share * n * (n + m)}
    if k == "cv":
        return {"bytes": row * n + 12.0 * n,
                "flops": per * share * n * n * case["folds"]}
    return {"bytes": row * (n + m) + 12.0 * n + 8.0 * m,
            "flops": per * share * n * (n + m)}


def tolerance(case):
    # predicting: fp32 kernel values of an fp32 dot product, fp64 sums (5e-7
    # to 1.4e-6 from 64 bits)
    if case["kind"] in ("serve", "predict", "pcsr"):
        return {"rel": 6e-6, "max": 1e-4}
    # training stops when the optimality gap is at most 1e-3, so two correct
    # runs (working sets of 16 and of 20) differ by 2e-4 in the decision
    # values and by up to 0.01 (0.4 in a single value) in alpha
    return {"rel": 0.03, "max": 0.9}


# ------------------------------------------------------------------ exact

def _kernel64(case, A, B):
    p = _params(case)
    g = p.get("gamma", 0.0) or 1.0 / case["d"]
    kern = case.get("kernel", "rbf")
    dot = A @ B.T
    if kern == "rbf":
        s = (A * A).sum(1)[:, None] + (B * B).sum(1)[None, :] - 2 * dot
        return torch.exp(-g * s.clamp_(min=0))
    if kern == "poly":
        return (g * dot + p["coef0"]) ** p["degree"]
    if kern == "sigmoid":
        return torch.tanh(g * dot)
    return dot


def _predict64(case, seed):
    X, _, Xt = _inputs(case, seed)
    if case["kind"] == "pcsr":
        X, Xt = X.to_dense(), Xt.to_dense()
    X, Xt = X.double(), Xt.double()
    a, y = _given_model(case, seed)
    y = y.double()
    c = a * y
    free = a < 1.0  # the bias: the mean over the free variables
    f = torch.cat([_kernel64(case, X[i:i + 4096], X) @ c
                   for i in range(0, len(X), 4096)])
    b = (y - f)[free].mean()
    D = torch.cat([_kernel64(case, Xt[i:i + 4096], X) @ c + b
                   for i in range(0, len(Xt), 4096)])
    return D[:, None] if case["kind"] == "serve" else D


def _smo64(K, y, p, C, tol=1e-6, most=400000):
    """Two-variable descent with second-order choice of the second one, in
    64 bits; -> (alpha, bias, objective).  Variable t belongs to row t mod n
    of K."""
    n, N = K.shape[0], len(y)
    a, v = np.zeros(N), -y * p          # v = -y * gradient
    smp = np.arange(N) % n
    diag = K[np.arange(n), np.arange(n)][smp]
    up, low = y > 0, y < 0
    reps = N // n
    for _ in range(most):
        i = int(np.argmax(np.where(up, v, -np.inf)))
        Ki = np.tile(K[smp[i]], reps)
        d = v[i] - v
        ok = low & (d > 0)
        if not ok.any() or d[ok].max() <= tol:
            break
        eta = np.maximum(diag[i] + diag - 2 * Ki, 1e-12)
        j = int(np.argmax(np.where(ok, d * d / eta, -np.inf)))
        t = d[j] / eta[j]
        t = min(t, C - a[i] if y[i] > 0 else a[i],
                a[j] if y[j] > 0 else C - a[j])
        for s, w in ((i, t), (j, -t)):
            a[s] += y[s] * w
            if a[s] < 1e-13 * C:
                a[s] = 0.0
            elif a[s] > C * (1 - 1e-13):
                a[s] = C
            up[s] = a[s] < C if y[s] > 0 else a[s] > 0
            low[s] = a[s] > 0 if y[s] > 0 else a[s] < C
        v -= t * (Ki - np.tile(K[smp[j]], reps))
    free = (a > 0) & (a < C)
    b = v[free].mean() if free.any() else 0.5 * (v[up].max() + v[low].min())
    return a, b, 0.5 * (a * (p - y * v)).sum()


def exact(case, seed):
    k = case["kind"]
    if k in ("serve", "predict", "pcsr"):
        return _predict64(case, seed)
    if k != "train" or case["n"] > 2500 or case["task"] != "svc" \
            or case["kernel"] != "rbf":
        return None
    X, y, Xt = _inputs(case, seed)
    X, Xt = X.double(), Xt.double()
    K = _kernel64(case, X, X)
    yn = y.double().cpu().numpy()
    a, b, obj = _smo64(K.cpu().numpy(), yn, -np.ones(len(yn)), 1.0)
    D = _kernel64(case, Xt, X) @ torch.as_tensor(a * yn, device=X.device) + b
    return {"decision": D, "alpha": a[None, :], "b_obj": np.array([[b, obj]])}
