"""The selection's bound over large row counts, against the CPU oracle.

From 640 blocks of the row kernel (81,793 rows at 128 a block) on, and up to
16 working variables, the bound on the candidates comes from the maxima of
the selection's waves; below, from those of its 16-lane rows.  The working
set, its order and the gap are exact: random responses, the alpha = 0 start
where every key of a side ties, keys ordered so that one wave's records hold
all the best, and sides with fewer candidates than half a working set.
"""
import numpy as np
import pytest

import oracle
from oracle import C_SVC, EPS_SVR, Params
from paper_1706_05544_amd import native as nv

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [81792, 81793, 130001])
@pytest.mark.parametrize("type_", [C_SVC, EPS_SVR])
def test_select_many_blocks(n, type_):
    rng = np.random.default_rng(n)
    X = rng.standard_normal((n, 3), dtype=np.float32)
    y = (np.where(rng.random(n) < 0.5, 1.0, -1.0) if type_ == C_SVC
         else rng.integers(0, 2, n)).astype(np.float32)
    p = Params(type_, C=1.0, eps=0.1, gamma=0.5, tol=1e-3)
    N = oracle.num_vars(type_, n)
    mid = rng.choice([0.0, 0.5, 1.0], N)
    few = np.zeros(N)
    if type_ == C_SVC:
        few[y < 0] = 0.0
        few[y > 0] = 1.0  # no up side but the three below
        few[np.nonzero(y > 0)[0][[5, n // 3, n // 2 - 999]]] = 0.5
    states = [(mid, rng.standard_normal(n)),
              (np.zeros(N), np.zeros(n)),
              (mid, np.linspace(-3, 3, n)),
              (few, np.round(rng.standard_normal(n), 1))]
    for q in (2, 10, 16):
        s = nv.Solver(X, y, type=type_, C=1.0, epsilon=0.1, gamma=0.5,
                      tol=1e-3, working_set=q)
        for alpha, F in states:
            s.set_state(alpha, F)
            B, m, M = s.select()
            Be, me, Me = oracle.select(y, p, alpha, F, q, d=3)
            assert (m, M) == (me, Me)
            assert list(B) == list(Be)
