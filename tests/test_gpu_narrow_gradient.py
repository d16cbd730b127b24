"""The gradient pass on narrow rows: one workgroup per chain and several, every count of lanes per row, against the
oracle."""
import numpy as np
import pytest

import halp_inputs as inp
import paper_1803_03383_amd as hp
from gpu_util import GpuProblem, rel_l2
from oracle import ref

pytestmark = pytest.mark.gpu

TOL = 1e-5  # rel-L2 of fp32 sums, as in test_gpu_parity.py


@pytest.mark.parametrize("loss,N,d,R,lam", [
    (hp.LOSS_SQUARED, 1, 3, 300, 1e-3), (hp.LOSS_LOGISTIC, 129, 100, 300, 1e-3),  # a chain per CU and more
    (hp.LOSS_SQUARED, 700, 64, 70, 0.0),                                          # 64 chains and more
    (hp.LOSS_SQUARED, 1024, 64, 1, 1e-3), (hp.LOSS_SQUARED, 1025, 64, 2, 1e-3),   # the edge for few chains
    (hp.LOSS_LOGISTIC, 512, 64, 1, 0.0), (hp.LOSS_LOGISTIC, 513, 64, 1, 1e-3),
    (hp.LOSS_SQUARED, 20001, 7, 1, 0.0), (hp.LOSS_LOGISTIC, 9001, 30, 2, 1e-4),   # 4, 8, 16, 32 lanes per row
    (hp.LOSS_SQUARED, 40003, 63, 1, 0.0), (hp.LOSS_LOGISTIC, 3001, 127, 3, 0.0),
])
def test_narrow_rows(loss, N, d, R, lam):
    gen = inp.logistic if loss == hp.LOSS_LOGISTIC else inp.linreg
    Rd = min(R, 3)
    data = [gen(N, d, seed=r) for r in range(Rd)]
    X = np.stack([data[r % Rd][0] for r in range(R)]).astype(np.float32)
    y = np.stack([data[r % Rd][1] for r in range(R)]).astype(np.float32)
    w = (0.3 * np.random.default_rng(1).standard_normal((R, 1, d))).astype(np.float32)
    P = GpuProblem(X, None, y, R=R, loss=loss, lam=lam, w0=w)
    P.h.full_gradient()
    phi, g, sc = P.get("phi"), P.get("g"), P.get("scales")
    for r in sorted({0, 1 % R, R // 2, R - 1}):
        prob = ref.make_problem(N, d, loss=loss, lam=lam)
        phi_r, g_r, f_r = ref.full_gradient(prob, X[r], y[r], w[r])
        assert rel_l2(phi[r].ravel(), np.asarray(phi_r).ravel()) <= TOL
        assert rel_l2(g[r].ravel(), np.asarray(g_r).ravel()) <= TOL
        assert abs(sc[r, 6] - f_r) <= TOL * max(1.0, abs(f_r))
