"""Inner loop of one row per step with eight and sixteen waves to a chain: bit for bit the oracle, past the step-indexed
draws' first refills, with L2 draws and with the margins of the sampled rows."""
import numpy as np
import pytest

import paper_1803_03383_amd as hp
from oracle import ref
from test_gpu_lpsvrg import _lp_case, _problem
from test_gpu_parity import _inner_case, _run_inner

pytestmark = pytest.mark.gpu

CASES = [
    # loss, N, d, b, lam, R, T, mu, waves asked for
    (hp.LOSS_LOGISTIC, 90, 4096, 16, 5e-2, 1, 530, 0.05, 0),   # eight waves of eight strips
    (hp.LOSS_LOGISTIC, 90, 2100, 16, 1e-3, 2, 271, 500.0, 0),  # ... of eight, the last waves empty; saturating
    (hp.LOSS_LOGISTIC, 60, 8000, 8, 5e-2, 1, 530, 0.05, 0),
    (hp.LOSS_LOGISTIC, 60, 3000, 8, 5e-2, 2, 270, 0.05, 16),   # sixteen waves of four strips
    (hp.LOSS_SQUARED, 60, 3001, 8, 5e-2, 1, 270, 0.05, 8),     # eight
    (hp.LOSS_SQUARED, 60, 5000, 8, 5e-2, 1, 100, 500.0, 0),
    (hp.LOSS_LOGISTIC, 40, 8000, 16, 5e-2, 1, 300, 0.05, 0),   # sixteen waves of eight strips
    (hp.LOSS_SQUARED, 40, 7992, 16, 5e-2, 1, 530, 0.05, 0),    # ... few chains with L2 draws
    (hp.LOSS_SQUARED, 40, 8192, 16, 1e-3, 2, 41, 500.0, 0),    # ... saturating
    (hp.LOSS_SQUARED, 40, 4104, 16, 5e-2, 130, 21, 0.05, 0),   # ... more chains
    (hp.LOSS_SQUARED, 40, 8000, 16, 0.0, 1, 270, 0.05, 0),
]


@pytest.mark.parametrize("loss,N,d,b,lam,R,T,mu,waves", CASES)
def test_wide_rows_bit_exact(loss, N, d, b, lam, R, T, mu, waves):
    seed = 810 + d + T
    case = _inner_case(loss, N, d, 1, 1, b, lam, R, T, seed, mu=mu)
    P = _run_inner(case, loss, 1, 1, b, lam, R, T, seed, 2, mu=mu)
    P.h.set_option(hp.OPT_INNER_WAVES, waves)
    P.h.inner_loop(3)
    z, w, cnt = P.get("z"), P.get("w"), P.get("counters")
    for r in {0, R // 2, R - 1}:
        prob = case["mk"](r)
        out = ref.inner_loop(prob, case["Xq"][r], case["phi"][r], case["y"][r], case["h"][r], case["scales"][r], 3, T)
        assert np.array_equal(z[r].astype(np.int32), out["z"]), f"chain {r}"
        assert np.array_equal(w[r], ref.apply_offset(prob, case["scales"][r], out["z"], case["w"][r]))
        assert np.array_equal(cnt[r].astype(np.uint64), out["counters"])
    if lam > 1e-2:
        assert cnt[0, 2] > 0
    if mu > 100:
        assert cnt[0, 0] > 0


@pytest.mark.parametrize("loss", [hp.LOSS_SQUARED, hp.LOSS_LOGISTIC])
@pytest.mark.parametrize("d,b", [(8000, 8), (4096, 16), (8000, 16)])
def test_wide_rows_algorithm_2(loss, d, b):
    """The margin is x^T w alone, and squared loss takes the margins of the sampled rows too."""
    N, T, seed = 60, 270, 13
    case = _lp_case(loss, N, d, 1, 1, b, 1, seed, 0.02, 2.0 ** -7)
    P = _problem(case, loss, 1, 1, b, 1, T, seed, 0.02, 2.0 ** -7)
    P.put("phi", case["phi"]); P.put("h", case["h"]); P.put("scales", case["scales"]); P.put("z", case["z"])
    P.h.inner_loop(3)
    out = ref.inner_loop(case["mk"](0), case["Xq"][0], case["phi"][0], case["y"][0], case["h"][0], case["scales"][0],
                         3, T, z0=case["z"][0])
    assert np.array_equal(P.get("z")[0].astype(np.int32), out["z"])
    assert np.array_equal(P.get("counters")[0].astype(np.uint64), out["counters"])
