"""The register-resident inner loop with one chain wave: its fused gamma against the fixed order of
roundings, bit for bit the oracle."""
import numpy as np
import pytest

import paper_1803_03383_amd as hp
from oracle import ref
from test_gpu_parity import _inner_case, _oracle_inner, _run_inner

pytestmark = pytest.mark.gpu

# Seeds (of chain 0) whose rounding draw of gamma at step 0 of epoch 3 lies within 2^-24 of 0 or 1, found by
# search.  z = 0 there, so that gamma = floor(rho) and the window is done again in the fixed order.
NEAR = {22397602: 0xFFFFFF64, 41644664: 0x5C, 44213804: 0x49, 59438199: 0xFFFFFFE1}


def _check(case, loss, d, b, lam, T, seed, alpha, mu, helpers):
    P = _run_inner(case, loss, 1, 1, b, lam, 1, T, seed, 2, alpha=alpha, mu=mu)
    P.h.set_option(hp.OPT_INNER_HELPERS, helpers)
    P.h.inner_loop(3)
    out = _oracle_inner(case, 0, T)
    assert np.array_equal(P.get("z")[0].astype(np.int32), out["z"])
    assert np.array_equal(P.get("counters")[0].astype(np.uint64), out["counters"])
    return out


@pytest.mark.parametrize("seed", sorted(NEAR))
@pytest.mark.parametrize("loss,d,lam", [(hp.LOSS_SQUARED, 40, 0.0), (hp.LOSS_SQUARED, 200, 0.0),
                                        (hp.LOSS_LOGISTIC, 500, 0.0), (hp.LOSS_SQUARED, 1000, 5e-2)])
def test_a_fraction_next_to_an_integer_is_settled_in_the_fixed_order(loss, d, lam, seed):
    assert ref.stream_word(seed, 1, 3, 0) == NEAR[seed]
    case = _inner_case(loss, 60, d, 1, 1, 8, lam, 1, 29, seed - 1000, mu=0.2)
    _check(case, loss, d, 8, lam, 29, seed - 1000, 0.02, 0.2, 3)


@pytest.mark.parametrize("loss,d,alpha,mu", [
    (hp.LOSS_SQUARED, 60, 50.0, 0.01),     # gammas far outside their range
    (hp.LOSS_SQUARED, 512, 500.0, 0.01),   # scales too large for the matrix instruction's sum: no step is fused
    (hp.LOSS_SQUARED, 1000, 500.0, 1e-4),
    (hp.LOSS_LOGISTIC, 130, 500.0, 0.01),
    (hp.LOSS_SQUARED, 130, 0.9, 2.0),      # -h~ / 2^b too large to ride in the records
    (hp.LOSS_SQUARED, 1000, 0.9, 8.0),
])
def test_steps_that_the_fused_form_does_not_cover(loss, d, alpha, mu):
    case = _inner_case(loss, 60, d, 1, 1, 8, 0.0, 1, 67, 7, alpha=alpha, mu=mu)
    out = _check(case, loss, d, 8, 0.0, 67, 7, alpha, mu, 3)
    if alpha >= 50 and loss == hp.LOSS_SQUARED:
        assert out["counters"][1] > 0
