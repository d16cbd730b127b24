"""The 8-bit softmax inner loop of one row per step: bit for bit the oracle with h~ in the records and in two parts,
with records of bytes and of 16-bit halves, with and without a row wave."""
import numpy as np
import pytest

import paper_1803_03383_amd as hp
from oracle import ref
from test_gpu_parity import _inner_case, _run_inner

pytestmark = pytest.mark.gpu

CASES = [
    # d, K, lam, R, T, mu
    (784, 10, 1e-2, 2, 150, 0.05),   # records of 16-bit halves, eight strips per lane, lanes past the row; L2 draws
    (1023, 15, 0.0, 1, 60, 500.0),   # ... the service wave takes the rows; odd row; saturating
    (1024, 16, 1e-2, 1, 60, 0.05),   # ... two classes to a wave
    (515, 13, 0.0, 8, 40, 500.0),
    (515, 13, 1e-2, 9, 40, 0.05),    # records of bytes
    (900, 7, 1e-2, 2, 90, 500.0),
    (513, 16, 0.0, 9, 30, 0.05),
    (1024, 16, 1e-2, 5, 30, 500.0),  # ... records of bytes from five chains on
    (300, 15, 1e-2, 1, 70, 0.05),    # four strips per lane, no row wave
    (129, 4, 1e-2, 1, 70, 500.0),    # two
    (3, 2, 1e-2, 2, 70, 0.05),       # one strip per lane, the row in two lanes
    (1, 3, 0.0, 1, 9, 0.05),
    (100, 3, 1e-2, 1030, 9, 0.05),   # without a row wave, for more chains to a CU: every class wave fetches for itself
    (200, 7, 0.0, 600, 9, 500.0),    # ... two strips
    (300, 4, 1e-2, 800, 9, 0.05),    # ... the service wave for all, four strips
    (600, 3, 1e-2, 520, 17, 500.0),  # ... eight
]


@pytest.mark.parametrize("large", ["none", "last chain", "one class"])
@pytest.mark.parametrize("d,K,lam,R,T,mu", CASES)
def test_softmax_8bit_bit_exact(d, K, lam, R, T, mu, large):
    loss, N, b, seed = hp.LOSS_SOFTMAX, 50, 8, 330 + d + K
    case = _inner_case(loss, N, d, K, 1, b, lam, R, T, seed, mu=mu)
    if large != "none":  # the last chain's h~ over all of its 16 bits, or one class's; the others' up to what the records hold
        rng = np.random.default_rng(seed)
        for r in range(R):
            rows = slice(0, K if large == "last chain" else 1)
            h = rng.integers(-16000, 16000, size=case["h"][r].shape)
            h.flat[0] = -16000
            h.flat[-1] = 15999
            if r == R - 1:
                h[rows] = rng.integers(-32768, 32768, size=h[rows].shape)
                h[rows].flat[0] = -32768
                h[rows].flat[-1] = 32767
            case["h"][r] = h
    P = _run_inner(case, loss, K, 1, b, lam, R, T, seed, 2, mu=mu)
    P.h.inner_loop(3)
    z, w, cnt = P.get("z"), P.get("w"), P.get("counters")
    for r in range(R):
        prob = case["mk"](r)
        out = ref.inner_loop(prob, case["Xq"][r], case["phi"][r], case["y"][r], case["h"][r], case["scales"][r], 3, T)
        assert np.array_equal(z[r].astype(np.int32), out["z"]), f"chain {r}"
        assert np.array_equal(w[r], ref.apply_offset(prob, case["scales"][r], out["z"], case["w"][r]))
        assert np.array_equal(cnt[r].astype(np.uint64), out["counters"])
    if mu > 100 or (large != "none" and d * K > 16):
        assert cnt[R - 1, 0] > 0


def test_softmax_8bit_over_several_segments():
    """More steps than one segment's records hold: the loop starts again from the z that it handed out."""
    loss, N, d, K, b, T, seed = hp.LOSS_SOFTMAX, 60, 1000, 14, 8, 3000, 77
    case = _inner_case(loss, N, d, K, 1, b, 1e-3, 1, T, seed, mu=0.5)
    P = _run_inner(case, loss, K, 1, b, 1e-3, 1, T, seed, 2, mu=0.5)
    P.h.inner_loop(3)
    out = ref.inner_loop(case["mk"](0), case["Xq"][0], case["phi"][0], case["y"][0], case["h"][0], case["scales"][0], 3, T)
    assert np.array_equal(P.get("z")[0].astype(np.int32), out["z"])
    assert np.array_equal(P.get("counters")[0].astype(np.uint64), out["counters"])
