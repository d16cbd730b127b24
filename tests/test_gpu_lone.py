"""The register-resident inner loop with one chain wave: its fused gamma against the fixed order of
roundings, bit for bit the oracle."""
import numpy as np
import pytest

import paper_1803_03383_amd as hp
import test_gpu_svrg
from gpu_util import GpuProblem
from oracle import ref
from test_gpu_lpsvrg import _lp_case
from test_gpu_parity import _inner_case, _oracle_inner, _run_inner

pytestmark = pytest.mark.gpu

# Seeds (of chain 0) whose rounding draw of gamma at step 0 of epoch 3 lies within 2^-24 of 0 or 1, found by
# search.  z = 0 there, so that gamma = floor(rho) and the window is done again in the fixed order.
NEAR = {22397602: 0xFFFFFF64, 41644664: 0x5C, 44213804: 0x49, 59438199: 0xFFFFFFE1}


def _check(case, loss, d, b, lam, R, T, seed, alpha, mu):
    P = _run_inner(case, loss, 1, 1, b, lam, R, T, seed, 2, alpha=alpha, mu=mu)
    if b == 8:
        P.h.set_option(hp.OPT_INNER_HELPERS, 3)  # (at 16 bits the library takes the form for few chains)
    P.h.inner_loop(3)
    z, w, cnt = P.get("z"), P.get("w"), P.get("counters")
    for r in range(R):
        out = _oracle_inner(case, r, T)
        assert np.array_equal(z[r].astype(np.int32), out["z"])
        assert np.array_equal(w[r], ref.apply_offset(case["mk"](r), case["scales"][r], out["z"], case["w"][r]))
        assert np.array_equal(cnt[r].astype(np.uint64), out["counters"])
    return out


@pytest.mark.parametrize("seed", sorted(NEAR))
@pytest.mark.parametrize("loss,d,b,lam", [
    (hp.LOSS_SQUARED, 40, 8, 0.0), (hp.LOSS_SQUARED, 200, 8, 0.0), (hp.LOSS_LOGISTIC, 500, 8, 0.0),
    (hp.LOSS_SQUARED, 1000, 8, 5e-2), (hp.LOSS_SQUARED, 64, 16, 0.0), (hp.LOSS_SQUARED, 300, 16, 1e-3),
])
def test_a_fraction_next_to_an_integer_is_settled_in_the_fixed_order(loss, d, b, lam, seed):
    assert ref.stream_word(seed, 1, 3, 0) == NEAR[seed]
    case = _inner_case(loss, 60, d, 1, 1, b, lam, 1, 29, seed - 1000, mu=0.2)
    _check(case, loss, d, b, lam, 1, 29, seed - 1000, 0.02, 0.2)


@pytest.mark.parametrize("loss,d,b,alpha,mu", [
    (hp.LOSS_SQUARED, 60, 8, 50.0, 0.01),      # gammas far outside their range
    (hp.LOSS_SQUARED, 512, 8, 500.0, 0.01),    # too large for the matrix instruction to do the multiply-add
    (hp.LOSS_SQUARED, 1000, 8, 500.0, 1e-4),
    (hp.LOSS_LOGISTIC, 130, 8, 500.0, 0.01),
    (hp.LOSS_SQUARED, 130, 8, 0.9, 2.0),       # -h~ / 2^b too large to ride in the records
    (hp.LOSS_SQUARED, 1000, 8, 0.9, 8.0),
    (hp.LOSS_SQUARED, 60, 16, 500.0, 0.01),
    (hp.LOSS_SQUARED, 500, 16, 500.0, 0.01),
    (hp.LOSS_LOGISTIC, 100, 16, 500.0, 0.01),
    (hp.LOSS_SQUARED, 64, 16, 0.9, 2.0),
    (hp.LOSS_SQUARED, 512, 16, 0.9, 8.0),
    (hp.LOSS_SQUARED, 130, 16, 1e-230, 1e-230),  # scales next to underflow: no step is fused
    (hp.LOSS_SQUARED, 130, 8, 1e-230, 1e-230),
])
def test_scales_at_the_ends_of_the_fused_form(loss, d, b, alpha, mu):
    case = _inner_case(loss, 60, d, 1, 1, b, 0.0, 1, 67, 7, alpha=alpha, mu=mu)
    out = _check(case, loss, d, b, 0.0, 1, 67, 7, alpha, mu)
    if alpha >= 50 and loss == hp.LOSS_SQUARED:
        assert out["counters"][1] > 0


@pytest.mark.parametrize("loss,d,lam,T", [
    (hp.LOSS_SQUARED, 1, 0.0, 40), (hp.LOSS_SQUARED, 63, 0.0, 8), (hp.LOSS_LOGISTIC, 64, 1e-3, 513),
    (hp.LOSS_SQUARED, 65, 0.0, 17), (hp.LOSS_SQUARED, 128, 1e-3, 264), (hp.LOSS_LOGISTIC, 129, 0.0, 16),
    (hp.LOSS_SQUARED, 256, 0.0, 257), (hp.LOSS_SQUARED, 257, 1e-3, 24), (hp.LOSS_SQUARED, 511, 0.0, 300),
    (hp.LOSS_LOGISTIC, 512, 0.0, 33), (hp.LOSS_SQUARED, 512, 0.0, 7), (hp.LOSS_SQUARED, 300, 0.0, 0),
])
@pytest.mark.parametrize("mu", [0.2, 300.0])
def test_sixteen_bits_one_to_eight_strips_per_lane(loss, d, lam, T, mu):
    """1, 2, 4 and 8 strips per lane, whole and ragged rows, L2 draws, epochs around windows and batches; the
    box far too small, so that z saturates and -h~ does not ride in the records."""
    case = _inner_case(loss, 90, d, 1, 1, 16, lam, 2, T, 5 + d + T, mu=mu)
    _check(case, loss, d, 16, lam, 2, T, 5 + d + T, 0.02, mu)


@pytest.mark.parametrize("loss,d,lam,R,T", [
    (hp.LOSS_SQUARED, 3, 0.0, 1, 9), (hp.LOSS_SQUARED, 255, 1e-3, 2, 264), (hp.LOSS_LOGISTIC, 256, 0.0, 1, 16),
    (hp.LOSS_SQUARED, 257, 0.0, 1, 513), (hp.LOSS_LOGISTIC, 511, 1e-3, 2, 31), (hp.LOSS_SQUARED, 512, 1e-2, 1, 257),
    (hp.LOSS_SQUARED, 513, 0.0, 2, 24), (hp.LOSS_LOGISTIC, 1000, 0.0, 1, 40), (hp.LOSS_SQUARED, 1024, 1e-3, 1, 25),
    (hp.LOSS_SQUARED, 30, 0.0, 300, 70), (hp.LOSS_LOGISTIC, 300, 1e-3, 260, 20),  # more chains than CUs
])
def test_full_precision_chain_wave(loss, d, lam, R, T):
    """One, two and four float4s per lane, whole and ragged rows, the L2 term, epochs around windows and batches."""
    test_gpu_svrg.test_inner_loop_matches_the_oracle(loss, 120, d, lam, R, T, 0)


@pytest.mark.parametrize("d,b", [(1024, 8), (512, 16)])
def test_more_than_two_to_the_32_clamped_coordinates(d, b):
    """Rows of zeros and an offset that pushes every coordinate out of the box in every step: d T clamps."""
    T = 2 ** 32 // d + 21
    P = GpuProblem(np.zeros((1, 4, d), np.float32), np.zeros((1, 4, d), np.int8), np.zeros((1, 4), np.float32),
                   b=b, T=T, alpha=0.02, mu=0.2, delta_d=1.0, seed=5)
    lowest = -2 ** (b - 1)
    P.put("z", np.full((1, 1, d), lowest))
    P.put("h", np.full((1, 1, d), 2 ** (2 * b - 1) - 1 if b == 8 else 2 ** 30))
    P.put("scales", np.full((1, 8), 1.0) * (np.arange(8) < 6))
    P.h.inner_loop(3)
    assert (P.get("z") == lowest).all()
    assert P.get("counters")[0].tolist() == [T * d, 0, 0, 0]


@pytest.mark.parametrize("loss,d,b", [
    (hp.LOSS_SQUARED, 40, 8), (hp.LOSS_SQUARED, 200, 8), (hp.LOSS_LOGISTIC, 500, 8), (hp.LOSS_SQUARED, 1000, 8),
    (hp.LOSS_SQUARED, 64, 16), (hp.LOSS_LOGISTIC, 120, 16), (hp.LOSS_SQUARED, 256, 16), (hp.LOSS_SQUARED, 500, 16),
])
@pytest.mark.parametrize("draw", [0.4, 1.0, 1.1, 10.0])
@pytest.mark.parametrize("inside", [True, False])
def test_l2_draws_at_the_edges_of_the_words(loss, d, b, draw, inside):
    """Every term of the update at its largest: rows of +-q_max and -2^(b-1), z at the ends of its box, gamma clamped,
    draws just below and above 32 (16 bits: 4096), where the fused steps end, and far above; high parts of -h~ at the
    ends of what rides in the records, and one past them."""
    N, T, seed = 40, 261, 11
    rng = np.random.default_rng(seed + d)
    q, largest = 2 ** (b - 1) - 1, 32 if b == 8 else 4096
    X = rng.choice(np.array([-1.0, 1.0], np.float32), size=(N, d))
    y = (X @ rng.standard_normal(d).astype(np.float32) * 50.0).astype(np.float32)
    if loss == hp.LOSS_LOGISTIC:
        y = np.where(y >= 0, 1.0, -1.0).astype(np.float32)
    Xq = ref.quantize_data(X, 1.0 / q, b)
    Xq[rng.random((N, d)) < 0.1] = -q - 1
    alpha, mu = 0.5, 2000.0
    lam = (draw * largest - 0.25) / (alpha * 2 ** b)
    prob = ref.make_problem(N, d, loss=loss, b=b, alpha=alpha, mu=mu, lam=lam, delta_d=1.0 / q, seed=seed)
    w = (rng.standard_normal((1, d)) * 3.0).astype(np.float32)
    phi, g, _ = ref.full_gradient(prob, X, y, w)
    phi = phi.astype(np.float32)
    sc, h, _ = ref.recenter(prob, g.astype(np.float32), 3)
    lo, hi = (-48, 46) if b == 8 else (-14000, 14000)
    hh = rng.choice([lo, lo, hi, hi, 0], size=d)
    if not inside:
        hh[rng.integers(d)] = rng.choice([lo - 1, hi + 1])
    h = -(hh * 2 ** b + rng.choice([0, 2 ** b - 1], size=d)).reshape(np.shape(h)).astype(np.asarray(h).dtype)
    out = ref.inner_loop(prob, Xq, phi, y, h, sc, 3, T)
    assert out["counters"][0] > 0 and (loss == hp.LOSS_LOGISTIC or out["counters"][1] > 0)
    assert out["counters"][2] == T
    P = GpuProblem(X, Xq, y, loss=loss, b=b, T=T, alpha=alpha, mu=mu, lam=lam, delta_d=1.0 / q, seed=seed, w0=w)
    P.put("phi", phi); P.put("h", h); P.put("scales", sc)
    P.h.set_option(hp.OPT_INNER_VARIANT, 2)
    if b == 8:
        P.h.set_option(hp.OPT_INNER_HELPERS, 3)
    P.h.inner_loop(3)
    assert np.array_equal(P.get("z")[0].astype(np.int32), out["z"])
    assert np.array_equal(P.get("counters")[0].astype(np.uint64), out["counters"])


@pytest.mark.parametrize("loss,d,b,lam", [
    (hp.LOSS_SQUARED, 64, 16, 0.0), (hp.LOSS_LOGISTIC, 50, 16, 1e-3),     # one strip per lane
    (hp.LOSS_SQUARED, 100, 16, 1e-3), (hp.LOSS_LOGISTIC, 128, 16, 0.0),   # two
    (hp.LOSS_SQUARED, 256, 16, 0.0), (hp.LOSS_LOGISTIC, 200, 16, 1e-3),   # four
    (hp.LOSS_LOGISTIC, 60, 8, 5e-2), (hp.LOSS_SQUARED, 100, 8, 5e-2),     # rows in 16 lanes; two strips
    (hp.LOSS_LOGISTIC, 256, 8, 0.0), (hp.LOSS_LOGISTIC, 512, 8, 5e-2),    # two, four
])
@pytest.mark.parametrize("lp", [False, True])
def test_more_chains_than_cus(loss, d, b, lam, lp):
    """The builds held to 128 registers, over shared data, the library's choice at 300 chains: every chain against one
    wave per chain, chains around the count of CUs against the oracle."""
    N, T, R, seed, alpha, delta = 100, 61, 300, 19, 0.02, 2.0 ** (-6 if b == 8 else -13)
    if lp:
        case = _lp_case(loss, N, d, 1, 1, b, 1, seed, alpha, delta)
        lam = 0.0
    else:
        case = _inner_case(loss, N, d, 1, 1, b, lam, 1, T, seed, mu=0.2)
    mk = lambda r: ref.make_problem(N, d, loss=loss, b=b, alpha=alpha, mu=0.2, lam=lam, delta_d=case["dd"], seed=900 + r,
                                    algorithm=ref.ALG_LPSVRG if lp else ref.ALG_HALP, delta=delta if lp else 0.0)
    X, Xq, y, phi, w = (case[k][0] for k in ("X", "Xq", "y", "phi", "w"))
    h, sc = case["h"][0], case["scales"][0]
    z0 = case["z"][0] if lp else np.zeros((1, d), np.int32)
    res = []
    for helpers in (0, 2):  # 2: no helper waves, i.e. not this form
        P = GpuProblem(X, Xq, y, R=R, loss=loss, b=b, T=T, alpha=alpha, mu=0.2, lam=lam, delta_d=case["dd"], seed=900,
                       share_data=True, w0=np.repeat(w[None], R, axis=0),
                       algorithm=hp.ALG_LPSVRG if lp else hp.ALG_HALP, delta=delta if lp else 0.0)
        for name, v in (("phi", phi), ("h", h), ("scales", sc), ("z", z0)):
            P.put(name, np.repeat(np.asarray(v)[None], R, axis=0))
        P.h.set_option(hp.OPT_INNER_HELPERS, helpers)
        P.h.inner_loop(3)
        res.append([P.get(k).copy() for k in ("z", "w", "counters")])
    for a, c in zip(*res):
        assert np.array_equal(a, c)
    for r in (0, 255, 256, R - 1):
        out = ref.inner_loop(mk(r), Xq, phi, y, h, sc, 3, T, z0=z0)
        assert np.array_equal(res[0][0][r].astype(np.int32), out["z"]), f"chain {r}"
        assert np.array_equal(res[0][2][r].astype(np.uint64), out["counters"])
