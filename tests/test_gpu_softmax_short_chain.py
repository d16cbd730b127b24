"""The short chain from x^T z to the gammas of a softmax step against the oracle, bit for bit, at the ends of the
bounds inside which it stands for the fixed order of roundings.  Each case is shown to leave them, by the oracle's trace."""
import numpy as np
import pytest

import paper_1803_03383_amd as hp
from gpu_util import GpuProblem
from oracle import ref
from test_gpu_parity import _inner_case

pytestmark = pytest.mark.gpu

SHAPES = [
    # N, d, K, B, b, T, seeds with which a fraction comes that close (searched for): each kernel that has the short chain
    (60, 100, 9, 1, 8, 700, (10, 17)),       # a row of z to a wave
    (60, 150, 10, 1, 16, 700, (5, 1)),
    (60, 100, 5, 8, 8, 200, (3, 1)),       # minibatches on the matrix cores
    (90, 64, 2, 130, 8, 40, (3, 4)),       # ... in chunks, two classes
    (90, 70, 11, 200, 8, 9, (2, 6)),       # ... four classes to a lane
    (50, 1100, 7, 1, 8, 300, (111, 10)),      # rows cut across workgroups
    (50, 1100, 6, 1, 16, 300, (25, 41)),
]
EPOCH = 3


@pytest.mark.parametrize("N,d,K,B,b,T,seeds", SHAPES)
@pytest.mark.parametrize("lp", [False, True])
@pytest.mark.parametrize("kind", ["near", "k2", "phi", "delta", "sum"])
def test_a_step_outside_the_bounds_is_done_in_the_fixed_order(N, d, K, B, b, T, seeds, lp, kind):
    loss, alpha, seed = hp.LOSS_SOFTMAX, 0.02, seeds[lp]
    T = T if kind == "near" else min(T, 40)
    rng = np.random.default_rng(seed)
    case = _inner_case(loss, N, d, K, B, b, 0.0, 1, T, seed, alpha=alpha, mu=0.05)
    Xq, y, h = case["Xq"][0], case["y"][0], case["h"][0]
    top = 100 if b == 8 else 20000
    z0 = rng.integers(-top, top + 1, size=(K, d)).astype(np.int32)
    D = Xq.astype(np.int64) @ z0.T.astype(np.int64)
    sc = case["scales"][0].copy()
    sc[0] = {"delta": 60.0, "sum": 6.0}.get(kind, 1.0) / (np.std(D) * case["dd"])  # of the margins' moves
    sc[5] = 2.0 ** (22 if kind == "k2" else 9) / (alpha / B)                        # (alpha / B) / delta_s
    moved = (case["dd"] * sc[0]) * D
    phi = rng.normal(0.0, 8.0 if kind == "sum" else 2.0, size=(N, K))
    if kind == "phi":
        phi[::3] *= 1500.0
    if lp:  # the margins are x^T w; phi is what they were measured from
        phi, start = moved + (moved if kind in ("delta", "sum") else 0.3 * phi), phi
        if kind == "phi":
            phi = phi + np.where(np.abs(start) > 1000.0, start, 0.0)
    phi = phi.astype(np.float32)
    prob = ref.make_problem(N, d, K=K, loss=loss, b=b, B=B, alpha=alpha, mu=0.05, delta_d=case["dd"], seed=77 + seed,
                            algorithm=ref.ALG_LPSVRG if lp else ref.ALG_HALP, delta=sc[0] if lp else 0.0)
    out = ref.inner_loop(prob, Xq, phi, y, h, sc, EPOCH, T, z0=z0, trace_steps=T, trace_z=False)

    ph = phi[out["idx"]].astype(np.float64)
    delta = (case["dd"] * sc[0]) * out["D"] - (ph if lp else 0.0)
    p0 = np.exp(ph - ph.max(-1, keepdims=True))
    p0 /= p0.sum(-1, keepdims=True)
    within = np.abs(delta).max(-1) <= 64.0
    if kind == "near":
        words = np.array([ref.stream_word(77 + seed, 1, EPOCH, n) for n in range(out["beta"].size)], np.float64)
        t = out["beta"] * sc[5] + words.reshape(out["beta"].shape) * 2.0 ** -32
        assert within.all() and (np.abs(t - np.rint(t)) < 2.0 ** -17).any()
    elif kind == "k2":
        assert alpha / B * sc[5] >= 2.0 ** 21
    elif kind == "phi":
        assert (np.abs(ph) > 1024.0).any()
    elif kind == "delta":
        assert not within.all()
    else:
        with np.errstate(over="ignore"):
            s = (p0 * np.exp(delta)).sum(-1)
        assert (within & (s <= 1 / 16)).any()

    P = GpuProblem(case["X"], case["Xq"], case["y"], K=K, loss=loss, b=b, B=B, T=T, alpha=alpha, mu=0.05,
                   delta_d=case["dd"], seed=77 + seed, w0=case["w"],
                   algorithm=hp.ALG_LPSVRG if lp else hp.ALG_HALP, delta=sc[0] if lp else 0.0)
    P.put("phi", phi); P.put("h", h); P.put("scales", sc); P.put("z", z0)
    P.h.inner_loop(EPOCH)
    assert P.h.get_stats(0).inner_variant == (1 if d > 1024 else 2)  # cut across workgroups in the general one's place
    assert np.array_equal(P.get("z")[0].astype(np.int32), out["z"])
    assert np.array_equal(P.get("counters")[0].astype(np.uint64), out["counters"])
