"""What a user of this library has it do, as a list of cases that can be timed and compared.

A case is one call through the public binding (paper_1803_03383_amd.Halp):

  epoch     one outer iteration from a given model: `w` is set to the model the epoch starts from,
            then Halp.epoch runs the gradient pass, bit centering and the T inner steps
  gradient  Halp.full_gradient alone: monitoring of f(w~) and ||g~||, the gradient of a shard
  quantize  Halp.quantize_data: the data set into its low-precision form, once per data set

listed() holds the repository's own configurations (the five of its baseline file, the
conditioning sweep, the ten-class ten-thousand-feature set, the gradient pass at an HBM-resident
row count); draw() gives further sizes of the same ranges, ragged ones and every option among
them.  Inputs are made on the GPU from the seed: Gaussian features for the linear models,
image-shaped features in [0,1] with 80 % zeros for softmax (dense Gaussian ones where rows are
wide), labels from a noisy random teacher.
"""
import math

import torch

import paper_1803_03383_amd as hp

LOSSES = {"squared": hp.LOSS_SQUARED, "logistic": hp.LOSS_LOGISTIC, "softmax": hp.LOSS_SOFTMAX}
ALGORITHMS = {"halp": hp.ALG_HALP, "lpsvrg": hp.ALG_LPSVRG, "svrg": hp.ALG_SVRG}
MODEL_SCALE = 4.0 / 127.0  # LP-SVRG's fixed lattice: teacher weights are N(0, 1)


def _case(call, loss, N, d, K=1, R=1, share=False, bits=8, B=1, T=0, algorithm="halp", alpha=0.1, mu=0.02,
          lam=0.0, grid=False, name=None):
    c = dict(call=call, loss=loss, N=N, d=d, K=K, R=R, share=share, bits=bits, B=B, T=T, algorithm=algorithm,
             alpha=alpha, mu=mu, lam=lam, grid=grid)
    return dict(c, name=name) if name else c


def listed():
    return [
        # the smallest call: gradient and loss of a 1000 x 64 least-squares problem, for a stopping rule
        _case("gradient", "squared", 1000, 64, name="gradient 1000x64"),
        # configuration 1: one short 8-bit chain, the latency of a step and of an epoch's launches
        _case("epoch", "squared", 1000, 64, T=2000, alpha=0.01, mu=1.0, name="epoch 1000x64 b8"),
        # configuration 2: one long 8-bit chain on wider rows, T = N
        _case("epoch", "squared", 100000, 1024, T=100000, alpha=1e-3, mu=0.3, name="epoch 100000x1024 b8"),
        # configuration 3: ten-class softmax on image-shaped data, T = N
        _case("epoch", "softmax", 60000, 784, K=10, T=60000, alpha=1e-2, mu=2.5, lam=1e-4,
              name="epoch 60000x784 K10 b8"),
        # the same data with 64 rows per step, one pass over them
        _case("epoch", "softmax", 60000, 784, K=10, B=64, T=938, alpha=1e-2, mu=2.5, lam=1e-4,
              name="epoch 60000x784 K10 b8 B64"),
        # configuration 4, the headline: 256 independent chains, each with its own data
        _case("epoch", "squared", 16384, 512, R=256, T=16384, name="epoch 256x16384x512 b8"),
        # full-precision SVRG on the same problems: the comparator a user measures against
        _case("epoch", "squared", 16384, 512, R=256, T=16384, algorithm="svrg", name="epoch 256x16384x512 svrg"),
        # configuration 5: binary logistic, 16 GB of data, 16 bits, 64 rows per step, one pass over the rows
        _case("epoch", "logistic", 1000000, 4096, bits=16, B=64, T=15625, alpha=0.05, mu=0.01, lam=1e-5,
              name="epoch 1000000x4096 b16 B64"),
        # the conditioning sweep: a grid of step sizes and mu as 504 short 16-bit chains
        _case("epoch", "squared", 1000, 64, R=504, bits=16, T=1000, grid=True, name="epoch 504x1000x64 b16 grid"),
        # the ten-class, ten-thousand-feature set, five seeds over the same data, T = N
        _case("epoch", "softmax", 7500, 10000, K=10, R=5, share=True, T=7500, alpha=2.0, mu=0.1, lam=1e-4,
              name="epoch 5x7500x10000 K10 b8"),
        # the softmax gradient pass where the data come from HBM
        _case("gradient", "softmax", 960000, 784, K=10, lam=1e-4, name="gradient 960000x784 K10"),
        # the data of configuration 5 into 16 bits
        _case("quantize", "logistic", 1000000, 4096, bits=16, name="quantize 1000000x4096 b16"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["linear", "chains", "softmax", "minibatch", "wide", "gradient", "quantize"])
    bits = rng.choice([8, 16])
    if kind == "linear":  # one chain, or a handful of seeds over the same data
        N, d, R = _log(rng, 500, 100000), _log(rng, 32, 4096), rng.choice([1, 1, 3, 8])
        return _case("epoch", rng.choice(["squared", "logistic"]), N, d, R=R, share=R > 1, bits=bits,
                     T=rng.choice([1, 2]) * min(N, 50000), algorithm=rng.choice(["halp", "halp", "lpsvrg", "svrg"]),
                     alpha=0.05, mu=0.3)
    if kind == "chains":  # many independent problems, or a grid over one
        N, d, R = _log(rng, 500, 16384), _log(rng, 32, 1024), _log(rng, 64, 1024)
        share = rng.choice([True, False]) or N * d * R > 2 ** 31
        algorithm = rng.choice(["halp", "halp", "halp", "lpsvrg", "svrg"])
        return _case("epoch", rng.choice(["squared", "squared", "logistic"]), N, d, R=R, share=share, bits=bits, T=N,
                     algorithm=algorithm, alpha=0.05, mu=0.1, grid=algorithm == "halp" and rng.choice([True, False]))
    if kind == "softmax":  # image-sized rows, a few to sixteen classes, one row per step or a minibatch
        N, d, B = _log(rng, 1000, 60000), _log(rng, 64, 1024), rng.choice([1, 1, 8, 32, 64])
        return _case("epoch", "softmax", N, d, K=rng.randint(2, 16), R=rng.choice([1, 1, 4]), share=True, bits=bits,
                     B=B, T=-(-min(N, 32768) // B), alpha=1e-2, mu=2.5, lam=rng.choice([0.0, 1e-4]))
    if kind == "minibatch":
        N, d, B = _log(rng, 5000, 400000), _log(rng, 128, 4096), rng.choice([4, 16, 32, 64, 128])
        return _case("epoch", rng.choice(["squared", "logistic"]), N, d, bits=bits, B=B, T=-(-N // B), alpha=0.05,
                     mu=0.05, lam=rng.choice([0.0, 1e-5]))
    if kind == "wide":  # softmax rows of thousands of features
        N, d = _log(rng, 1000, 7500), _log(rng, 1100, 10000)
        return _case("epoch", "softmax", N, d, K=rng.randint(2, 10), R=rng.choice([1, 3, 5]), share=True, bits=bits,
                     T=N, alpha=2.0, mu=0.1, lam=rng.choice([0.0, 1e-4]))
    N, d = _log(rng, 500, 1000000), _log(rng, 32, 4096)
    if kind == "gradient":
        loss = rng.choice(["squared", "logistic", "softmax"])
        if loss == "softmax":
            d = _log(rng, 32, 1024)
        return _case("gradient", loss, N, d, K=rng.randint(2, 16) if loss == "softmax" else 1, lam=1e-4)
    return _case("quantize", "squared", N, d, bits=bits)


def _pad(n, m):
    return (n + m - 1) // m * m


def _data(case, gen):
    """X [Rd, N, d] (rows padded to whole 16-byte groups), labels, and the teacher they come from."""
    N, d, K = case["N"], case["d"], case["K"]
    Rd = 1 if case["share"] else case["R"]
    f = dict(dtype=torch.float32, device="cuda")
    full = torch.zeros((Rd, N, _pad(d, 4)), **f)
    X = full[:, :, :d]
    soft = case["loss"] == "softmax"
    sparse = soft and d <= 1024
    teacher = torch.empty((Rd, d, K), **f).normal_(generator=gen)
    out = torch.empty((Rd, N, K), **f)
    rows = max(1, (1 << 28) // d)
    for r in range(Rd):
        for s in range(0, N, rows):  # bounded temporaries
            x = torch.empty((min(N, s + rows) - s, d), **f)
            if sparse:
                x.uniform_(generator=gen)
                x = torch.relu(x - 0.8) * 5.0
            else:
                x.normal_(0.0, d ** -0.5, generator=gen)
            if case["grid"]:  # Hessian eigenvalues from 1 to kappa over the columns, kappa by chain
                x *= math.sqrt(d) * torch.logspace(0.0, 0.5 * (r % 6), d, **f)
            X[r, s:s + rows] = x
            out[r, s:s + rows] = x @ teacher[r]
    if soft:
        u = torch.empty_like(out).uniform_(1e-7, 1.0 - 1e-7, generator=gen)
        y = torch.argmax((1.0 if sparse else 4.0) * out - torch.log(-torch.log(u)), dim=2).to(torch.int32)
    else:
        noise = torch.empty_like(out).normal_(0.0, 0.5 if case["loss"] == "logistic" else 0.1, generator=gen)
        y = (out + noise)[:, :, 0].contiguous()
        if case["loss"] == "logistic":
            y = torch.where(y >= 0, 1.0, -1.0)
    return X, y, teacher


def prepare(case, seed):
    N, d, K, R, bits = case["N"], case["d"], case["K"], case["R"], case["bits"]
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    X, y, teacher = _data(case, gen)
    Rd = X.shape[0]
    qmax = float(2 ** (bits - 1) - 1)
    top = max(float(X[r].max()) for r in range(Rd)), max(-float(X[r].min()) for r in range(Rd))
    h = hp.Halp(N, d, K=K, R=R, loss=LOSSES[case["loss"]], b=bits, B=case["B"], T=case["T"], alpha=case["alpha"],
                mu=case["mu"], lam=0.0 if case["algorithm"] == "lpsvrg" else case["lam"], delta_d=max(top) / qmax,
                seed=seed, share_data=case["share"], algorithm=ALGORITHMS[case["algorithm"]],
                delta=MODEL_SCALE * 127.0 / qmax if case["algorithm"] == "lpsvrg" else 0.0)
    st = hp.alloc_state(N, d, K=K, R=R, b=bits) if case["call"] != "quantize" else {}
    Xq = None
    if case["call"] == "quantize" or (case["call"] == "epoch" and case["algorithm"] != "svrg"):
        Xq = torch.zeros((Rd, N, _pad(d, 8)), dtype=torch.int8 if bits == 8 else torch.int16, device="cuda")
    h.bind(X=X, Xq=Xq, y=y, **st)
    s = dict(case=case, h=h, X=X, y=y, Xq=Xq, st=st)
    if case["call"] == "quantize":
        return s
    # a model some epochs in: the teacher and what training has not removed yet
    w0 = torch.empty((R, K, d), dtype=torch.float32, device="cuda").normal_(0.0, 0.3, generator=gen)
    w0 += teacher.transpose(1, 2)
    st["w"].copy_(w0)
    if case["call"] == "epoch":
        s["w0"] = w0
        if case["grid"]:
            h.set_chain_hyper(alpha=[10.0 ** (-0.5 * (3 + (r // 6) % 12)) for r in range(R)],
                              mu=[0.5 * 4.0 ** ((r // 72) % 7) for r in range(R)])
        if Xq is not None:
            h.quantize_data()
    return s


def run(s):
    h, st, call = s["h"], s["st"], s["case"]["call"]
    if call == "quantize":
        h.quantize_data()
        return {"Xq": s["Xq"]}
    if call == "gradient":
        h.full_gradient()
        return {"phi": st["phi"], "g": st["g"], "loss": st["scales"][:, 6]}
    st["w"].copy_(s["w0"])
    h.epoch(0)
    out = {"w": st["w"], "phi": st["phi"], "g": st["g"], "loss": st["scales"][:, 6]}
    if s["case"]["algorithm"] != "svrg":
        out["z"], out["h"], out["counters"] = st["z"], st["h"], st["counters"]
    return out


def work(case):
    N, d, K, R, B, T = (case[k] for k in ("N", "d", "K", "R", "B", "T"))
    Rd = 1 if case["share"] else R
    size = case["bits"] // 8
    if case["call"] == "quantize":
        return {"bytes": Rd * N * d * (4 + size), "flops": Rd * N * d}
    # gradient pass: X and y read, the margins, g and w once each; two products per element and class
    nbytes = Rd * N * (4 * d + 4) + R * (4 * N * K + 8 * K * d)
    flops = 4 * R * N * d * K
    if case["call"] == "epoch":
        # inner loop: the sampled rows (from memory at most once per data set and pass over it) and their margins;
        # a dot product and an update of d coordinates per row and class
        row = d * (4 if case["algorithm"] == "svrg" else size)
        nbytes += min(R * T * B, Rd * N) * row + 4 * min(T * B, N) * R * K
        nbytes += R * K * d * (4 + (0 if case["algorithm"] == "svrg" else 3 * size))
        flops += 4 * R * T * B * d * K
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    if case["call"] == "quantize":
        return "exact"
    if case["algorithm"] == "svrg":
        # fp32 iterates: every step rounds a dot product and d updates, and the steps' errors add like sqrt(T)
        return {"rel": 3e-5, "max": 5e-3}
    # fp32 sums; everything behind the gradient is whole numbers on a given gradient and stays the same
    return {"rel": 1e-5}
