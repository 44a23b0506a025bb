"""Performance cases of the call-auction ensemble engine and its calibration surrogate.

Each case is one call (or the short fixed sequence of calls) that a program built on this package
repeats: stepping an ensemble it holds, recording traced series, exact calibration statistics,
clearing books it aggregated itself, surrogate inference and the two forms of a training step.
Sizes come from ``workloads``, the benchmark's legs and the tests.
"""
import math

import numpy as np
import torch

from paper_2606_21784_amd import dynamics, engine, mlp, surrogate, workloads

# Kinds and their plain fields:
#   step     M, L, A, K, Q, S, noise, mom, mid, splitmix, overlap: ``Ensemble.step(S)`` on a held
#            handle.  L = 0: the uneven mixture of ``workloads.uneven`` (L, A and K drawn per
#            market, A at most the given A).  overlap > 0: the handle was made with the tuned
#            schedule (waves per market, overlap); 0: the library's own choice.
#   trace    the agent-mix sweep (``dynamics.composition_descs``) through ``step_traced``.
#   calib    ``surrogate.exact_stats`` of fresh parameter rows (ensemble made, stepped, read).
#   clear    M books of L ticks aggregated by the caller, cleared by ``clear_books``.
#   predict  surrogate inference on N rows.
#   train    the fused training step on a batch of N rows gathered from a sample set.
#   unfused  forward, loss gradient, backward and Adam of a network of any allowed width.


def listed():
    return [
        # an interactive loop on a handful of markets: one step per call, launch latency
        dict(name="step_one_M4_L64_A128", **_step(M=4, L=64, A=128, K=8, Q=10, S=1)),
        # the latency experiment: a few steps per call over 4096 live markets
        dict(name="step_live_M4096_L128_A256", **_step(M=4096, L=128, A=256, K=8, Q=10, S=11)),
        # the fixed standard workload in the library's own schedule
        dict(name="step_fixed_M1024_L256_A1024", **_step(M=1024, L=256, A=1024, K=16, Q=100, S=1000)),
        # small populations, the agent-count sweep's first point
        dict(name="step_small_M8192_L128_A16", **_step(M=8192, L=128, A=16, K=8, Q=10, S=500)),
        # few large markets, the market-count sweep's small-count regime
        dict(name="step_large_M64_L512_A4096", **_step(M=64, L=512, A=4096, K=32, Q=100, S=500)),
        # markets of uneven size in one launch
        dict(name="step_uneven_M1024", **_step(M=1024, L=0, A=16384, K=0, Q=100, S=200)),
        # the paper's own agent rules, traced: one mix sweep with its price and volume series
        dict(name="trace_mix_M960_A256", kind="trace", per_mix=64, A=256, L=128, K=8, Q=10, S=1000,
             mid=True, p_mkt=0.05),
        # exact statistics of 32 calibration draws in the tuned schedule
        dict(name="calib_32_draws", kind="calib", draws=32, per_draw=64, S=1000, overlap=4),
        # external order flow: books aggregated elsewhere, cleared in one pass
        dict(name="clear_M16384_L256", kind="clear", M=16384, L=256, qmax=100),
        # the held-out sweep through the surrogate
        dict(name="predict_N6553_H256", kind="predict", d_in=4, H=256, d_out=3, N=6553),
        # one training step of the surrogate at its training batch
        dict(name="train_N1024_H256", kind="train", d_in=4, H=256, d_out=3, N=1024, huber=0.05),
        # a wider network than the fused step takes
        dict(name="train_wide_N4096_H1024", kind="unfused", d_in=64, H=1024, d_out=16, N=4096, huber=0.05),
    ]


def _step(M, L, A, K, Q, S, noise=1.0, mom=0.0, mid=False, splitmix=False, overlap=0):
    return dict(kind="step", M=M, L=L, A=A, K=K, Q=Q, S=S, noise=noise, mom=mom, mid=mid, splitmix=splitmix,
                overlap=overlap)


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


# Work of one call of the stepping kinds: order events plus a clearing's ticks, and the longest
# chain of steps (a single market's), both at most those of the listed cases.
_MOST_WORK, _MOST_CHAIN = 1.2e9, 2.0e6


def draw(rng):
    kind = rng.choice(["step", "step", "step", "trace", "calib", "clear", "predict", "train", "unfused"])
    if kind == "step":
        A = _log_int(rng, 16, 16384)
        L = rng.choice([64, 128, 256, 512, 1024, rng.randint(16, 1024), rng.randint(16, 1024)])
        M = _log_int(rng, 1, 8192)
        S = _log_int(rng, 1, 1000)
        M = max(1, min(M, int(_MOST_WORK / (A + 2 * L))))
        S = max(1, min(S, int(_MOST_WORK / (M * (A + 2 * L))), int(_MOST_CHAIN / (A + 2 * L))))
        q = max(1, min(100, int(2**31 / (A * S)) // 8))
        pure = rng.random() < 0.5
        noise = 1.0 if pure else rng.uniform(0.2, 0.9)
        return _step(M=M, L=L, A=A, K=max(1, L // 16), Q=min(q, rng.choice([10, 100, 37])), S=S,
                     noise=round(noise, 3), mom=0.0 if pure else round(rng.uniform(0.0, 1.0 - noise), 3),
                     mid=rng.random() < 0.25, splitmix=rng.random() < 0.15,
                     overlap=rng.choice([0, 0, 0, 3]) if A >= 256 else 0)
    if kind == "trace":
        A = rng.choice([16, 64, 256, rng.randint(20, 400)])
        return dict(kind="trace", per_mix=rng.randint(4, 64), A=A, L=128, K=8, Q=10, S=_log_int(rng, 50, 1000),
                    mid=rng.random() < 0.5, p_mkt=0.05)
    if kind == "calib":
        return dict(kind="calib", draws=rng.randint(1, 32), per_draw=64, S=_log_int(rng, 50, 1000),
                    overlap=rng.choice([0, 4]))
    if kind == "clear":
        L = rng.choice([5, 64, 128, 256, 512, 1024, rng.randint(1, 1024), rng.randint(1, 1024)])
        return dict(kind="clear", M=_log_int(rng, 1, max(1, 16384 * 256 // L)), L=L, qmax=100)
    if kind == "predict":
        H = rng.choice([64, 256, 256, 16 * rng.randint(1, 31)])
        return dict(kind="predict", d_in=rng.choice([4, rng.randint(1, 64)]), H=H, d_out=rng.randint(1, 16),
                    N=_log_int(rng, 1, 65536))
    if kind == "train":
        return dict(kind="train", d_in=rng.choice([4, rng.randint(1, 32)]), H=rng.choice([256, 32 * rng.randint(1, 8)]),
                    d_out=rng.randint(1, 16), N=_log_int(rng, 16, 8192), huber=rng.choice([0.0, 0.05]))
    return dict(kind="unfused", d_in=rng.randint(1, 64), H=16 * rng.randint(1, 64), d_out=rng.randint(1, 16),
                N=_log_int(rng, 16, 4096), huber=rng.choice([0.0, 0.05]))


# ------------------------------------------------------------------------------------------
# Inputs
# ------------------------------------------------------------------------------------------
def _flags(case):
    return engine.model_flags(1 if case.get("mid") else 0, case.get("p_mkt", 0.0) if case.get("mid") else 0.0,
                              1 if case.get("splitmix") else 0)


def _descs(case, seed):
    if case["kind"] == "trace":
        return dynamics.composition_descs(A=case["A"], L=case["L"], K=case["K"], Q=case["Q"],
                                          markets=case["per_mix"], flags=_flags(case))
    if case["L"] == 0:
        d = workloads.uneven(case["M"], seed=4)["descs"]  # the same mixture; the seed draws the orders
        d["A"] = np.minimum(d["A"], case["A"])
        d["n_noise"] = d["A"]
        return d
    A = case["A"]
    n_noise = int(round(case["noise"] * A))
    n_mom = min(A - n_noise, int(round(case["mom"] * A)))
    return engine.markets(case["L"], A, case["K"], case["Q"], M=case["M"], n_noise=n_noise, n_mom=n_mom,
                          h=min(2, case["L"] - 1), flags=_flags(case))


def _tuned(case, L, A):
    """A schedule as the autotuner returns it for one size class: four waves per market, orders
    generated while the step clears."""
    if not case["overlap"]:
        return None
    c = engine.size_class(L, A)
    return {"waves_per_group": 4, "waves_per_market": {c: 4}, "overlap": {c: case["overlap"]}}


def _held(case, seed):
    d = _descs(case, seed)
    ens = engine.Ensemble(d, 1000 + seed, tuning=_tuned(case, case["L"], case["A"]) if "overlap" in case else None)
    limit = (2**32 - 1) // int((d["A"].astype(np.int64) * d["Q"].astype(np.int64)).max())
    return {"ens": ens, "limit": limit, "steps": 0, "S": case["S"], "opening": (ens.read_state(), ens.read_books())}


def _network(case, seed, batch):
    net = mlp.MLP(case["d_in"], case["H"], case["d_out"], max_batch=batch, seed=seed)
    p, (d_in, H, d_out) = net.get_params(), net.dims
    rng = np.random.default_rng(seed)
    o1, o2 = d_in * H, d_in * H + H + H * H
    p[o1:o1 + H] = rng.normal(0, 0.1, H)  # a trained network's biases are not zero
    p[o2:o2 + H] = rng.normal(0, 0.1, H)
    net.set_params(p)
    return net


def _samples(case, seed):
    """Sample set of a training case and the rows of its batch."""
    rng = np.random.default_rng(seed + 77)
    rows = case["N"] if case["kind"] == "unfused" else 2 * case["N"]
    x = rng.uniform(-1, 1, (rows, case["d_in"])).astype(np.float32)
    mix = rng.normal(0, 1, (case["d_in"], case["d_out"]))
    t = (np.sin(x @ mix) + 0.05 * rng.normal(0, 1, (rows, case["d_out"]))).astype(np.float32)
    return x, t, rng.permutation(rows)[:case["N"]].astype(np.int32)


def prepare(case, seed):
    kind = case["kind"]
    if kind in ("step", "trace"):
        return dict(_held(case, seed), kind=kind)
    if kind == "calib":
        theta = workloads.calibration_params(case["draws"], seed=100 + seed)
        return {"kind": kind, "theta": theta, "ids": np.arange(case["draws"]) + 64 * (seed % 1000), "S": case["S"],
                "per_draw": case["per_draw"], "tuning": _tuned(case, workloads.CALIB_L, workloads.CALIB_A)}
    if kind == "clear":
        g = torch.Generator(device="cuda")
        g.manual_seed(seed)
        M, L = case["M"], case["L"]
        # orders around a price near the middle: bids thin out above it, asks below it
        tick = torch.arange(L, device="cuda", dtype=torch.float32)
        mid = L / 2 + (torch.rand((M, 1), generator=g, device="cuda") - 0.5) * L / 4
        near = torch.exp(-((tick[None, :] - mid) / max(1.0, L / 8)) ** 2)
        q = torch.rand((M, 2, L), generator=g, device="cuda") * case["qmax"]
        side = torch.stack([torch.sigmoid((mid - tick) / max(1.0, L / 32)),
                            torch.sigmoid((tick - mid) / max(1.0, L / 32))], dim=1)
        orders = (q * near[:, None, :] * (0.2 + side)).to(torch.int32).reshape(-1).contiguous()
        return {"kind": kind, "orders": orders, "book": torch.empty_like(orders), "L": L, "M": M}
    if kind == "predict":
        net = _network(case, seed, 16)
        g = torch.Generator(device="cuda")
        g.manual_seed(seed)
        x = torch.rand((case["N"], case["d_in"]), generator=g, device="cuda") * 2 - 1
        return {"kind": kind, "net": net, "x": x}
    net = _network(case, seed, case["N"])
    x, t, idx = _samples(case, seed)
    return {"kind": kind, "net": net, "x": torch.from_numpy(x).cuda(), "t": torch.from_numpy(t).cuda(),
            "idx": torch.from_numpy(idx).cuda(), "huber": case["huber"] or None}


# ------------------------------------------------------------------------------------------
# One pass
# ------------------------------------------------------------------------------------------
def run(state):
    kind = state["kind"]
    if kind in ("step", "trace"):
        ens = state["ens"]
        if state["steps"] + state["S"] > state["limit"]:  # 32-bit books are full: back to the opening
            ens.write_state(*state["opening"])
            state["steps"] = 0
        state["steps"] += state["S"]
        if kind == "step":
            ens.step(state["S"])
            return {"book": ens.book, "state": ens.state}
        price, volume = ens.step_traced(state["S"])
        return {"price": price, "volume": volume, "book": ens.book, "state": ens.state}
    if kind == "calib":
        return surrogate.exact_stats(state["theta"], state["ids"], S=state["S"], markets_per_draw=state["per_draw"],
                                     tuning=state["tuning"])
    if kind == "clear":
        state["book"].copy_(state["orders"])
        p, v = engine.clear_books(state["book"], state["L"], state["M"])
        return {"book": state["book"], "price": p, "volume": v}
    net = state["net"]
    if kind == "predict":
        return net.predict(state["x"])
    if kind == "train":
        loss = net.train_step_fused(state["x"], state["t"], 1e-3, idx=state["idx"], huber_delta=state["huber"])
        return {"loss": loss, "params": net.params, "m": net.m, "v": net.v}
    loss = net.train_step(state["x"], state["t"], 1e-3, huber_delta=state["huber"])
    return {"loss": loss, "grads": net.grads, "params": net.params, "m": net.m, "v": net.v}


# ------------------------------------------------------------------------------------------
# Work: bytes and operations a pass cannot do without
# ------------------------------------------------------------------------------------------
# Least VALU operations of an order event (Philox4x32-10 with the agent-independent products
# hoisted: 16 products, 18 xors; two range reductions; one word) and of a clearing's tick.
_OPS_EVENT, _OPS_TICK = 37.0, 6.0


def _engine_work(d, S, traced):
    A, L = float(d["A"].astype(np.float64).sum()), float(d["L"].astype(np.float64).sum())
    b = 16.0 * L + 160.0 * len(d) + 48.0 * len(d) + (8.0 * len(d) * S if traced else 0.0)
    return {"bytes": b, "flops": S * (_OPS_EVENT * A + _OPS_TICK * L)}


def work(case):
    kind = case["kind"]
    if kind in ("step", "trace"):
        return _engine_work(_descs(case, 0), case["S"], kind == "trace")
    if kind == "calib":
        M = case["draws"] * case["per_draw"]
        return _engine_work(engine.markets(workloads.CALIB_L, workloads.CALIB_A, 8, 10, M=M), case["S"], False)
    if kind == "clear":
        return {"bytes": 16.0 * case["M"] * case["L"] + 8.0 * case["M"], "flops": 6.0 * case["M"] * case["L"]}
    d_in, H, d_out, N = case["d_in"], case["H"], case["d_out"], case["N"]
    w = d_in * H + H * H + H * d_out
    p = w + 2 * H + d_out
    if kind == "predict":
        return {"bytes": 4.0 * N * (d_in + d_out) + 2.0 * w, "flops": 2.0 * N * w}
    # x and targets; parameters and both moments read and written, bfloat16 copies read and written
    return {"bytes": 4.0 * N * (d_in + d_out) + 24.0 * p + 4.0 * w + (4.0 * p if kind == "unfused" else 0.0),
            "flops": 6.0 * N * w - 2.0 * N * d_in * H}


# ------------------------------------------------------------------------------------------
# The same results in 64 bits (networks; the engine's results are whole numbers)
# ------------------------------------------------------------------------------------------
def _split(p, dims):
    d_in, H, d_out = dims
    out, o = [], 0
    for shape in ((d_in, H), (H,), (H, H), (H,), (H, d_out), (d_out,)):
        n = int(np.prod(shape))
        out.append(p[o:o + n].reshape(shape))
        o += n
    return out


def _forward64(p, dims, x):
    W1, b1, W2, b2, W3, b3 = _split(p, dims)
    z1 = x @ W1 + b1
    h1 = z1 * torch.sigmoid(z1)
    z2 = h1 @ W2 + b2
    h2 = z2 * torch.sigmoid(z2)
    return z1, h1, z2, h2, h2 @ W3 + b3


def exact(case, seed):
    kind = case["kind"]
    if kind not in ("predict", "train", "unfused"):
        return None
    state = prepare(case, seed)
    dims = (case["d_in"], case["H"], case["d_out"])
    p = state["net"].params.double().clone()
    if kind == "predict":
        return _forward64(p, dims, state["x"].double())[4]
    x, t = state["x"].double(), state["t"].double()
    if kind == "train":
        x, t = x[state["idx"].long()], t[state["idx"].long()]
    z1, h1, z2, h2, y = _forward64(p, dims, x)
    r, n, delta = y - t, y.numel(), state["huber"]
    if delta is None:
        loss, dy = (r * r).mean(), 2.0 * r / n
    else:
        a = r.abs()
        loss = torch.where(a <= delta, 0.5 * r * r, delta * (a - 0.5 * delta)).mean()
        dy = r.clamp(-delta, delta) / n
    W1, b1, W2, b2, W3, b3 = _split(p, dims)

    def slope(z):
        s = torch.sigmoid(z)
        return s * (1.0 + z * (1.0 - s))

    dz2 = (dy @ W3.t().contiguous()) * slope(z2)
    dz1 = (dz2 @ W2.t().contiguous()) * slope(z1)
    g = torch.cat([v.reshape(-1) for v in (x.t().contiguous() @ dz1, dz1.sum(0), h1.t().contiguous() @ dz2,
                                           dz2.sum(0), h2.t().contiguous() @ dy, dy.sum(0))])
    m, v = 0.1 * g, 0.001 * g * g
    new = p - 1e-3 * (m / 0.1) / (torch.sqrt(v / 0.001) + 1e-8)
    out = {"loss": loss.reshape(1), "params": new, "m": m, "v": v}
    return dict(out, grads=g) if kind == "unfused" else out
