"""What is timed when the speed of this library is at stake: the calls that a training program makes,
over the range of models, batches and precisions that the library takes.

Three kinds of case:

  round  The simulated training loop (driver.run_async, bench.py): every one of k workers, each on a
         stream of its own (at most four streams, as bench.py runs them), makes n local steps
         (forward, backward, AdamW) on its own batches, and the server then takes all of them in
         with one Delayed Nesterov group and restarts them.  One pass is one such round; a local
         step has both directions, and the group pass the outer step.
  outer  The outer step alone on flat vectors (k_dn_group): G pseudo-gradients, with or without the
         restart of the workers.
  adamw  The inner optimiser alone on flat vectors (k_adamw), with the bf16 working copy.

A state is what a program holds between calls: the context with its arena (or the flat vectors),
the token batches of its workers on the GPU, and the learning rate.  Passes change the state, as
training does."""
from __future__ import annotations

import ctypes
import math

import torch

import paper_2401_09135_amd as A

DEVICE = "cuda:0"
LR = 1e-3
OUTER_LR, OUTER_BETA = 0.7, 0.9


def _round(name, L, d, h, dh, ff, V, S, B, dtype, k, n, norm="rms", N=4, c=0.0):
    return dict(kind="round", name=name, L=L, d=d, h=h, dh=dh, ff=ff, V=V, S=S, B=B, dtype=dtype, norm=norm,
                k=k, n=n, N=N, c=c)


def listed():
    return [
        # the fp32 correctness workload ("tiny"): what a user steps first and debugs with; launches and latency only
        _round("tiny_f32", 2, 64, 2, 32, 256, 256, 32, 8, "f32", 4, 2),
        # the reduced bf16 workload ("mini_bf16"), four workers with little work per kernel
        _round("mini_bf16", 2, 256, 4, 64, 1024, 1024, 128, 4, "bf16", 4, 2),
        # sizes that are no multiples of anything: a vocabulary as a tokeniser leaves it, an odd batch of sequences of
        # an odd length
        _round("ragged_bf16", 4, 320, 5, 64, 1280, 5003, 200, 3, "bf16", 2, 1, N=2),
        # heads of 32, momentum activation c > 0
        _round("heads32_bf16", 4, 256, 8, 32, 1024, 4096, 256, 8, "bf16", 2, 1, N=2, c=0.25),
        # fp32 reference mode on a model of ordinary width, layer normalisation
        _round("reference_f32", 4, 256, 4, 64, 1024, 2000, 128, 8, "f32", 1, 1, norm="layer", N=1),
        # the 150M-class model on one sequence per worker step ("lm150m_b1")
        _round("lm150m_b1", 12, 896, 14, 64, 3584, 32000, 1024, 1, "bf16", 2, 1, N=2),
        # the paper's 20M model (vocabulary 32000 on a width of 256) at a small per-worker batch
        _round("paper20m_b32", 6, 256, 4, 64, 1024, 32000, 256, 32, "bf16", 2, 1, N=2),
        # the 20M-class workload, four workers ("lm20m")
        _round("lm20m", 6, 512, 8, 64, 2048, 8192, 512, 32, "bf16", 4, 1),
        # the 150M-class workload, four workers ("lm150m"): the largest, and the headline of bench.py
        _round("lm150m", 12, 896, 14, 64, 3584, 32000, 1024, 16, "bf16", 4, 1),
        # one asynchronous sync event of a 20M-class model, whose parameter count is odd
        dict(kind="outer", name="event_20m", P=27_484_675, G=1, N=4, t0=0, c=0.0, restart=False, bf16=True),
        # sixteen workers that finish together, with their restart (20M-class model)
        dict(kind="outer", name="group16_20m", P=27_484_672, G=16, N=16, t0=0, c=0.0, restart=True, bf16=True),
        # the inner optimiser on the vector of the outer-step microbenchmark
        dict(kind="adamw", name="adamw_150m", P=150_000_000, decay=149_995_904, bf16=True),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    r = rng.random()
    if r < 0.15:
        G = rng.choice((1, 1, 2, 3, 4, 8, 16))
        P = min(_log(rng, 1_000, 150_000_000), 450_000_000 // G)
        N = rng.choice((1, 4, 8, 16))
        return dict(kind="outer", P=P, G=G, N=N, t0=rng.randrange(N), c=rng.choice((0.0, 0.0, 0.5 / N)),
                    restart=rng.random() < 0.6, bf16=rng.random() < 0.8)
    if r < 0.25:
        P = _log(rng, 1_000, 150_000_000)
        return dict(kind="adamw", P=P, decay=P - 64 * rng.randrange(0, 1 + min(64, P // 128)), bf16=rng.random() < 0.8)
    while True:
        dtype = "f32" if rng.random() < 0.25 else "bf16"
        whole = rng.random() < 0.6     # round sizes throughout, as configurations are mostly written
        unit = 128 if whole else 64
        d = unit * _log(rng, 1, 1024 // unit)
        dh = 64 if whole else rng.choice((32, 64))
        h = d // dh
        if rng.random() < 0.2:         # an attention width that is not the model width
            h = _log(rng, 1, 1024 // unit) * (unit // dh)
        ff = unit * int(round(d / unit * rng.uniform(1.0, 4.0)))
        V, S = (128 * _log(rng, 1, 312), 128 * _log(rng, 1, 8)) if whole else (_log(rng, 64, 40_000), _log(rng, 16, 1024))
        B = _log(rng, 1, 64)
        c = _round(None, rng.randint(1, 12), d, h, dh, ff, V, S, B, dtype, rng.randint(1, 4), rng.randint(1, 2),
                   norm=rng.choice(("rms", "rms", "layer")), N=rng.choice((1, 2, 4)))
        del c["name"]
        # reference mode and odd sizes belong to small runs; no draw is larger than the largest listed case
        most = 6e13 if whole and dtype == "bf16" else 2e11
        if work(c)["flops"] <= most and _arena_bytes(c) <= 6e10:
            return c


def _config(c):
    return A.Config(n_layers=c["L"], d_model=c["d"], n_heads=c["h"], d_ff=c["ff"], vocab=c["V"], seq_len=c["S"], batch=c["B"],
                    dtype=A.ALS_DTYPE_BF16 if c["dtype"] == "bf16" else A.ALS_DTYPE_F32, n_workers=c["k"], dn_N=c["N"],
                    max_local_steps=c["n"], flags=0, head_dim=c["dh"], norm_kind={"rms": 0, "layer": 1}[c["norm"]],
                    adam_beta1=0.9, adam_beta2=0.999, adam_eps=1e-8, weight_decay=0.1, outer_lr=OUTER_LR,
                    outer_beta=OUTER_BETA, dn_c=c["c"], norm_eps=1e-5)


def _sizes(c):
    """(parameters, decayed parameters) of a round's model."""
    d, a = c["d"], c["h"] * c["dh"]
    decayed = 2 * c["V"] * d + c["S"] * d + c["L"] * (4 * d * a + 2 * d * c["ff"])
    return decayed + (2 * c["L"] + 1) * d, decayed


def _arena_bytes(c):
    return int(A.lib.als_arena_bytes(ctypes.byref(_config(c))))


def _gen(seed):
    return torch.Generator(device=DEVICE).manual_seed(int(seed))


def _tokens(c, gen):
    """Bounded Zipf(1.1) token ids by inverse CDF: [k workers][n steps, B, S + 1]."""
    p = torch.arange(1, c["V"] + 1, dtype=torch.float64, device=DEVICE) ** -1.1
    cdf = torch.cumsum(p, 0)
    cdf = (cdf / cdf[-1]).float()
    out = []
    for _ in range(c["k"]):
        u = torch.rand(c["n"], c["B"], c["S"] + 1, device=DEVICE, generator=gen)
        out.append(torch.searchsorted(cdf, u).clamp_(max=c["V"] - 1).to(torch.int32))
    return out


def _prepare_round(c, seed):
    gen = _gen(seed)
    P, decayed = _sizes(c)
    theta0 = torch.empty(P, device=DEVICE)
    theta0[:decayed].normal_(0.0, 0.02, generator=gen)
    theta0[decayed:] = 1.0
    cfg = _config(c)
    ctx = A.Context(cfg, theta0.cpu().numpy(), n_streams=min(c["k"], 4), device=DEVICE)
    toks = _tokens(c, gen)
    # Views of the vectors that a program reads back with Context.get_vector, where they lie in the context's arena (each
    # at a multiple of 256 bytes): theta, momentum, Delta, and at the head of each worker's equal share its replica,
    # snapshot, AdamW moments and gradient.
    flat = ctx.arena[:ctx.arena.numel() // 4 * 4].view(torch.float32)
    at = (-ctx.arena.data_ptr() % 256) // 4
    step = (4 * P + 255) // 256 * 64
    share = (_arena_bytes(dict(c, k=2)) - _arena_bytes(dict(c, k=1))) // 4
    server = [flat[at + i * step:][:P] for i in range(3)]
    workers = [[flat[at + 3 * step + w * share + i * step:][:P] for i in range(5)] for w in range(c["k"])]
    assert all(torch.equal(v, theta0) for v in [server[0]] + [x for w in workers for x in w[:2]])
    # The second moments of a run under way: with the zeros of a new one, a worker's first updates have the size of the
    # learning rate wherever the gradient has any sign at all, and rounding decides the sign of many.
    v = torch.rand(P, device=DEVICE, generator=gen).add_(0.5).mul_(1e-6).cpu().numpy()
    for w in range(c["k"]):
        ctx.set_vector("adam_v", w, v)
    return dict(c=c, ctx=ctx, toks=toks, group=list(range(c["k"])), server=server, workers=workers)


def _vector(P, gen, sigma):
    return torch.empty(P, device=DEVICE).normal_(0.0, sigma, generator=gen)


def _prepare_outer(c, seed):
    gen, P = _gen(seed), c["P"]
    start = [_vector(P, gen, 0.02) for _ in range(c["G"])]
    return dict(c=c, theta=_vector(P, gen, 0.02), m=_vector(P, gen, 1e-3), delta=torch.zeros(P, device=DEVICE), start=start,
                worker=[s + _vector(P, gen, 1e-3) for s in start],
                bf16=[torch.zeros(P, dtype=torch.bfloat16, device=DEVICE) for _ in range(c["G"])] if c["bf16"] else None)


def _prepare_adamw(c, seed):
    gen, P = _gen(seed), c["P"]
    return dict(c=c, theta=_vector(P, gen, 0.02), grad=_vector(P, gen, 1e-3), m=_vector(P, gen, 1e-3),
                v=_vector(P, gen, 1e-3).square_(), bf16=torch.zeros(P, dtype=torch.bfloat16, device=DEVICE) if c["bf16"] else None,
                step=0)


def prepare(case, seed):
    state = {"round": _prepare_round, "outer": _prepare_outer, "adamw": _prepare_adamw}[case["kind"]](case, seed)
    torch.cuda.synchronize()
    return state


def _run_round(s):
    ctx = s["ctx"]
    for w, tok in enumerate(s["toks"]):
        ctx.worker_local_steps(w, tok, LR)
    ctx.outer_apply_dn(s["group"], restart=True)
    names = ("replica", "snapshot", "adam_m", "adam_v", "grad")
    return dict(zip(("theta", "momentum", "delta"), s["server"]), workers=[dict(zip(names, w)) for w in s["workers"]])


def _run_outer(s):
    c = s["c"]
    A.k_dn_group(s["theta"], s["m"], s["delta"], s["start"], s["worker"], s["bf16"], c["N"], c["t0"], OUTER_LR, OUTER_BETA,
                 c["c"], restart=c["restart"])
    return dict(theta=s["theta"], m=s["m"], delta=s["delta"], start=s["start"], worker=s["worker"],
                bf16=s["bf16"] if c["restart"] else None)


def _run_adamw(s):
    s["step"] += 1
    A.k_adamw(s["theta"], s["grad"], s["m"], s["v"], s["bf16"], s["c"]["decay"], s["step"], LR)
    return dict(theta=s["theta"], m=s["m"], v=s["v"], bf16=s["bf16"])


def run(state):
    return {"round": _run_round, "outer": _run_outer, "adamw": _run_adamw}[state["c"]["kind"]](state)


def work(case):
    c = case
    if c["kind"] == "outer":
        # per event start and replica read; theta and Delta read and written, m too on an N-th event (or read, for c > 0);
        # a restart writes replica, snapshot and bf16 copy
        nth = any((c["t0"] + j + 1) % c["N"] == 0 for j in range(c["G"]))
        per = 8 * c["G"] + 16 + (8 if nth else 4 if c["c"] else 0) + (c["G"] * (10 if c["bf16"] else 8) if c["restart"] else 0)
        return dict(bytes=per * c["P"], flops=8 * c["G"] * c["P"])
    if c["kind"] == "adamw":
        return dict(bytes=(30 if c["bf16"] else 28) * c["P"], flops=15 * c["P"])
    P, _ = _sizes(c)
    steps, T, d, a = c["k"] * c["n"], c["B"] * c["S"], c["d"], c["h"] * c["dh"]
    # the matrix products and causal attention (half of the S x S scores), backward twice the forward
    token = 3.0 * (c["L"] * (8.0 * d * a + 4.0 * d * c["ff"] + 2.0 * c["S"] * a) + 2.0 * d * c["V"])
    # per step: replica and moments read and written, the gradient and the bf16 copy written, the tokens read; per worker
    # and round: start and replica read, replica, start and copy written; theta, m, Delta read and written
    lp = 2 if c["dtype"] == "bf16" else 0
    return dict(bytes=steps * ((28 + lp) * P + 4 * c["B"] * (c["S"] + 1)) + (c["k"] * (16 + lp) + 24) * P, flops=steps * T * token)


def tolerance(case):
    if case["kind"] != "round":
        # a handful of fp32 roundings per element; a value of the bf16 copy may round the other way (2^-8 of it)
        return dict(rel=1e-6, max=1e-2)
    if case["dtype"] == "f32":
        # Against the numpy oracle in 64 bits: rel 9.7e-6 at most (the momentum, a sum of small differences of
        # parameters) and max 7.8e-4, the same as the oracle in 32 bits.
        return dict(rel=4e-5, max=4e-3)
    # The matrix-core kernels against the generic ones (als_config.flags = 1: other summation orders, probabilities not
    # rounded to bf16), on every listed model and sixteen drawn ones: rel 1.9e-3 and max 0.27 at most, both in the
    # gradient.  max sets a single element against the root mean square of the whole vector, whose tensors have
    # gradients of very different sizes; bf16 against fp32 on the same models: rel 1.0e-2, max 1.0.
    return dict(rel=8e-3, max=0.99)
