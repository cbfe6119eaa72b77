"""Performance cases of the dual-step LABS library: calls a search program makes.

Each case is one pass through public entry points (paper_2409_07222_amd.labs and
.learn) at the sizes the benchmark and the tests use: first-step walks (tabu and
Bloom filter, with and without the pool, one length or many), the second step
(odd and even lengths, with rotations), the exact energies and flip changes, and
the learned proposal's log, training step, logits and walk.
"""
import math

import numpy as np
import torch

from paper_2409_07222_amd import labs, learn

DEV = "cuda"
NO_LIMIT = 1 << 62          # T_u of the second step: stop on the expansion budget only


# ------------------------------------------------------------------ the cases
def listed():
    return [
        # exact energies, C tables and both neighbourhoods of a batch of sequences
        dict(name="score_501", kind="score", L=501, p=16, n=4096),
        # a short walk of a few walkers: launch latency
        dict(name="walk_101_small", kind="walk", L=101, p=8, n=256, steps=408),
        # the L = 101 configuration (65,536 walkers, F >= 6 sieve), shortened; top 1024
        dict(name="pool_101", kind="pool", L=101, p=8, n=65536, steps=1000, tau=6, best=False, cap=1 << 20),
        # the headline first step (16,384 walkers at L = 501, F >= 8 sieve, walker
        # bests offered), shortened; top 1024
        dict(name="pool_501", kind="pool", L=501, p=16, n=16384, steps=8192, tau=8, best=True, cap=1 << 20),
        # Algorithm 1 as the paper runs it: Bloom filter, T_i = 4(L+1) steps
        dict(name="bloom_451", kind="bloom", L=451, p=16, n=16384, steps=1808, log2_bits=15, n_hash=8),
        # every odd length of 301..449 in one launch, little work per length
        dict(name="batch_301_449", kind="batch", L_lo=301, L_hi=449, p=12, n=256, steps=1000),
        # the second step from the first step's top 1024
        dict(name="step2_501", kind="step2", L=501, batch=1024, queue=1 << 20, pops=200_000, T_r=0, seeds=1024),
        # the end operators to even lengths, then the second step with rotations
        dict(name="even_500_rot4", kind="even", L=501, batch=1024, queue=1 << 20, pops=100_000, T_r=4, seeds=1025),
        # logging a plain walk's states and moves for training
        dict(name="log_501", kind="log", L=501, p=16, n=16384, steps=245, every=7),
        # one training step at the training batch
        dict(name="train_501", kind="train", L=501, hidden=256, n=4096),
        # logits of held-out states
        dict(name="logits_501", kind="logits", L=501, hidden=256, n=20480),
        # the learned walk: top 8 of the network, a full scan every 64 steps
        dict(name="learned_501", kind="learned", L=501, p=16, n=16384, steps=256, hidden=256, top_m=8, every=64),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _odd(rng, lo, hi):
    return rng.randrange(lo | 1, hi + 1, 2)


def draw(rng):
    kind = rng.choice(["score", "walk", "pool", "bloom", "batch", "step2", "even", "log", "train", "logits",
                       "learned"])
    p = rng.choice([8, 12, 16])
    hidden = rng.choice([64, 128, 256])
    if kind == "score":
        return dict(kind=kind, L=_odd(rng, 37, 639), p=rng.choice([0, 8, 16]), n=_log_int(rng, 16, 4096))
    if kind in ("walk", "pool", "bloom", "log", "learned"):
        L = _odd(rng, 101, 527)
        n = _log_int(rng, 64, 16384)
        if kind == "walk":
            return dict(kind=kind, L=L, p=p, n=n, steps=_log_int(rng, 200, 4000))
        if kind == "pool":
            return dict(kind=kind, L=L, p=p, n=n, steps=_log_int(rng, 400, 4000), tau=rng.choice([4, 5, 6]),
                        best=rng.random() < 0.5, cap=_log_int(rng, 1 << 12, 1 << 20))
        if kind == "bloom":
            return dict(kind=kind, L=L, p=p, n=n, steps=_log_int(rng, 200, 2000),
                        log2_bits=rng.choice([12, 13, 14, 15, 16]), n_hash=rng.randint(2, 12))
        if kind == "log":
            every = rng.randint(1, 16)
            return dict(kind=kind, L=L, p=p, n=n, steps=rng.randint(64, 245), every=every)
        return dict(kind=kind, L=L, p=p, n=n, steps=rng.randint(100, 256), hidden=hidden, top_m=rng.choice([4, 8, 16]),
                    every=rng.choice([16, 32, 64]))
    if kind == "batch":
        lo = _odd(rng, 101, 401)
        return dict(kind=kind, L_lo=lo, L_hi=lo + 2 * rng.randint(8, 60), p=p, n=_log_int(rng, 16, 256),
                    steps=_log_int(rng, 200, 1000))
    if kind in ("step2", "even"):
        L = rng.randint(96, 640) if kind == "step2" else _odd(rng, 97, 599)
        return dict(kind=kind, L=L, batch=_log_int(rng, 256, 1024), queue=_log_int(rng, 1 << 16, 1 << 20),
                    pops=_log_int(rng, 20_000, 100_000), T_r=rng.choice([0, 0, 1, 4]),
                    seeds=_log_int(rng, 64, 1025))
    L = _odd(rng, 101, 527)
    if kind == "train":
        return dict(kind=kind, L=L, hidden=hidden, n=_log_int(rng, 64, 8192))
    return dict(kind=kind, L=L, hidden=hidden, n=_log_int(rng, 64, 20480))


# ------------------------------------------------------------------ inputs
def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(seed)


def _skew(g, n, L, p):
    """n random skew-symmetric sequences of odd length L (+1 / -1, int8 [n, L]),
    the first element +1 when a prefix is held."""
    k = (L - 1) // 2
    h = torch.randint(0, 2, (n, k + 1), generator=g, device=DEV, dtype=torch.int8) * 2 - 1
    if p >= 1:
        h[:, 0] = 1
    i = torch.arange(1, k + 1, device=DEV)
    sign = (1 - 2 * (i % 2)).to(torch.int8)
    return torch.cat([h, sign * h.flip(1)[:, 1:]], 1)


def _pack(s):
    """The library's wire format: 32 elements a word, the first in the top bit."""
    n, L = s.shape
    W = (L + 31) // 32
    b = torch.zeros((n, 32 * W), dtype=torch.int64, device=s.device)
    b[:, :L] = (s > 0)
    v = (b.view(n, W, 32) << torch.arange(31, -1, -1, device=s.device)).sum(2)
    return torch.where(v >= 1 << 31, v - (1 << 32), v).to(torch.int32).contiguous()


def _net_arrays(seed, L, hidden):
    """U(-1/sqrt(fan_in), 1/sqrt(fan_in)) weights, small biases."""
    k = (L - 1) // 2
    g = np.random.Generator(np.random.PCG64(seed))
    d_in, d_out = L + k, k + 1

    def u(*shape):
        b = 1.0 / math.sqrt(shape[-1])
        return g.uniform(-b, b, size=shape).astype(np.float32)
    return {"W1": u(hidden, d_in), "b1": 0.1 * u(hidden), "W2": u(hidden, hidden), "b2": 0.1 * u(hidden),
            "W3": u(d_out, hidden), "b3": 0.1 * u(d_out)}


def _moments(seed, L, hidden):
    """Adam moments of a training run under way."""
    P = _net_arrays(seed, L, hidden)
    g = np.random.Generator(np.random.PCG64(seed + 1))
    m = {q: (1e-4 * g.standard_normal(v.shape)).astype(np.float32) for q, v in P.items()}
    v = {q: (1e-8 * g.uniform(0.5, 2.0, size=v.shape)).astype(np.float32) for q, v in P.items()}
    return m, v


TRAIN_T = 100               # the training step's Adam count before the pass
LR = 1e-3


def _batch(g, L, n):
    """States, admissible masks (a tenure of the last moved positions out, and the
    prefix of 16) and the chosen moves, as a plain walk logs them."""
    k = (L - 1) // 2
    p = 16 if k > 40 else 0
    s = _skew(g, n, L, p)
    order = torch.rand((n, k + 1), generator=g, device=DEV)
    order[:, :p] = 2.0
    rank = order.argsort(1).argsort(1)
    nf = k + 1 - p
    ten = torch.randint(L // 10, min(L // 5, nf - 2) + 1, (n, 1), generator=g, device=DEV)
    ok = (rank < nf - ten)
    label = (rank == 0).to(torch.int32).argmax(1).to(torch.int32)
    mw = (k + 1 + 31) // 32
    b = torch.zeros((n, 32 * mw), dtype=torch.int64, device=DEV)
    b[:, :k + 1] = ok
    v = (b.view(n, mw, 32) << torch.arange(32, device=DEV)).sum(2)
    mask = torch.where(v >= 1 << 31, v - (1 << 32), v).to(torch.int32).contiguous()
    return s, ok, mask, label


def _tenure(c):
    nf = (c["L"] - 1) // 2 + 1 - c["p"]
    hi = min(c["L"] // 5, nf - 1)
    return min(c["L"] // 10, hi), hi


def _seeds_for_step2(L, n, seed):
    """Candidates of the second step: the best sequences of a short first step (for
    an even length, shortened by their last element)."""
    Lo = L | 1
    pool = labs.PoolBuffers.empty(Lo, 4096)
    nf = (Lo - 1) // 2 + 1
    labs.walk_step1(Lo, 0, 4 * (Lo + 1), min(Lo // 10, nf - 1), min(Lo // 5, nf - 1), seed, 2048, pool=pool,
                    e_max=-1, pool_walker_best=True)
    s, _ = labs.pool_topk(pool, n)
    if L != Lo:
        s = labs.length_operators(Lo, s.contiguous())[0][1::2]
    return s.contiguous()


def prepare(case, seed):
    c = dict(case)
    kind, L = c["kind"], c.get("L")
    st = {"case": c, "seed": seed}
    if kind == "score":
        st["seqs"] = _pack(_skew(_gen(seed), c["n"], L, c["p"]))
    elif kind == "pool":
        st["pool"] = labs.PoolBuffers.empty(L, c["cap"])
        st["e_max"] = (L * L) // (2 * c["tau"])
    elif kind == "batch":
        cfgs = []
        for x in range(c["L_lo"], c["L_hi"] + 1, 2):
            lo, hi = _tenure(dict(c, L=x))
            cfgs.append(dict(L=x, p=c["p"], steps=c["steps"], tenure_lo=lo, tenure_hi=hi, seed=seed, n_walkers=c["n"]))
        st["cfgs"], st["res"], st["ws"] = cfgs, None, None
    elif kind in ("step2", "even"):
        st["seqs"] = _seeds_for_step2(L, c["seeds"], seed)
    elif kind == "logits":
        st["net"] = learn.Network(L, _net_arrays(seed, L, c["hidden"]), c["hidden"], device=DEV)
        st["seqs"] = _pack(_skew(_gen(seed), c["n"], L, 0))
    elif kind == "train":
        net = learn.Network(L, _net_arrays(seed, L, c["hidden"]), c["hidden"], device=DEV)
        m, v = _moments(seed, L, c["hidden"])
        net.m.copy_(torch.from_numpy(labs.mlp_blob_from_dict(net.lay, m)))
        net.v.copy_(torch.from_numpy(labs.mlp_blob_from_dict(net.lay, v)))
        net.t = TRAIN_T
        s, _, mask, label = _batch(_gen(seed), L, c["n"])
        st["net"], st["seqs"], st["mask"], st["label"] = net, _pack(s), mask, label
    elif kind == "learned":
        st["net"] = learn.Network(L, _net_arrays(seed, L, c["hidden"]), c["hidden"], device=DEV)
    return st


# ------------------------------------------------------------------ one pass
def _walk_out(r):
    return {"final_seqs": r.final_seqs, "final_E": r.final_E, "best_seqs": r.best_seqs, "best_E": r.best_E,
            "best_step": r.best_step, "flip_evals": r.flip_evals}


def _step2_out(r):
    out = {q: r[q] for q in ("expansions", "pushes", "dup_skips", "evictions", "rounds", "open_count", "best_E",
                             "best_round")}
    out["best_seq"] = r["best_seq"]
    return out


def run(st):
    c = st["case"]
    kind, L = c["kind"], c.get("L")
    if kind == "score":
        E, C = labs.energy(L, st["seqs"], want_c=True)
        return {"E": E, "C": C, "dE": labs.flip_deltas(L, st["seqs"]),
                "dE_skew": labs.flip_deltas(L, st["seqs"], skew=True, p=c["p"])}
    if kind == "walk":
        lo, hi = _tenure(c)
        return _walk_out(labs.walk_step1(L, c["p"], c["steps"], lo, hi, st["seed"], c["n"]))
    if kind == "pool":
        lo, hi = _tenure(c)
        pool = st["pool"]
        pool.count.zero_()
        pool.dropped.zero_()
        r = labs.walk_step1(L, c["p"], c["steps"], lo, hi, st["seed"], c["n"], e_max=st["e_max"], pool=pool,
                            pool_walker_best=c["best"])
        top_s, top_E = labs.pool_topk(pool, 1024)
        return dict(_walk_out(r), top_seqs=top_s, top_E=top_E, count=pool.count, dropped=pool.dropped,
                    pool_E=pool.E, pool_seqs=pool.seqs, pool_walker=pool.walker, pool_step=pool.step)
    if kind == "bloom":
        return _walk_out(labs.walk_step1(L, c["p"], c["steps"], 0, 0, st["seed"], c["n"],
                                         bloom=(c["log2_bits"], c["n_hash"])))
    if kind == "batch":
        st["res"], st["ws"] = labs.walk_step1_batch(st["cfgs"], workspace=st["ws"], results=st["res"])
        outs = [_walk_out(r) for r in st["res"]]     # collated over the lengths
        return {q: torch.cat([o[q].reshape(-1) for o in outs]) for q in outs[0]}
    if kind == "step2":
        return _step2_out(labs.refine_step2(L, st["seqs"], c["batch"], c["queue"], c["pops"], NO_LIMIT, T_r=c["T_r"]))
    if kind == "even":
        minus, Em, plus, Ep = labs.length_operators(L, st["seqs"])
        r = labs.refine_step2(L - 1, minus, c["batch"], c["queue"], c["pops"], NO_LIMIT, T_r=c["T_r"])
        return dict(_step2_out(r), minus=minus, E_minus=Em, plus=plus, E_plus=Ep)
    if kind == "log":
        lo, hi = _tenure(c)
        seqs, mask, label = learn.log_plain(L, c["p"], c["steps"], lo, hi, st["seed"], c["n"], c["every"], device=DEV)
        return {"seqs": seqs, "mask": mask, "label": label}
    if kind == "train":
        net = st["net"]
        loss = net.train_step(st["seqs"], st["mask"], st["label"], lr=LR)
        return {"loss": loss, "grads": net.grads, "params": net.params, "m": net.m, "v": net.v,
                "params_bf16": net.params_bf16}
    if kind == "logits":
        return st["net"].logits(st["seqs"])[:, :(L - 1) // 2 + 1]
    lo, hi = _tenure(c)
    r = labs.learned_walk(L, c["p"], c["steps"], lo, hi, st["seed"], c["n"], top_m=c["top_m"], fallback_every=c["every"],
                          device=DEV, **st["net"].proposer_args())
    out = {q: r[q] for q in ("final_seqs", "final_E", "best_seqs", "best_E", "best_step", "flip_evals")}
    out["logits"] = st["net"].logits(r["final_seqs"])[:, :(L - 1) // 2 + 1]
    return out


# ------------------------------------------------------------------ what a pass cannot do without
def _mlp_flops(L, hidden):
    k = (L - 1) // 2
    return 2 * (hidden * (L + k) + hidden * hidden + hidden * (k + 1))


def work(case):
    c = case
    kind = c["kind"]
    L = c.get("L", 0)
    W, k = (L + 31) // 32, (L - 1) // 2
    n = c.get("n", 0)

    def walk(x, steps, walkers):
        # 4 operations a free position and even lag; sequences and energies out
        kx = (x - 1) // 2
        nf = kx + 1 - c["p"]
        return {"bytes": walkers * (8 * ((x + 31) // 32) + 12), "flops": 4 * kx * nf * steps * walkers}
    if kind == "score":
        nf = k + 1 - c["p"]
        return {"bytes": 4 * n * (3 * W + 1 + (L - 1) + L + nf), "flops": n * (L * L + 4 * (L - 1) * (L + nf))}
    if kind in ("walk", "bloom", "pool"):
        return walk(L, c["steps"], n)
    if kind == "batch":
        ws = [walk(x, c["steps"], n) for x in range(c["L_lo"], c["L_hi"] + 1, 2)]
        return {"bytes": sum(w["bytes"] for w in ws), "flops": sum(w["flops"] for w in ws)}
    if kind in ("step2", "even"):
        # every popped sequence, its key and energy once; 4 operations a neighbour and lag
        return {"bytes": c["pops"] * (4 * W + 16), "flops": c["pops"] * (L + 2 * c["T_r"]) * 4 * (L - 1)}
    if kind == "log":
        recs = n * (c["steps"] // c["every"])
        w = walk(L, c["steps"], n)
        return {"bytes": w["bytes"] + recs * 4 * (W + (k + 32) // 32 + 1), "flops": w["flops"]}
    f = _mlp_flops(L, c["hidden"])
    if kind == "train":
        return {"bytes": n * 4 * (W + (k + 32) // 32 + 1) + f // 2 * (4 * 7 + 2 * 2), "flops": 3 * f * n}
    if kind == "logits":
        return {"bytes": n * (4 * W + 4 * (k + 1)) + f, "flops": f * n}
    full = -(-c["steps"] // c["every"])
    nf = k + 1 - c["p"]
    return {"bytes": n * (8 * W + 12) + f + n * 4 * (k + 1),
            "flops": n * ((c["steps"] - full + 1) * f + 4 * k * (full * nf + (c["steps"] - full) * c["top_m"]))}


# ------------------------------------------------------------------ 64-bit values
def _autocorr(s):
    """C_1..C_{L-1} of +1/-1 rows by FFT in double (rounded: they are whole numbers)."""
    L = s.shape[1]
    F = torch.fft.rfft(s.double(), 2 * L)
    return torch.fft.irfft(F * F.conj(), 2 * L)[:, 1:L].round()


def _deltas(s, C, pairs):
    """dE of flipping each set {a, b} (0-based; a == b: one element)."""
    n, L = s.shape
    a = torch.tensor([x for x, _ in pairs], device=s.device)
    b = torch.tensor([y for _, y in pairs], device=s.device)
    d = torch.arange(1, L, device=s.device)
    pad = torch.nn.functional.pad(s.double(), (L, L))

    def t(x, skip):
        f, g = x[:, None] + d, x[:, None] - d
        return pad[:, f + L] * (f != skip[:, None]) + pad[:, g + L] * (g != skip[:, None])
    none = torch.full_like(a, -10 * L)
    dc = -2 * s.double()[:, a, None] * t(a, torch.where(a == b, none, b))
    dc = dc + torch.where(a == b, 0.0, 1.0)[None, :, None] * (-2 * s.double()[:, b, None] * t(b, torch.where(a == b, none, a)))
    return (dc * (2 * C[:, None, :] + dc)).sum(2)


def _exact_score(c, seed):
    L, p = c["L"], c["p"]
    k = (L - 1) // 2
    s = _skew(_gen(seed), c["n"], L, p)
    C = _autocorr(s)
    single = [(i, i) for i in range(L)]
    skew = [(i, L - 1 - i) for i in range(p, k + 1)]
    step = max(1, int(2e7 // (L * L)))
    dE, dS = [], []
    for i in range(0, c["n"], step):
        dE.append(_deltas(s[i:i + step], C[i:i + step], single))
        dS.append(_deltas(s[i:i + step], C[i:i + step], skew))
    return {"E": (C * C).sum(1), "C": C, "dE": torch.cat(dE), "dE_skew": torch.cat(dS)}


def _features(s):
    L = s.shape[1]
    C = _autocorr(s)[:, 1::2]
    m = torch.arange(1, (L - 1) // 2 + 1, device=s.device)
    return torch.cat([s.double(), C / (L - 2 * m)], 1)


def _gelu(x):
    return torch.nn.functional.gelu(x, approximate="tanh")


def _forward(P, X):
    h = _gelu(X @ P["W1"].T + P["b1"])
    h = _gelu(h @ P["W2"].T + P["b2"])
    return h @ P["W3"].T + P["b3"]


def _to64(d):
    return {q: torch.from_numpy(v).to(DEV).double() for q, v in d.items()}


def _blob(L, hidden, d):
    """The parameter blob of include/labs.h (each slice at a multiple of 64 elements,
    padded columns and rows zero)."""
    k = (L - 1) // 2
    ld_in, ld_out = -(-(L + k) // 64) * 64, -(-(k + 1) // 64) * 64
    out = []
    for q, rows, cols in (("W1", hidden, ld_in), ("b1", 1, hidden), ("W2", hidden, hidden), ("b2", 1, hidden),
                          ("W3", ld_out, hidden), ("b3", 1, ld_out)):
        full = torch.zeros((rows, cols), dtype=torch.float64, device=DEV)
        v = d[q] if d[q].dim() == 2 else d[q][None, :]
        full[:v.shape[0], :v.shape[1]] = v
        out.append(full.reshape(-1))
    return torch.cat(out)


def _exact_train(c, seed):
    L, hidden, n = c["L"], c["hidden"], c["n"]
    s, ok, _, label = _batch(_gen(seed), L, n)
    P = {q: v.requires_grad_(True) for q, v in _to64(_net_arrays(seed, L, hidden)).items()}
    z = _forward(P, _features(s))
    z = torch.where(ok, z, torch.full_like(z, -float("inf")))
    lab = label.long()[:, None]
    loss = (torch.logsumexp(z, 1) - z.gather(1, lab)[:, 0]).mean()
    loss.backward()
    m0, v0 = (_to64(x) for x in _moments(seed, L, hidden))
    t, b1, b2, eps = TRAIN_T + 1, 0.9, 0.999, 1e-8
    g = {q: P[q].grad for q in P}
    m = {q: b1 * m0[q] + (1 - b1) * g[q] for q in g}
    v = {q: b2 * v0[q] + (1 - b2) * g[q] * g[q] for q in g}
    new = {q: P[q].detach() - LR * (m[q] / (1 - b1 ** t)) / ((v[q] / (1 - b2 ** t)).sqrt() + eps) for q in g}
    return {"loss": loss.detach().reshape(1), "grads": _blob(L, hidden, g), "params": _blob(L, hidden, new),
            "m": _blob(L, hidden, m), "v": _blob(L, hidden, v), "params_bf16": None}


def exact(case, seed):
    if case["kind"] == "score":
        return _exact_score(case, seed)
    if case["kind"] == "train":
        return _exact_train(case, seed)
    if case["kind"] == "logits":
        s = _skew(_gen(seed), case["n"], case["L"], 0)
        with torch.no_grad():
            return _forward(_to64(_net_arrays(seed, case["L"], case["hidden"])), _features(s))
    return None
