"""The work that users of the library have it do, as cases that can be timed.

Each case goes through the public entry points (pulda.Plan, pulda.FoldIn,
server.serve, and the C ABI's device-to-device exports where the Python
binding would copy to the host).  Sizes are those of the synthetic
configurations in synth.CONFIGS, or parts of them.

Kinds of case:
  sweep     Algorithm 2 (or Algorithm 1's Phi-step) over a resident corpus:
            Phi-step, z-step with the count rebuild, log joint
  phi       a Phi-step from counts held elsewhere (a serving model's)
  loglik    the log joint of a state, from the counts and z
  foldin    theta of new documents: one request alone, or a closed loop of
            requests through the continuous-batching server
  heldout   left-to-right held-out log-likelihood of new documents

Inputs are drawn on the GPU from the LDA generative model (Zipf topic-word
rows, Polya-urn document topics), and a chain starts from the generating
topics, so that it is near its stationary state from the first pass on.
"""
import ctypes
import math

import numpy as np
import torch

from paper_1704_03581_amd import pulda, server

ALPHA, BETA, ZIPF = 0.1, 0.01, 1.07   # the priors and the word law of synth.py
DEV = "cuda"


# --------------------------------------------------------------------------
# the cases
# --------------------------------------------------------------------------
def _sweep(D, V, K, law, mean, sigma=0.0, n_long=0, max_len=0, n=1, method="polya_urn", priors="symmetric",
           graph=False, tune=False):
    return dict(kind="sweep", D=D, V=V, K=K, law=law, mean=mean, sigma=sigma, n_long=n_long, max_len=max_len, n=n,
                method=method, priors=priors, graph=graph, tune=tune)


def listed():
    return [
        # the smallest corpus a user samples (synth "tiny"): one sweep a call,
        # watching the log joint; launches and latency count
        dict(_sweep(1000, 5000, 20, "poisson", 50.0), name="sweep_tiny"),
        # long articles, few topics (synth "small"): several sweeps a call,
        # replayed as a graph
        dict(_sweep(1500, 12400, 100, "lognormal", 1200.0, 0.329, n=4, graph=True), name="sweep_small_graph"),
        # mail-like corpus whose longest documents have up to 20,000 tokens
        # (synth "medium"), schedule autotuned once
        dict(_sweep(40000, 28000, 1000, "lognormal", 120.0, 0.70, n_long=40, max_len=20000, tune=True),
             name="sweep_medium"),
        # abstracts (an eighth of synth "large"): the bulk throughput case,
        # schedule autotuned once
        dict(_sweep(1025000, 141000, 1000, "poisson", 90.0, tune=True), name="sweep_large"),
        # the paper's comparison: Algorithm 1's Dirichlet Phi-step, default
        # schedule
        dict(_sweep(100000, 28000, 1000, "poisson", 90.0, method="dirichlet"), name="sweep_dirichlet"),
        # vector priors alpha_k and beta_v, odd sizes, ragged lengths
        dict(_sweep(20011, 9973, 257, "lognormal", 150.0, 0.9, priors="vector"), name="sweep_vector_priors"),
        # building a serving model's Phi from counts (synth "large" sizes)
        dict(kind="phi", V=141000, K=1000, tokens=738000000, method="polya_urn", name="phi_large"),
        # evaluating a state: the log joint alone
        dict(kind="loglik", D=200000, V=28000, K=1000, law="poisson", mean=90.0, sigma=0.0, n_long=0, max_len=0,
             name="loglik"),
        # one new document of ordinary length, alone: latency
        dict(kind="foldin", V=141000, K=1000, tokens=738000000, requests=1, median=200.0, sigma=0.0, max_len=5000,
             sweeps=50, slots=64, name="foldin_one"),
        # a closed loop of requests through the server (lengths of synth's
        # fold-in requests)
        dict(kind="foldin", V=141000, K=1000, tokens=738000000, requests=2000, median=200.0, sigma=1.0, max_len=2000,
             sweeps=50, slots=1024, name="foldin_serve"),
        # held-out check of a few short documents with every particle's
        # normalisers; and the benchmark's: 1,000 documents of the fold-in
        # length law
        dict(kind="heldout", V=12400, K=100, tokens=1900000, docs=37, median=60.0, sigma=0.3, max_len=150,
             particles=20, group=32, want_Z=True, name="heldout_small"),
        dict(kind="heldout", V=141000, K=1000, tokens=738000000, docs=1000, median=200.0, sigma=1.0, max_len=500,
             particles=10, group=32, want_Z=False, name="heldout_large"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the listed ranges."""
    kind = rng.choice(["sweep", "sweep", "sweep", "phi", "loglik", "foldin", "foldin", "heldout"])
    K = _log_int(rng, 5, 1000)
    V = _log_int(rng, 500, 60000)
    if kind in ("sweep", "loglik"):
        mean = float(_log_int(rng, 20, 1200))
        tokens = _log_int(rng, 50000, 12000000)
        D = max(50, int(tokens / mean))
        law = rng.choice(["poisson", "lognormal"])
        sigma = round(rng.uniform(0.3, 0.9), 3) if law == "lognormal" else 0.0
        n_long = rng.choice([0, 0, 1, 7])
        if kind == "loglik":
            return dict(kind="loglik", D=D, V=V, K=K, law=law, mean=mean, sigma=sigma, n_long=n_long,
                        max_len=_log_int(rng, 3000, 20000))
        return _sweep(D, V, K, law, mean, sigma, n_long=n_long, max_len=_log_int(rng, 3000, 20000),
                      n=rng.choice([1, 1, 3]), method=rng.choice(["polya_urn", "polya_urn", "dirichlet"]),
                      priors=rng.choice(["symmetric", "symmetric", "vector"]), graph=rng.random() < 0.3,
                      tune=rng.random() < 0.25)
    if kind == "phi":
        return dict(kind="phi", V=V, K=K, tokens=_log_int(rng, 100000, 300000000),
                    method=rng.choice(["polya_urn", "polya_urn", "dirichlet"]))
    tokens = _log_int(rng, 1000000, 300000000)
    if kind == "foldin":
        return dict(kind="foldin", V=V, K=K, tokens=tokens, requests=rng.choice([1, 3, _log_int(rng, 10, 2000)]),
                    median=float(_log_int(rng, 15, 400)), sigma=round(rng.uniform(0.0, 1.0), 3),
                    max_len=_log_int(rng, 500, 2000), sweeps=rng.choice([20, 50]), slots=rng.choice([256, 1024]))
    return dict(kind="heldout", V=V, K=K, tokens=tokens, docs=_log_int(rng, 5, 1000),
                median=float(_log_int(rng, 15, 150)), sigma=round(rng.uniform(0.0, 0.8), 3),
                max_len=_log_int(rng, 150, 400), particles=rng.choice([1, 5, 10]), group=rng.choice([16, 32, 64]),
                want_Z=rng.random() < 0.3)


# --------------------------------------------------------------------------
# inputs, drawn on the GPU
# --------------------------------------------------------------------------
def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed) & 0x7FFFFFFF)


def _topic_word(V, K, g):
    """Generating topic-word rows (K x V): Dirichlet around a Zipf law whose
    ranks are scattered over the word ids."""
    f = (torch.arange(V, device=DEV, dtype=torch.float64) + 1.0) ** (-ZIPF)
    base = torch.empty_like(f)
    base[torch.randperm(V, device=DEV, generator=g)] = f / f.sum()
    rows = torch.empty(K, V, dtype=torch.float32, device=DEV)
    conc = (BETA * V * base).float()
    for k in range(0, K, 256):
        part = torch._standard_gamma(conc.expand(min(256, K - k), V).contiguous(), generator=g)
        part[:, int(base.argmax())] += 1e-30        # no row is empty
        rows[k:k + 256] = part / part.sum(1, keepdim=True)
    return rows


def _length_gen(case):
    """Document lengths belong to the case, not to the seed: every seed's
    inputs have the same sizes."""
    return _gen(sum(ord(c) * 31 ** (i % 5) for i, c in enumerate(repr(sorted(case.items())))))


def _doc_lengths(law, mean, sigma, D, g, n_long=0, max_len=0):
    if law == "poisson":
        lens = torch.poisson(torch.full((D,), mean, device=DEV), generator=g).long()
    else:
        lens = torch.exp(torch.randn(D, device=DEV, generator=g) * sigma + math.log(mean)).round().long().clamp_(min=1)
        lens.clamp_(max=20000)
    if n_long:
        # a few far longer documents, spaced geometrically up to max_len
        j = torch.arange(n_long, device=DEV, dtype=torch.float64) / max(1, n_long - 1)
        tail = (max_len * 10.0 ** (j - 1.0)).round().long() if n_long > 1 else torch.tensor([max_len], device=DEV)
        lens[torch.randperm(D, device=DEV, generator=g)[:n_long]] = tail
    return lens


def _documents(lens, rows, g):
    """(doc_off, words, z): topics by the Polya-urn sequence (a token copies
    an earlier token's topic, or draws a fresh one), words from the topics'
    rows."""
    K, V = rows.shape
    off = torch.zeros(len(lens) + 1, dtype=torch.int64, device=DEV)
    off[1:] = torch.cumsum(lens, 0)
    N = int(off[-1])
    start = torch.repeat_interleave(off[:-1], lens)
    i = torch.arange(N, device=DEV)
    j = i - start
    fresh = torch.rand(N, device=DEV, generator=g) * (K * ALPHA + j) < K * ALPHA
    parent = start + (torch.rand(N, device=DEV, generator=g, dtype=torch.float64) * j).long()
    parent = torch.where(fresh | (j == 0), i, parent)
    del start, j, fresh, i
    while True:
        up = parent[parent]
        if torch.equal(up, parent):
            break
        parent = up
    z = torch.randint(0, K, (N,), device=DEV, generator=g)[parent]
    del parent, up
    # word: the first whose cumulative row passes a uniform; the K rows'
    # cumulative sums lie one after the other, row k in [k, k + 1]
    cdf = torch.cumsum(rows, 1, dtype=torch.float64)
    cdf /= cdf[:, -1:].clone()
    cdf += torch.arange(K, device=DEV, dtype=torch.float64)[:, None]
    words = torch.empty(N, dtype=torch.int32, device=DEV)
    for a in range(0, N, 1 << 25):
        zz = z[a:a + (1 << 25)]
        u = torch.rand(len(zz), device=DEV, generator=g, dtype=torch.float64)
        w = torch.searchsorted(cdf.view(-1), zz + u, right=True) - zz * V
        words[a:a + (1 << 25)] = w.clamp_(0, V - 1).int()
    return off, words, z.to(torch.int16)


def _corpus(case, seed):
    g = _gen(seed)
    rows = _topic_word(case["V"], case["K"], g)
    lens = _doc_lengths(case["law"], case["mean"], case["sigma"], case["D"], _length_gen(case), case["n_long"],
                        case["max_len"])
    return _documents(lens, rows, g)


def _priors(case):
    if case.get("priors", "symmetric") == "symmetric":
        return ALPHA, BETA
    r = np.random.default_rng(case["K"] * 100003 + case["V"])
    return r.uniform(0.02, 0.3, case["K"]), r.uniform(0.002, 0.05, case["V"])


def _model(case, seed):
    """A plan without a corpus whose counts are those of a trained model of
    `tokens` tokens, and the generating rows."""
    g = _gen(seed)
    V, K = case["V"], case["K"]
    rows = _topic_word(V, K, g)
    share = torch._standard_gamma(torch.ones(K, device=DEV), generator=g)
    share = share / share.sum() * case["tokens"]
    plan = pulda.Plan(K, V, 0, 0, alpha=ALPHA, beta=BETA, seed=int(seed) % 1000003 + 1)
    n = torch.empty(V, K, dtype=torch.int32, device=DEV)
    for k in range(0, K, 256):
        n[:, k:k + 256] = torch.poisson(rows[k:k + 256] * share[k:k + 256, None], generator=g).int().t()
    plan.set_counts(n.view(-1))
    return plan, rows, g


def _new_documents(case, count, rows, g):
    """Documents as host word lists, lengths LogNormal in [10, max_len]."""
    lens = torch.exp(torch.randn(count, device=DEV, generator=_length_gen(case)) * case["sigma"] +
                     math.log(case["median"]))
    off, words, _ = _documents(lens.round().long().clamp_(10, case["max_len"]), rows, g)
    off, words = off.cpu().numpy(), words.cpu().numpy()
    return [words[off[i]:off[i + 1]].copy() for i in range(count)]


# the C ABI's exports into device memory
_abi = ctypes.CDLL(pulda.LIB_PATH)
_abi.pulda_get_z.argtypes = [ctypes.c_void_p] * 3
_abi.pulda_get_phi.argtypes = [ctypes.c_void_p, ctypes.POINTER(pulda.PhiView), ctypes.c_void_p]


def _call(fn, *args):
    status = fn(*args)
    if status != pulda.PULDA_OK:
        raise RuntimeError(f"pulda status {status}")


def prepare(case, seed):
    kind = case["kind"]
    if kind in ("sweep", "loglik"):
        off, words, z = _corpus(case, seed)
        alpha, beta = _priors(case)
        plan = pulda.Plan(case["K"], case["V"], case["D"], int(off[-1]), alpha=alpha, beta=beta,
                          seed=int(seed) % 1000003 + 1)
        plan.upload(off, words)
        plan.init(z.cpu().numpy().view(np.uint16))
        if kind == "loglik":
            return dict(kind=kind, plan=plan)
        plan.set_phi_method(case["method"])
        if case["tune"]:
            plan.phi_step(1)
            plan.autotune(1)
        plan.set_graph(case["graph"])
        return dict(kind=kind, plan=plan, t=1, n=case["n"], z=z)
    plan, rows, g = _model(case, seed)
    if kind == "phi":
        plan.set_phi_method(case["method"])
        V, K = case["V"], case["K"]
        cap = V * K
        out = dict(colptr=torch.zeros(V + 1, dtype=torch.int64, device=DEV),
                   topic=torch.zeros(cap, dtype=torch.int16, device=DEV),
                   gamma=torch.zeros(cap, dtype=torch.int32, device=DEV),
                   phi=torch.zeros(cap, dtype=torch.float32, device=DEV),
                   alias_thr=torch.zeros(cap, dtype=torch.int32, device=DEV),
                   alias_topic=torch.zeros(cap, dtype=torch.int16, device=DEV),
                   sigma_a=torch.zeros(V, dtype=torch.float64, device=DEV),
                   S=torch.zeros(K, dtype=torch.int64, device=DEV))
        view = pulda.PhiView(*[out[f].data_ptr() for f, _ in pulda.PhiView._fields_])
        if case["method"] == "dirichlet":
            view.S = None          # the urn's integer row sums are not this step's
        return dict(kind=kind, plan=plan, t=1, out=out, view=view)
    plan.phi_step(1)
    if kind == "foldin":
        reqs = _new_documents(case, case["requests"], rows, g)
        fi = pulda.FoldIn(plan, sweeps=case["sweeps"], burn_in=case["sweeps"] // 2, max_slots=case["slots"],
                          arena_tokens=case["slots"] * 600 + case["max_len"], max_len=case["max_len"], seed=7)
        return dict(kind=kind, plan=plan, server=fi, reqs=reqs)
    return dict(kind=kind, plan=plan, docs=_new_documents(case, case["docs"], rows, g), particles=case["particles"],
                group=case["group"], want_Z=case["want_Z"])


def run(state):
    kind, plan = state["kind"], state["plan"]
    if kind == "sweep":
        ll = plan.sweep(state["t"], state["n"])
        state["t"] += state["n"]
        z = state["z"]
        _call(_abi.pulda_get_z, plan._h, z.data_ptr(), torch.cuda.current_stream().cuda_stream)
        return dict(ll=ll, z=z)
    if kind == "phi":
        plan.phi_step(state["t"])
        state["t"] += 1
        _call(_abi.pulda_get_phi, plan._h, ctypes.byref(state["view"]), torch.cuda.current_stream().cuda_stream)
        return state["out"]
    if kind == "loglik":
        return dict(ll=plan.loglik())
    if kind == "foldin":
        reqs = state["reqs"]
        if len(reqs) == 1:
            res = [state["server"].run_one(0, reqs[0])]
        else:
            rep = server.serve(state["server"], reqs)
            res = [rep.results[i] for i in range(len(reqs))]
        return dict(theta=np.stack([r["theta"] for r in res]), loglik=np.array([r["loglik"] for r in res]),
                    kept=np.array([r["kept"] for r in res]))
    got = plan.heldout_loglik(state["docs"], particles=state["particles"], group=state["group"],
                              want_Z=state["want_Z"])
    out = dict(ll=got[0], kept=got[1])
    if state["want_Z"]:
        # every document's particles x kept array (zeros for dropped tokens)
        out["Z"] = np.concatenate([np.pad(Z, ((0, 0), (0, len(d) - Z.shape[1]))).reshape(-1)
                                   for Z, d in zip(got[2], state["docs"])])
    return out


# --------------------------------------------------------------------------
# the least work, and exact values
# --------------------------------------------------------------------------
def _topics_in(length, K):
    """Expected topics of a document of that many tokens (Polya urn)."""
    A = K * ALPHA
    return min(float(K), A * math.log1p(length / A)) if length > 0 else 0.0


def work(case):
    kind, V, K = case["kind"], case["V"], case["K"]
    if kind in ("sweep", "loglik"):
        N = case["D"] * case["mean"] * math.exp(case["sigma"] ** 2 / 2)
        if kind == "loglik":
            # word ids are in the counts: z, offsets and the counts are read
            return dict(bytes=2 * N + 8 * case["D"] + 4.0 * V * K, flops=2.0 * min(N, float(V) * K))
        # per sweep: word id, z read and written, the counts read and written,
        # a product and a sum per topic of the token's document
        per = 8 * N + 8 * case["D"] + 8.0 * V * K
        return dict(bytes=case["n"] * per, flops=case["n"] * 2 * N * _topics_in(case["mean"], K))
    if kind == "phi":
        # counts read once; the nonzeros of Phi and their alias entries
        nnz = min(float(V) * K, 0.12 * V * K if case["method"] == "polya_urn" else 0.6 * V * K)
        return dict(bytes=4.0 * V * K + 16 * nnz + 16.0 * V, flops=20.0 * nnz)
    mean = min(case["median"] * math.exp(case["sigma"] ** 2 / 2), float(case["max_len"]))
    if kind == "foldin":
        draws = case["requests"] * mean * case["sweeps"]
        return dict(bytes=case["requests"] * (4 * mean + 4.0 * K) + 4 * draws, flops=2 * draws * _topics_in(mean, K))
    draws = case["docs"] * case["particles"] * mean * (mean + 1) / 2
    return dict(bytes=case["docs"] * (4 * mean + 16) + 2 * draws, flops=2 * draws * _topics_in(mean / 2, K))


def exact(case, seed):
    """The log joint by its definition in fp64.  The other outputs are random
    draws keyed by the seed: only the sampler itself gives their values."""
    if case["kind"] != "loglik":
        return None
    off, words, z = _corpus(case, seed)
    K, V, A = case["K"], case["V"], case["K"] * ALPHA
    z = z.long() & 0xFFFF
    n = torch.bincount(words.long() * K + z, minlength=V * K).double().view(V, K)
    ll = K * math.lgamma(V * BETA) - torch.lgamma(n.sum(0) + V * BETA).sum()
    used = n[n > 0]
    ll = ll + (torch.lgamma(used + BETA) - math.lgamma(BETA)).sum()
    lens = off[1:] - off[:-1]
    doc = torch.repeat_interleave(torch.arange(case["D"], device=DEV), lens)
    _, m = torch.unique(doc * K + z, return_counts=True)
    ll = ll + (torch.lgamma(m.double() + ALPHA) - math.lgamma(ALPHA)).sum()
    ll = ll + (math.lgamma(A) - torch.lgamma(lens.double() + A)).sum()
    return dict(ll=float(ll))
