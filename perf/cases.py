"""Workloads whose speed matters to a user of the sampler, as calls of its public entry points.

``listed()`` names the standing ones, ``draw(rng)`` gives further ones of the same ranges; ``prepare`` makes what a
program has in hand before the call (a corpus and a sampler built on it), ``run`` is one pass of the call and returns
everything that call computes, ``work`` the bytes and operations no implementation can do without, ``tolerance`` and
``exact`` what the results may be compared with.

Corpora are drawn on the GPU from the LDA generative process with planted topics (Zipf-ordered vocabulary, sparse
document mixtures, lognormal or constant document lengths); the shapes are those of the benchmark's corpora and of
document prefixes of them, plus small and odd ones.
"""
import math

import numpy as np
import torch

import paper_1610_02496_amd as pk

BETA = 0.01


def _case(name, kind, D, V, T, sigma, K_true, K, n=0, zipf=1.07, doc_conc=0.05, workers=0, chunks=0, m=0):
    """D documents with T tokens over V words (lengths lognormal with `sigma`, 0: equal), drawn from K_true planted
    topics, fitted with K; n: iterations (training) or fold-in iterations (holdout); workers, chunks: host streaming;
    m: tokens inspected."""
    c = {"kind": kind, "D": D, "V": V, "T": T, "sigma": sigma, "K_true": K_true, "K": K, "n": n, "zipf": zipf,
         "doc_conc": doc_conc, "workers": workers, "chunks": chunks, "m": m}
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # Training, ten iterations and a checkpoint of the assignments.
        # A first experiment on a thousand short texts: a chain of short launches.
        _case("train_unit", "train", 1000, 5000, 100_000, 0.0, 100, 100, n=10, zipf=1.1, doc_conc=0.1),
        # A newsgroup- or abstract-sized collection with an odd number of topics.
        _case("train_small", "train", 18_846, 30_011, 2_261_513, 0.9, 100, 777, n=10),
        # A tenth of the NYTimes-shaped corpus at a moderate number of topics.
        _case("train_news_prefix", "train", 30_000, 100_000, 10_000_000, 0.8, 1000, 1000, n=10),
        # The NYTimes-shaped corpus in full in the sparse regime (the benchmark's workload and number of iterations).
        _case("train_news_full", "train", 300_000, 100_000, 100_000_000, 0.8, 1000, 10_000, n=20),
        # A prefix of the PubMed-shaped corpus: many short documents, a large share of the tokens on the dense term.
        _case("train_abstracts", "train", 400_000, 141_000, 36_000_000, 0.6, 1000, 5000, n=10, zipf=1.05),
        # A prefix of the web-shaped corpus: long, heavy-tailed documents, and more topics than a workgroup's usual
        # share of LDS takes.
        _case("train_web", "train", 41_001, 100_000, 15_006_366, 1.0, 1000, 20_011, n=10, zipf=1.05, doc_conc=0.03),
        # More topics than 16 bits number: 32-bit assignments, rows that do not fit LDS.
        _case("train_many_topics", "train", 12_007, 4001, 1_500_875, 0.8, 500, 70_000, n=5),
        # A corpus that is streamed from the host in chunks.
        _case("train_streamed", "train", 60_000, 60_000, 20_000_000, 0.8, 500, 2000, n=10, workers=3, chunks=4),
        # The quality metric a training loop asks for every few iterations.
        _case("loglik", "loglik", 30_000, 100_000, 10_000_000, 0.8, 1000, 1000),
        # Scoring of held-out documents on a trained model: layout, ten fold-in iterations, score.
        _case("holdout", "holdout", 20_000, 50_000, 6_600_000, 0.8, 500, 1000, n=10),
        # Export of a trained model: A in CSR, B, topic totals.
        _case("export", "export", 20_000, 20_000, 5_000_000, 0.8, 500, 500),
        # Inspection: normalisers of a sample of the tokens, the topic distribution of a few hundred words.
        _case("inspect", "inspect", 20_000, 50_000, 5_000_000, 0.8, 500, 1500, m=100_000),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["train"] * 7 + ["loglik", "holdout", "export", "inspect"])
    T = _log_uniform(rng, 50_000, 30_000_000 if kind == "train" else 8_000_000)
    mean_len = _log_uniform(rng, 30, 600)
    D = max(50, T // mean_len)
    V = _log_uniform(rng, 2000, 100_000)
    K = _log_uniform(rng, 20, 16_000 if kind in ("train", "loglik") else 2000)
    if kind == "train" and rng.random() < 0.15:        # beyond LDS, beyond 16 bits
        K, V, T = _log_uniform(rng, 30_000, 80_000), _log_uniform(rng, 2000, 4000), min(T, 2_000_000)
        D = max(50, T // mean_len)
    if kind in ("loglik", "holdout", "inspect"):       # (these are also computed densely in 64 bits)
        V = min(V, 40_000)
        K = min(K, 4000)
    K_true = max(8, min(K, _log_uniform(rng, 20, 1000)))
    stream = kind == "train" and K < 16_000 and rng.random() < 0.15
    return _case("", kind, D, V, T, round(rng.uniform(0.0, 1.0), 3), K_true, max(K, K_true),
                 n=rng.randint(5, 10) if kind == "train" else rng.choice([0, 5, 10]) if kind == "holdout" else 0,
                 zipf=round(rng.uniform(1.05, 1.1), 4), doc_conc=round(rng.uniform(0.03, 0.1), 4),
                 workers=3 if stream else 0, chunks=rng.randint(2, 6) if stream else 0,
                 m=_log_uniform(rng, 100, 100_000) if kind == "inspect" else 0)


def _corpus(c, seed):
    """(doc_ptr int64 [D+1], word_ids int32 [T], planted topics int32 [T]) as host arrays, from the seed alone."""
    dev = torch.device("cuda")
    g = torch.Generator(device=dev)
    g.manual_seed(seed)
    D, V, T, Kt = c["D"], c["V"], c["T"], c["K_true"]
    raw = np.exp(c["sigma"] * np.random.default_rng(D).standard_normal(D))   # lengths belong to the case, not the seed
    doc_ptr = np.zeros(D + 1, dtype=np.int64)
    doc_ptr[1:] = np.rint(np.cumsum(raw) * (T / raw.sum())).astype(np.int64)
    doc_ptr[D] = T
    # planted topics: Dirichlet(0.01 V m), m Zipf over the vocabulary; as one ascending sequence, topic k in (k, k+1]
    m = torch.arange(1, V + 1, device=dev, dtype=torch.float64) ** -c["zipf"]
    shape = (0.01 * V * m / m.sum()).float()
    words = torch.empty((Kt, V), device=dev, dtype=torch.float64)
    for k in range(0, Kt, 128):
        rows = torch._standard_gamma(shape.expand(min(128, Kt - k), V).contiguous(), generator=g).double().cumsum(1)
        words[k:k + 128] = rows / rows[:, -1:]
    words += torch.arange(Kt, device=dev, dtype=torch.float64)[:, None]
    words = words.view(-1)
    lengths = torch.from_numpy(np.diff(doc_ptr)).to(dev)
    word_ids, planted = np.empty(T, dtype=np.int32), np.empty(T, dtype=np.int32)
    block = max(1, 20_000_000 // Kt)                       # documents at a time
    for d in range(0, D, block):
        n = min(block, D - d)
        mix = torch._standard_gamma(torch.full((n, Kt), c["doc_conc"], device=dev), generator=g).double().cumsum(1)
        mix = mix / mix[:, -1:] + torch.arange(n, device=dev, dtype=torch.float64)[:, None]
        doc = torch.repeat_interleave(torch.arange(n, device=dev), lengths[d:d + n])
        u = torch.rand((2, doc.numel()), device=dev, dtype=torch.float64, generator=g)
        k = (torch.searchsorted(mix.view(-1), doc + u[0]) - doc * Kt).clamp_(0, Kt - 1)
        w = (torch.searchsorted(words, k + u[1]) - k * V).clamp_(0, V - 1)
        a, b = int(doc_ptr[d]), int(doc_ptr[d + n])
        planted[a:b] = k.int().cpu().numpy()
        word_ids[a:b] = w.int().cpu().numpy()
    return doc_ptr, word_ids, planted


def _alpha(c):
    return 50.0 / c["K"]


def _export_topics(c, doc_ptr, seed):
    """Assignments with as many distinct topics per document as the case fixes (a third of its tokens, some frequent, many
    rare): what is exported then has the same size for every seed."""
    r = np.random.default_rng(seed)
    length = np.diff(doc_ptr)
    i = (np.arange(c["T"]) - np.repeat(doc_ptr[:-1], length)) / np.repeat(np.maximum(length, 1), length)
    kd = np.clip(length // 3, 1, c["K"])
    first, step = r.integers(0, c["K"], c["D"]), 1
    while step == 1 or math.gcd(step, c["K"]) > 1:
        step = int(r.integers(2, c["K"] + 2))
    return ((np.repeat(first, length) + (np.repeat(kd, length) * i * i).astype(np.int64) * step) % c["K"]).astype(np.int32)


def _held_out(c, doc_ptr, word_ids, planted):
    """The last sixth of the documents as held-out ones, every second token of them observed."""
    d0 = c["D"] - max(1, c["D"] // 6)
    t0 = int(doc_ptr[d0])
    hp = doc_ptr[d0:] - t0
    T = int(hp[-1])
    observed = ((np.arange(T) - np.repeat(hp[:-1], np.diff(hp))) % 2 == 0).astype(np.uint8)
    return doc_ptr[:d0 + 1], t0, hp, word_ids[t0:], observed, planted[t0:][observed != 0]


def prepare(case, seed):
    """The corpus and a sampler on it: at its initial assignment for training, at a trained model's (the planted
    topics) for the calls that look at a model."""
    c = case
    doc_ptr, word_ids, planted = _corpus(c, seed)
    state = {"case": c}
    if c["kind"] == "train":
        opts = {"stream_workers": c["workers"], "n_chunks": c["chunks"]} if c["workers"] else {}
        state["sampler"] = pk.Saber(doc_ptr, word_ids, c["V"], c["K"], _alpha(c), BETA, seed, **opts)
        return state
    if c["kind"] == "holdout":
        doc_ptr, t0, state["hp"], state["hw"], state["observed"], z0 = _held_out(c, doc_ptr, word_ids, planted)
        word_ids, planted = word_ids[:t0], planted[:t0]
        state["z_init"] = z0 if c["n"] == 0 else None
        state["seed"] = seed + 1
    if c["kind"] == "export":
        planted = _export_topics(c, doc_ptr, seed)
    s = pk.Saber(doc_ptr, word_ids, c["V"], c["K"], _alpha(c), BETA, seed)
    s.set_z(planted, 10)
    state["sampler"] = s
    if c["kind"] == "inspect":
        state["tok"], state["words"] = _inspected(c, seed)
    return state


def _inspected(c, seed):
    """Tokens and words looked at: a sample of all tokens; the most frequent words and some of the others."""
    r = np.random.default_rng(seed)
    return r.integers(0, c["T"], c["m"]), np.r_[np.arange(200), r.integers(200, c["V"], 200)].astype(np.int32)


def run(state):
    c, s = state["case"], state["sampler"]
    if c["kind"] == "train":
        s.iterate(c["n"])
        return {"z": s.get_z()}
    if c["kind"] == "loglik":
        return {"ll": s.loglik()}
    if c["kind"] == "holdout":
        ll, scored, z = s.holdout_loglik(state["hp"], state["hw"], state["observed"], c["n"], state["seed"],
                                         state["z_init"])
        return {"ll": ll, "scored": scored, "z": z}
    if c["kind"] == "export":
        cd_ptr, topic, count, cwk, ck = s.counts()
        return {"cd_ptr": cd_ptr, "topic": topic, "count": count, "cwk": cwk, "ck": ck}
    S, Q, p = s.token_probs(state["tok"])
    phi, prefix = s.get_phi(state["words"])
    return {"S": S, "Q": Q, "p": p, "phi": phi, "prefix": prefix}


def work(case):
    """Each input read once, each output written once.  A training iteration reads the token list and the assignments,
    writes the new ones, and writes and reads the non-zero counts of A and B with Bhat beside them (at most one per
    token and cell); a token's product loop takes two operations per topic of its document (about half as many as
    the document has tokens)."""
    c = case
    T, D, V, K = c["T"], c["D"], c["V"], c["K"]
    zb = 2 if K <= 65536 else 4
    per_token = min(K, max(1.0, 0.5 * T / D))
    nnz_a, nnz_b = min(0.5 * T, float(D) * K), min(0.5 * T, float(V) * K)
    sweep = T * (4 + 2 * zb) + 8 * D + 8 * nnz_a + 12 * nnz_b
    if c["kind"] == "train":
        return {"bytes": c["n"] * sweep + 4 * T, "flops": c["n"] * T * (2 * per_token + 20)}
    if c["kind"] == "loglik":
        return {"bytes": 4 * T + 8 * D + 4 * nnz_a + 8 * nnz_b, "flops": T * (2 * per_token + 20)}
    if c["kind"] == "holdout":
        H = T / 6
        return {"bytes": H * 5 + 8 * nnz_b + max(1, c["n"]) * H / 2 * (4 + 2 * zb), "flops": (c["n"] + 1) * H / 2 * per_token}
    if c["kind"] == "export":
        return {"bytes": 16 * nnz_a + 4.0 * V * K + 8 * K + 8 * D + zb * T, "flops": T}
    return {"bytes": 20 * c["m"] + 4 * per_token * c["m"] + 400 * 12.0 * K, "flops": 2 * per_token * c["m"] + 400 * 2.0 * K}


def tolerance(case):
    """Assignments and counts are whole numbers of a path that is deterministic from the seed on, so they stay the same.
    Floating results are binary32 sums of at most a few thousand positive terms (S, Q), single-rounded quotients and
    running sums (Bhat and its prefixes), or binary64 means of their logarithms."""
    if case["kind"] in ("train", "export"):
        return "exact"
    if case["kind"] in ("loglik", "holdout"):
        return {"rel": 3e-7, "max": 3e-7, "differ": 0.0}
    return {"rel": 3e-7, "max": 3e-6}


def _model64(c, doc_ptr, word_ids, planted):
    """(A, Bhat, doc of every token) of the planted assignment, dense, in 64 bits."""
    dev = torch.device("cuda")
    D, V, K = len(doc_ptr) - 1, c["V"], c["K"]
    beta = float(np.float32(BETA))
    w = torch.from_numpy(word_ids.astype(np.int64)).to(dev)
    z = torch.from_numpy(planted.astype(np.int64)).to(dev)
    d = torch.repeat_interleave(torch.arange(D, device=dev), torch.from_numpy(np.diff(doc_ptr)).to(dev))
    B = torch.bincount(w * K + z, minlength=V * K).view(V, K).double()
    return (d, w, z), (B + beta) / (B.sum(0) + V * beta)


def _dots64(A, phi, doc, word):
    """sum_k A[doc, k] phi[word, k] for the tokens given, by blocks of documents."""
    out = torch.empty(doc.numel(), device=A.device, dtype=torch.float64)
    block = max(1, 200_000_000 // phi.shape[0])
    for d in range(0, A.shape[0], block):
        sel = torch.nonzero((doc >= d) & (doc < d + block)).view(-1)
        if sel.numel():
            out[sel] = (A[d:d + block] @ phi.T)[doc[sel] - d, word[sel]]
    return out


def exact(case, seed):
    c = case
    if c["kind"] not in ("loglik", "holdout", "inspect") or (c["kind"] == "holdout" and c["n"]):
        return None
    dev = torch.device("cuda")
    doc_ptr, word_ids, planted = _corpus(c, seed)
    alpha, K = float(np.float32(_alpha(c))), c["K"]
    if c["kind"] == "holdout":
        doc_ptr, t0, hp, hw, observed, z0 = _held_out(c, doc_ptr, word_ids, planted)
        _, phi = _model64(c, doc_ptr, word_ids[:t0], planted[:t0])
        H = len(hp) - 1
        hd = torch.repeat_interleave(torch.arange(H, device=dev), torch.from_numpy(np.diff(hp)).to(dev))
        o = torch.from_numpy(observed != 0).to(dev)
        A = torch.bincount(hd[o] * K + torch.from_numpy(z0.astype(np.int64)).to(dev), minlength=H * K).view(H, K).double()
        sd, sw = hd[~o], torch.from_numpy(hw.astype(np.int64)).to(dev)[~o]
        ll = torch.log(_dots64(A, phi, sd, sw) + alpha * phi.sum(1)[sw]) - torch.log(A.sum(1) + K * alpha)[sd]
        return {"ll": float(ll.sum() / max(1, ll.numel())), "scored": None, "z": None}
    (d, w, z), phi = _model64(c, doc_ptr, word_ids, planted)
    A = torch.bincount(d * K + z, minlength=c["D"] * K).view(c["D"], K).double()
    if c["kind"] == "loglik":
        ll = torch.log(_dots64(A, phi, d, w) + alpha * phi.sum(1)[w]) - torch.log(A.sum(1) + K * alpha)[d]
        return {"ll": float(ll.mean())}
    tok, words = _inspected(c, seed)
    t = torch.from_numpy(tok).to(dev)
    S = _dots64(A, phi, d[t], w[t])
    Q = alpha * phi.sum(1)[w[t]]
    rows = phi[torch.from_numpy(words.astype(np.int64)).to(dev)]
    return {"S": S, "Q": Q, "p": S / (S + Q), "phi": rows, "prefix": rows.cumsum(1)}
