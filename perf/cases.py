"""Measured workloads of the LDA sampler, through its public entry points.

A case is one call pattern of a fitting program on one corpus shape:

  step     a running fit goes on: ``iterate(n)``, the LLPT that watches the
           convergence (where ``llpt`` is set) and the assignment and topic
           totals to keep (``counts``)
  resume   a checkpoint is loaded into a handle (``set_assignments``), goes on
           for ``n`` iterations, is scored, and the whole model is exported
           (assignment, document-topic and word-topic tables)
  scratch  a whole fit of a new corpus: construct, ``iterate(n)``, LLPT, export

Corpora are planted mixtures made on the GPU from the seed alone: document
lengths are Poisson or lognormal, a document mixes a few of the planted topics,
words follow a Zipf law whose frequent words all topics share and whose rarer
words belong to a sixteenth of them.  The shapes are those of the repository's
workloads (news articles of about 330 tokens, abstracts of about 90, a skewed
web-scale collection, K = 16 to 32,768), at sizes that prepare in a second or
two, and generic ragged ones between them.

``exact`` recomputes the small ones in 64-bit torch, without this package.
"""
import math

import numpy as np
import torch

import paper_2007_08725_amd as lda

BETA = 0.01


def _case(name, kind, docs, mean, V, K, alpha, iters, *, sigma=0.0, cap=0, zipf=1.1, planted=200, start="random",
          warm=5, shuffle=False, chunks=0, g=2, two_branch=False, llpt=True):
    c = dict(kind=kind, docs=docs, mean=float(mean), sigma=float(sigma), cap=cap, V=V, zipf=float(zipf),
             planted=planted, K=K, alpha=float(alpha), iters=iters, start=start, warm=warm, shuffle=shuffle,
             chunks=chunks, g=g, two_branch=two_branch, llpt=llpt)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # one interactive iteration on a thousand short notes: launches and latency
        _case("notes_k16", "step", 1000, 50, 2000, 16, 50.0 / 16, 1, zipf=1.0, planted=20, llpt=False),
        # a mailbox in arrival order (tokens not sorted by document), odd sizes
        _case("mail_k101_unsorted", "step", 7919, 77, 9973, 101, 50.0 / 101, 10, sigma=1.0, planted=40, shuffle=True),
        # very short documents
        _case("posts_k2000", "step", 500_000, 18, 50_000, 2000, 0.025, 10, planted=300),
        # a new corpus fitted from nothing and exported
        _case("reviews_k256_scratch", "scratch", 60_000, 90, 40_000, 256, 50.0 / 256, 10, sigma=0.8, planted=100,
              warm=0),
        # a checkpoint loaded, continued by one iteration, scored and exported
        _case("checkpoint_k500_export", "resume", 60_000, 100, 60_000, 500, 0.1, 1, sigma=0.8, start="planted",
              warm=3),
        # news articles, K = 1,000: the early iterations of a fit
        _case("news_k1000", "step", 150_000, 330, 102_000, 1000, 0.05, 10, zipf=1.07),
        # abstracts, K = 1,000: the early iterations of the largest fit here
        _case("abstracts_k1000", "step", 1_600_000, 90, 141_000, 1000, 0.05, 10, sigma=0.8, planted=500),
        # the same shape near convergence, where many tokens skip
        _case("abstracts_k1000_late", "step", 500_000, 90, 141_000, 1000, 0.05, 10, sigma=0.8, planted=500,
              start="planted", warm=12),
        # a skewed web collection: documents from one token to 50,000, a million words
        _case("web_k1000_skewed", "step", 200_000, 150, 1_000_000, 1000, 0.05, 10, sigma=1.5, cap=50_000, zipf=1.2,
              planted=1000),
        # many topics
        _case("news_k10000", "step", 100_000, 330, 102_000, 10_000, 0.1, 5, zipf=1.07),
        # the most topics
        _case("news_k32768", "step", 60_000, 330, 102_000, 32_768, 0.05, 5, zipf=1.07),
        # the corpus kept in host memory and streamed in chunks
        _case("abstracts_k1000_chunked", "step", 300_000, 90, 141_000, 1000, 0.05, 5, sigma=0.8, planted=500,
              chunks=8),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step", "step", "step", "step", "resume", "scratch"])
    K = min(32_768, max(2, _log_uniform(rng, 16, 40_000)))
    tokens = _log_uniform(rng, 30_000, 30_000_000 if kind == "step" else 4_000_000)
    mean = _log_uniform(rng, 12, 400)
    sigma = rng.choice([0.0, 0.8, 1.5])
    docs = max(20, tokens // mean)
    V = _log_uniform(rng, 1000, 200_000)
    alpha = rng.choice([50.0 / K, 0.05, 0.1])
    start = rng.choice(["random", "planted"])
    chunks = rng.choice([0, 0, 0, 0, 3, 8]) if docs > 1000 and K <= 4000 else 0
    return _case(None, kind, docs, mean, V, K, alpha, rng.choice([1, 3, 10]) if K < 8000 else 3, sigma=sigma,
                 cap=20_000 if sigma > 1.0 else 0, zipf=rng.choice([1.0, 1.07, 1.2]), planted=rng.choice([20, 200]),
                 start=start, warm=0 if kind == "scratch" else rng.choice([2, 5, 9]),
                 shuffle=chunks == 0 and rng.random() < 0.25, chunks=chunks, g=rng.choice([1, 2, 2, 2, 3]),
                 two_branch=chunks == 0 and rng.random() < 0.1, llpt=True)


# ------------------------------------------------------------- corpora ----
def _tokens(case):
    return int(case["docs"] * case["mean"])


def _corpus(case, seed):
    """Token list and planted topics (int32, on the GPU): word, doc, topic."""
    g = torch.Generator(device="cuda").manual_seed(1_000_003 * (seed + 1))
    M, V, J = case["docs"], case["V"], case["planted"]

    def rand(*shape):
        return torch.rand(*shape, generator=g, device="cuda", dtype=torch.float32)

    if case["sigma"] > 0:
        mu = math.log(case["mean"]) - 0.5 * case["sigma"] ** 2
        lens = torch.exp(mu + case["sigma"] * torch.randn(M, generator=g, device="cuda")).round()
    else:
        lens = torch.poisson(torch.full((M,), case["mean"], device="cuda"), generator=g)
    lens = lens.clamp(1, case["cap"] or 60_000)
    # scaled to the case's token count, the remainder to random documents
    extra = torch.floor((lens - 1).double() * ((_tokens(case) - M) / max(1.0, float((lens - 1).sum())))).to(torch.int64)
    left = _tokens(case) - M - int(extra.sum())
    extra += left // M
    extra[torch.randperm(M, generator=g, device="cuda")[:left % M]] += 1
    lens = extra + 1
    doc = torch.repeat_interleave(torch.arange(M, device="cuda", dtype=torch.int32), lens)
    N = doc.numel()
    # a document mixes six slots of planted topics with falling weights
    slots = torch.randint(0, J, (M, 6), generator=g, device="cuda", dtype=torch.int32)
    wts = rand(M, 6) ** 3 + 1e-3
    cum = torch.cumsum(wts, 1) / wts.sum(1, keepdim=True)
    cdf = torch.cumsum((torch.arange(V, device="cuda", dtype=torch.float64) + 1.0) ** (-case["zipf"]), 0)
    cdf /= cdf[-1].clone()
    perm = torch.randperm(V, generator=g, device="cuda").to(torch.int32)
    word = torch.empty(N, dtype=torch.int32, device="cuda")
    topic = torch.empty(N, dtype=torch.int32, device="cuda")
    for b in range(0, N, 1 << 24):
        e = min(N, b + (1 << 24))
        dd = doc[b:e].long()
        pick = (rand(e - b, 1) > cum[dd]).sum(1).clamp(max=5)
        j = slots[dd, pick].long()
        rank = torch.searchsorted(cdf, torch.rand(e - b, generator=g, device="cuda", dtype=torch.float64))
        r1 = rank.clamp(max=V - 1) + 1
        # past the 64 most frequent words a topic uses a sixteenth of each octave of ranks
        octave = torch.floor(torch.log2(r1.double() + 0.5)).long()
        size = torch.bitwise_left_shift(torch.ones_like(octave), octave)
        size = torch.minimum(size, V + 1 - size)
        off = (r1 - torch.bitwise_left_shift(torch.ones_like(octave), octave)) % torch.clamp(size // 16, min=1)
        off = (off + (j * 7919 + octave * 104_729) * 2654435761 % 4294967296 % torch.clamp(size, min=1)) % size
        r2 = torch.where(octave >= 6, torch.bitwise_left_shift(torch.ones_like(octave), octave) + off, r1)
        word[b:e] = perm[r2 - 1]
        topic[b:e] = (j % case["K"]).to(torch.int32)
    if case["shuffle"]:
        p = torch.randperm(N, generator=g, device="cuda")
        word, doc, topic = word[p], doc[p], topic[p]
    return word, doc, topic


def _key(seed):
    return 42 + 7 * seed


T_PLANTED = 100  # the iteration count that a planted (late) start stands at


def prepare(case, seed):
    word, doc, topic = _corpus(case, seed)
    state = dict(case=case, word=word.cpu().numpy(), doc=doc.cpu().numpy(), key=_key(seed))
    del word, doc
    z0 = topic.cpu().numpy() if case["start"] == "planted" else None
    del topic
    torch.cuda.empty_cache()
    if case["kind"] != "scratch":
        m = _handle(state)
        if z0 is not None:
            m.set_assignments(z0, T_PLANTED)
        m.iterate(case["warm"])
        state["m"] = m
        if case["kind"] == "resume":
            got = m.counts(z=True, D=False, W=False)
            state["z"], state["t"] = got["z"], got["iteration"]
        state.pop("word"), state.pop("doc")
    if case["kind"] != "step":
        # the program's own arrays for an exported model: as many entries as a table of N tokens can have
        state["tables"] = {t + k: np.zeros(_tokens(case), np.int32) for t in "DW" for k in ("_topic", "_count")}
    return state


def _handle(state):
    c = state["case"]
    return lda.LDA(state["word"], state["doc"], c["V"], c["K"], c["alpha"], BETA, state["key"], g=c["g"],
                   two_branch=c["two_branch"], chunks=c["chunks"])


def run(state):
    c = state["case"]
    if c["kind"] == "scratch":
        with _handle(state) as m:
            m.iterate(c["iters"])
            return _answer(m, c, state["tables"])
    m = state["m"]
    if c["kind"] == "resume":
        m.set_assignments(state["z"], state["t"])
    m.iterate(c["iters"])
    return _answer(m, c, state.get("tables"))


def _answer(m, c, tables):
    out = {}
    if c["llpt"]:
        out["llpt"] = np.float64(m.loglik())
    got = m.counts(z=True, D=tables is not None, W=tables is not None)
    out.update({k: v for k, v in got.items() if k not in ("iteration", "M")})
    for k, a in (tables or {}).items():
        n = got[k].shape[0]
        a[:n] = got[k]
        a[n:] = 0
        out[k] = a
    return out


# ---------------------------------------------------------------- work ----
def _shape(case):
    """Tokens, expected entries of the D and of the W table."""
    N, K = _tokens(case), case["K"]
    topics = K * (1.0 - (1.0 - 1.0 / K) ** case["mean"])  # of a document whose topics spread over all of them
    row = topics if case["start"] == "random" else min(topics, 0.5 * case["mean"])
    return N, case["docs"] * row, min(N * 0.5, case["V"] * float(K)), row


def work(case):
    """Per iteration: word and document of each token read (8 B), its topic read and written (2 x 2 B), the count
    tables read and written (4 B an entry); two operations per token and entry of its document's row.  Scoring
    reads the tokens and tables once more; the outputs are written once (4 B a value)."""
    N, nd, nw, row = _shape(case)
    export = case["kind"] != "step"
    per_iter = 12.0 * N + 8.0 * (nd + nw)
    b = case["iters"] * per_iter + (8.0 * N + 4.0 * (nd + nw) if case["llpt"] else 0.0) + 4.0 * N
    if export:
        b += 8.0 * (nd + nw) + 4.0 * N
    return {"bytes": b, "flops": 2.0 * N * row * (case["iters"] + (1 if case["llpt"] else 0))}


def tolerance(case):
    """The draws are inverse-CDF decisions on 64-bit sums: another order of the sums moves an edge by a few 2^-53 of
    the total, so that a draw differs in about one of 1e12.  The LLPT is a 64-bit sum over the tokens: this path's
    and torch's, in another order, differed by up to 3e-16 at a million tokens, and region sums like the largest
    case's added one after another instead of in 256 strands by up to 5e-14."""
    return {"rel": 2e-13, "max": 2e-13, "differ": 1e-8}


# --------------------------------------------------------------- exact ----
_M32 = 0xFFFFFFFF


def _philox(i, t, purpose, key):
    """First two words of Philox4x32-10 for counters (i, 0, t, purpose), as int64 tensors."""
    c0, c1 = i.clone(), torch.zeros_like(i)
    c2, c3 = torch.full_like(i, t), torch.full_like(i, purpose)
    k0, k1 = key & _M32, (key >> 32) & _M32
    for _ in range(10):
        p0, p1 = c0 * 0xD2511F53, c2 * 0xCD9E8D57  # 64-bit products, wrapping
        h0, l0 = (p0 >> 32) & _M32, p0 & _M32
        h1, l1 = (p1 >> 32) & _M32, p1 & _M32
        c0, c1, c2, c3 = h1 ^ c1 ^ k0, l1, h0 ^ c3 ^ k1, l0
        k0, k1 = (k0 + 0x9E3779B9) & _M32, (k1 + 0xBB67AE85) & _M32
    return c0, c1


def exact(case, seed):
    word, doc, topic = (x.long() for x in _corpus(case, seed))
    N, M, V, K, alpha = word.numel(), case["docs"], case["V"], case["K"], case["alpha"]
    iters = case["warm"] + case["iters"]
    M = int(doc.max()) + 1
    if float(N) * K * (iters + 1) > 6e10 or float(max(M, V)) * K > 2e9:
        return None
    key, dev = _key(seed), word.device
    idx = torch.arange(N, device=dev)
    if case["start"] == "planted" and case["kind"] != "scratch":
        z, t = topic, T_PLANTED
    else:
        z, t = (_philox(idx, 0, 1, key)[0] * K) >> 32, 0
    step = max(1, 100_000_000 // K)

    def tables(z):
        D = torch.bincount(doc * K + z, minlength=M * K).view(M, K).to(torch.int32)
        W = torch.bincount(word * K + z, minlength=V * K).view(V, K).to(torch.int32)
        return D, W, torch.bincount(z, minlength=K)

    for _ in range(iters):
        D, W, T = tables(z)
        den = T.double() + V * BETA
        hi, lo = _philox(idx, t, 0, key)
        u = (((hi << 32) | lo) >> 11 & ((1 << 53) - 1)).double() * 2.0 ** -53
        new = torch.empty_like(z)
        cols = torch.arange(K, device=dev)
        for b in range(0, N, step):
            w = (W[word[b:b + step]].double() + BETA) / den
            d = D[doc[b:b + step]].double()
            if case["two_branch"]:
                m = torch.zeros(w.shape[0], 1, device=dev, dtype=torch.float64)
                k1 = torch.full((w.shape[0], 1), -1, device=dev)
            else:
                a1 = w.max(1, keepdim=True).values
                k1 = torch.where(w == a1, cols, K).min(1, keepdim=True).values  # the lowest id among equals
                m = a1 * (d.gather(1, k1) + alpha)
                w.scatter_(1, k1, 0.0)
            cs, cq = torch.cumsum(d * w, 1), torch.cumsum(alpha * w, 1)
            S, Q = cs[:, -1:], cq[:, -1:]
            x = u[b:b + step, None] * ((m + S) + Q)
            ks = (m + cs <= x).sum(1, keepdim=True)
            kq = ((m + S) + cq <= x).sum(1, keepdim=True)
            k = torch.where(x < m + S, ks, kq.clamp(max=K - 1))
            new[b:b + step] = torch.where(x < m, k1, k)[:, 0]
        z, t = new, t + 1
    D, W, T = tables(z)
    out = {"z": z.to(torch.int32), "T": T}
    if case["llpt"]:
        den = T.double() + V * BETA
        lens = torch.bincount(doc, minlength=M).double()
        total = 0.0
        for b in range(0, N, step):
            w = (W[word[b:b + step]].double() + BETA) / den
            dd = doc[b:b + step]
            p = ((D[dd].double() + alpha) * w).sum(1) / (lens[dd] + K * alpha)
            total += float(torch.log2(p).sum())
        out["llpt"] = np.float64(total / N)
    if case["kind"] != "step":
        for name, A in (("D", D), ("W", W)):
            r, k = torch.nonzero(A, as_tuple=True)
            out[name + "_off"] = torch.cat([torch.zeros(1, dtype=torch.int64, device=dev),
                                            torch.cumsum((A != 0).sum(1), 0)])
            for what, v in (("_topic", k.to(torch.int32)), ("_count", A[r, k])):
                out[name + what] = torch.zeros(N, dtype=torch.int32, device=dev)
                out[name + what][:v.numel()] = v
    return out
