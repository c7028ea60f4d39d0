"""The per-word precompute by topic list below K = 4,096 (small words by 16 lanes, larger ones by a wave), against the oracle."""
import numpy as np
import pytest

import lda_synth
import oracle
from gpu_common import SEED, compare_draws, corpus_kw, make_lda, oracle_step, say

pytestmark = pytest.mark.gpu


# K = 500 and 512: the list is every topic; 513: one more; 4,095 and 4,096: the counted list's last K and the sorted
# list's first.  Enough words for the list to be used (4M table entries).
@pytest.mark.parametrize("K", [500, 512, 513, 1000, 4095, 4096])
def test_records_by_topic_list_follow_the_oracle(K):
    rng = np.random.default_rng(K)
    V = (5 << 20) // K
    counts = rng.integers(1, 9, V)
    counts[:12] = [64, 65, 63, 1, 16, 17, 200, K - 1, K, K, 2, 40]  # K tokens: the largest sparse word
    word = np.repeat(np.arange(V, dtype=np.int32), counts)
    n_docs = max(40, word.size // 60)
    doc = rng.integers(0, n_docs, word.size).astype(np.int32)
    doc[0] = n_docs - 1
    order = np.argsort(doc, kind="stable")
    word, doc = word[order], doc[order]
    spec = lda_synth.CorpusSpec("records", n_docs, ("poisson", 1.0), V, 0.0, K, K, 0.05)
    c = lda_synth.Corpus(spec, word, doc, V, n_docs)
    # few topics for most tokens (ties of T among the many unused ones); one word whose row holds every topic but two
    # (no topic of a 512-topic list is outside it), one whose row holds all of them
    z = rng.integers(0, 30, c.N).astype(np.int32)
    for w, skip in ((8, 2), (9, 0)):
        at = np.nonzero(word == w)[0]
        z[at] = np.arange(at.size) % (K - skip)
    with make_lda(c, always_skip_test=True) as m:
        for t in (3, 4):
            say("word records K=%d V=%d t=%d" % (K, V, t))
            m.set_assignments(z, t)
            want, flags, ost = oracle_step(c, z, t)
            st = m.iterate(1, stats=True)[0]
            got = m.counts(D=False, W=False)["z"]
            compare_draws(got, want, flags, max(c.N, 10 ** 6))
            assert st["skip_step3"] <= ost["skip3"] <= st["skip_step3"] + max(2, c.N // 1000)
            assert m.loglik() == pytest.approx(oracle.llpt(c.word, c.doc, got, **corpus_kw(c)), rel=1e-12)
            z = got


# beta so large that every W^ is the same number: K1 is topic 0 for every word, whatever T is
@pytest.mark.parametrize("K", [1000, 4096])
@pytest.mark.parametrize("beta", [1e18, 1e300])
def test_equal_w_hat_takes_the_lowest_topic(K, beta):
    import paper_2007_08725_amd as lda
    rng = np.random.default_rng(K)
    V, M, alpha = (5 << 20) // K, 300, 0.05
    word = np.repeat(np.arange(V, dtype=np.int32), rng.integers(1, 9, V))
    word = np.r_[word, np.full(K - 10, 7, np.int32)]  # one word past 64 tokens
    doc = np.sort(rng.integers(0, M, word.size)).astype(np.int32)
    doc[-1] = M - 1
    z = rng.integers(0, K, word.size).astype(np.int32)
    say("equal W^ K=%d beta=%g" % (K, beta))
    with lda.LDA(word, doc, V, K, alpha, beta, SEED) as m:
        m.set_assignments(z, 3)
        want, flags, _ = oracle.iterate(word, doc, z, M=M, V=V, K=K, alpha=alpha, beta=beta, seed=SEED, t=3)
        m.iterate(1)
        compare_draws(m.counts(D=False, W=False)["z"], want, flags, max(word.size, 10 ** 6))


def _records(word, doc, z, V, K, alpha, beta, two, dense_cutoff=0):
    """(a1, Q', sum W^, K1) per word id as the kernels left them in device memory after a scoring call."""
    import ctypes

    import torch

    import paper_2007_08725_amd as lda
    live = {}

    def alloc(nbytes, ctx):
        t = torch.empty(int(nbytes), dtype=torch.uint8, device="cuda")
        live[t.data_ptr()] = t
        return t.data_ptr()

    def free(ptr, ctx):
        live.pop(ptr, None)

    fa, ff = lda.ALLOC_FN(alloc), lda.FREE_FN(free)
    o = lda.Options()
    o.dev_alloc, o.dev_free, o.two_branch, o.dense_cutoff = fa, ff, int(two), dense_cutoff
    lib, h, ll = lda.load_library(), ctypes.c_void_p(), ctypes.c_double()
    w, d, z = (np.ascontiguousarray(x, np.int32) for x in (word, doc, z))
    ptr = lambda a: ctypes.c_void_p(a.ctypes.data)  # noqa: E731
    assert lib.lda_create(ptr(w), ptr(d), w.size, V, K, alpha, beta, SEED, ctypes.byref(o), ctypes.byref(h)) == 0
    try:
        assert lib.lda_set_assignments(h, ptr(z), 1) == 0
        assert lib.lda_loglik(h, ctypes.byref(ll)) == 0
        # 48 bytes a word (a1, a2, a3, Q', sum, K1 | K2 << 32), words by descending count, lowest id first on ties
        size = (48 * V + 255) & ~255
        found = [t for t in live.values() if t.numel() == size]
        assert len(found) == 1
        raw = found[0].cpu().numpy()[:48 * V].view(np.float64).reshape(V, 6)
    finally:
        lib.lda_destroy(h)
    order = np.lexsort((np.arange(V), -np.bincount(w, minlength=V)))
    out = np.empty((V, 4))
    out[order] = np.stack([raw[:, 0], raw[:, 3], raw[:, 4], raw[:, 5].view(np.uint64) & 0xFFFFFFFF], 1)
    return out


# words of one to 60 tokens (16 lanes each) and of 65 to 200 (a wave each), nearly all of one topic, so that W^[v][K1]
# is nearly the whole sum; and a topic with two tokens, whose beta/den[k] is a large part of the sum over all topics, in two rows
@pytest.mark.parametrize("K,beta,two", [(1000, 1e-6, False), (1000, 1e-9, False), (1000, 0.01, False),
                                        (1000, 1e-6, True), (4096, 1e-6, False)])
def test_q_prime_of_a_word_held_by_one_topic(K, beta, two):
    rng = np.random.default_rng(K)
    V, alpha = max((5 << 20) // K + 1, 2 * K), 0.1  # enough words for the list, and two or more per topic
    counts = rng.integers(1, 61, V)
    counts[:40] = rng.integers(65, 200, 40)
    word = np.repeat(np.arange(V, dtype=np.int32), counts)
    doc = np.sort(rng.integers(0, 900, word.size)).astype(np.int32)
    doc[-1] = 899
    z = (word % (K - 1)).astype(np.int32)
    first = np.r_[0, np.cumsum(counts)[:-1]]
    z[first[100:400]] = rng.integers(0, K - 1, 300)  # rows of two topics
    z[first[[5, 50]]] = K - 1                        # the topic of two tokens
    say("Q' K=%d beta=%g two_branch=%s" % (K, beta, two))
    got = _records(word, doc, z, V, K, alpha, beta, two)
    W = np.bincount(word.astype(np.int64) * K + z, minlength=V * K).reshape(V, K)
    den = W.sum(0) + np.float64(V * beta)
    wh = ((W + beta) / den).astype(np.longdouble)  # the fp64 values, summed in 80 bits
    k1 = np.argmax(wh, 1)
    total = wh.sum(1)
    top = wh[np.arange(V), k1].copy()
    wh[np.arange(V), k1] = 0
    q = wh.sum(1)
    # the exact sums rounded once, times alpha
    bound = 2.5 * 2.0 ** -53
    if not two:
        assert np.array_equal(got[:, 3], k1) and np.array_equal(got[:, 0], top.astype(np.float64))
    want = np.longdouble(alpha) * (total if two else q)
    assert np.max(np.abs(got[:, 1] - want) / want) < bound
    assert np.max(np.abs(got[:, 2] - total) / total) < bound
    # the same bits from dense rows (of which out-of-core handles are made), and without a list of few topics
    for cutoff in (-1, 1 << 30):
        assert np.array_equal(_records(word, doc, z, V, K, alpha, beta, two, cutoff), got)
