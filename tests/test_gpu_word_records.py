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
