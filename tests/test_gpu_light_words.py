"""The light-word sampler: batches of whole words with at most 64 tokens, against the oracle."""
import numpy as np
import pytest

import lda_synth
from gpu_common import compare_draws, make_lda, oracle_step, say

pytestmark = pytest.mark.gpu


def _corpus(counts, n_docs, K, seed):
    """Word w has counts[w] tokens, spread over n_docs documents (sorted by document, none empty at the end)."""
    rng = np.random.default_rng(seed)
    word = np.repeat(np.arange(len(counts), dtype=np.int32), counts)
    doc = rng.integers(0, n_docs, word.shape[0]).astype(np.int32)
    doc[0] = n_docs - 1
    order = np.lexsort((rng.random(word.shape[0]), doc))
    spec = lda_synth.CorpusSpec("light", n_docs, ("poisson", 1.0), len(counts), 0.0, K, K, 0.07)
    return lda_synth.Corpus(spec, word[order], doc[order], len(counts), n_docs)


# K = 2,127 and 2,128: the last K with a light sampler and the first without; 16: light words that are dense
@pytest.mark.parametrize("K", [2, 16, 1000, 2127, 2128])
@pytest.mark.parametrize("opts", [{}, {"two_branch": True}, {"region_tokens": 7}, {"dense_cutoff": -1}, {"chunks": 3}])
def test_light_batches_follow_the_oracle(K, opts):
    # one to 64 tokens (batches of many words, of one word, words that just end a batch), 65 and more beside them
    counts = [1] * 200 + [2, 3, 15, 16, 17, 31, 32, 33, 47, 48, 49, 63, 64, 65] * 5 + [64] * 9 + [200, 700, 2500]
    c = _corpus(counts, 40, K, 11)  # 40 documents: rows of several lengths, runs of a word in a document
    branches = 2 if opts.get("two_branch") else 3
    with make_lda(c, **opts) as m:
        z = m.counts(D=False, W=False)["z"]
        for t in range(2):
            say("light words K=%d %s t=%d" % (K, opts, t))
            want, flags, _ = oracle_step(c, z, t, **({"branches": 2} if branches == 2 else {}))
            m.iterate(1)
            z = m.counts(D=False, W=False)["z"]
            compare_draws(z, want, flags, max(c.N, 10 ** 6))
