"""The document kernels' batches and grids at small and ragged document counts, against the oracle."""
import numpy as np
import pytest

import lda_synth
from gpu_common import check_counts_are_histograms, compare_draws, make_lda, oracle_step, say

pytestmark = pytest.mark.gpu


# one document; around one workgroup set (8 workgroups of 4 waves); one past every wave of the D rebuild's grid; two
# batches of two per wave and a remainder
@pytest.mark.parametrize("n_docs", [1, 7, 31, 32, 33, 4097, 16385, 40001])
@pytest.mark.parametrize("opts", [{}, {"chunks": 3}])
def test_every_document_is_walked_once(n_docs, opts):
    rng = np.random.default_rng(n_docs)
    lens = rng.integers(0, 9, n_docs)  # some empty
    lens[-1] = 5000 if n_docs in (33, 4097) else 3  # a heavy document among light ones
    doc = np.repeat(np.arange(n_docs, dtype=np.int32), lens)
    word = rng.integers(0, 50, doc.shape[0]).astype(np.int32)
    K = 24
    spec = lda_synth.CorpusSpec("docs", n_docs, ("poisson", 4.0), 50, 0.0, K, K, 0.3)
    c = lda_synth.Corpus(spec, word, doc, 50, n_docs)
    with make_lda(c, always_skip_test=True, **opts) as m:
        z = m.counts(D=False, W=False)["z"]
        for t in range(2):
            say("doc batches M=%d %s t=%d" % (n_docs, opts, t))
            want, flags, _ = oracle_step(c, z, t)
            m.iterate(1)
            cnt = m.counts()
            z = cnt["z"]
            compare_draws(z, want, flags, max(c.N, 10 ** 6))
            check_counts_are_histograms(c, cnt, K)
