"""lda_get_counts on results large enough for the pinned buffers, the host threads and several slabs of rows."""
import numpy as np
import pytest

import lda_synth
from gpu_common import check_counts_are_histograms, make_lda, say

pytestmark = pytest.mark.gpu


# more entries of D and of W than one slab (2^23), input in another order than by document, out of core; and one
# token more and one fewer than the largest result that is read without the pinned buffers (2^19 topics)
@pytest.mark.parametrize("n_docs,mean,V,K,opts", [
    (330_000, 30, 60_000, 1000, {}),
    (40_000, 30, 5_000, 200, {"shuffle": True}),
    (40_000, 30, 5_000, 200, {"chunks": 3}),
    (2, ((1 << 19) + 1), 300, 30, {"tokens": (1 << 19) + 1}),
    (2, ((1 << 19) - 1), 300, 30, {"tokens": (1 << 19) - 1}),
])
def test_large_exports_are_the_histograms_of_z(n_docs, mean, V, K, opts):
    rng = np.random.default_rng(K)
    if "tokens" in opts:
        n_docs = 9
        doc = np.sort(np.arange(opts["tokens"], dtype=np.int64) % n_docs).astype(np.int32)
    else:
        doc = np.repeat(np.arange(n_docs, dtype=np.int32), rng.integers(0, 2 * mean + 1, n_docs))
    word = rng.integers(0, V, doc.shape[0]).astype(np.int32)
    if opts.get("shuffle"):
        p = rng.permutation(doc.shape[0])
        word, doc = word[p], doc[p]
    n_docs = int(doc.max()) + 1
    spec = lda_synth.CorpusSpec("export", n_docs, ("poisson", 1.0), V, 0.0, K, K, 0.1)
    c = lda_synth.Corpus(spec, word, doc, V, n_docs)
    say("export N=%d K=%d %s" % (c.N, K, opts))
    with make_lda(c, **({"chunks": 3} if "chunks" in opts else {})) as m:
        if "tokens" not in opts:
            m.iterate(1)
        for _ in range(2):  # the second call has the pinned buffers already
            cnt = m.counts()
            sz = m.sizes()
            assert (sz["nnz_D"], sz["nnz_W"]) == (cnt["D_topic"].shape[0], cnt["W_topic"].shape[0])
            check_counts_are_histograms(c, cnt, K)
        only = m.counts(D=False, W=False)
        assert np.array_equal(only["z"], cnt["z"]) and only["iteration"] == cnt["iteration"] and only["M"] == n_docs
