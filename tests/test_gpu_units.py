"""The sampler's units (regions cut finer for small corpora) and the folded statistics: the same draws and counts."""
import numpy as np
import pytest

import lda_synth
from gpu_common import compare_draws, make_lda, oracle_step, say

pytestmark = pytest.mark.gpu


# token counts of one frequent word around the least unit (256 threads, or 2 K = 2,000) and its multiples
@pytest.mark.parametrize("K,counts", [(16, [255, 256, 257, 511, 512, 513, 5000, 20001]), (1000, [1999, 2001, 4000, 12001])])
@pytest.mark.parametrize("opts", [{}, {"region_tokens": 300}, {"sampler_block": 1024}, {"chunks": 2}])
def test_cut_regions_draw_the_same_and_are_counted_once(K, counts, opts):
    rng = np.random.default_rng(K)
    word = np.repeat(np.arange(len(counts) + 40, dtype=np.int32), counts + [3] * 40)
    n_docs = 300
    doc = rng.integers(0, n_docs, word.size).astype(np.int32)
    doc[0] = n_docs - 1
    order = np.argsort(doc, kind="stable")
    spec = lda_synth.CorpusSpec("units", n_docs, ("poisson", 1.0), len(counts) + 40, 0.0, K, K, 0.1)
    c = lda_synth.Corpus(spec, word[order], doc[order], len(counts) + 40, n_docs)
    with make_lda(c, always_skip_test=True, **opts) as m:
        z = m.counts(D=False, W=False)["z"]
        for t in range(2):
            say("units K=%d %s t=%d" % (K, opts, t))
            want, flags, ost = oracle_step(c, z, t)
            st = m.iterate(1, stats=True)[0]
            z = m.counts(D=False, W=False)["z"]
            compare_draws(z, want, flags, max(c.N, 10 ** 6))
            assert st["sampled"] + st["skip_step3"] == c.N
            assert st["skip_step3"] <= ost["skip3"] <= st["skip_step3"] + max(2, c.N // 1000)
            R = opts.get("region_tokens", 10_000)
            if "chunks" not in opts:  # regions, not units: a dense word (count > K) has ceil(count / R), a sparse one one
                per_word = [-(-n // R) if n > K else 1 for n in counts] + [1] * 40
                assert st["regions"] == sum(per_word)
                assert st["dense_regions"] == sum(r for r, n in zip(per_word, counts) if n > K)
