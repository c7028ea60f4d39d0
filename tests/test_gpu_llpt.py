"""The LLPT kernels at their edges against the oracle: light batches, long rows and runs, the tiled rows of large K."""
import numpy as np
import pytest

import lda_synth
import oracle
from gpu_common import corpus_kw, make_lda, say

pytestmark = pytest.mark.gpu


# K: the light kernel's last (2,127), a 1,024-thread workgroup (5,000, 16,384), tiled rows (17,500: the second tile
# ends inside a chunk; 32,768); lengths: rows around 512 and 1,024 slots and past 16 chunks of 128
@pytest.mark.parametrize("K", [2, 50, 2127, 5000, 16384, 17500, 32768])
@pytest.mark.parametrize("opts", [{}, {"region_tokens": 100}, {"dense_cutoff": -1}, {"chunks": 2}])
def test_llpt_follows_the_oracle(K, opts):
    rng = np.random.default_rng(K)
    lens = np.array([1, 2, 31, 32, 127, 128, 255, 256, 510, 511, 512, 513, 700, 1023, 1024, 2100, 3500])
    doc = np.repeat(np.arange(lens.size, dtype=np.int32), lens)
    # one frequent word (runs of it in the long documents), words of 1 to 70 tokens
    word = rng.choice(300, doc.size, p=np.r_[0.4, np.full(299, 0.6 / 299)]).astype(np.int32)
    spec = lda_synth.CorpusSpec("llpt", lens.size, ("poisson", 1.0), 300, 0.0, K, K, 0.05)
    c = lda_synth.Corpus(spec, word, doc, 300, lens.size)
    with make_lda(c, **opts) as m:
        for it in range(2):
            say("LLPT K=%d %s iteration %d" % (K, opts, it))
            z = m.counts(D=False, W=False)["z"]
            want = oracle.llpt(c.word, c.doc, z, **corpus_kw(c))
            got = m.loglik()
            # 64-bit sums of at most 3,500 + K terms of one sign in another order
            assert got == pytest.approx(want, rel=1e-12)
            assert m.loglik_noalloc() == got and m.loglik() == got  # bit for bit
            m.iterate(1)
