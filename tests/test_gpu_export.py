"""lda_get_counts on results large enough for the pinned buffers, the host threads and several slabs of rows."""
import numpy as np
import pytest

import lda_synth
from gpu_common import SEED, check_counts_are_histograms, make_lda, say

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


# the topics and tables of a handle whose allocator has nothing left after construction, resident and out of core, over several
# slabs of rows and with results on either side of the threads' threshold
@pytest.mark.parametrize("n_docs,mean,V,K,chunks", [
    (330_000, 30, 60_000, 1000, 0),
    (40_000, 30, 5_000, 200, 3),
    (300, 20, 500, 30, 0),
])
def test_tables_are_exported_without_device_memory_to_spare(n_docs, mean, V, K, chunks):
    import ctypes

    import torch

    import paper_2007_08725_amd as lda
    rng = np.random.default_rng(K)
    doc = np.repeat(np.arange(n_docs, dtype=np.int32), rng.integers(1, 2 * mean, n_docs))
    word = rng.integers(0, V, doc.shape[0]).astype(np.int32)
    n, live, refused = doc.shape[0], {}, []

    def alloc(nbytes, ctx):
        if alloc.closed:
            refused.append(int(nbytes))
            return None
        t = torch.empty(int(nbytes), dtype=torch.uint8, device="cuda")
        live[t.data_ptr()] = t
        return t.data_ptr()

    alloc.closed = False

    def free(ptr, ctx):
        live.pop(ptr, None)

    fa, ff = lda.ALLOC_FN(alloc), lda.FREE_FN(free)
    o = lda.Options()
    o.dev_alloc, o.dev_free = fa, ff
    if chunks:
        o.chunks = chunks
    lib, h = lda.load_library(), ctypes.c_void_p()
    say("export without device memory N=%d K=%d chunks=%d" % (n, K, chunks))

    def ptr(a):
        return ctypes.c_void_p(a.ctypes.data)

    assert lib.lda_create(ptr(word), ptr(doc), n, V, K, 50.0 / K, 0.01, SEED, ctypes.byref(o), ctypes.byref(h)) == 0
    try:
        assert lib.lda_iterate(h, 1, None) == 0

        def tables():
            c = lda.Counts()
            assert lib.lda_get_counts(h, ctypes.byref(c)) == 0
            a = dict(z=np.empty(n, np.int32), T=np.empty(K, np.int64), D_off=np.empty(c.M + 1, np.int64), D_topic=np.empty(c.nnz_D, np.int32),
                     D_count=np.empty(c.nnz_D, np.int32), W_off=np.empty(c.V + 1, np.int64),
                     W_topic=np.empty(c.nnz_W, np.int32), W_count=np.empty(c.nnz_W, np.int32))
            for name, arr in a.items():
                setattr(c, name, arr.ctypes.data)
            assert lib.lda_get_counts(h, ctypes.byref(c)) == 0, lib.lda_last_error(h)
            return a

        ref, kept = tables(), len(live)
        alloc.closed = True
        got = tables()
        assert len(refused) == 6 if not chunks else len(refused) >= 5  # every array of the export was refused
        assert len(live) == kept
        for name in ref:
            assert np.array_equal(ref[name], got[name]), name
        # topics out of range are LDA_E_ARG with their place, topics in range LDA_E_NOMEM; both leave the state alone
        if not chunks:
            z = ref["z"].copy()
            assert lib.lda_set_assignments(h, ptr(z), 5) == lda.LDA_E_NOMEM
            z[n // 2] = K
            assert lib.lda_set_assignments(h, ptr(z), 5) == lda.LDA_E_ARG
            assert b"topic out of range at token %d" % (n // 2) in lib.lda_last_error(h)
            assert np.array_equal(tables()["z"], ref["z"])
    finally:
        lib.lda_destroy(h)
    assert not live
