"""The sampler with a single-precision W^ row: every draw is the fp64 one (decided within its bounds, or redone in fp64)."""
import numpy as np
import pytest

import lda_synth
import oracle
from gpu_common import SEED, compare_draws, say

pytestmark = pytest.mark.gpu


def _corpus(K, seed, tokens=60_000):
    """Rows of every bucket and past it, documents around the longest that reads counts as f16, runs of one word."""
    rng = np.random.default_rng(seed)
    lens = [1, 2, 31, 32, 33, 63, 64, 95, 96, 127, 128, 129, 191, 192, 255, 256, 383, 384, 511, 512, 513, 640, 1023, 1100,
            2046, 2047, 2048, 2049, 2600, 3300]
    while sum(lens) < tokens:
        lens.append(int(rng.integers(1, 700)))
    doc = np.repeat(np.arange(len(lens), dtype=np.int32), lens)
    p = 1.0 / np.arange(1, 2001) ** 1.1
    word = rng.choice(2000, doc.size, p=p / p.sum()).astype(np.int32)
    z = rng.integers(0, K, doc.size).astype(np.int32)
    # the documents of 2,046 to 2,600 tokens hold one topic thousands of times (counts at and past 2^11)
    z[(doc >= 24) & (doc <= 28) & (rng.random(doc.size) < 0.999)] = min(7, K - 1)
    return word, doc, z, len(lens)


def _check(K, alpha, beta, opts, seed=3, two=False):
    import paper_2007_08725_amd as lda
    word, doc, z, M = _corpus(K, seed)
    kw = dict(M=M, V=2000, K=K, alpha=alpha, beta=beta)
    with lda.LDA(word, doc, 2000, K, alpha, beta, SEED, two_branch=two, **opts) as m:
        for t in (1, 2):
            say("certified K=%d alpha=%g beta=%g %s t=%d" % (K, alpha, beta, opts, t))
            m.set_assignments(z, t)
            want, flags, _ = oracle.iterate(word, doc, z, seed=SEED, t=t, branches=2 if two else 3, **kw)
            m.iterate(1)
            got = m.counts(D=False, W=False)["z"]
            compare_draws(got, want, flags, max(word.size, 10 ** 6))
            z = got


# 2,300: the first K of this sampler; 2,304, 4,095, 4,096, 17,000: whole and ragged blocks of 32; 32,768: the largest
# row.  Below it, the workgroup sizes that are its own.
@pytest.mark.parametrize("K,opts", [(2299, {}), (2300, {}), (2304, {}), (4095, {}), (4096, {}), (10_000, {}), (17_000, {}),
                                    (32_768, {}), (3, {"sampler_block": 512}), (33, {"sampler_block": 1024}),
                                    (1000, {"sampler_block": 512}), (5000, {"sampler_block": 256}),
                                    (2500, {"region_tokens": 100}), (2500, {"dense_cutoff": -1}),
                                    (2500, {"dense_cutoff": 1 << 30}), (2500, {"chunks": 2}), (2500, {"skip_marks": 2})])
def test_draws_are_the_fp64_ones(K, opts):
    _check(K, 0.05, 0.01, opts)


# priors far from 1: counts of sparse rows searched instead of recovered (beta above 10^6), W^ of unheld topics that
# underflows in single precision, a Q' that takes nearly every draw (many topics within the bound of an edge)
@pytest.mark.parametrize("alpha,beta", [(0.05, 3.0e7), (0.05, 1e-42), (1e-30, 0.01), (200.0, 0.01), (1e-3, 1e-3)])
@pytest.mark.parametrize("K", [2500, 32_768])
def test_extreme_priors(K, alpha, beta):
    _check(K, alpha, beta, {})


@pytest.mark.parametrize("K", [2500, 20_000])
def test_two_branch(K):
    _check(K, 0.05, 0.01, {}, two=True)


def test_rows_of_many_chunks():
    """Rows past 16 chunks of 128 slots (a lane's total covers several), whole and ragged, with runs of one word."""
    import paper_2007_08725_amd as lda
    rng = np.random.default_rng(8)
    K = 20_000
    lens = [1900, 2040, 2300, 4100, 6200, 9000, 16_500, 30_000]
    doc = np.repeat(np.arange(len(lens), dtype=np.int32), lens)
    word = rng.choice(60, doc.size, p=np.r_[0.5, np.full(59, 0.5 / 59)]).astype(np.int32)
    z = rng.integers(0, K, doc.size).astype(np.int32)
    kw = dict(M=len(lens), V=60, K=K, alpha=0.05, beta=0.01)
    with lda.LDA(word, doc, 60, K, 0.05, 0.01, SEED) as m:
        m.set_assignments(z, 1)
        want, flags, _ = oracle.iterate(word, doc, z, seed=SEED, t=1, **kw)
        m.iterate(1)
        compare_draws(m.counts(D=False, W=False)["z"], want, flags, max(word.size, 10 ** 6))


# rows of several hundred entries a word, spread over the blocks of the Q' prefix and over the waves of a workgroup
@pytest.mark.parametrize("K,alpha", [(2500, 0.05), (2500, 20.0), (20_000, 0.05)])
def test_determinism_and_resume(K, alpha):
    """The same topics on every run, from a resumed state, and however the regions are cut and the workgroups sized."""
    import paper_2007_08725_amd as lda
    rng = np.random.default_rng(K)
    doc = np.repeat(np.arange(900, dtype=np.int32), rng.integers(100, 500, 900))
    word = rng.choice(400, doc.size).astype(np.int32)

    def fit(start=None, t=0, iters=6, **opts):
        with lda.LDA(word, doc, 400, K, alpha, 0.01, SEED, **opts) as m:
            if start is not None:
                m.set_assignments(start, t)
            m.iterate(iters)
            return m.counts(D=False, W=False)["z"]

    say("determinism K=%d alpha=%g" % (K, alpha))
    want, half = fit(), fit(iters=3)
    assert np.array_equal(fit(), want)
    assert np.array_equal(fit(start=half, t=3, iters=3), want)
    assert np.array_equal(fit(region_tokens=150), want)
    if K <= 4000:
        for block in (256, 512, 1024):
            assert np.array_equal(fit(sampler_block=block), want)
