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


EPS = 9.5 * 2.0 ** -24  # the bound on the single-precision error of S', of S'; the CPU checks see up to 4 of 9.5


def _edges(word, doc, z, u, M, V, K, alpha, beta):
    """Per token in fp64, by brute force: branch (0 M, 1 S', 2 Q'), the distance of x from the nearest edge, S' and Q'."""
    import torch
    dev = "cuda"
    word, doc, z = (torch.as_tensor(a, device=dev).long() for a in (word, doc, z))
    D = torch.bincount(doc * K + z, minlength=M * K).view(M, K).double()
    W = torch.bincount(word * K + z, minlength=V * K).view(V, K).double()
    den = W.sum(0) + V * beta
    u = torch.as_tensor(u, device=dev)
    out = [torch.empty(word.numel(), dtype=torch.float64, device=dev) for _ in range(4)]
    step = max(1, 20_000_000 // K)
    for b in range(0, word.numel(), step):
        w = (W[word[b:b + step]] + beta) / den
        d = D[doc[b:b + step]]
        a1, k1 = w.max(1, keepdim=True)
        m = a1 * (d.gather(1, k1) + alpha)
        w.scatter_(1, k1, 0.0)
        S, Q = (d * w).sum(1, keepdim=True), (alpha * w).sum(1, keepdim=True)
        x = u[b:b + step, None] * ((m + S) + Q)
        inside = torch.where(x < m + S, m + torch.cumsum(d * w, 1), (m + S) + torch.cumsum(alpha * w, 1))
        near = torch.minimum((inside - x).abs().min(1, keepdim=True).values,
                             torch.minimum((x - m).abs(), (x - (m + S)).abs()))
        near = torch.where(x < m, m - x, near)
        for o, v in zip(out, (torch.where(x < m, 0.0, torch.where(x < m + S, 1.0, 2.0)), near, S, Q)):
            o[b:b + step] = v[:, 0]
    return [o.cpu().numpy() for o in out]


def _uniforms(t, n):
    return np.array([oracle.uniform(SEED, t, i) for i in range(n)])


@pytest.mark.parametrize("K", [2500, 10_000, 32_768])
def test_both_ways_are_taken(K):
    """The corpus of these tests has tokens within the bound of an edge of S' and of Q', which are redone in fp64, and
    at least 95% of its tokens further from every edge than the bound and its own error, which are not."""
    word, doc, z, M = _corpus(K, 3)
    say("both ways K=%d" % K)
    branch, near, S, Q = _edges(word, doc, z, _uniforms(1, word.size), M, 2000, K, 0.05, 0.01)
    eq = EPS * S * Q / (S + Q)
    # the single-precision x and edge are each off by at most 4 of the 9.5 units
    assert np.sum((branch == 1) & (near < EPS * S)) >= 1
    assert np.sum((branch == 2) & (near < 0.5 * eq)) >= 1
    # inside a block of 32 topics the walk's own bound is below (32 + 4) * 2^-23 of the block, here at most of Q'
    far = np.where(branch == 2, near > 2.5 * eq + 36 * 2.0 ** -23 * Q, near > 3 * EPS * S)
    assert far.mean() > 0.95 if K < 30_000 else far.mean() > 0.5


@pytest.mark.parametrize("K", [2500, 20_000])
def test_draws_next_to_the_max_topic_edge(K):
    """alpha chosen so that one token's x falls beside M by half the bound, on either side: redone in fp64, and right
    (an edge of the max-topic branch is within the bound of one x in a million, so no corpus holds it by itself)."""
    import paper_2007_08725_amd as lda
    word, doc, z, M = _corpus(K, 5, tokens=20_000)
    t, V, beta = 4, 2000, 0.01
    u = _uniforms(t, word.size)
    D = np.bincount(doc.astype(np.int64) * K + z, minlength=M * K).reshape(M, K)
    W = np.bincount(word.astype(np.int64) * K + z, minlength=V * K).reshape(V, K)
    den = W.sum(0) + V * beta
    tried = 0
    for i in np.random.default_rng(1).permutation(word.size):
        w = (W[word[i]] + beta) / den
        k1 = int(np.argmax(w))
        a1, rest = w[k1], np.delete(w, k1).sum()
        S = float(np.dot(D[doc[i]], w) - D[doc[i], k1] * a1)
        # M - x = a1 (C1 + alpha) (1 - u) - u (S + alpha rest) = side * kEps S / 2, linear in alpha
        for side in (1.0, -1.0):
            slope = a1 * (1 - u[i]) - u[i] * rest
            alpha = (side * 0.5 * EPS * S - a1 * D[doc[i], k1] * (1 - u[i]) + u[i] * S) / slope
            Z = a1 * (D[doc[i], k1] + alpha) + S + alpha * rest
            # a usable prior, with the edge further than the oracle's own margin (1e-9 of Z)
            if not (1e-3 < alpha < 50.0) or 0.5 * EPS * S < 1e-8 * Z:
                continue
            say("edge of M K=%d token %d side %+d alpha=%.6g" % (K, i, side, alpha))
            with lda.LDA(word, doc, V, K, alpha, beta, SEED) as m:
                m.set_assignments(z, t)
                want, flags, _ = oracle.iterate(word, doc, z, M=M, V=V, K=K, alpha=alpha, beta=beta, seed=SEED, t=t)
                m.iterate(1)
                got = m.counts(D=False, W=False)["z"]
            assert not flags[i] & 1 and got[i] == want[i] and (want[i] == k1) == (side > 0)
            compare_draws(got, want, flags, max(word.size, 10 ** 6))
            tried += 1
        if tried >= 6:
            break
    assert tried >= 6


@pytest.mark.parametrize("block,last", [(256, 17_743), (512, 17_071), (1024, 16_384)])
def test_sizes_that_can_be_asked_for(block, last):
    import paper_2007_08725_amd as lda
    word, doc = np.array([0, 1, 0], np.int32), np.array([0, 0, 1], np.int32)
    with lda.LDA(word, doc, 2, last, 0.05, 0.01, SEED, sampler_block=block) as m:
        assert m.iterate(1, stats=True)[0]["sampler_block"] == block
    with pytest.raises(lda.LDAError) as e:
        lda.LDA(word, doc, 2, last + 1, 0.05, 0.01, SEED, sampler_block=block)
    assert e.value.status == lda.LDA_E_RANGE
    with lda.LDA(word, doc, 2, last + 1, 0.05, 0.01, SEED) as m:
        assert m.iterate(1, stats=True)[0]["sampler_block"] in (256, 512, 1024)
