"""Small minibatches: keys grouped by one launch (up to 65 536 of either side, 80 000 in all), against the oracle,
at the sizes and vocabularies where the grouping takes another way, in every form that a step has."""
import numpy as np
import pytest
import torch

import oracle
from paper_1606_08495_amd import w2v, workloads
from util import all_rows, dev, vec_error

pytestmark = pytest.mark.gpu


def words(V, skew, n, rng):
    return workloads.zipf_draw(workloads.zipf_cdf(V, skew), n, rng)


# (V, skew, n, k): places counted pairwise (up to 256 keys a bucket), digit by digit, keys written out by themselves
# (more than 512 of a bucket in a wavefront's stretch), both sides of the lines to the radix sort, single keys
SHAPES = [(100_000, 1.0, 1999, 5), (100_000, 1.0, 10_922, 5), (100_000, 1.0, 10_923, 5), (3000, 1.2, 10_000, 5),
          (300, 1.5, 9000, 6), (2, 1.0, 10_922, 5), (5, 0.5, 26_666, 1), (5, 0.5, 26_667, 1), (70, 3.0, 40_000, 0), (70, 3.0, 40_001, 0),
          (40_000, 1.2, 20_000, 2), (1000, 1.0, 1, 0), (1000, 1.0, 97, 1), (65_537, 0.0, 8192, 7)]


@pytest.mark.parametrize("V,skew,n,k", SHAPES)
def test_small_minibatch_in_every_form(V, skew, n, k):
    print("small", V, skew, n, k, flush=True)
    d, seed = 8, 77
    rng = np.random.default_rng(n + k)
    counts = workloads.analytic_counts(V, skew, 10 ** 7)
    th, al = oracle.build_alias(counts)
    a, b = words(V, skew, n, rng), words(V, skew, n, rng)
    alpha = float(min(0.05, 0.2 / max(1, np.bincount(b, minlength=V).max() * (k + 1), np.bincount(a, minlength=V).max() * (k + 1))))
    rows = np.arange(V, dtype=np.uint32)
    U, W = oracle.init_rows(3, d, 0, d, 0, rows), oracle.init_rows(3, d, 0, d, 1, rows)
    oracle.train_minibatch([U], [W], a, b, k, seed, th, al, alpha)
    da, db = dev(a), dev(b)
    got = {}
    for form in ("plain", "announced", "captured", "two calls"):
        sh = w2v.Shard(V, d, 3, init_mode=1)
        sh.set_counts(counts)
        if form in ("announced", "two calls"):
            sh.prefetch_minibatch(da, db, k, seed)
        if form == "captured":
            w2v.StepGraph(sh, n, k).run(da, db, seed, alpha)
        elif form == "two calls":
            f = sh.dotprod(da, db, k, seed)
            sh.adjust(da, db, k, seed, sh.coeffs([f], k), alpha)
        else:
            w2v.train_minibatch([sh], da, db, k, seed, alpha)
        sh.status()
        got[form] = (all_rows(sh, 0), all_rows(sh, 1))
        # a minibatch's bound (1e-5 of a row's largest component)
        assert vec_error(got[form][0], U) <= 1e-5 and vec_error(got[form][1], W) <= 1e-5, form
        torch.cuda.synchronize()
        sh.destroy()
    for form in ("announced", "captured"):
        assert np.array_equal(got[form][0], got["plain"][0]) and np.array_equal(got[form][1], got["plain"][1]), form


def words_of_one_bucket(n, rng):
    """Different words whose bytes fold to the same bucket (of 256: more than 12 288 keys)."""
    hi, mid = np.divmod(rng.permutation(1 << 16)[:n].astype(np.uint32), 256)
    return (hi << 16 | mid << 8 | (hi ^ mid ^ 77)).astype(np.uint32)


def some_twice(n, rng):
    a = words_of_one_bucket(n, rng)
    a[rng.integers(0, n, n // 3)] = a[:n // 3]
    return a


def one_often(n, rng):
    a = words_of_one_bucket(n, rng)
    a[rng.random(n) < 0.4] = a[0]
    a[rng.random(n) < 0.3] = 12_345                             # another bucket's
    return a


@pytest.mark.parametrize("make", [words_of_one_bucket, some_twice, one_often])
@pytest.mark.parametrize("n", [40_000, 39_937, 13_000])
def test_many_words_of_one_bucket(make, n):
    """All of a minibatch's words in one bucket of the grouping: the same result, in the time of a few passes, not of
    one for every word."""
    print("one bucket", make.__name__, n, flush=True)
    V, d, alpha = 1 << 24, 4, 0.05
    rng = np.random.default_rng(n)
    a, b = make(n, rng), make(n, rng)
    da, db = dev(a), dev(b)
    ra, rb = np.unique(a), np.unique(b)
    for form in ("plain", "announced", "adjust"):
        sh = w2v.Shard(V, d, 3, init_mode=1)
        U, W = (sh.get_rows(which, dev(r)).cpu().numpy().astype(np.float64) for which, r in ((0, ra), (1, rb)))
        ia, ib = np.searchsorted(ra, a), np.searchsorted(rb, b)
        g = 1.0 / (1.0 + np.exp(np.sum(U[ia] * W[ib], axis=1)))
        if form == "adjust":
            sh.adjust(da, db, 0, 1, torch.from_numpy(g.astype(np.float32)).cuda().reshape(n, 1), alpha)
        else:
            if form == "announced":
                sh.prefetch_minibatch(da, db, 0, 1)
            w2v.train_minibatch([sh], da, db, 0, 1, alpha)
        dU, dW = np.zeros_like(U), np.zeros_like(W)
        np.add.at(dU, ia, alpha * g[:, None] * W[ib])
        np.add.at(dW, ib, alpha * g[:, None] * U[ia])
        assert vec_error(sh.get_rows(0, dev(ra)).cpu().numpy(), U + dU) <= 1e-5, form
        assert vec_error(sh.get_rows(1, dev(rb)).cpu().numpy(), W + dW) <= 1e-5, form
        t0, t1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        t0.record()
        w2v.train_minibatch([sh], da, db, 0, 2, 0.0)
        t1.record()
        torch.cuda.synchronize()
        print("  ", form, t0.elapsed_time(t1), "ms", flush=True)
        assert t0.elapsed_time(t1) < 20                         # (some hundreds with a pass for every word)
        sh.status()
        sh.destroy()
