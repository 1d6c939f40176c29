"""Row kernels at the edges of their batches: slots per pair that fill a batch, several, or part of one, at every number of
float4 a lane holds; runs of the output side that end at the edges of chunks, windows and cells."""
import numpy as np
import pytest
import torch

import oracle
from paper_1606_08495_amd import w2v, workloads
from util import all_rows, dev, vec_error

pytestmark = pytest.mark.gpu

BOUND = 1e-5                 # of a row's largest component, as for every minibatch


def oracle_step(V, d, a, b, k, seed, counts, alpha):
    th, al = oracle.build_alias(counts)
    rows = np.arange(V, dtype=np.uint32)
    U, W = oracle.init_rows(3, d, 0, d, 0, rows), oracle.init_rows(3, d, 0, d, 1, rows)
    oracle.train_minibatch([U], [W], a, b, k, seed, th, al, alpha)
    return U, W


# float4 of a row: 1, 15, 16, 17, 25, 32, 33, 50, 64, 65, 75, 128, 129, 192, 193, 256
@pytest.mark.parametrize("d,cuts,k", [(3, 1, 8), (60, 1, 5), (60, 1, 10), (60, 1, 9), (64, 1, 25), (66, 1, 3), (100, 1, 5), (100, 1, 12),
                                      (128, 1, 10), (130, 1, 25), (200, 1, 5), (200, 1, 26), (256, 1, 17), (260, 1, 5), (300, 1, 5),
                                      (300, 1, 10), (300, 1, 11), (512, 1, 4), (514, 1, 5), (768, 1, 7), (770, 1, 3), (1024, 1, 6),
                                      (100, 3, 5), (300, 5, 5), (300, 5, 12), (130, 2, 21), (700, 2, 7), (300, 1, 0), (60, 2, 64)])
def test_slots_of_a_pair_in_whole_and_part_batches(d, cuts, k, n=1203):
    print("batches", d, cuts, k, n, flush=True)
    V, seed = 4000, 9
    rng = np.random.default_rng(d + k)
    counts = workloads.analytic_counts(V, 1.0, 10 ** 7)
    cdf = workloads.zipf_cdf(V, 1.0)
    a, b = (workloads.zipf_draw(cdf, n, rng) for _ in range(2))
    alpha = 0.2 / (n * 0.12 * (k + 1))
    U, W = oracle_step(V, d, a, b, k, seed, counts, alpha)
    edges = [d * s // cuts for s in range(cuts + 1)]
    for form in ("one step", "two calls"):
        shards = [w2v.Shard(V, hi - lo, 3, d_total=d, col_begin=lo, init_mode=1) for lo, hi in zip(edges, edges[1:])]
        for sh in shards:
            sh.set_counts(counts)
        if form == "one step":
            w2v.train_minibatch(shards, dev(a), dev(b), k, seed, alpha)
        else:
            g = shards[0].coeffs([sh.dotprod(dev(a), dev(b), k, seed) for sh in shards], k)
            for sh in shards:
                sh.adjust(dev(a), dev(b), k, seed, g, alpha)
        got = [np.concatenate([all_rows(sh, which) for sh in shards], axis=1) for which in (0, 1)]
        for sh in shards:
            sh.status()
            sh.destroy()
        assert vec_error(got[0], U) <= BOUND and vec_error(got[1], W) <= BOUND, form


# chunks of two pairs up to 98 303, three from there on: of rows of 17 to 32 float4 the latter are refilled; of more than 64 up to
# 16 384 pairs are, of more than 128 up to 8192; one matrix or slices
@pytest.mark.parametrize("d,cuts,k,n", [(100, 1, 10, 98_303), (100, 1, 10, 98_304), (100, 1, 7, 98_305), (128, 1, 12, 98_306), (68, 1, 25, 98_304),
                                        (100, 1, 1, 98_307), (100, 2, 10, 98_304), (60, 1, 10, 98_306), (7, 1, 20, 98_305), (300, 1, 9, 16_384),
                                        (300, 1, 9, 16_385), (260, 3, 7, 16_385), (700, 1, 7, 8192), (700, 1, 7, 8193), (700, 2, 9, 8193),
                                        (1000, 1, 6, 8193)])
def test_longer_chunks_in_whole_and_part_batches(d, cuts, k, n):
    test_slots_of_a_pair_in_whole_and_part_batches(d, cuts, k, n)


# a chunk is 16 contributions, a window two, a cell 32 (64 from 2^19 contributions on)
LENGTHS = [1, 2, 15, 16, 17, 30, 31, 32, 33, 34, 47, 48, 49, 62, 63, 64, 65, 66, 79, 80, 81, 95, 96, 97, 127, 128, 129, 300]


@pytest.mark.parametrize("d,repeats,lead", [(8, 1, 0), (8, 1, 7), (100, 1, 3), (130, 1, 15), (300, 1, 1), (8, 290, 0), (8, 290, 11)])
def test_runs_that_end_at_the_edges_of_chunks_and_cells(d, repeats, lead):
    """Output words (no negatives) named as often as the list says, after a few others; a bag of words has the same walk
    on its input side."""
    print("runs", d, repeats, lead, flush=True)
    rng = np.random.default_rng(lead)
    lengths = np.concatenate([[1] * lead] + [rng.permutation(LENGTHS) for _ in range(repeats)]).astype(int)
    V = lengths.size
    b = np.repeat(np.arange(V, dtype=np.uint32), lengths)
    n = b.size
    assert (n > 1 << 19) == (repeats > 1)
    b = b[rng.permutation(n)]
    a = rng.integers(0, V, n).astype(np.uint32)
    counts = np.ones(V, np.uint64)
    alpha = 0.002
    U, W = oracle_step(V, d, a, b, 0, 5, counts, alpha)
    sh = w2v.Shard(V, d, 3, init_mode=1)
    sh.set_counts(counts)
    w2v.train_minibatch([sh], dev(a), dev(b), 0, 5, alpha)
    sh.status()
    assert vec_error(all_rows(sh, 0), U) <= BOUND and vec_error(all_rows(sh, 1), W) <= BOUND
    sh.destroy()


@pytest.mark.parametrize("d", [8, 100, 200, 300, 600, 900])
@pytest.mark.parametrize("most", [0, 1, 15, 16, 17, 33])
def test_hidden_vectors_of_any_number_of_context_words(d, most):
    """Context lengths 0 .. most: none, part of sixteen, whole sixteens."""
    print("hidden", d, most, flush=True)
    V, n, k, seed, alpha = 500, 300, 3, 4, 0.001
    rng = np.random.default_rng(d + most)
    counts = workloads.analytic_counts(V, 1.0, 10 ** 6)
    th, al = oracle.build_alias(counts)
    lens = rng.integers(0, most + 1, n)
    lens[:2] = 0, most
    off = np.concatenate([[0], np.cumsum(lens)]).astype(np.uint32)
    ctx = rng.integers(0, V, int(off[-1])).astype(np.uint32)
    out = rng.integers(0, V, n).astype(np.uint32)
    rows = np.arange(V, dtype=np.uint32)
    U, W = oracle.init_rows(3, d, 0, d, 0, rows), oracle.init_rows(3, d, 0, d, 1, rows)
    oracle.cbow_train_minibatch([U], [W], off, ctx, out, k, seed, th, al, alpha)
    sh = w2v.Shard(V, d, 3, init_mode=1)
    sh.set_counts(counts)
    w2v.cbow_train_minibatch([sh], dev(off), dev(ctx), dev(out), k, seed, alpha)
    sh.status()
    assert vec_error(all_rows(sh, 0), U) <= BOUND and vec_error(all_rows(sh, 1), W) <= BOUND
    torch.cuda.synchronize()
    sh.destroy()
