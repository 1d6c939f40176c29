"""Steps whose keys are sorted in tiles of every shape, on both sides of the sizes where the shape changes."""
import numpy as np
import pytest
import torch

import oracle
from paper_1606_08495_amd import w2v, workloads
from util import all_rows, dev, vec_error

pytestmark = pytest.mark.gpu


# n (k + 2) keys in all, k = 5: 300 000, 2^20, 2 500 000
@pytest.mark.parametrize("n", [42_857, 42_858, 149_796, 149_797, 357_142, 357_143])
@pytest.mark.parametrize("V", [3000, 1 << 17])                 # two passes, three
def test_step_at_the_edges_of_the_tile_shapes(n, V):
    print("sort shapes", n, V, flush=True)
    d, k, alpha = 4, 5, 0.0005
    rng = np.random.default_rng(n + V)
    counts = workloads.analytic_counts(V, 1.0, 10 ** 7)
    th, al = oracle.build_alias(counts)
    a, b = (workloads.zipf_draw(workloads.zipf_cdf(V, 1.0), n, rng) for _ in range(2))
    rows = np.arange(V, dtype=np.uint32)
    U, W = oracle.init_rows(3, d, 0, d, 0, rows), oracle.init_rows(3, d, 0, d, 1, rows)
    sh = w2v.Shard(V, d, 3, init_mode=1)
    sh.set_counts(counts)
    for step in range(2):                                       # the second on states the first has left
        w2v.train_minibatch([sh], dev(a), dev(b), k, 40 + step, alpha)
        oracle.train_minibatch([U], [W], a, b, k, 40 + step, th, al, alpha)
    sh.status()
    assert vec_error(all_rows(sh, 0), U) <= 2e-5 and vec_error(all_rows(sh, 1), W) <= 2e-5      # 1e-5 a minibatch
    sh.destroy()


# n (k + 2) keys: 1 500 000, up to which both sides' keys are sorted by the same launches
@pytest.mark.parametrize("n", [214_285, 214_286])
def test_adjust_where_the_sides_keys_are_sorted_apart(n):
    print("sorted together or apart", n, flush=True)
    V, d, k, alpha = 3000, 4, 5, 0.0005
    rng = np.random.default_rng(n)
    counts = workloads.analytic_counts(V, 1.0, 10 ** 7)
    th, al = oracle.build_alias(counts)
    a, b = (workloads.zipf_draw(workloads.zipf_cdf(V, 1.0), n, rng) for _ in range(2))
    rows = np.arange(V, dtype=np.uint32)
    U, W = oracle.init_rows(3, d, 0, d, 0, rows), oracle.init_rows(3, d, 0, d, 1, rows)
    sh = w2v.Shard(V, d, 3, init_mode=1)
    sh.set_counts(counts)
    for step in range(2):
        g = workloads.uniform_coeffs(n, k + 1, step)
        sh.adjust(dev(a), dev(b), k, 40 + step, torch.from_numpy(g).cuda(), alpha)
        oracle.adjust(U, W, a, b, k, 40 + step, th, al, g, alpha)
    sh.status()
    assert vec_error(all_rows(sh, 0), U) <= 2e-5 and vec_error(all_rows(sh, 1), W) <= 2e-5      # 1e-5 a minibatch
    sh.destroy()
