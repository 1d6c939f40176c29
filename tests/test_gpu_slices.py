"""Several column shards trained in one process as one matrix of joint rows, against the same step through
dotprod, coefficients and adjust of each shard, and against the oracle."""
import ctypes

import numpy as np
import pytest
import torch

import oracle
from paper_1606_08495_amd import w2v
from util import all_rows, dev, vec_error, zipf_counts

pytestmark = pytest.mark.gpu

# fp32 sums in another order.  A dot of up to 1025 terms of unit rows is off by some sqrt(1025) 2^-24 = 2e-6, a coefficient
# by a quarter of that, and a row moves by less than its size: 5e-7; as much again for the order of a row's contributions.
TOL = 2e-6
ORACLE_TOL = 1e-5           # a minibatch against sums in double


def make_shard(V, d, seed, counts, d_total=None, col_begin=0):
    sh = w2v.Shard(V, d, seed, d_total=d_total, col_begin=col_begin, init_mode=1)
    sh.set_counts(counts, 0.0)
    return sh


def steps(shards, ins, outs, k, form):
    losses, alpha = [], min(0.03, 3.0 / ins[0].numel())      # (frequent rows move by less than their size)
    for h, (a, b) in enumerate(zip(ins, outs)):
        if form == "joint":
            loss = torch.zeros(1, dtype=torch.float64, device="cuda")
            w2v.train_minibatch(shards, a, b, k, 70 + h, alpha, loss=loss)
        else:
            dots = [s.dotprod(a, b, k, 70 + h) for s in shards]
            g, loss = shards[0].coeffs(dots, k, want_loss=True)
            for s in shards:
                s.adjust(a, b, k, 70 + h, g, alpha)
        losses.append(float(loss))
    return losses


# widths: padded and unpadded strides, a slice in two lane groups' float4, one to four float4 a lane, the widest
# joint row and one past it (of 1024 floats with the rows' padding: 16 x 64, and 17), more slices than lanes of a float4
CASES = [([60] * 16, 400, 5), ([60] * 17, 400, 5), ([60] * 5, 3001, 5), ([1, 2], 17, 5), ([7, 143, 150], 1500, 5), ([30, 30], 999, 5), ([102, 103, 102, 103, 102], 700, 3),
         ([300, 400], 500, 12), ([512, 512], 300, 1), ([512, 513], 300, 1), ([4] * 32, 800, 5), ([33] * 7, 2500, 0),
         ([60, 100, 140], 180_000, 5)]


@pytest.mark.parametrize("widths,n,k", CASES)
def test_joint_step_matches_each_shard_on_its_own(widths, n, k):
    print("slices", widths, n, k, flush=True)
    rng = np.random.default_rng(n)
    V, d = 2500, sum(widths)
    begins = np.concatenate([[0], np.cumsum(widths)[:-1]])
    counts = zipf_counts(V)
    sets = [[make_shard(V, w, 5, counts, d_total=d, col_begin=int(b)) for w, b in zip(widths, begins)] for _ in range(2)]
    ins = [dev(np.minimum(rng.zipf(1.3, n), V) - 1) for _ in range(2)]
    outs = [dev(rng.integers(0, V, n)) for _ in range(2)]
    for s in sets[0] + sets[1]:                     # rows of unit size: the dots count
        for which in (0, 1):
            rows = torch.arange(V, dtype=torch.int32, device="cuda")
            g = torch.Generator(device="cuda").manual_seed(7 + which)
            x = torch.randn(V, d, device="cuda", generator=g) * d ** -0.5
            i = (sets[0] + sets[1]).index(s) % len(widths)
            s.set_rows(which, rows, x[:, begins[i]:begins[i] + widths[i]].contiguous())
    whole = [np.concatenate([all_rows(s, which) for s in sets[0]], axis=1) for which in (0, 1)]
    la, lb = steps(sets[0], ins, outs, k, "joint"), steps(sets[1], ins, outs, k, "apart")
    assert np.allclose(la, lb, rtol=1e-6)
    th, al = oracle.build_alias(counts)
    for h, (a, b) in enumerate(zip(ins, outs)):
        ref = oracle.train_minibatch([whole[0]], [whole[1]], w2v.index_to_numpy(a), w2v.index_to_numpy(b), k, 70 + h, th, al, min(0.03, 3.0 / n))
        assert abs(la[h] - ref) <= 1e-5 * ref
    for which in (0, 1):
        assert vec_error(np.concatenate([all_rows(s, which) for s in sets[0]], axis=1), whole[which]) <= 2 * ORACLE_TOL
    for a, b in zip(*sets):
        for which in (0, 1):
            assert vec_error(all_rows(a, which), all_rows(b, which)) <= TOL
        a.status()
    for s in sets[0] + sets[1]:
        s.destroy()


def test_a_shard_listed_twice_is_updated_twice():
    rng = np.random.default_rng(3)
    V, n, k = 300, 900, 5
    counts = zipf_counts(V)
    a, b = make_shard(V, 40, 5, counts), make_shard(V, 40, 5, counts)
    ins, outs = [dev(rng.integers(0, V, n))], [dev(rng.integers(0, V, n))]
    assert steps([a, a], ins, outs, k, "joint") == steps([b, b], ins, outs, k, "apart")
    for which in (0, 1):
        assert np.array_equal(all_rows(a, which), all_rows(b, which))
    a.destroy()
    b.destroy()


def test_joint_step_leaves_a_prepared_step_valid():
    """Joint rows take more scratch than one shard after the other, which had room in what the prepared step reserved."""
    rng = np.random.default_rng(4)
    V, n, k = 500, 4000, 5
    counts = zipf_counts(V)
    sets = [[make_shard(V, 60, 5, counts, d_total=120, col_begin=60 * i) for i in range(2)] for _ in range(2)]
    a, b = dev(rng.integers(0, V, n)), dev(rng.integers(0, V, n))
    graph = w2v.StepGraph(sets[0][0], n, k)
    for one, shards in zip((lambda: graph.run(a, b, 9, 0.01), lambda: w2v.train_minibatch(sets[1][:1], a, b, k, 9, 0.01)), sets):
        w2v.train_minibatch(shards, a, b, k, 8, 0.01)
        one()
    for x, y in zip(*sets):
        for which in (0, 1):
            assert np.array_equal(all_rows(x, which), all_rows(y, which))
    graph.destroy()
    for s in sets[0] + sets[1]:
        s.destroy()


def test_without_memory_for_joint_rows_the_shards_are_trained_apart():
    """Scratch of joint rows (16 x 64 columns, some 2.5 GB) that cannot be had: the step takes each shard on its own,
    and the scratch that a prepared step reserved stays."""
    rng = np.random.default_rng(5)
    V, n, k, S = 2000, 1 << 19, 5, 16
    counts = zipf_counts(V)
    sets = [[make_shard(V, 64, 5, counts, d_total=64 * S, col_begin=64 * i) for i in range(S)] for _ in range(2)]
    a, b = dev(rng.integers(0, V, n)), dev(rng.integers(0, V, n))
    big = dev(rng.integers(0, V, 2 * n))
    loss = [torch.zeros(1, dtype=torch.float64, device="cuda") for _ in range(2)]
    graph = w2v.StepGraph(sets[0][0], 2 * n, k)
    w2v.train_minibatch(sets[1], a, b, k, 7, 1e-4, loss=loss[1])
    w2v.train_minibatch(sets[1][:1], big, big, k, 8, 1e-4)
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    hog = torch.empty(torch.cuda.mem_get_info()[0] - (1 << 30), dtype=torch.uint8, device="cuda")
    free = []
    for h in range(3):
        w2v.train_minibatch(sets[0], a, b, k, 7, 1e-4 if h == 0 else 0.0, loss=loss[0] if h == 0 else None)
        free.append(torch.cuda.mem_get_info()[0])
    graph.run(big, big, 8, 1e-4)
    torch.cuda.synchronize()
    del hog
    torch.cuda.empty_cache()
    assert free[0] == free[1] == free[2] and free[0] > 1 << 29        # (joint rows would have left less)
    assert abs(float(loss[0]) - float(loss[1])) <= 1e-6 * abs(float(loss[1]))
    for x, y in zip(*sets):
        for which in (0, 1):
            assert vec_error(all_rows(x, which), all_rows(y, which)) <= TOL
        x.status()
    graph.destroy()
    for s in sets[0] + sets[1]:
        s.destroy()


def test_a_captured_step_over_shards_grows_nothing():
    """Scratch that holds one shard after the other, but not joint rows: under capture the step makes do with it."""
    rng = np.random.default_rng(6)
    V, n, k = 500, 1500, 5
    counts = zipf_counts(V)
    sets = [[make_shard(V, 60, 5, counts, d_total=300, col_begin=60 * i) for i in range(5)] for _ in range(2)]
    a, b = dev(rng.integers(0, V, n)), dev(rng.integers(0, V, n))
    more = dev(rng.integers(0, V, 2 * n))
    w2v.train_minibatch(sets[0][:1], more, more, k, 8, 0.0)      # one shard's scratch for twice the pairs, a fifth of the columns
    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph):
        w2v.train_minibatch(sets[0], a, b, k, 9, 0.01)
    for replay in range(3):
        graph.replay()
        torch.cuda.synchronize()
        w2v.train_minibatch(sets[1], a, b, k, 9, 0.01)
        for x, y in zip(*sets):
            for which in (0, 1):
                assert vec_error(all_rows(x, which), all_rows(y, which)) <= (replay + 1) * TOL
    for s in sets[0] + sets[1]:
        s.destroy()


class Rows:
    """All of a shard's matrix as it lies in memory, padding included (a host function, by its linker name)."""
    def __init__(self, shard, which):
        fn = ctypes.CDLL(w2v.LIB_PATH)._ZN3w2v10shard_rowsEPK9w2v_shardiPj
        fn.restype, fn.argtypes = ctypes.c_void_p, [ctypes.c_void_p, ctypes.c_int, ctypes.POINTER(ctypes.c_uint32)]
        stride = ctypes.c_uint32()
        at = fn(shard.h, which, ctypes.byref(stride))
        self.__cuda_array_interface__ = dict(shape=(shard.V, stride.value), typestr="<f4", data=(at, False), version=2)


# up to four float4 a lane, padding of a whole float4 and of parts of one; the last: the write-back has a launch of its own
@pytest.mark.parametrize("widths,n,k", [([60] * 5, 3001, 5), ([60] * 16, 400, 5), ([30, 30], 999, 5), ([27, 59, 122], 1500, 3),
                                        ([58, 300], 700, 12), ([60, 60], 300_000, 5), ([300, 300], 180_000, 5)])
def test_padding_stays_zero(widths, n, k):
    """Matrices are written in whole strides; a step over several shards holds anything in the lanes of the padding."""
    print("padding", widths, n, k, flush=True)
    V, d = 3000, sum(widths)
    counts = zipf_counts(V)
    rng = np.random.default_rng(n)
    begins = np.concatenate([[0], np.cumsum(widths)[:-1]])
    shards = [make_shard(V, w, 5, counts, d_total=d, col_begin=int(b)) for w, b in zip(widths, begins)]
    views = [torch.as_tensor(Rows(s, which), device="cuda")[:, w:] for s, w in zip(shards, widths) for which in (0, 1)]
    assert any(v.shape[1] for v in views)
    for h in range(3):
        a, b = dev(np.minimum(rng.zipf(1.3, n), V) - 1), dev(rng.integers(0, V, n))
        w2v.train_minibatch(shards, a, b, k, 70 + h, 1e-4)
        for s in shards:
            s.status()
        assert all(bool((v.view(torch.int32) == 0).all()) for v in views), h
    for s in shards:
        s.destroy()
