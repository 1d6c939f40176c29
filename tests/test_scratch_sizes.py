"""Sizes of the library's scratch: what one call reserves must hold every launch it may make.

The size rules are host functions inside the library (namespace w2v, not part of the C ABI); the CPU
tests here call them by their linker names and compare them with the arithmetic of the launches.  The
GPU tests run the calls at the sizes where the rules change.
"""
import ctypes

import numpy as np
import pytest
import torch

import oracle
from paper_1606_08495_amd import w2v, workloads
from util import all_rows, dev, vec_error

SMALL = 1 << 19              # elements from which the sort's scratch is reserved by large tiles
TILES = [(300_000, 2048), (1 << 20, 4096), (1 << 32, 8192)]      # below how many elements in all: elements of a tile


def rule(mangled, n_args, restype=ctypes.c_size_t):
    fn = getattr(ctypes.CDLL(w2v.LIB_PATH), mangled)
    fn.restype, fn.argtypes = restype, [ctypes.c_uint32] * n_args
    return fn


def sort_scratch(n0, n1=0):
    return rule("_ZN3w2v16sort_scratch_u32Ejj", 2)(n0, n1)


def sort_need(n0, n1=0):
    """uint32 words that a sort of n0 keys, or of n0 and n1 together, touches: digit totals, tickets, two rows of states
    per tile."""
    tile = next(t for below, t in TILES if n0 + n1 < below)
    return 2 * 4 * 256 + 8 + 2 * 2 * 256 * (-(-n0 // tile) - (-n1 // tile))


@pytest.mark.parametrize("n0,n1", [(SMALL - 1, 1), (SMALL - 1, 0), (SMALL - 1, SMALL - 1), (480_000, 80_000), (522_000, 3_000),
                                   (300_000, 300_000), (6_000, 522_000), (SMALL, 5), (3_000_000, 400_000), (1, 1),
                                   (299_999, 0), (250_000, 49_999), (299_999, 1), (299_999, 299_999), (SMALL - 1, SMALL),
                                   ((1 << 20) - 1, 0), (1 << 20, 0), ((1 << 20) - 1, 1), (299_999, (1 << 20) - 299_999),
                                   ((1 << 20) - 1, 1_500_000), (2_499_999, 0), (2_499_999, 1), (2_500_000, 299_999)])
def test_joint_sort_scratch_holds_each_array_alone(n0, n1):
    have = sort_scratch(n0, n1)
    assert have >= max(sort_need(n0, n1), sort_need(n0), sort_need(n1))
    assert sort_scratch(n0) >= sort_need(n0)


def test_sort_scratch_holds_every_smaller_sort():
    edges = steps_of(300_000, SMALL, 1 << 20, 2_500_000)
    most = 0
    for n in [s for s in edges if s < 1 << 24]:
        most = max(most, sort_need(n))
        assert sort_scratch(n) >= most
        for n1 in (1, 2047, 299_999, 700_000):
            assert sort_scratch(n, n1) >= max(most, sort_need(n, n1))


# n (k + 1) < 2^19 <= n (k + 2), both sides sorted by the same launches; n (k + 2) > 1 500 000, each by its own from given
# coefficients (over two shards as one matrix of joint rows: the same launches): n (k + 1) and n in the three shapes
SORT_EDGES = [(80_000, 5), (87_381, 5), (500_000, 0), (750_001, 0), (500_001, 1), (524_288, 1), (299_999, 5), (300_000, 5),
              (416_666, 5), (416_667, 5)]


@pytest.mark.gpu
@pytest.mark.parametrize("n,k", SORT_EDGES)
@pytest.mark.parametrize("form", ["adjust", "two shards"])
def test_both_sides_sorted_at_the_edges_of_the_tiles(n, k, form):
    print("sorts", n, k, form, flush=True)
    V, d, alpha = 3000, 8, 0.001
    rng = np.random.default_rng(n + k)
    counts = workloads.analytic_counts(V, 1.0, 10 ** 7)
    th, al = oracle.build_alias(counts)
    a, b = (workloads.zipf_draw(workloads.zipf_cdf(V, 1.0), n, rng) for _ in range(2))
    rows = np.arange(V, dtype=np.uint32)
    U, W = oracle.init_rows(3, d, 0, d, 0, rows), oracle.init_rows(3, d, 0, d, 1, rows)
    cuts = [(0, d)] if form == "adjust" else [(0, 3), (3, 5)]
    shards = [w2v.Shard(V, w, 3, d_total=d, col_begin=c, init_mode=1) for c, w in cuts]
    for sh in shards:
        sh.set_counts(counts)
    for step in range(2):                                       # the second on states the first has left
        if form == "adjust":
            g = workloads.uniform_coeffs(n, k + 1, step)
            shards[0].adjust(dev(a), dev(b), k, 40 + step, torch.from_numpy(g).cuda(), alpha)
            oracle.adjust(U, W, a, b, k, 40 + step, th, al, g, alpha)
        else:
            w2v.train_minibatch(shards, dev(a), dev(b), k, 40 + step, alpha)
            oracle.train_minibatch([U], [W], a, b, k, 40 + step, th, al, alpha)
    for sh in shards:
        sh.status()
    got = [np.concatenate([all_rows(sh, which) for sh in shards], axis=1) for which in (0, 1)]
    assert vec_error(got[0], U) <= 2e-5 and vec_error(got[1], W) <= 2e-5      # 1e-5 a minibatch
    for sh in shards:
        sh.destroy()


@pytest.mark.gpu
@pytest.mark.parametrize("n,k,m", [(87_000, 5, 3_000), (80_000, 5, 200_000), (60_000, 5, 500_000)])
def test_bag_of_words_sorts_apart_at_the_edge_of_the_small_tiles(n, k, m):
    print("bag of words, sorts apart", n, k, m, flush=True)
    V, d, alpha = 3000, 8, 0.001
    rng = np.random.default_rng(m)
    counts = workloads.analytic_counts(V, 1.0, 10 ** 7)
    th, al = oracle.build_alias(counts)
    cdf = workloads.zipf_cdf(V, 1.0)
    ctx, out = workloads.zipf_draw(cdf, m, rng), workloads.zipf_draw(cdf, n, rng)
    off = np.concatenate([[0], np.sort(rng.integers(0, m + 1, n - 1)), [m]]).astype(np.uint32)
    rows = np.arange(V, dtype=np.uint32)
    U, W = oracle.init_rows(3, d, 0, d, 0, rows), oracle.init_rows(3, d, 0, d, 1, rows)
    sh = w2v.Shard(V, d, 3, init_mode=1)
    sh.set_counts(counts)
    for step in range(2):
        w2v.cbow_train_minibatch([sh], dev(off), dev(ctx), dev(out), k, 60 + step, alpha)
        oracle.cbow_train_minibatch([U], [W], off, ctx, out, k, 60 + step, th, al, alpha)
    g = workloads.uniform_coeffs(n, k + 1, 7)
    sh.cbow_adjust(dev(off), dev(ctx), dev(out), k, 70, torch.from_numpy(g).cuda(), alpha)
    oracle.cbow_adjust(U, W, off, ctx, out, k, 70, th, al, g, alpha)
    sh.status()
    assert vec_error(all_rows(sh, 0), U) <= 3e-5 and vec_error(all_rows(sh, 1), W) <= 3e-5    # 1e-5 a minibatch
    sh.destroy()


def slots_after(entries, per_chunk):
    return 2 * (-(-entries // per_chunk) - 1) if entries else 0


def steps_of(*edges):
    """Sizes around the edges and between them, increasing."""
    return sorted({max(1, e + o) for e in edges for o in (-1, 0, 1)} | {int(1.31 ** i) for i in range(1, 70)})


def test_scratch_of_a_minibatch_holds_every_smaller_one():
    """A region grown by a large minibatch serves smaller ones without growing again: what the rules of
    the chunk sizes ask for at any smaller size is within what is reserved, and that never falls."""
    most_w, cell = rule("_ZN3w2v15wseg_slots_mostEj", 1, ctypes.c_uint32), rule("_ZN3w2v22wseg_entries_per_chunkEj", 1, ctypes.c_uint32)
    sizes = [s for s in steps_of(1 << 19, 1 << 20) if s < 1 << 28]
    held = needed = 0
    for M in sizes:
        needed = max(needed, slots_after(M, cell(M)))
        assert most_w(M) >= max(needed, held)
        held = most_w(M)
    most_u, chunk = rule("_ZN3w2v15useg_slots_mostEjj", 2, ctypes.c_uint32), rule("_ZN3w2v20useg_pairs_per_chunkEjjj", 3, ctypes.c_uint32)
    held_T = {}
    for T in (1, 2, 3, 6, 11, 17, 24, 25, 26, 65):
        held = needed = 0
        for n in [s for s in steps_of(*(32768 * c for c in range(1, 34))) if s < 1 << 25]:
            needed = max([needed] + [slots_after(n, chunk(T, d4, n)) for d4 in (1, 16, 17, 32, 33, 64, 256)])
            assert most_u(T, n) >= max(needed, held, held_T.get(n, 0)), (T, n)
            held = held_T[n] = most_u(T, n)
    loss = rule("_ZN3w2v27coeffs_loss_scratch_doublesEjj", 2)
    held = needed = 0
    for n in [s for s in steps_of(1 << 24) if s < 1 << 30]:
        needed = max(needed, -(-n // (1024 if n <= 1 << 24 else 16384)))
        assert loss(n, 1) >= max(needed, held)
        held = loss(n, 1)
    for n1 in (0, 1, 5000, 700_000):
        held = 0
        for n0 in [s for s in steps_of(SMALL, SMALL - n1 if n1 < SMALL else SMALL) if s < 1 << 28]:
            assert sort_scratch(n0, n1) >= held
            held = sort_scratch(n0, n1)


@pytest.mark.parametrize("free,asked,held_after", [(10_000, 50_000, 10_000), (60_000, 50_000, 50_000), (100_000, 50_000, 60_346)])
@pytest.mark.parametrize("same_address", [False, True])
def test_a_region_that_cannot_grow_is_left_as_large_as_it_was(free, asked, held_after, same_address):
    """What a prepared step was promised stays there: against an allocator of `free` bytes, of which 10 000 are held,
    that gives out new addresses or the first that is free again."""
    alloc_t = ctypes.CFUNCTYPE(ctypes.c_int, ctypes.POINTER(ctypes.c_void_p), ctypes.c_size_t)
    release_t = ctypes.CFUNCTYPE(ctypes.c_int, ctypes.c_void_p)
    blocks, made = {4096: 10_000}, [0]

    def alloc(p, n):
        if sum(blocks.values()) + n > free:
            return 2
        made[0] += 1
        at = 4096 if same_address else 4096 + (made[0] << 32)
        assert at not in blocks
        blocks[at], p[0] = n, at
        return 0

    def release(p):
        del blocks[p]
        return 0

    fn = ctypes.CDLL(w2v.LIB_PATH)._ZN3w2v11grow_regionEPPcPmmPFiPPvmEPFiS3_EPi
    fn.argtypes = [ctypes.POINTER(ctypes.c_void_p), ctypes.POINTER(ctypes.c_size_t), ctypes.c_size_t, alloc_t, release_t,
                   ctypes.POINTER(ctypes.c_int)]
    region, cap, error = ctypes.c_void_p(4096), ctypes.c_size_t(10_000), ctypes.c_int(0)
    rc = fn(region, cap, asked, alloc_t(alloc), release_t(release), error)
    assert (rc == 0) == (held_after >= asked) and (rc == 0 or error.value == 2)
    assert cap.value == held_after and blocks == {region.value: held_after}


@pytest.mark.gpu
@pytest.mark.parametrize("d,big,small,k", [(300, 20_165, 20_164, 25), (300, 98_304, 98_303, 5)])
def test_a_smaller_minibatch_leaves_a_captured_step_valid(d, big, small, k):
    """(n (k+1) just past 2^19, where the cells of long runs double; n where the input side's chunks grow)"""
    print("captured", big, "then plain", small, flush=True)
    V = 2000
    rng = np.random.default_rng(1)
    a, b = dev(rng.integers(0, V, big).astype(np.uint32)), dev(rng.integers(0, V, big).astype(np.uint32))
    sh = w2v.Shard(V, d, 3)
    sh.set_counts(np.ones(V, np.uint64))
    graph = w2v.StepGraph(sh, big, k)
    w2v.train_minibatch([sh], a[:small].contiguous(), b[:small].contiguous(), k, 5, 0.001)
    graph.run(a, b, 6, 0.001)
    sh.status()
    graph.destroy()
    sh.destroy()


@pytest.mark.parametrize("Q,N,d", [(1, 10_000, 300), (1, 20_000, 300), (1, 1 << 19, 512), (4, 5000, 300), (7, 3000, 512),
                                   (32, 3000, 512), (33, 5000, 300), (100, 200_003, 100), (128, 1 << 20, 1000)])
def test_few_queries_take_the_stream_screen_with_the_default_workspace(Q, N, d):
    """Its query tiles are 32, 64 or 128 rows: the rounded queries fit a workspace for rounds of 32768."""
    fn = ctypes.CDLL(w2v.LIB_PATH)._ZN3w2v11topk_screenEjjjm
    fn.restype, fn.argtypes = ctypes.c_uint32, [ctypes.c_uint32] * 3 + [ctypes.c_size_t]
    assert fn(Q, N, d, w2v.lib().w2v_topk_cosine_workspace(Q, N, 32768)) == 1
