"""GPU parity of vector export (bit exact) and of the top-K cosine retrieval against the CPU oracle,
through the C ABI.

Retrieval tolerance: the GPU forms each similarity in fp32 (d products accumulated in fp32, two
inverse norms), the oracle in double.  The error of an fp32 dot product is at most about d * 2^-24
times |q||c| and in practice a few times sqrt(d) * 2^-24, so similarities must agree within
TOL = 1e-5 (d <= 1000).  Where the oracle's ranking is decided by a margin wider than 2 TOL the
indices must be identical; inside such a margin any order of the tied candidates is accepted, as
long as every returned candidate's true similarity fits its rank.
"""
import ctypes

import numpy as np
import pytest
import torch

import oracle
from paper_1606_08495_amd import w2v, workloads
from util import dev

pytestmark = pytest.mark.gpu

TOL = 1e-5


def say(*a):
    print(*a, flush=True)


def check_topk(Qm, C, K, tau, gi, gs, gc):
    """gi, gs, gc: GPU index / score / count arrays (numpy)."""
    oi, os_, oc = oracle.topk_cosine(Qm, C, K, tau)
    full_i, full_s, _ = oracle.topk_cosine(Qm, C, min(C.shape[0], K + 8), -2.0)   # a little beyond rank K
    exact = 0
    for q in range(Qm.shape[0]):
        n = int(gc[q])
        # counts differ only if a similarity sits within TOL of tau
        if n != int(oc[q]):
            edge = full_s[q][(np.abs(full_s[q] - tau) <= TOL)]
            assert edge.size >= abs(n - int(oc[q])), (q, n, oc[q])
        assert np.all(gi[q, n:] == 0xFFFFFFFF) and np.all(gs[q, n:] == 0)
        assert np.all(np.diff(gs[q, :n]) <= 0)                            # ranked
        assert np.unique(gi[q, :n]).size == n                             # no candidate twice
        assert np.all(gs[q, :n] > tau)
        m = min(n, int(oc[q]))
        assert np.all(np.abs(gs[q, :m] - os_[q, :m]) <= TOL), (q, np.abs(gs[q, :m] - os_[q, :m]).max())
        # every returned candidate's true similarity (oracle arithmetic) fits its rank
        cq = C[gi[q, :n]].astype(np.float64)
        qv = Qm[q].astype(np.float64)
        den = np.linalg.norm(cq, axis=1) * np.linalg.norm(qv)
        true = np.divide(cq @ qv, den, out=np.zeros(n), where=den > 0)
        assert np.all(np.abs(true - gs[q, :n]) <= TOL)
        # ranks decided by a clear margin must carry the oracle's index
        s = full_s[q]
        for r in range(m):
            above = s[r - 1] - s[r] if r > 0 else np.inf
            below = s[r] - s[r + 1] if r + 1 < s.size else np.inf
            if above > 2 * TOL and below > 2 * TOL:
                assert gi[q, r] == oi[q, r], (q, r)
                exact += 1
    return exact


def run_gpu(Qm, C, K, tau, round_candidates):
    gi, gs, gc = w2v.topk_cosine(torch.from_numpy(Qm).cuda(), torch.from_numpy(C).cuda(), K, tau,
                                 round_candidates=round_candidates)
    torch.cuda.synchronize()
    return w2v.index_to_numpy(gi), gs.cpu().numpy(), w2v.index_to_numpy(gc)


@pytest.mark.parametrize("Q,N,d,K,tau", [(5, 1000, 300, 30, -2.0), (300, 5000, 60, 10, 0.2),
                                         (130, 20011, 100, 64, -2.0), (257, 12800, 37, 1, -2.0),
                                         (1, 3, 7, 5, -2.0), (129, 129, 1000, 30, 0.65), (3, 300, 1, 4, -2.0)])
def test_topk_parity(Q, N, d, K, tau):
    say("topk", Q, N, d, K, tau)
    Qm = workloads.embedding_like(Q, d, 1, n_clusters=50)
    C = workloads.embedding_like(N, d, 2, n_clusters=50)
    ref = None
    for rounds in (128, 1024, 0):
        gi, gs, gc = run_gpu(Qm, C, K, tau, rounds)
        if ref is None:
            exact = check_topk(Qm, C, K, tau, gi, gs, gc)
            say("  ranks with an exact index check:", exact, "of", int(gc.sum()))
            if d >= 30:
                assert exact >= 0.5 * int(gc.sum())
            ref = (gi, gs, gc)
        else:   # the round length never changes the result
            assert np.array_equal(gi, ref[0]) and np.array_equal(gs, ref[1]) and np.array_equal(gc, ref[2])


def test_topk_equal_similarities_rank_by_index_and_zero_vectors_score_zero():
    rng = np.random.default_rng(3)
    N, d, K = 2000, 60, 40
    C = workloads.embedding_like(N, d, 4, n_clusters=20)
    C[1000:] = C[:1000]                     # every candidate twice: bitwise equal similarities
    C[7] = 0; C[1007] = 0
    Qm = workloads.embedding_like(6, d, 5, n_clusters=20)
    Qm[5] = 0                               # an all-zero query: similarity 0 with everyone
    gi, gs, gc = run_gpu(Qm, C, K, -2.0, 256)
    for q in range(5):
        a, b = gi[q, 0::2], gi[q, 1::2]
        assert np.all(b == a + 1000), "a candidate and its copy must come as (lower index, higher index)"
        assert np.all(gs[q, 0::2] == gs[q, 1::2])
    assert gi[5].tolist() == list(range(K)) and np.all(gs[5] == 0)
    oi, os_, oc = oracle.topk_cosine(Qm, C, K)
    assert np.array_equal(gi[5], oi[5])
    check_topk(Qm[:5], C, K, -2.0, gi[:5], gs[:5], gc[:5])


def test_topk_similarities_rising_with_the_index_fill_every_pending_list():
    # candidate i is the query direction plus noise that shrinks with i: every round, most
    # candidates beat the current K-th best, so the pending lists run full.
    rng = np.random.default_rng(6)
    N, d, K = 4096, 64, 30
    Qm = rng.standard_normal((4, d)).astype(np.float32)
    noise = rng.standard_normal((N, d)).astype(np.float32)
    scale = np.linspace(3.0, 0.05, N).astype(np.float32)[:, None]
    C = (Qm[0][None, :] + scale * noise).astype(np.float32)
    for rounds in (128, 1024):
        gi, gs, gc = run_gpu(Qm, C, K, -2.0, rounds)
        check_topk(Qm, C, K, -2.0, gi, gs, gc)
    assert gi[0].min() > N // 2


def test_topk_argument_errors():
    q = torch.zeros((4, 8), dtype=torch.float32, device="cuda")
    c = torch.zeros((10, 8), dtype=torch.float32, device="cuda")
    with pytest.raises(w2v.W2VError) as e:
        w2v.topk_cosine(q, c, 0)
    assert e.value.code == -2
    with pytest.raises(w2v.W2VError):
        w2v.topk_cosine(q, c, 65)
    with pytest.raises(w2v.W2VError) as e:
        w2v.topk_cosine(q, c, 3, workspace=torch.empty(1024, dtype=torch.uint8, device="cuda"))
    assert e.value.code == -2
    ws = torch.empty(1 << 20, dtype=torch.uint8, device="cuda")
    with pytest.raises(w2v.W2VError):
        w2v.topk_cosine(q, c, 3, workspace=ws[4:])
    gi, gs, gc = w2v.topk_cosine(q, c, 3, workspace=ws)        # all zeros: similarity 0, index order
    assert w2v.index_to_numpy(gi).tolist() == [[0, 1, 2]] * 4


def test_topk_full_size_sampled_queries():
    # the benchmark's shape; the oracle checks a sample of the queries
    Q, N, d, K = 4096, 1 << 20, 300, 30
    C = workloads.embedding_like(N, d, 7)
    Qm = workloads.embedding_like(Q, d, 8)
    gi, gs, gc = run_gpu(Qm, C, K, -2.0, 8192)
    pick = np.array([0, 127, 128, 2049, 4095])
    exact = check_topk(Qm[pick], C, K, -2.0, gi[pick], gs[pick], gc[pick])
    say("  full size: exact index checks", exact, "of", pick.size * K)
    assert np.all(gc == K)
    gi2, gs2, gc2 = run_gpu(Qm, C, K, -2.0, 8192)
    assert np.array_equal(gi, gi2) and np.array_equal(gs, gs2)      # reproducible bit for bit


# --- export ---------------------------------------------------------------------------------------------

def test_export_rows_bit_exact():
    V, dt = 1000, 300
    widths = [60, 100, 40, 96, 4]
    begins = np.concatenate([[0], np.cumsum(widths)[:-1]])
    counts = np.ones(V, np.uint64)
    shards = [w2v.Shard(V, w, 9, d_total=dt, col_begin=int(b), init_mode=1) for w, b in zip(widths, begins)]
    for sh in shards:
        sh.set_counts(counts, 0.0)
    rng = np.random.default_rng(10)
    a = dev(rng.integers(0, V, 500).astype(np.uint32))
    b = dev(rng.integers(0, V, 500).astype(np.uint32))
    w2v.train_minibatch(shards, a, b, 5, 77, 0.05)               # move the vectors off their start
    rows = rng.integers(0, V, 333).astype(np.uint32)
    rd = dev(rows)
    for which in (0, 1):
        got = w2v.export_rows(shards[::-1], which, rd).cpu().numpy()      # any shard order
        parts = [sh.get_rows(which, rd).cpu().numpy() for sh in shards]
        assert np.array_equal(got, oracle.export_rows(parts, begins, dt, np.arange(rows.size)))
    whole = oracle.init_rows(9, dt, 0, dt, 0, np.arange(V, dtype=np.uint32))
    fresh = [w2v.Shard(V, w, 9, d_total=dt, col_begin=int(b), init_mode=1) for w, b in zip(widths, begins)]
    allr = torch.arange(V, dtype=torch.int32, device="cuda")
    assert np.array_equal(w2v.export_rows(fresh, 0, allr).cpu().numpy(), whole)
    with pytest.raises(w2v.W2VError) as e:
        w2v.export_rows(fresh[:-1], 0, allr)                      # columns missing
    assert e.value.code == -7
    with pytest.raises(w2v.W2VError):
        w2v.export_rows(fresh + fresh[:1], 0, allr)               # a slice twice
    w2v.export_rows(fresh, 0, dev(np.array([1, V + 5], np.uint32)))
    with pytest.raises(w2v.W2VError) as e:
        fresh[0].status()
    assert e.value.code == -6
    for sh in shards + fresh:
        sh.destroy()


# ---- the screens: which pairs are looked at must not show in the results --------------------------


def screen_of(Q, N, d, nbytes):
    """0 fp32, 1 stream, 2 wide: the library's own rule (a host function, by its linker name)."""
    fn = ctypes.CDLL(w2v.LIB_PATH)._ZN3w2v11topk_screenEjjjm
    fn.restype, fn.argtypes = ctypes.c_uint32, [ctypes.c_uint32] * 3 + [ctypes.c_size_t]
    return fn(Q, N, d, nbytes)


def screens_agree(Qm, C, K, tau):
    """A workspace with room for the 16-bit screen of that many queries (stream up to 128; wide for more
    than 256, and from 129 on where rows are short and few), the default one and the smallest (fp32 scores,
    rounds of 128): same bits."""
    (Q, d), N = Qm.shape, C.shape[0]
    q, c = torch.from_numpy(Qm).cuda(), torch.from_numpy(C).cuda()
    size = lambda r: int(w2v.lib().w2v_topk_cosine_workspace(Q, N, r))
    large, small = size(0) + (Q + N + 512) * (2 * d + 128), size(128)
    assert screen_of(Q, N, d, large) == (2 if Q > 256 or (Q > 128 and N <= 65536 and d <= 320) else 1)
    assert screen_of(Q, N, d, small) == 0
    a, b, e = ([t.cpu().numpy() for t in w2v.topk_cosine(q, c, K, tau, workspace=ws)]
               for ws in (torch.empty(large, dtype=torch.uint8, device="cuda"), torch.empty(small, dtype=torch.uint8, device="cuda"), None))
    for x, y, z in zip(a, b, e):
        assert np.array_equal(x.view(np.uint32), y.view(np.uint32)) and np.array_equal(x.view(np.uint32), z.view(np.uint32))
    return a[0].view(np.uint32), a[1], a[2]


@pytest.mark.parametrize("Q", [1, 31, 33, 65, 128, 129, 257])          # tiles of 32, 64, 128 (stream), 256 (wide)
@pytest.mark.parametrize("N,d", [(129, 3), (1025, 16), (5000, 300), (20001, 102), (3000, 324), (1500, 1000)])
def test_screens_list_every_pair_that_counts(Q, N, d):
    Qm = workloads.embedding_like(Q, d, 11, n_clusters=40)
    C = workloads.embedding_like(N, d, 12, n_clusters=40)
    gi, gs, gc = screens_agree(Qm, C, 30, -2.0)
    if N * Q * d < 10 ** 9:
        check_topk(Qm, C, 30, -2.0, gi, gs, gc)
    screens_agree(Qm, C, 64, 0.2)


# a fold's wavefronts read rows 32 columns at a time, whole or in part, four columns to an access or one; lanes read rows of up to
# 16 (of four to an access 40) columns on their own, of a list up to 24 (48)
@pytest.mark.parametrize("d", [1, 3, 4, 12, 16, 17, 24, 25, 28, 31, 32, 33, 36, 40, 44, 48, 52, 61, 64, 65, 100, 255, 257])
@pytest.mark.parametrize("tau", [-2.0, 0.02])
def test_topk_folds_agree(d, tau):
    """How many wavefronts fold a list, or the bits of a few queries, goes by the number of queries: a
    similarity has the same bits in all.  Similarities rise with the index, so that lists are longer than a wavefront; with
    a threshold no round is formed in fp32, without one the first."""
    say("fold", d, tau)
    K, N = 30, 6000
    rng = np.random.default_rng(d)
    base = 1.0 + rng.random(d)
    Qm = (base + 0.1 * rng.standard_normal((2048, d))).astype(np.float32)
    C = (base + np.linspace(8.0, 0.3, N)[:, None] * rng.standard_normal((N, d))).astype(np.float32)
    C[-50:-25] = C[-25:]                                       # equal similarities, ranked by index
    c, first = torch.from_numpy(C).cuda(), None
    for Q in (2048, 2047, 1024, 1023, 300, 9):
        nbytes = int(w2v.lib().w2v_topk_cosine_workspace(Q, N, 0)) + (Q + N + 512) * (2 * d + 128) + 32768 * Q
        assert screen_of(Q, N, d, nbytes) == (2 if Q > 256 else 1)
        ws = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
        got = [t.cpu().numpy() for t in w2v.topk_cosine(torch.from_numpy(Qm[:Q]).cuda(), c, K, tau, workspace=ws)]
        if first is None:
            first = got
            check_topk(Qm[:40], C, K, tau, got[0][:40].view(np.uint32), got[1][:40], got[2][:40])
        assert all(np.array_equal(a[:Q].view(np.uint32), b.view(np.uint32)) for a, b in zip(first, got)), Q


# long rows that are no multiple of four columns: lanes read them where few are expected (up to 128 queries, more than 96 columns,
# up to 100 candidates of a round: (5000 - 1024) K / 1024 is 97 and 101 for K = 25 and 26, in the first round any threshold)
@pytest.mark.parametrize("Q,d", [(3, 95), (3, 97), (128, 97), (129, 97), (3, 98), (3, 100), (40, 257), (1, 1001)])
@pytest.mark.parametrize("K,tau", [(1, -2.0), (25, -2.0), (26, -2.0), (1, 0.3), (64, 0.3), (10, 0.65)])
def test_few_candidates_of_long_rows(Q, d, K, tau):
    say("few", Q, d, K, tau)
    Qm, C = (workloads.embedding_like(n, d, seed, n_clusters=20) for n, seed in ((Q, 11), (5000, 12)))
    screens_agree(Qm, C, K, tau)


@pytest.mark.parametrize("Q,N", [(7, 9000), (7, 40_000), (200, 9000), (500, 9000)])
@pytest.mark.parametrize("spread", [0.0, 1e-4, 1e-2])
def test_crowded_similarities(Q, N, spread):
    """Similarities closer together than the 16-bit margin, down to equal ones (ranked by index): blocks
    that form them in fp32 after all, rounds that do not screen, early rounds in fp32 (500 queries)."""
    rng = np.random.default_rng(5)
    base = rng.standard_normal(60)
    Qm = (base + spread * rng.standard_normal((Q, 60))).astype(np.float32)
    C = (base + spread * rng.standard_normal((N, 60))).astype(np.float32)
    gi, gs, _ = screens_agree(Qm, C, 30, -2.0)
    C[N // 2:] = rng.standard_normal((N - N // 2, 60))         # the second half is not crowded
    screens_agree(Qm, C, 30, -2.0)
    if spread == 0.0:
        assert np.array_equal(gi, np.tile(np.arange(30, dtype=np.uint32), (Q, 1)))


@pytest.mark.parametrize("Q,N,d", [(512, 60_160, 100), (512, 60_160, 7), (512, 60_160, 300), (512, 21_760, 400), (100, 148_480, 100)])
def test_crowded_rounds_stay_counted(Q, N, d):
    """Every block that screens or might have, from the second round on, is counted as crowded where all similarities are:
    by itself, or by the first block of a round that does not screen.  (The count lies behind the flag word in the
    workspace.)  Rows with and without the next round's rounding beside the products, and few queries."""
    say("crowded", Q, N, d)
    rng = np.random.default_rng(8)
    base = rng.standard_normal(d)
    q, c = (torch.from_numpy((base + 1e-4 * rng.standard_normal((n, d))).astype(np.float32)).cuda() for n in (Q, N))
    ws = torch.zeros(int(w2v.lib().w2v_topk_cosine_workspace(Q, N, 32768)), dtype=torch.uint8, device="cuda")
    w2v.topk_cosine(q, c, 30, 0.5, workspace=ws)
    up = lambda n: (n + 255) // 256 * 256
    at = 2 * up(4 * Q) + up(4 * N) + 2 * up(4 * Q)              # 1 / |query|, 1 / |candidate|, thresholds, two counts
    counted = int(ws[at + 4:at + 8].view(torch.int32).item())
    wide = screen_of(Q, N, d, ws.numel()) == 2
    begin, tiles = (256, -(-Q // 256)) if wide else (1024, -(-Q // 128))
    assert (N - begin) % 128 == 0 and counted == tiles * (N - begin) // 128


# rounds of 1024, 16 384 and the rest: of one block to a query, of two to sixteen; past 32 queries a block for every 32 768
# candidates
@pytest.mark.parametrize("Q,N,d", [(1, 120_000, 12), (7, 34_000, 12), (31, 1 << 18, 12), (128, 120_000, 12), (129, 120_000, 12),
                                   (256, 120_001, 12), (129, 120_000, 13), (1, 120_000, 44), (31, 120_000, 37), (100, 120_000, 52),
                                   (200, 120_000, 33)])
def test_long_rounds_of_rising_similarities(Q, N, d):
    """Nearly all of a round passes the thresholds of the one before: its candidates are shared by several blocks."""
    say("rising", Q, N, d)
    rng = np.random.default_rng(9)
    Qm = (rng.standard_normal(d) + 0.02 * rng.standard_normal((Q, d))).astype(np.float32)
    C = (Qm[0] + np.linspace(3.0, 0.05, N)[:, None] * rng.standard_normal((N, d))).astype(np.float32)
    C[-50:-25] = C[-25:]                                       # equal similarities, ranked by index
    gi, _, gc = screens_agree(Qm, C, 30, -2.0)
    assert gi.min() > N // 2 and np.all(gc == 30)
    screens_agree(Qm, C, 64, 0.9)


@pytest.mark.parametrize("Q", [40, 140])
def test_rows_without_a_usable_length(Q):
    """Zero, tiny, huge, infinite and NaN rows on either side."""
    rng = np.random.default_rng(6)
    d, N = 50, 4000
    Qm, C = rng.standard_normal((Q, d)).astype(np.float32), rng.standard_normal((N, d)).astype(np.float32)
    for M in (Qm, C):
        M[1] = 0
        M[2] *= 1e-17                      # squares underflow in part
        M[3] *= 1e-25                      # and altogether
        M[4] *= 3e19                       # squares overflow
        M[5, 7] = np.inf
        M[6, 7] = np.nan
        M[7, :] = 1e-44
        M[8] *= 1e18
        M[9, 3:] = 0
        M[10, 1:] *= 1e-9
    C[2000:2100] = C[100]
    C[3000:] = 0
    for tau in (-2.0, 0.0, 0.1):
        _, gs, _ = screens_agree(Qm, C, 40, tau)
        assert not np.isnan(gs).any()


def test_more_queries_than_one_launch_holds():
    """2^24 queries and one more: the fold (a block per query) and the stream screen (a block per 128) go
    in slices.  Queries on both sides of the slices' borders must get what they get on their own."""
    Q, N, d, K = (1 << 24) + 1, 1000, 4, 2
    say("queries", Q)
    g = torch.Generator(device="cuda").manual_seed(3)
    q, c = torch.randn(Q, d, device="cuda", generator=g), torch.randn(N, d, device="cuda", generator=g)
    got = w2v.topk_cosine(q, c, K, 0.2, round_candidates=256)
    pick = torch.tensor([0, 127, (1 << 21) - 1, 1 << 21, (1 << 22) - 1, 1 << 22, (1 << 23) + 5, Q - 2, Q - 1], device="cuda")
    want = w2v.topk_cosine(q[pick].contiguous(), c, K, 0.2)
    for x, y in zip(got, want):
        assert torch.equal(x[pick], y)
    assert int(got[2].min()) >= 0 and int((got[2] == K).sum()) > Q // 2
