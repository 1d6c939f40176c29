"""Pair formation where a sum of sums, or a block's list of centers, is exceeded."""
import numpy as np
import pytest
import torch

import oracle
from paper_1606_08495_amd import w2v, workloads
from util import dev

pytestmark = pytest.mark.gpu


# whole and cut blocks of centers; blocks of more than 6144 pairs; the longest text whose blocks add up the counts before
# them, and one of which these are scanned
@pytest.mark.parametrize("n_tok,B,sentence", [(65_536, 2, 30), (65_537, 2, 7), (200_001, 1, 25), (9000, 40, 500), (5000, 13, 5000),
                                              (1 << 22, 1, 19), ((1 << 22) + 1, 1, 19)])
def test_long_texts_and_wide_windows(n_tok, B, sentence):
    print("formation", n_tok, B, sentence, flush=True)
    rng = np.random.default_rng(n_tok + B)
    V = 300
    tokens = workloads.zipf_draw(workloads.zipf_cdf(V, 1.0), n_tok, rng)
    off = np.append(np.arange(0, n_tok, sentence), n_tok).astype(np.uint64)
    sh = w2v.Shard(V, 4, 1)
    sh.set_counts(np.maximum(1, workloads.counted(tokens, V)), 0.0)        # every token survives
    doff = torch.from_numpy(off.astype(np.int64)).cuda()
    gi, go = (torch.empty(n_tok * 2 * B, dtype=torch.int32, device="cuda") for _ in range(2))
    for inter in (False, True):
        cnt = sh.make_pairs(dev(tokens), doff, 9, 0, 3, B, gi, go, interleaved=inter)
        oi, oo, ocnt = oracle.make_pairs(tokens, off, 9, 0, 3, B, None, interleaved=inter)
        assert cnt == ocnt
        assert np.array_equal(w2v.index_to_numpy(gi[:cnt]), oi) and np.array_equal(w2v.index_to_numpy(go[:cnt]), oo)
    co, ce = torch.empty(n_tok + 1, dtype=torch.int32, device="cuda"), torch.empty(n_tok, dtype=torch.int32, device="cuda")
    n_ex, n_ctx = sh.make_cbow_examples(dev(tokens), doff, 9, 0, 3, B, co, go, ce)
    ooff, octx, oout, ocnt, onctx = oracle.make_cbow_examples(tokens, off, 9, 0, 3, B, None)
    assert (n_ex, n_ctx) == (ocnt, onctx)
    assert np.array_equal(w2v.index_to_numpy(co[:n_ex + 1]), ooff) and np.array_equal(w2v.index_to_numpy(ce[:n_ex]), oout)
    assert np.array_equal(w2v.index_to_numpy(go[:n_ctx]), octx)
    sh.status()
    sh.destroy()
