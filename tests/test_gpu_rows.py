"""Row get / set / export at the widths, counts and alignments where the moves change their access
width or their rows per block.  Whole words move: everything is compared bit for bit."""
import numpy as np
import pytest
import torch

import oracle
from paper_1606_08495_amd import w2v
from util import dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [1, 2, 3, 4, 6, 61, 64, 300, 1023, 1024])
@pytest.mark.parametrize("m", [1, 2047, 2048, 6001])
def test_get_and_set_rows_move_whole_rows(d, m):
    V, seed = 3000, 4
    sh = w2v.Shard(V, d, seed, init_mode=1)
    rng = np.random.default_rng(d * 10007 + m)
    rows = rng.integers(0, V, m).astype(np.uint32)
    U = oracle.init_rows(seed, d, 0, d, 0, np.arange(V, dtype=np.uint32))
    assert np.array_equal(sh.get_rows(0, dev(rows)).cpu().numpy(), U[rows])
    some = rng.permutation(V)[:min(m, V)].astype(np.uint32)      # (distinct: two writers of a row would race)
    src = torch.from_numpy(rng.standard_normal(some.size * d + 1).astype(np.float32)).cuda()
    x = src[1:].view(some.size, d)                               # four bytes off the allocation's alignment
    sh.set_rows(0, dev(some), x)
    U[some] = x.cpu().numpy()
    assert np.array_equal(sh.get_rows(0, dev(np.arange(V, dtype=np.uint32))).cpu().numpy(), U)
    sh.status()
    sh.destroy()


def test_rows_outside_are_reported_and_not_written():
    V, d = 50, 12
    sh = w2v.Shard(V, d, 1, init_mode=1)
    rows = np.array([3, V, 0xFFFFFFFF, 7], np.uint32)
    before = sh.get_rows(0, dev(np.arange(V, dtype=np.uint32)))
    got = sh.get_rows(0, dev(rows))
    with pytest.raises(w2v.W2VError):
        sh.status()
    assert torch.equal(got, before[[3, 0, 0, 7]])
    sh.set_rows(0, dev(rows), torch.ones(4, d, device="cuda"))
    with pytest.raises(w2v.W2VError):
        sh.status()
    before[[3, 7]] = 1.0
    assert torch.equal(sh.get_rows(0, dev(np.arange(V, dtype=np.uint32))), before)
    sh.destroy()


@pytest.mark.parametrize("widths", [(4, 8, 4), (60,) * 5, (3, 4, 5), (2, 2), (1, 7), (100,)])
def test_export_joins_slices_of_any_alignment(widths):
    V, seed, total = 700, 9, sum(widths)
    shards, col = [], 0
    for w in widths:
        shards.append(w2v.Shard(V, w, seed, d_total=total, col_begin=col, init_mode=1))
        col += w
    rows = np.random.default_rng(1).integers(0, V, 2500).astype(np.uint32)
    want = oracle.init_rows(seed, total, 0, total, 1, rows)
    assert np.array_equal(w2v.export_rows(shards, 1, dev(rows)).cpu().numpy(), want)
    odd = torch.zeros(rows.size * total + 1, device="cuda")[1:].view(rows.size, total)
    assert np.array_equal(w2v.export_rows(shards, 1, dev(rows), out=odd).cpu().numpy(), want)


@pytest.mark.parametrize("widths,m", [((60,) * 5, 1), ((60,) * 5, 273), ((1, 7), 8 * 256 + 1), ((4,) * 32, 4099), ((32,) * 4, 5001),
                                      ((512, 512), (1 << 18) * 16 + 5), ((7, 8), 8 * 256 + 1), ((60, 100, 140), 166_666), ((60, 100, 140), 166_667)])
def test_export_at_the_edges_of_the_grid(widths, m):
    """Blocks of several parts' rows in groups of eight, the last one not full; past 2^18 of them in a second row of the grid.
    Unequal widths one after the other, together from 200 MB on."""
    print("export", widths, m, flush=True)
    V, total = 64, sum(widths)
    shards, col = [], 0
    for w in widths:
        shards.append(w2v.Shard(V, w, 5, d_total=total, col_begin=col, init_mode=1))
        col += w
    table = torch.from_numpy(oracle.init_rows(5, total, 0, total, 0, np.arange(V, dtype=np.uint32))).cuda()
    rows = torch.randint(0, V, (m,), dtype=torch.int32, device="cuda", generator=torch.Generator(device="cuda").manual_seed(m))
    got = w2v.export_rows(shards, 0, rows)
    for lo in range(0, m, 1 << 18):
        assert torch.equal(got[lo:lo + (1 << 18)], table[rows[lo:lo + (1 << 18)].long()])
    for sh in shards:
        sh.status()
        sh.destroy()
