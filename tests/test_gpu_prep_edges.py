"""Preprocessing at the edges of its tiles (1024 entries in lists below 2^20, 4096 in longer ones; 8192 in the sort) and
digits, bit for bit against the oracle."""
import numpy as np
import pytest
import torch

import oracle
from paper_2308_12093_amd import binding as B
from paper_2308_12093_amd import graphs as G
from tests._util import assert_close, dev, host

pytestmark = pytest.mark.gpu


def pattern(n, nnz, hub, seed):
    """Sorted rows without duplicates: `hub` of the entries in row n // 2, the others spread; empty rows at both ends."""
    rng = np.random.default_rng(seed)
    keys = set((n // 2) * n + rng.choice(n, min(hub, n), replace=False).astype(np.int64))
    lo, hi = (n // 4, n - n // 4) if n > 8 else (0, n)
    while len(keys) < nnz:
        r, c = rng.integers(lo, hi, nnz), rng.integers(0, n, nnz)
        for k in r * n + c:
            keys.add(int(k))
            if len(keys) == nnz:
                break
    keys = np.sort(np.fromiter(keys, np.int64, len(keys)))
    rowptr = np.zeros(n + 1, np.int32)
    np.cumsum(np.bincount(keys // n, minlength=n), out=rowptr[1:])
    return rowptr, (keys % n).astype(np.int32)


@pytest.mark.parametrize("n,nnz,hub", [
    (1, 1, 0), (2, 1, 0), (257, 4095, 257), (300, 4096, 0), (300, 4097, 0), (256, 8192, 256), (70000, 8191, 8000),
    (20000, 8193, 8193), (65536, 40960, 20000), (65537, 3, 0), (128, 4096, 0), (300, 12288, 0),
])
def test_tile_and_digit_edges(n, nnz, hub):
    rowptr, col = pattern(n, nnz, hub, seed=n + nnz)
    rp_o, c_o, deg_o = oracle.add_self_loops_degree(rowptr, col)
    rp, c, deg = G.add_self_loops(n, dev(rowptr), dev(col))
    for got, ref in ((rp, rp_o), (c, c_o), (deg, deg_o)):
        np.testing.assert_array_equal(host(got), ref)
    val = torch.empty(c.numel(), device="cuda")
    B.gnn_gcn_normalize(n, rp, c, deg, val)
    assert_close(host(val), oracle.gcn_normalize(rp_o, c_o, deg_o), "val", tol=1e-6)
    for ptr, idx in ((rowptr, col), (rp_o, c_o)):          # with empty rows, and with none
        np.testing.assert_array_equal(host(G.expand(n, dev(ptr), idx.size)), np.repeat(np.arange(n), np.diff(ptr)))
        for got, ref in zip(G.transpose(n, dev(ptr), dev(idx)), oracle.csr_transpose(ptr, idx)):
            np.testing.assert_array_equal(host(got), ref)


@pytest.mark.parametrize("count", [1, 4095, 4096, 4097, 1 << 20, (1 << 20) + 1])
def test_scan_tiles(count):
    """Row pointers after the insertion of the diagonal into an empty pattern: the scan of `count` ones and a zero."""
    rp, c, deg = G.add_self_loops(count, dev(np.zeros(count + 1, np.int32)), dev(np.zeros(0, np.int32)))
    np.testing.assert_array_equal(host(rp), np.arange(count + 1))
    np.testing.assert_array_equal(host(c), np.arange(count))
    assert int(deg.min()) == int(deg.max()) == 1


@pytest.mark.parametrize("said", [0, 1, 5000])
def test_expand_writes_what_the_pointers_say(said):
    """The entry count that goes with the call only sizes the launch."""
    rowptr, _ = pattern(3000, 9001, 2000, seed=1)
    out = torch.full((9001,), -1, dtype=torch.int32, device="cuda")
    B.gnn_expand_ptr(3000, said, dev(rowptr), out)
    np.testing.assert_array_equal(host(out), np.repeat(np.arange(3000), np.diff(rowptr)))


def check_setup(n, rowptr, col):
    """Every preprocessing step of a pattern, bit for bit."""
    rp_o, c_o, deg_o = oracle.add_self_loops_degree(rowptr, col)
    rp, c, deg = G.add_self_loops(n, dev(rowptr), dev(col))
    for got, ref in ((rp, rp_o), (c, c_o), (deg, deg_o)):
        np.testing.assert_array_equal(host(got), ref)
    for got, ref in zip(G.transpose(n, dev(rowptr), dev(col)), oracle.csr_transpose(rowptr, col)):
        np.testing.assert_array_equal(host(got), ref)
    rows = np.repeat(np.arange(n), np.diff(rowptr))
    np.testing.assert_array_equal(host(G.expand(n, dev(rowptr), col.size)), rows)
    val, ones = torch.empty(col.size, device="cuda"), torch.arange(1, n + 1, dtype=torch.int32, device="cuda")
    B.gnn_aggregator_weights(B.GNN_AGG_MEAN, 0.0, n, dev(rowptr), dev(col), ones, val)
    np.testing.assert_array_equal(host(val), np.float32(1) / (rows + 1).astype(np.float32))


def stretched(nnz, gaps, seed):
    """Rows of one to nine entries, with `gaps` (place among them, number) of empty rows in between."""
    rng = np.random.default_rng(seed)
    lens = rng.integers(1, 10, nnz // 4)
    lens = lens[np.cumsum(lens) < nnz]
    lens = np.append(lens, nnz - lens.sum())
    lens = np.insert(lens, np.repeat([int(at * lens.size) for at, _ in gaps], [k for _, k in gaps]), 0)
    n = lens.size
    rowptr = np.zeros(n + 1, np.int32)
    np.cumsum(lens, out=rowptr[1:])
    j = np.arange(nnz) - np.repeat(rowptr[:-1], lens)       # ascending: a random start and a step that fits
    step = n // (int(lens.max()) + 1)
    col = np.repeat(rng.integers(0, step, n), lens) + j * step
    return n, rowptr, col.astype(np.int32)


# a long run of empty rows inside one tile (of 1024, of 4096 and of 8192 entries): in front, between, at the end; a few beside it
@pytest.mark.parametrize("nnz", [700, 8200, (1 << 20) + 4100])
@pytest.mark.parametrize("gaps", [[(0, 40000)], [(0.5, 40000)], [(1, 40000)], [(0.3, 5), (0.31, 33000), (0.6, 70000), (1, 1)]])
def test_long_runs_of_empty_rows(nnz, gaps):
    check_setup(*stretched(nnz, gaps, seed=nnz))


def test_empty_rows_cost_no_more_than_others():
    """2^21 nodes without an edge against as many with one each."""
    n = 1 << 21
    ids = torch.arange(n + 1, dtype=torch.int32, device="cuda")
    cases = [(torch.zeros_like(ids), ids[:0]), (ids, ids[:n].flip(0).contiguous())]
    times = []
    for rowptr, col in cases:
        best = float("inf")
        for _ in range(4):
            start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            start.record()
            G.add_self_loops(n, rowptr, col)
            end.record()
            end.synchronize()
            best = min(best, start.elapsed_time(end))
        times.append(best)
    assert times[0] < 3 * times[1], times


# lists of 2^20 entries and more, in tiles of 4096: around the line, whole tiles, one entry more and less; empty rows here and there
@pytest.mark.parametrize("nnz", [(1 << 20) - 1, 1 << 20, (1 << 20) + 1, (1 << 20) + 4095, (1 << 20) + 4097])
def test_edges_of_long_lists(nnz):
    check_setup(*stretched(nnz, [(0, 3), (0.25, 1), (0.5, 5000), (1, 2)], seed=nnz))


def test_hub_rows_of_long_lists():
    """Rows that fill several tiles of 4096 entries, and one that ends with one."""
    lens = np.zeros(100000, np.int64)
    lens[::7] = 70
    lens[[0, 5, 50001, 99999]] = 40000, 8192, 12289, 4096
    rowptr = np.zeros(lens.size + 1, np.int32)
    np.cumsum(lens, out=rowptr[1:])
    col = np.concatenate([np.arange(k) + i % (lens.size - k + 1) for i, k in enumerate(lens) if k]).astype(np.int32)
    assert col.size > 1 << 20
    check_setup(lens.size, rowptr, col)


@pytest.mark.parametrize("count", [(1 << 24) - 1, 1 << 24, (1 << 24) + 4097])
def test_scans_of_many_tiles(count):
    """4096 tiles of 4096 elements, up to which the second kernel sums the tile totals, and more, where they are scanned: `count`
    row lengths and a zero, an entry in every third row."""
    entries = torch.arange(0, count, 3, device="cuda")
    rowptr = (torch.arange(count + 1, device="cuda") + 2).div(3, rounding_mode="floor").int()
    rp, c, deg = G.add_self_loops(count, rowptr, (entries == 0).int())
    # row 3 i holds column 0 (row 0: column 1): a diagonal and an entry there, a diagonal elsewhere
    at = torch.arange(count + 1, device="cuda")
    assert bool((rp == at + (at + 2).div(3, rounding_mode="floor")).all())
    has = at[:-1] % 3 == 0
    assert bool((deg == 1 + has.int()).all()) and c.numel() == count + entries.numel()
    first = c[rp[:-1].long()]
    assert bool((first == torch.where(has, 0, at[:-1])).all())
    assert bool((c[rp[:-1][has].long() + 1] == torch.where(at[:-1][has] == 0, 1, at[:-1][has])).all())
