"""The product with a wavefront per row: widths that fill lanes or not, rows around what wavefronts share, counts of rows around
a block's, many entries, with and without expanded rows, against float64.  (The lines to the segments: test_gpu_spmm_hubs_small.py.)"""
import pytest
import torch

from paper_2308_12093_amd import binding as B

pytestmark = pytest.mark.gpu


def pattern(lengths, n, gen):
    rowptr = torch.zeros(n + 1, dtype=torch.int32, device="cuda")
    rowptr[1:] = torch.tensor(lengths, device="cuda").cumsum(0).int()
    q = int(rowptr[-1])
    col = torch.randint(0, n, (q,), generator=gen, device="cuda", dtype=torch.int32)
    erow = torch.repeat_interleave(torch.arange(n, device="cuda"), torch.tensor(lengths, device="cuda")).int()
    return rowptr, col, erow, q


def check(n, f, lengths, expanded=True, relu=False):
    gen = torch.Generator(device="cuda").manual_seed(n + f)
    rowptr, col, erow, q = pattern(lengths, n, gen)
    val, X = torch.randn(q, generator=gen, device="cuda"), torch.randn(n, f, generator=gen, device="cuda")
    bias, C = torch.randn(f, generator=gen, device="cuda"), torch.full((n, f), float("nan"), device="cuda")
    ws = B.alloc(B.gnn_spmm_workspace_bytes(n, q, f))
    B.gnn_spmm_csr(n, q, rowptr, col, val, erow if expanded else None, X, f, C, bias=bias, relu=relu, workspace=ws)
    ref, size = (torch.zeros(n, f, dtype=torch.float64, device="cuda") for _ in range(2))
    term = val.double()[:, None] * X.double()[col.long()]
    ref.index_add_(0, erow.long(), term)
    size.index_add_(0, erow.long(), term.abs())
    ref += bias.double()
    if relu:
        ref = torch.relu(ref)
    # a rounding per entry at the most, and a few for the sums of the slots and the bias
    bound = (torch.tensor(lengths, device="cuda").double()[:, None] + 16) * 2.0 ** -24 * (size + bias.abs())
    assert bool(((C.double() - ref).abs() <= bound).all())


@pytest.mark.parametrize("f", [1, 2, 3, 4, 5, 7, 8, 16, 17, 32, 33, 47, 64, 65, 100, 128])
def test_widths(f):
    slots = 64 // max(1, 1 << ((f + 3) // 4 - 1).bit_length())
    rows = [0, 1, 2, 16 * slots - 1, 16 * slots, 16 * slots + 1, 0, 129 * slots, 1000, 3, 0]
    check(len(rows), f, rows)
    check(len(rows), f, rows, relu=True)


@pytest.mark.parametrize("n", [1, 7, 8, 9, 16384, 16385])
def test_rows(n):
    check(n, 16, [i % 5 for i in range(n)])


@pytest.mark.parametrize("f,q", [(16, 412500), (16, 412501), (32, 206250), (32, 206251), (33, 75757), (33, 75758), (128, 19531)])
def test_lines(f, q):
    n = 512
    check(n, f, [q // n + (i < q % n) for i in range(n)])


@pytest.mark.parametrize("f", [3, 16, 130, 300])
def test_without_expanded_rows(f):
    check(40, f, [0, 700, 1, 0, 5000] * 8, expanded=False)
