"""Dense products with rows = nodes: tile, step and alignment edges of the three kernels (one wavefront per tile, three
bf16 parts per float, fp32 instruction), and what the parts cannot hold."""
import numpy as np
import pytest
import torch

from paper_2308_12093_amd import binding as B

pytestmark = pytest.mark.gpu

# (M, N, K): below and above the size (1024 tiles of 32 x 32) up to which a tile has a wavefront of its own, edges of the
# 128-row, 32/64/128-column tiles and 32-index steps, widths that are no multiple of 4
SHAPES = [(1, 1, 1), (33, 31, 3), (64, 32, 32), (2048, 16, 512), (3001, 7, 203), (32768, 16, 128), (32769, 16, 128), (65600, 32, 3),
          (66000, 33, 31), (65281, 64, 47), (32000, 200, 5), (65281, 65, 33), (33000, 129, 36), (32769, 256, 64),
          (65536, 128, 16), (66001, 100, 101), (65664, 32, 4)]


def product(M, N, K, A, Bm, tb, bias=None, relu=0, C=None, workspace=True):
    C = torch.empty(M, N, device="cuda") if C is None else C
    ws = B.alloc(B.gnn_gemm_workspace_bytes(0, tb, M, N, K)) if workspace else None
    B.gnn_gemm(0, tb, M, N, K, A, Bm.t().contiguous() if tb else Bm, C, bias, relu, ws)
    return C


@pytest.mark.parametrize("tb", [0, 1])
@pytest.mark.parametrize("M,N,K", SHAPES)
def test_against_float64(M, N, K, tb):
    gen = torch.Generator(device="cuda").manual_seed(M + N + K)
    A, Bm = torch.randn(M, K, generator=gen, device="cuda"), torch.randn(K, N, generator=gen, device="cuda")
    bias = torch.randn(N, generator=gen, device="cuda")
    held = torch.randn(M, N, generator=gen, device="cuda")
    ref = A.double() @ Bm.double()
    # at most eight roundings of the sum per 16 indices, the dropped products (2^-26) and the rounding of bias and held value
    bound = (8 * ((K + 15) // 16) + 4) * 2.0 ** -24 * (A.abs().double() @ Bm.abs().double())
    runs = [(product(M, N, K, A, Bm, tb), ref, 0.0)]
    runs.append((product(M, N, K, A, Bm, tb, bias, 1 | 4, held.clone()), torch.relu(ref + bias + held),
                 2.0 ** -22 * (ref.abs() + bias.abs() + held.abs())))
    if tb:
        runs.append((product(M, N, K, A, Bm, tb, workspace=False), ref, 0.0))
    for got, want, more in runs:
        assert bool(((got.double() - want).abs() <= bound + more).all())


@pytest.mark.parametrize("M", [96, 70000])                 # a wavefront per tile, and the parts
def test_values_the_parts_cannot_hold(M):
    N, K = 40, 70
    gen = torch.Generator(device="cuda").manual_seed(M)
    A, Bm = torch.randn(M, K, generator=gen, device="cuda"), torch.randn(K, N, generator=gen, device="cuda").abs() + 0.5
    A[3, 7] = float("inf")
    A[5, 1] = float("nan")
    A[40] = 0.0
    A[40, 2] = 3.4e38                                       # rounds to infinity in bf16
    A[M - 1] *= 1e-34                                       # third parts below the bf16 range
    Bm[:, 33] *= 1e-34
    Bm[40:, 33] = 0.0
    A[40, 2:] *= 0.5
    got = product(M, N, K, A, Bm, 0)
    ref = A.double() @ Bm.double()
    assert bool(torch.isinf(got[3]).all()) and bool((got[3] > 0).all())
    assert bool(torch.isnan(got[5]).all())
    keep = torch.ones(M, dtype=torch.bool, device="cuda")
    keep[3] = keep[5] = False
    bound = K * 2.0 ** -23 * (A.abs().double() @ Bm.abs().double()) + 2.0 ** -140
    fits = keep[:, None] & (ref.abs() < 3.4e38)
    assert bool(((got.double() - ref).abs() <= bound)[fits].all())
    assert bool(torch.isinf(got[40][ref[40] > 3.5e38]).all())


@pytest.mark.parametrize("tb", [0, 1])
@pytest.mark.parametrize("side", ["A", "B"])
@pytest.mark.parametrize("N,K", [(40, 70), (128, 33)])
def test_small_operands_beside_large_ones(side, tb, N, K):
    """Rows and columns whose sum hangs on an element of 2^-100 .. 2^-149 (its third part is below the bf16 range from 2^-110
    on): what is larger in its row or column meets zero."""
    M = 70000
    gen = torch.Generator(device="cuda").manual_seed(N)
    small = torch.empty(M if side == "A" else N, device="cuda").uniform_(1, 2, generator=gen)
    small *= 2.0 ** -(100.0 + torch.arange(small.numel(), device="cuda") % 46)
    A, Bm = torch.zeros(M, K, device="cuda"), torch.zeros(K, N, device="cuda")
    if side == "A":
        A[:, 0], A[:, 3], Bm[3] = 1.0, small, torch.empty(N, device="cuda").uniform_(1, 2, generator=gen) * 2.0 ** 112
        A[5], A[6, 3] = 0.0, 0.0
    else:
        Bm[0], Bm[3], A[:, 3] = 1.0, small, torch.empty(M, device="cuda").uniform_(1, 2, generator=gen) * 2.0 ** 112
        Bm[:, 7] = 0.0
    ref = A.double() @ Bm.double()
    # one product a result: its rounding; the parts' dropped products 3 2^-26 and the roundings of three sums
    assert bool(((product(M, N, K, A, Bm, tb).double() - ref).abs() <= 2.0 ** -22 * ref.abs()).all())


def test_small_operands_that_do_not_matter():
    """Saturated probabilities beside ordinary gradients, and decayed weights: the results stay those of the parts."""
    M, N, K = 66000, 64, 48
    gen = torch.Generator(device="cuda").manual_seed(1)
    A, Bm = torch.randn(M, K, generator=gen, device="cuda"), torch.randn(K, N, generator=gen, device="cuda")
    A[::3, 5], A[1::3], Bm[11] = 1e-36, 0.0, 3e-39
    A0, B0 = A.clone(), Bm.clone()
    A0[::3, 5], B0[11] = 0.0, 0.0
    assert bool((product(M, N, K, A, Bm, 0) == product(M, N, K, A0, B0, 0)).all())


# long reductions of a narrow output; 32 columns; fewer, few rows or a large first operand; 64 columns and few rows
@pytest.mark.parametrize("tb,M,N,K", [(1, 12288, 32, 128), (0, 9000, 24, 384), (0, 8225, 7, 1000), (1, 40000, 32, 4), (0, 262144, 32, 64),
                                      (1, 40001, 16, 64), (1, 33000, 1, 4), (0, 420000, 20, 160), (1, 50000, 64, 128)])
def test_fp32_instruction_where_it_is_faster(tb, M, N, K):
    gen = torch.Generator(device="cuda").manual_seed(M + N + K)
    A, Bm = torch.randn(M, K, generator=gen, device="cuda"), torch.randn(K, N, generator=gen, device="cuda")
    C = product(M, N, K, A, Bm, tb)
    assert bool((torch.relu(C) == product(M, N, K, A, Bm, tb, relu=1)).all())      # the same sums as before an activation
    bound = (K + 4) * 2.0 ** -24 * (A.abs().double() @ Bm.abs().double())
    assert bool(((C.double() - A.double() @ Bm.double()).abs() <= bound).all())


@pytest.mark.parametrize("tb", [0, 1])
@pytest.mark.parametrize("N,K", [(70, 40), (256, 33), (33, 200)])
def test_rows_of_tiny_values(N, K, tb):
    """Rows of 2^-85 .. 2^-149, some with larger values later on, beside ordinary rows and rows of zeros."""
    M = 70000
    gen = torch.Generator(device="cuda").manual_seed(N)
    A, Bm = torch.randn(M, K, generator=gen, device="cuda"), torch.randn(K, N, generator=gen, device="cuda")
    A[::3] *= 2.0 ** -(85.0 + torch.arange(A[::3].shape[0], device="cuda") % 65)[:, None]
    A[1::21] = 0.0
    A[2::33, :32] *= 2.0 ** -100                            # tiny in the first 32 places only
    A[4::33, :32] *= 2.0 ** -140
    A[5::1000, 0], A[6::1000, K - 1] = float("inf"), 1e38
    C, ref = product(M, N, K, A, Bm, tb).double(), A.double() @ Bm.double()
    bound = (8 * ((K + 15) // 16) + 4) * 2.0 ** -24 * (A.abs().double() @ Bm.abs().double()) + K * 2.0 ** -149
    fine = torch.isfinite(ref) & (ref.abs() < 3e38)
    assert bool(((C - ref).abs() <= bound)[fine].all())
    assert bool((torch.isinf(C) | torch.isnan(C))[5::1000].all())
