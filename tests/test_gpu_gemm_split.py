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
