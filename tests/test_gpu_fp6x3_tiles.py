"""The MX FP6 product over smaller tiles: the same bits as the 256 x 256 tiles where a tile's
K range is not divided, integer products exact everywhere, at tile edges, remainders of the K
blocks, odd leading dimensions and with non-finite values."""
import numpy as np
import pytest

import synth
from gpu_util import gamma, host, say

pytestmark = pytest.mark.gpu

# 64 x 64 tiles with K divided between two groups of waves; 64 x 64 undivided and 128 x 128; K slices
DIVIDED = [(1, 1, 1), (63, 65, 128), (129, 130, 200), (257, 191, 640), (700, 900, 1300)]
WHOLE = [(1500, 1530, 200), (1601, 1345, 129), (2048, 1985, 1000), (1921, 2050, 1409), (3000, 2500, 1500)]
SLICED = [(100, 128, 4100), (64, 65, 8000)]


def place(x, pad):
    import torch
    buf = torch.full((x.shape[0], x.shape[1] + pad), float("nan"), device="cuda")[:, pad:]
    buf.copy_(torch.from_numpy(x))
    return buf


def product(A, B, C0=None, alpha=1.0, beta=0.0, pad=0, big=False):
    """(C, kernels that ran); big: the unsplit 256 x 256 tiles"""
    import torch
    import paper_2311_03543_amd as pa
    C0 = np.full((A.shape[0], B.shape[1]), np.nan, np.float32) if C0 is None else C0
    say(f"  fp6x3 tiles {A.shape} {B.shape} alpha={alpha} beta={beta} pad={pad} big={big}")
    with pa.Compar(0) as cx:
        if big:
            cx.set_split_k(1)
        a, b, c = place(A, pad), place(B, pad), place(C0, pad)
        cx.kernel_timing(True)
        cx.gemm_variant(cx.register_builtin("fp6x3"), a, b, c, alpha, beta)
        torch.cuda.synchronize()
        cx.kernel_timing(False)
        return host(c), set(cx.kernel_stats())


@pytest.mark.parametrize("pad", [0, 3])
@pytest.mark.parametrize("M,N,K", DIVIDED + WHOLE + SLICED)
def test_integer_exact(M, N, K, pad):
    A, B = synth.int_matrix(M, K, 31), synth.int_matrix(K, N, 32)
    C, ran = product(A, B, pad=pad)
    assert "gemm_fp6x3_tiles" in ran and ("splitk_reduce" in ran) == ((M, N, K) in SLICED), ran
    assert np.array_equal(C.astype(np.float64), A.astype(np.float64) @ B.astype(np.float64))


@pytest.mark.parametrize("M,N,K", DIVIDED + WHOLE + SLICED)
def test_as_large_tiles(M, N, K):
    A, B = synth.gemm_operands(M, N, K, seed=M + K)
    A *= np.exp2(synth.rng(1).integers(-6, 7, (M, 1))).astype(np.float32)      # scales differ between tiles
    C0 = synth.normal_matrix(M, N, 33)
    C, ran = product(A, B, C0, -0.75, 1.5, pad=1)
    ref, large = product(A, B, C0, -0.75, 1.5, pad=1, big=True)
    assert "gemm_fp6x3_tiles" in ran and "gemm_fp6x3_tn" in large
    if (M, N, K) in WHOLE:
        assert np.array_equal(C.view(np.uint32), ref.view(np.uint32))
        return
    # two FP32 sums of the same MFMA results (three products; |hi| and |lo| <= 1.1 |x|), one
    # rounding per MFMA and scaling; an MFMA's own truncation falls on other running sums: 2^-21
    # of the magnitudes it adds
    nmfma = 3 * (-(-K // 64) + 1)
    mag = np.abs(A).astype(np.float64) @ np.abs(B).astype(np.float64) * 3.7
    bound = 0.75 * (2 * gamma(nmfma + 8) + nmfma * 2.0 ** -21) * mag + 2 * gamma(2) * np.abs(1.5 * C0)
    viol = np.abs(C.astype(np.float64) - ref) - bound
    assert np.all(viol <= 0), float(viol.max())


@pytest.mark.parametrize("M,N,K", [(129, 130, 200), (1601, 1345, 129), (3000, 2500, 1500), (100, 128, 4100)])
def test_non_finite_as_large_tiles(M, N, K):
    A, B = synth.gemm_operands(M, N, K, seed=K)
    A[M // 2, K // 2], A[0, 0], B[K - 1, N // 3] = np.inf, np.nan, -np.inf
    C, ran = product(A, B)
    ref, _ = product(A, B, big=True)
    assert "gemm_fp6x3_tiles" in ran
    assert np.array_equal(np.isnan(C), np.isnan(ref)) and np.isnan(C[0]).all()
