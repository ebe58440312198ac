"""The bf16 and bf16x3 products taken straight from the FP32 operands: integer products are exact
and random ones within the entrywise rounding bound for each tile (64 and 128 wide, one and more
groups over K, K slices), at tile and K-stage edges, odd leading dimensions and bases that are not
16-byte aligned; non-finite and overflowing values give what the operand images give; overlapping
outputs keep the image form."""
import numpy as np
import pytest

import oracle
import synth
from gpu_util import gamma, host, say

pytestmark = pytest.mark.gpu
NAMES = ["bf16", "bf16x3"]

# the first four rows: one 64-wide tile per CU at most; then several per CU, one 128-wide tile per
# CU, K slices of each, and (one term) several sliced 128-wide tiles per CU
SHAPES = [(1, 1, 1), (64, 63, 31), (65, 128, 33), (129, 127, 257), (191, 65, 1000), (1090, 1100, 97), (1100, 1087, 96),
          (2047, 1999, 609), (130, 260, 4100), (300, 1500, 4097), (300, 4000, 8191)]


def place(x, pad):
    """Device copy of x as the right columns of a buffer `pad` wider (base at 4 * pad bytes)."""
    import torch
    buf = torch.full((x.shape[0], x.shape[1] + pad), float("nan"), device="cuda")[:, pad:]
    buf.copy_(torch.from_numpy(x))
    return buf


def product(name, A, B, C0=None, alpha=1.0, beta=0.0, pad=0, images=False):
    """(C, kernels that ran)"""
    import torch
    import paper_2311_03543_amd as pa
    C0 = np.full((A.shape[0], B.shape[1]), np.nan, np.float32) if C0 is None else C0
    say(f"  direct {name} {A.shape} {B.shape} alpha={alpha} beta={beta} pad={pad} images={images}")
    with pa.Compar(0) as cx:
        if images:
            cx.set_split_k(1)
        a, b, c = place(A, pad), place(B, pad), place(C0, pad)
        cx.kernel_timing(True)
        cx.gemm_variant(cx.variant_find(name), a, b, c, alpha, beta)
        torch.cuda.synchronize()
        cx.kernel_timing(False)
        return host(c), set(cx.kernel_stats())


@pytest.mark.parametrize("pad", [0, 3])
@pytest.mark.parametrize("M,N,K", SHAPES)
@pytest.mark.parametrize("name", NAMES)
def test_integer_exact(name, M, N, K, pad):
    A, B = synth.int_matrix(M, K, 11), synth.int_matrix(K, N, 12)
    C, ran = product(name, A, B, pad=pad)
    assert f"gemm_{name}_direct" in ran, ran
    assert np.array_equal(C.astype(np.float64), A.astype(np.float64) @ B.astype(np.float64))


@pytest.mark.parametrize("M,N,K", SHAPES)
@pytest.mark.parametrize("name", NAMES)
def test_random_alpha_beta_within_bound(name, M, N, K):
    A, B = synth.gemm_operands(M, N, K, seed=M + N + K)
    C0 = synth.normal_matrix(M, N, 13)
    alpha, beta = -0.75, 1.5
    C, ran = product(name, A, B, C0, alpha, beta, pad=1)
    assert f"gemm_{name}_direct" in ran, ran
    rows = np.unique(np.r_[0:min(M, 3), min(M - 1, 63):min(M, 66), M // 2, max(M - 2, 0):M])
    f = lambda x: oracle.bf16_to_float(x).astype(np.float64)
    if name == "bf16":
        pairs, terms = [(f(oracle.bf16_rne(A[rows])), f(oracle.bf16_rne(B)))], 1
    else:
        (ah, al), (bh, bl) = [[f(y) for y in oracle.split_bf16(x)] for x in (np.ascontiguousarray(A[rows]), B)]
        pairs, terms = [(ah, bh), (ah, bl), (al, bh)], 3
    ref = alpha * sum(x @ y for x, y in pairs) + beta * C0[rows].astype(np.float64)
    mag = sum(np.abs(x) @ np.abs(y) for x, y in pairs)
    # the K sum's roundings plus the scaling's, on the products; the last FMA's on beta C
    bound = abs(alpha) * gamma(terms * K + 4) * mag + gamma(2) * np.abs(beta * C0[rows].astype(np.float64))
    viol = np.abs(C[rows].astype(np.float64) - ref) - bound
    assert np.all(viol <= 0), float(viol.max())


@pytest.mark.parametrize("M,N,K", [(70, 66, 70), (1090, 1100, 97), (130, 260, 4100), (1500, 1900, 609)])
@pytest.mark.parametrize("name", NAMES)
def test_special_values_as_images(name, M, N, K):
    g = synth.rng(M + K)
    A, B = synth.gemm_operands(M, N, K, seed=M)
    top = np.float32(3.4e38)                               # hi rounds to infinity, lo to minus infinity
    for X, along in ((A, 0), (B, 1)):                      # a few rows of A and columns of B
        for v in (np.inf, -np.inf, np.nan, top, -top, np.float32(1e-42), np.float32(-1e-39)):
            r, k = g.integers(0, X.shape[along]), g.integers(0, K)
            X[(r, k) if along == 0 else (k, r)] = v
    C, ran = product(name, A, B, pad=2)
    I, by_images = product(name, A, B, pad=2, images=True)
    assert f"gemm_{name}_direct" in ran and f"gemm_{name}_tn" in by_images
    assert np.array_equal(np.isnan(C), np.isnan(I))
    inf = np.isinf(I)
    assert np.array_equal(np.isinf(C), inf) and np.array_equal(C[inf], I[inf])
    ok = np.isfinite(I)
    mag = np.abs(np.where(np.isfinite(A), A, 0).astype(np.float64)) @ np.abs(np.where(np.isfinite(B), B, 0).astype(np.float64))
    # two FP32 sums of the same products (|hi| + |lo| <= (1 + 2^-7) |x|), each within its own bound
    assert np.all(np.abs(C[ok].astype(np.float64) - I[ok]) <= 2 * gamma(3 * K) * 1.02 * mag[ok])


def test_repeatable_bits():
    A, B = synth.gemm_operands(300, 1500, 4097, seed=3)
    c1, c2 = product("bf16x3", A, B)[0], product("bf16x3", A, B)[0]
    assert np.array_equal(c1.view(np.uint32), c2.view(np.uint32))


@pytest.mark.parametrize("name", NAMES)
def test_output_over_an_operand(name):
    import torch
    import paper_2311_03543_amd as pa
    A, B = synth.int_matrix(200, 200, 21), synth.int_matrix(200, 200, 22)
    ref = A.astype(np.float64) @ B.astype(np.float64)
    with pa.Compar(0) as cx:
        vid = cx.variant_find(name)
        for over in "ab":
            say(f"  output over {over} {name}")
            a, b = torch.from_numpy(A).cuda(), torch.from_numpy(B).cuda()
            c = a if over == "a" else b
            cx.gemm_variant(vid, a, b, c)
            assert np.array_equal(host(c).astype(np.float64), ref)
