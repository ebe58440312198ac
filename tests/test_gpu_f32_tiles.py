"""The FP32 variant's tiles: every entry of C is the chain of FP32 FMAs over k in increasing
order, bit for bit, for each tile shape the launch picks, at tile and K-stage edges, for 16-byte
and 4-byte operand copies, with subnormal, infinite and NaN values, and for leading dimensions
whose offsets pass 32 bits.  Tolerance: none (the chain defines every bit; NaN payloads aside)."""
import numpy as np
import pytest

import synth
from gpu_util import host, say

pytestmark = pytest.mark.gpu


def fma32(a, b, c):
    """Correctly rounded FP32 a * b + c: the product is exact in binary64, the sum is rounded to
    odd there (53 bits >= 24 + 2), so the final rounding to FP32 is the only one."""
    with np.errstate(invalid="ignore", over="ignore"):
        p = a.astype(np.float64) * b.astype(np.float64)
        c = np.broadcast_to(c.astype(np.float64), p.shape)
        s = p + c
        bb = s - p
        err = (p - (s - bb)) + (c - bb)                    # exact: s + err = p + c
        even = (s.view(np.int64) & 1) == 0
        fix = np.isfinite(s) & (err != 0) & even
        s = np.where(fix, np.nextafter(s, np.where(err > 0, np.inf, -np.inf)), s)
        return s.astype(np.float32)


def chain(A, B, alpha, beta, C0):
    acc = np.zeros((A.shape[0], B.shape[1]), np.float32)
    for k in range(A.shape[1]):
        acc = fma32(A[:, k:k + 1], B[k:k + 1, :], acc)
    with np.errstate(invalid="ignore", over="ignore"):
        v = np.float32(alpha) * acc
    return fma32(np.full_like(C0, beta), C0, v) if beta else v


def values(shape, kind, g):
    x = g.standard_normal(shape, dtype=np.float32)
    if kind == "wide":                                     # products from subnormal to large
        x = np.ldexp(x, g.integers(-75, 40, shape)).astype(np.float32)
    elif kind == "special":
        pick = g.random(shape)
        x[pick < 0.02] = np.inf
        x[(pick > 0.02) & (pick < 0.04)] = np.nan
        x[(pick > 0.04) & (pick < 0.2)] = -0.0
        x[(pick > 0.2) & (pick < 0.3)] = np.float32(1e-42)
    return x


def check(M, N, K, pad, kind, alpha=1.0, beta=0.0, seed=0, lda=None, ldb=None):
    import torch
    import paper_2311_03543_amd as pa
    g = synth.rng(seed)
    A, B, C0 = values((M, K), kind, g), values((K, N), kind, g), values((M, N), "normal", g)

    def padded(x, ld):
        buf = torch.empty((x.shape[0], ld), device="cuda")[:, ld - x.shape[1]:] if ld < 4096 + 64 else \
            torch.empty((x.shape[0], ld), device="cuda")[:, :x.shape[1]]
        buf.copy_(torch.from_numpy(x))
        return buf

    say(f"  f32 tiles M={M} N={N} K={K} pad={pad} kind={kind} lda={lda} ldb={ldb}")
    with pa.Compar(0) as cx:
        dA, dB, dC = padded(A, lda or K + pad), padded(B, ldb or N + pad), padded(C0, N + pad)
        cx.gemm_variant(0, dA, dB, dC, alpha, beta)
        got = host(dC)
    rows = np.arange(M) if M <= 150 else np.unique(np.r_[0:3, 31:34, 63:66, 127:130, 255:258, M // 2, M - 33:M])
    rows = rows[rows < M]
    ref = chain(A[rows], B, alpha, beta, C0[rows])
    got = got[rows]
    same = (got.view(np.uint32) == ref.view(np.uint32)) | (np.isnan(got) & np.isnan(ref))
    assert same.all(), (int((~same).sum()), np.argwhere(~same)[:4], got[~same][:4], ref[~same][:4])


# one row per tile shape of the launch: 32 x 32, 64 x 64, 128 x 128, 128 x 256; K around the
# stage depths (16, 32, 64) and past the ring depth
@pytest.mark.parametrize("pad", [0, 4, 3])
@pytest.mark.parametrize("M,N,K", [(1, 1, 1), (33, 31, 63), (64, 64, 64), (32, 96, 257), (130, 36, 448),
                                   (1001, 1000, 15), (960, 1023, 113), (2000, 2048, 33), (2047, 1999, 96),
                                   (4096, 4092, 16), (4089, 4096, 67)])
def test_fma_chain(M, N, K, pad):
    check(M, N, K, pad, "normal", seed=M + K + pad)


@pytest.mark.parametrize("kind", ["wide", "special"])
@pytest.mark.parametrize("M,N,K", [(65, 63, 130), (1000, 1001, 70), (2000, 2040, 37)])
def test_fma_chain_values(M, N, K, kind):
    check(M, N, K, 0, kind, alpha=-0.75, beta=0.5, seed=K)


@pytest.mark.parametrize("lda,ldb", [(1 << 25, None), (None, 1 << 24)])
def test_fma_chain_far_rows(lda, ldb):
    check(3 if lda else 40, 37, 70, 0, "normal", seed=5, lda=lda, ldb=ldb)
