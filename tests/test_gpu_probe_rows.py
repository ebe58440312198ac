"""The residual probe at the shapes where its kernels branch: one and four rows per wave (from 8192
rows on, with a ragged last group), 16-byte and 4-byte row reads, tails of both, more rows than
one pass of the grid, beta and alpha zero; each against numpy in FP64, and repeated bit for bit.
Tolerance: both sides sum the same FP64 terms in different orders, n 2^-53 of their magnitudes'
sum, and w - z loses at most that against ||z||: 1e-10 absolute on an estimate of order one."""
import numpy as np
import pytest

import synth
from gpu_util import dev, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("alpha,beta", [(1.0, 0.0), (-0.5, 2.0), (0.0, 1.0)])
@pytest.mark.parametrize("M,N,K,pad", [(1, 1, 1, 0), (5, 63, 66, 0), (64, 260, 255, 1), (70, 1028, 516, 4),
                                       (8193, 33, 40, 0), (8200, 36, 8195, 4), (9001, 64, 64, 3)])
def test_probe_matches_oracle(M, N, K, pad, alpha, beta):
    import paper_2311_03543_amd as pa
    g = synth.rng(M + N + K)
    A, B, C, C0 = (g.standard_normal(s, dtype=np.float32) for s in ((M, K + pad), (K, N + pad), (M, N + pad), (M, N + pad)))
    x = np.where(g.random(N) < 0.5, -1.0, 1.0)
    say(f"  probe M={M} N={N} K={K} pad={pad} alpha={alpha} beta={beta}")
    with pa.Compar(0) as cx:
        args = [dev(t)[:, pad:] for t in (A, B, C)]
        d0 = dev(C0)[:, pad:] if beta else None
        est = [cx.freivalds(*args, x, alpha=alpha, beta=beta, C0=d0) for _ in range(2)]
    assert est[0] == est[1]
    A, B, C, C0 = (t[:, pad:].astype(np.float64) for t in (A, B, C, C0))
    z = alpha * (A @ (B @ x)) + beta * (C0 @ x)
    ref = np.linalg.norm(C @ x - z) / np.linalg.norm(z)
    assert abs(est[0] - ref) <= 1e-10 * max(1.0, ref)
