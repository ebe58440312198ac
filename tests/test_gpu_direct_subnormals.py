"""bf16 and bf16x3 products straight from FP32 operands whose values are subnormal, or so small that
hi or lo is a subnormal bf16: the split keeps what the operand images keep (large values on the
other side bring the products back to ordinary size)."""
import numpy as np
import pytest

import synth
from gpu_util import gamma, say
from test_gpu_direct import product

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("side", "AB")
@pytest.mark.parametrize("low,high", [(-149, -126), (-133, -118), (-126, -110)])
@pytest.mark.parametrize("M,N,K", [(70, 66, 70), (1090, 1100, 97), (1500, 1900, 609)])
@pytest.mark.parametrize("name", ["bf16", "bf16x3"])
def test_as_images(name, M, N, K, low, high, side):
    g = synth.rng(M + K - low)
    tiny = lambda s: np.ldexp(g.standard_normal(s), g.integers(low, high, s)).astype(np.float32)
    big = lambda s: np.ldexp(g.standard_normal(s), 120).astype(np.float32)
    A, B = (tiny((M, K)), big((K, N))) if side == "A" else (big((M, K)), tiny((K, N)))
    say(f"  {name} {M} x {N} x {K}, {side} in 2^{low} .. 2^{high}")
    C, ran = product(name, A, B)
    I, by_images = product(name, A, B, images=True)
    assert f"gemm_{name}_direct" in ran and f"gemm_{name}_tn" in by_images
    assert np.any(I != 0)
    mag = np.abs(A.astype(np.float64)) @ np.abs(B.astype(np.float64))
    # two FP32 sums of the same products; hi of a subnormal may be up to twice it, lo at most |x|
    assert np.all(np.abs(C.astype(np.float64) - I) <= 2 * gamma(3 * K) * 3 * mag)
