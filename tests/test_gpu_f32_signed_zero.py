"""FP32 products whose sums are all -0 (every product underflows from below): the chain of FMAs over
k stays -0, so C is -0 for every tile shape and stage depth (16, 32 and 64), with and without a
partial last stage, in single and in grouped launches."""
import numpy as np
import pytest

from gpu_util import host, say

pytestmark = pytest.mark.gpu


def operands(M, N, K):
    import torch
    return [torch.full(s, v, device="cuda") for s, v in (((M, K), -2.0 ** -100), ((K, N), 2.0 ** -100), ((M, N), 1.0))]


# 32 x 32 tiles (stages of 64), 64 x 64 (16), 128 x 128 (32), 128 x 256 (16)
@pytest.mark.parametrize("K", [1, 16, 33, 96])
@pytest.mark.parametrize("M,N", [(33, 31), (960, 1023), (2000, 2048), (4096, 4092)])
def test_single(M, N, K):
    import paper_2311_03543_amd as pa
    say(f"  -0 sums {M} x {N} x {K}")
    A, B, C = operands(M, N, K)
    with pa.Compar(0) as cx:
        cx.gemm_variant(0, A, B, C)
        assert np.all(host(C).view(np.uint32) == 0x80000000)


@pytest.mark.parametrize("config", range(10))
def test_grouped(config):
    import paper_2311_03543_amd as pa
    say(f"  -0 sums, grouped configuration {config}")
    probs = [operands(70, 66, K) for K in (1, 16, 33, 96)]
    with pa.Compar(0) as cx:
        plan = cx.grouped_plan([(A, B, C, 1.0, 0.0) for A, B, C in probs], config=config)
        try:
            plan.launch()
            assert all(np.all(host(C).view(np.uint32) == 0x80000000) for _, _, C in probs)
        finally:
            plan.destroy()
