"""bf16 and bf16x3 products from the FP32 operands that take more K slices than the 256 x 256 tiles
would (the count that split_k reports), with the workspace reserved for exactly that shape and
variant: the partial sums fit in it and the integer products are exact."""
import numpy as np
import pytest

import synth
from gpu_util import host, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name,M,N,K,reported", [("bf16", 601, 658, 1545, 5), ("bf16x3", 64, 4622, 7069, 13),
                                                 ("bf16x3", 1301, 6311, 3246, 1)])
def test_slices_in_a_reserved_workspace(name, M, N, K, reported):
    import torch
    import paper_2311_03543_amd as pa
    A, B = synth.int_matrix(M, K, 7), synth.int_matrix(K, N, 8)
    say(f"  {name} {M} x {N} x {K} in a reserved workspace")
    with pa.Compar(0) as cx:
        vid = cx.variant_find(name)
        cx.set_variant_mask(1 << vid)                      # the reservation sizes enabled variants only
        cx.reserve(M, N, K)
        assert cx.split_k(vid, M, N, K) == reported
        a, b, c = (torch.from_numpy(x).cuda() for x in (A, B, np.full((M, N), np.nan, np.float32)))
        for _ in range(2):
            cx.kernel_timing(True)
            cx.gemm_variant(vid, a, b, c)
            torch.cuda.synchronize()
            cx.kernel_timing(False)
            assert {f"gemm_{name}_direct", "splitk_reduce"} <= set(cx.kernel_stats(reset=True))
            assert np.array_equal(host(c).astype(np.float64), A.astype(np.float64) @ B.astype(np.float64))
