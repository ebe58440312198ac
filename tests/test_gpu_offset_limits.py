"""Leading dimensions on both sides of the limits of 32-bit byte offsets inside a tile: each FP32
tile's rows of A and of B (16-byte and 4-byte copies below the limit, per-lane addresses from it
on), a grouped FP32 piece, and the bf16 and bf16x3 products from the FP32 operands, which leave
larger ones to the operand images.  Integer products, exact."""
import numpy as np
import pytest

import synth
from gpu_util import host, say

pytestmark = pytest.mark.gpu


def spread(x, ld):
    """Device copy of x with leading dimension ld."""
    import torch
    t = torch.empty(x.shape[0] * ld, device="cuda").view(x.shape[0], ld)[:, :x.shape[1]]
    t.copy_(torch.from_numpy(x))
    return t


def exact(A, B):
    return A.astype(np.float64) @ B.astype(np.float64)


# tile, limit of lda (BM lda = 2^30) and of ldb (BK ldb = 2^30)
@pytest.mark.parametrize("below", [4, 1, 0])
@pytest.mark.parametrize("M,N,lda,ldb", [(64, 16384, 1 << 24, None), (128, 32768, 1 << 23, None),
                                         (128, 65536, 1 << 23, None), (40, 37, None, 1 << 24),
                                         (64, 16384, None, 1 << 26), (128, 32768, None, 1 << 25),
                                         (128, 65536, None, 1 << 26)])
def test_f32_tiles(M, N, lda, ldb, below):
    import torch
    import paper_2311_03543_amd as pa
    K = 70
    A, B = synth.int_matrix(M, K, 1), synth.int_matrix(K, N, 2)
    say(f"  f32 {M} x {N} lda={lda} ldb={ldb} less {below}")
    with pa.Compar(0) as cx:
        C = torch.full((M, N), float("nan"), device="cuda")
        cx.gemm_variant(0, spread(A, lda - below if lda else K), spread(B, ldb - below if ldb else N), C)
        assert np.array_equal(host(C).astype(np.float64), exact(A, B))
    torch.cuda.empty_cache()


@pytest.mark.parametrize("below", [1, 0])
@pytest.mark.parametrize("config,bm", [(0, 64), (4, 128)])
def test_grouped_piece(config, bm, below):
    import torch
    import paper_2311_03543_amd as pa
    lda = (1 << 30) // bm - below
    ops = [(synth.int_matrix(m, k, 3 + m), synth.int_matrix(k, n, 4 + n)) for m, n, k in ((bm, 200, 70), (33, 40, 50))]
    say(f"  grouped configuration {config} lda={lda}")
    with pa.Compar(0) as cx:
        C = [torch.full((a.shape[0], b.shape[1]), float("nan"), device="cuda") for a, b in ops]
        dA = [spread(ops[0][0], lda), spread(ops[1][0], 50)]
        plan = cx.grouped_plan([(a, spread(b, b.shape[1]), c, 1.0, 0.0) for a, (_, b), c in zip(dA, ops, C)], config=config)
        try:
            plan.launch()
            for (a, b), c in zip(ops, C):
                assert np.array_equal(host(c).astype(np.float64), exact(a, b))
        finally:
            plan.destroy()
    torch.cuda.empty_cache()


@pytest.mark.parametrize("M,N,K,lda,ldb", [(200, 16384, 300, 1 << 23, None), (150, 150, 70, None, 1 << 25)])
@pytest.mark.parametrize("below", [1, 0])
@pytest.mark.parametrize("name", ["bf16", "bf16x3"])
def test_direct(name, M, N, K, lda, ldb, below):
    import torch
    import paper_2311_03543_amd as pa
    A, B = synth.int_matrix(M, K, 5), synth.int_matrix(K, N, 6)
    say(f"  {name} {M} x {N} lda={lda} ldb={ldb} less {below}")
    with pa.Compar(0) as cx:
        C = torch.full((M, N), float("nan"), device="cuda")
        cx.kernel_timing(True)
        cx.gemm_variant(cx.variant_find(name), spread(A, lda - below if lda else K), spread(B, ldb - below if ldb else N), C)
        torch.cuda.synchronize()
        cx.kernel_timing(False)
        assert (f"gemm_{name}_direct" if below else f"gemm_{name}_tn") in cx.kernel_stats()
        assert np.array_equal(host(C).astype(np.float64), exact(A, B))
    torch.cuda.empty_cache()
