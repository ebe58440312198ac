"""Products with more than 2^29 rows or columns, where the smaller tiles would need launches of 2^32
threads or more: a tile that can be launched is taken.  Integer values, so every bit is known."""
import pytest

from gpu_util import say

pytestmark = pytest.mark.gpu
SIDE = 2 ** 29 + 5


@pytest.mark.parametrize("name,M,N,need_gib", [("f32_simt", SIDE, 1, 8), ("f32_simt", 1, SIDE, 8),
                                               ("bf16x3", SIDE, 1, 180)])
def test_huge_side(name, M, N, need_gib):
    import torch
    import paper_2311_03543_amd as pa
    torch.cuda.empty_cache()
    if torch.cuda.mem_get_info()[0] < need_gib << 30:     # bf16x3: the workspace is that of the images
        pytest.skip(f"needs {need_gib} GiB of free device memory")
    say(f"  huge side {name} {M} x {N} x 1")
    long = torch.arange(SIDE, device="cuda", dtype=torch.int32).remainder_(251).sub_(125).float()
    A, B = (long.view(M, 1), torch.full((1, 1), 3.0, device="cuda")) if N == 1 else \
        (torch.full((1, 1), 3.0, device="cuda"), long.view(1, N))
    C = torch.full((M, N), float("nan"), device="cuda")
    with pa.Compar(0) as cx:
        cx.gemm_variant(cx.variant_find(name), A, B, C)
        torch.cuda.synchronize()
        assert torch.equal(C.view(-1), long.mul_(3.0))
    torch.cuda.empty_cache()
