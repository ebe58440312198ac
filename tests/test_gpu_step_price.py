"""The price of a K block of the 256 x 256 tiles, which sets the split-K counts, comes from the
times of shapes that run these tiles: a shape whose calls take another form (the FP32 operands
directly, or smaller tiles) does not move it, however fast it was."""
import pytest

from gpu_util import say

pytestmark = pytest.mark.gpu

COUNTED = [(m, m, k) for m in (256, 512, 768, 1024, 1536, 2048) for k in (2048, 4096, 8192, 16384)]


@pytest.mark.parametrize("name", ["bf16", "bf16x3", "fp8r", "fp6x3"])
def test_rows_of_other_forms_do_not_move_the_price(name):
    import torch
    import paper_2311_03543_amd as pa
    M, N, K = 300, 33000, 4100                             # 258 tiles of 256 x 256, at least 64 K blocks
    with pa.Compar(0) as cx:
        vid = cx.register_builtin(name) if name == "fp6x3" else cx.variant_find(name)
        A, B, C = (torch.ones(s, device="cuda") for s in ((M, K), (K, N), (M, N)))
        say(f"  {name} {M} x {N} x {K}: form and price")
        cx.kernel_timing(True)
        cx.gemm_variant(vid, A, B, C)
        torch.cuda.synchronize()
        cx.kernel_timing(False)
        assert f"gemm_{name}_tn" not in cx.kernel_stats()
        before = [cx.split_k(vid, *s) for s in COUNTED]
        for ms in (0.4, 100.0):                            # far below and above the constant's time
            cx.history_clear()
            cx.history_add(M, N, K, vid, 1, ms)
            assert [cx.split_k(vid, *s) for s in COUNTED] == before
        cx.history_clear()
        cx.history_add(8192, 8192, 8192, vid, 1, 10.0)     # runs the 256 x 256 tiles
        assert [cx.split_k(vid, *s) for s in COUNTED] != before
