"""The selector network's gradient and Adam kernels at the row counts where their split can go
wrong: fewer rows than one workgroup's 32 (or one wave's 16), whole and ragged last workgroups,
more workgroup records than one batch of the update's sum (64 records = 2048 rows), the largest.
Tolerances: every value is a chain of at most 32 + 256 FP32 roundings (2^-24 each) of terms that
partly cancel, a few 1e-5 of the gradient's norm; 1e-5 for the loss, a mean of squares."""
import numpy as np
import pytest

import synth
from gpu_util import say
from oracle import mlp as omlp

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 15, 16, 17, 31, 32, 33, 2048, 2049, 4127, 8192])
def test_gradient_and_step(n):
    import paper_2311_03543_amd as pa
    g = synth.rng(n)
    X, Y = (g.standard_normal((n, 4)).astype(np.float32) for _ in range(2))
    p0 = synth.mlp_init(3)
    say(f"  mlp gradient and one step n={n}")
    with pa.Compar(0) as cx:
        cx.mlp_set_params(p0)
        loss, grad = cx.mlp_grad(X, Y)
        rl, rg = omlp.loss_and_grad(p0.astype(np.float64), X.astype(np.float64), Y.astype(np.float64))
        assert abs(loss - rl) <= 1e-5 * abs(rl)
        assert np.linalg.norm(grad - rg) <= 5e-5 * np.linalg.norm(rg)
        again = cx.mlp_grad(X, Y)
        assert again[0] == loss and np.array_equal(again[1].view(np.uint32), grad.view(np.uint32))
        if n > 1:                                   # training standardises its rows (deviation 0 for one)
            trace = cx.mlp_train(X, Y, 2, 1e-3)
            mx, sx = omlp.standardize_stats(X.astype(np.float64))
            my, sy = omlp.standardize_stats(Y.astype(np.float64))
            _, losses = omlp.train(p0.astype(np.float64), (X - mx) / sx, (Y - my) / sy, 2, 1e-3)
            assert np.allclose(trace, losses, rtol=2e-5)
