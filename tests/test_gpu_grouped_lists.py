"""The per-XCD tile lists of grouped launches: groups with fewer tiles than lists, one problem that
holds most of the work (cut into pieces), K = 0 and alpha = 0 among ordinary problems, more tiles
than workgroups.  Every launch of a plan (its counters are left zero by the launch before) and
every replay of its graph gives the bits of one launch per problem."""
import numpy as np
import pytest

import synth
from gpu_util import dev, host, say

pytestmark = pytest.mark.gpu

GROUPS = {
    "one tile": [(20, 30, 40)],
    "three tiles": [(64, 64, 65), (1, 1, 1), (5, 64, 17)],
    "one large": [(900, 1100, 70), (3, 4, 5), (40, 40, 300)],
    "large and many": [(1500, 700, 260)] + [(33 + i, 65, 31 + 3 * i) for i in range(40)],
    "empty K": [(70, 50, 0), (130, 130, 33), (0, 9, 9), (64, 70, 0)],
}


@pytest.mark.parametrize("config", [0, 4, 7, 10])
@pytest.mark.parametrize("name", list(GROUPS))
def test_lists(name, config):
    import torch
    import paper_2311_03543_amd as pa
    shapes = GROUPS[name]
    if config == 10 and any(k == 0 for _, _, k in shapes):
        pytest.skip("the bf16x3 configuration refuses K = 0")
    g = synth.rng(len(shapes) + config)
    ops = [(dev(g.standard_normal((m, k), dtype=np.float32)), dev(g.standard_normal((k, n), dtype=np.float32)),
            g.standard_normal((m, n), dtype=np.float32)) for m, n, k in shapes]
    say(f"  grouped lists: {name}, configuration {config}")
    with pa.Compar(0) as cx:
        cx.set_split_k(1)
        ref = [dev(c) for _, _, c in ops]
        for (A, B, _), C in zip(ops, ref):
            cx.gemm_variant(pa.grouped_config_variant(config), A, B, C, 1.5, 0.5)
        C = [dev(c) for _, _, c in ops]
        plan = cx.grouped_plan([(A, B, c, 1.5, 0.5) for (A, B, _), c in zip(ops, C)], config=config)
        try:
            assert plan.info()["problems"] == sum(m > 0 and n > 0 for m, n, _ in shapes)
            for launch in (plan.launch, plan.graph_launch, plan.launch, plan.graph_launch, plan.graph_launch):
                for (_, _, c0), c in zip(ops, C):
                    c.copy_(torch.from_numpy(c0))
                launch()
                for c, r in zip(C, ref):
                    assert np.array_equal(host(c).view(np.uint32), host(r).view(np.uint32))
        finally:
            plan.destroy()
