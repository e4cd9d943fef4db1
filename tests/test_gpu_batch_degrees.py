"""GPU: untuned plans of de Casteljau batches of low, middle and high degrees, at
sizes on both sides of the rule for their layout: the results of explicitly
configured layouts bit for bit (the same lerps)."""
import numpy as np
import pytest
import torch

import bz_synth
import paper_2603_15447_amd as bz
from tests._gpu import to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("deg_hi,n", [(7, 123300), (7, 123400), (12, 123300), (12, 123400), (15, 370000), (15, 370200),
                                      (8, 986900), (8, 987000)])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_default_layout(deg_hi, n, dtype):
    b = bz_synth.mixed_batch(n_bezier=n, n_nurbs=n // 16, n_t=16, deg_hi=deg_hi, seed=n, knots_hi=12)
    plan = bz.BatchPlan(torch.from_numpy(b.kind_degree.astype(np.int16)).cuda(), torch.from_numpy(b.cp_offset).cuda(),
                        to_dev(b.ctrl).to(dtype), to_dev(b.w).to(dtype), 3, torch.from_numpy(b.knot_offset).cuda(),
                        to_dev(b.knots), 16, "decasteljau")
    t = to_dev(b.t)
    got = plan(t)
    assert bool(torch.isfinite(got).all())
    for sub_tiles, lanes in ((4, 4), (1, 1)):
        plan.configure(4096, sub_tiles, "static", lanes, 0)
        assert torch.equal(plan(t), got)
    plan.close()
