"""GPU: untuned plans of de Casteljau batches -- the layout that the plan
chooses, at sizes on both sides of its rule, gives the results of explicitly
configured layouts bit for bit (four queries per lane or one: the same lerps)."""
import numpy as np
import pytest
import torch

import bz_synth
import paper_2603_15447_amd as bz
from tests._gpu import to_dev

pytestmark = pytest.mark.gpu


def _ints(x):
    return torch.from_numpy(x).cuda()


@pytest.mark.parametrize("n,n_t", [(1, 16), (40, 16), (3000, 16), (700, 24), (90, 32), (300, 20), (530000, 16)])
@pytest.mark.parametrize("dtype", [torch.float32, torch.float16])
def test_default_layout(n, n_t, dtype):
    b = bz_synth.mixed_batch(n_bezier=n, n_nurbs=n // 16, n_t=n_t, seed=n + n_t, n_patches=n // 20)
    plan = bz.BatchPlan(_ints(b.kind_degree.astype(np.int16)), _ints(b.cp_offset), to_dev(b.ctrl).to(dtype),
                        to_dev(b.w).to(dtype), 3, _ints(b.knot_offset), to_dev(b.knots), n_t, "decasteljau")
    t, v = to_dev(b.t), (to_dev(b.v) if n // 20 else None)
    got = plan(t, v=v)
    assert bool(torch.isfinite(got).all())
    for sub_tiles, lanes, window in ((4, 4, 0), (2, 1, 1 << 15)):
        plan.configure(2048, sub_tiles, "static", lanes, window)
        assert torch.equal(plan(t, v=v), got), (sub_tiles, lanes, window)
    plan.close()
