"""GPU: the autotuner keeps a plan's own configuration where that is the fastest,
though its search does not hold it (200,000 curves x 33 in windows of 2^11
objects: 57.5 us, 62.4 with the best that is searched)."""
import numpy as np
import pytest
import torch

import bz_synth
import paper_2603_15447_amd as bz
from tests._gpu import to_dev

pytestmark = pytest.mark.gpu


def _time(f, launches=20, rounds=7):
    """Shortest average time per launch, in microseconds."""
    best = 1e30
    a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    for _ in range(rounds):
        a.record()
        for _ in range(launches):
            f()
        b.record()
        b.synchronize()
        best = min(best, a.elapsed_time(b) * 1e3 / launches)
    return best


def test_keeps_the_plans_own_configuration():
    b = bz_synth.mixed_batch(n_bezier=200000, n_nurbs=0, n_t=33)
    dev = lambda x: torch.from_numpy(x).cuda()
    plan = bz.BatchPlan(dev(b.kind_degree.astype(np.int16)), dev(b.cp_offset), to_dev(b.ctrl), to_dev(b.w), 3,
                        dev(b.knot_offset), to_dev(b.knots), b.n_t)
    t = to_dev(b.t)
    out = plan(t)
    ref = out.clone()
    ratios = []
    for _ in range(3):
        plan.configure(16384, 4, "static", 1, 1 << 11)
        before = _time(lambda: plan(t, out=out))
        plan.autotune(t, out)
        ratios.append(_time(lambda: plan(t, out=out)) / before)
        assert torch.equal(plan(t), ref)
    # the best of the search alone is 8 % slower, timings of one launch differ by 1 %
    assert sorted(ratios)[1] <= 1.04, ratios
    plan.close()
