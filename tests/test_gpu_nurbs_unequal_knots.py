"""GPU: batched NURBS whose knots lie at very unequal distances -- spans far
shorter than the knots around them reach, down to denormal ones, ranges beyond
FP32's largest number, an infinite end -- at parameters on every span, against
the FP64 oracle."""
import numpy as np
import pytest
import torch

import paper_2603_15447_amd as bz
from tests._gpu import TOL_F32, to_dev

pytestmark = pytest.mark.gpu

KNOTS = {
    "tiny span in a wide range": [0, 0, 0, 0, 1e-25, 1e20, 1e20, 1e20, 1e20],
    "tiny span, large interior knot": [0, 0, 0, 0, 1e-27, 2e18, 3e18, 3e18, 3e18, 3e18],
    "denormal span": [0, 0, 0, 0, 1e-42, 1e-3, 1, 1e30, 1e30, 1e30, 1e30],
    "rising by 2^12": [0.0] * 4 + [2.0 ** e for e in range(-140, 120, 12)] + [2.0 ** 120] * 4,
    "falling by 2^12": [-(2.0 ** 120)] * 4 + [-(2.0 ** e) for e in range(108, -141, -12)] + [0.0] * 4,
    "beyond the largest number": [-3e38] * 4 + [-1e38, -1.0, 0.0, 1e-38, 1.0, 2e38] + [3.4e38] * 4,
    "beyond it in one span": [-3e38] * 4 + [3.4e38] * 4,
    "repeated": [0, 0, 0, 0, 1e-30, 1e-30, 1e-10, 1e-10, 1e-10, 1e25, 1e25, 1e30, 1e30, 1e30, 1e30],
    "infinite end": [0, 0, 0, 0, 1, 2, 3, np.inf, np.inf, np.inf, np.inf],
}


@pytest.mark.parametrize("dim,dtype", [(3, torch.float32), (2, torch.float16), (4, torch.bfloat16), (1, torch.float32)])
@pytest.mark.parametrize("name", sorted(KNOTS))
def test_unequal_knots(orc, name, dim, dtype):
    rng = np.random.default_rng(11)
    knots = np.asarray(KNOTS[name], np.float32)
    ncp = len(knots) - 4
    P = torch.from_numpy(rng.uniform(-1, 1, (dim, ncp)).astype(np.float32)).to(dtype)
    w = torch.from_numpy(np.exp2(rng.uniform(-2, 2, ncp)).astype(np.float32)).to(dtype)
    u = []
    for a, b in zip(knots[3:ncp].astype(np.float64), knots[4:ncp + 1].astype(np.float64)):
        if a < b:  # (on a span without an end, parameters of the size of the others)
            c = b if np.isfinite(b) else 2 * a + 1
            f = np.concatenate([[0.0, 0.5, 1.0 - 2.0 ** -24], rng.random(12), np.exp2(-100 * rng.random(4))])
            u.append(np.clip((1 - f) * a + f * c, a, c).astype(np.float32))
    u = np.concatenate(u)
    u = u[u < knots[-1]]
    off = torch.tensor([0, ncp], dtype=torch.int64, device="cuda")
    koff = torch.tensor([0, len(knots)], dtype=torch.int64, device="cuda")
    kd = torch.tensor([2 << 8 | 3], dtype=torch.int16, device="cuda").view(torch.uint16)
    plan = bz.BatchPlan(kd, off, P.reshape(-1).cuda(), w.cuda(), dim, koff, to_dev(knots), len(u))
    got = plan(to_dev(u[None])).cpu().numpy()
    far = np.where(np.isfinite(knots), knots.astype(np.float64), 1e300)  # an end that far off has the limit's values
    P, w = P.double().numpy(), w.double().numpy()
    assert np.isfinite(got).all()
    assert np.abs(got - orc.nurbs_eval(P, w, far, u)).max() <= TOL_F32 * max((P.max(axis=1) - P.min(axis=1)).max(), 1e-3)
    plan.close()
