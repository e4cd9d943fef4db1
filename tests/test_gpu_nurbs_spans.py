"""GPU: knot span lookup and evaluation of batched NURBS where they can go
wrong -- one span, repeated knots, many knots in one bucket of the span table,
parameters on knots, at and beyond the ends, NaN, knots of extreme size and
distance, more control points than the table numbers -- against the FP64
oracle, in every storage type."""
import numpy as np
import pytest
import torch

import paper_2603_15447_amd as bz
from tests._gpu import TOL_F32, to_dev

pytestmark = pytest.mark.gpu


def _knots(inner, scale=1.0, shift=0.0):
    inner = np.sort(np.asarray(inner, np.float64))
    return ((np.concatenate([np.zeros(4), inner, np.ones(4)]) + shift) * scale).astype(np.float32)


def _vectors():
    rng = np.random.default_rng(3)
    v = {"one span": _knots([]), "uniform": _knots(np.arange(1, 40) / 40), "random": _knots(rng.random(56)),
         "double": _knots(np.repeat(rng.random(9), 2)), "triple": _knots(np.repeat(rng.random(7), 3)),
         "quadruple": _knots(np.repeat([0.25, 0.5], 4)),
         "crowded": _knots(0.5 + 1e-4 * rng.random(40)), "crowded at the start": _knots(1e-6 * rng.random(30)),
         "geometric": _knots(2.0 ** -np.arange(1, 60)), "large": _knots(rng.random(20), 1e30, 0.5),
         "small": _knots(rng.random(20), 1e-35), "shifted": _knots(rng.random(30), 1.0, -7.0)}
    return v


def _evaluate(knots, dim, n_t, dtype, seed):
    rng = np.random.default_rng(seed)
    ncp = len(knots) - 4
    P = torch.from_numpy(rng.uniform(-1, 1, (dim, ncp)).astype(np.float32)).to(dtype)
    w = torch.from_numpy(np.exp2(rng.uniform(-2, 2, ncp)).astype(np.float32)).to(dtype)
    lo, hi = float(knots[3]), float(knots[ncp])
    u = (lo + (hi - lo) * rng.random(n_t)).astype(np.float32)
    special = np.concatenate([[lo, hi, lo - abs(hi - lo), hi + abs(hi - lo)], rng.choice(knots, 8)]).astype(np.float32)
    m = min(len(special), n_t)
    u[:m] = special[:m]
    off = torch.tensor([0, ncp], dtype=torch.int64, device="cuda")
    koff = torch.tensor([0, len(knots)], dtype=torch.int64, device="cuda")
    kd = torch.tensor([2 << 8 | 3], dtype=torch.int16, device="cuda").view(torch.uint16)
    plan = bz.BatchPlan(kd, off, P.reshape(-1).cuda(), w.cuda(), dim, koff, to_dev(knots), n_t)
    got = plan(to_dev(u[None])).cpu().numpy()
    return P.float().numpy(), w.float().numpy(), u, got, plan


@pytest.mark.parametrize("name", sorted(_vectors()))
@pytest.mark.parametrize("dim,n_t,dtype", [(3, 1000, torch.float32), (2, 37, torch.float16), (4, 64, torch.bfloat16),
                                           (1, 300, torch.float32)])
def test_spans(orc, name, dim, n_t, dtype):
    knots = _vectors()[name]
    P, w, u, got, plan = _evaluate(knots, dim, n_t, dtype, seed=n_t + dim)
    uc = np.clip(u, knots[3], knots[-4])
    ref = orc.nurbs_eval(P, w, knots, uc)
    ext = max((P.max(axis=1) - P.min(axis=1)).max(), 1e-3)
    if name == "quadruple":  # the curve may jump at a knot of multiplicity 4: either side's point there
        on = np.isin(uc, [0.25, 0.5])
        got, ref = got[:, ~on], ref[:, ~on]
    assert np.abs(got - ref).max() <= TOL_F32 * ext
    assert plan.info()["n_segments"] == np.count_nonzero(np.diff(knots))
    for v in (np.nan,):
        bad = u.copy()
        bad[-1] = v
        out = plan(to_dev(bad[None])).cpu().numpy()
        assert np.isnan(out[:, -1]).all()
        np.testing.assert_array_equal(out[:, :-1], plan(to_dev(u[None])).cpu().numpy()[:, :-1])


def test_more_points_than_the_table_numbers(orc):
    rng = np.random.default_rng(4)
    knots = _knots(np.arange(1, 70000) / 70000)
    P, w, u, got, plan = _evaluate(knots, 3, 4096, torch.float32, seed=5)
    pick = np.arange(4, 4096, 61)
    uc = np.clip(u, 0, 1)
    for a in pick:  # each point from the dozen control points around its span
        i = int(np.clip(np.searchsorted(knots, uc[a], side="right") - 1, 3, len(knots) - 5))
        b = max(0, min(i - 6, len(knots) - 4 - 13))
        e = b + 13
        if i < 4 or i > len(knots) - 10:
            continue
        local = np.concatenate([np.full(4, knots[b + 3]), knots[b + 4:e], np.full(4, knots[e])])
        # the curve on span i depends on knots i-2..i+3 and points i-3..i only
        Q, ww = P[:, b:e], w[b:e]
        ref = orc.nurbs_eval(Q, ww, local, uc[a:a + 1])[:, 0]
        assert np.abs(got[:, a] - ref).max() <= TOL_F32 * 2
    assert plan.info()["n_segments"] == 70000
