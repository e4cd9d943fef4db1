"""GPU: curves staged per workgroup -- chunk edges, chunks over many and over
parts of curves, planes that do and don't lie alike to the 64-byte lines,
outputs off a cache line, the switch to per-query loading below 8 parameters --
against the FP64 oracle, and the count of recomputed rational points."""
import numpy as np
import pytest
import torch

import bz_synth
import paper_2603_15447_amd as bz
from tests._gpu import TOL_F32, bbox_err, extents, host, to_dev

pytestmark = pytest.mark.gpu

SHAPES = [(1, 7), (1, 8), (3, 33), (31, 33), (32, 33), (1000, 9), (1001, 63), (524, 1001), (20001, 27), (5242, 100),
          (8191, 65), (16400, 33), (2, 2047)]


@pytest.mark.parametrize("n,nt", SHAPES)
@pytest.mark.parametrize("degree,dim", [(3, 3), (15, 4), (4, 1)])
def test_integral(orc, n, nt, degree, dim):
    ctrl, t = bz_synth.random_curves(n, degree, dim, nt, seed=n + nt + degree)
    ref = orc.bezier_decasteljau(ctrl, t, per_object=True)
    cd, td = to_dev(ctrl), to_dev(t)
    for m in ("decasteljau", "bernstein", "seiler"):
        assert bbox_err(host(bz.eval_bezier(cd, td, m)), ref, extents(ctrl), nt) <= TOL_F32, m
    sc = bz.bezier_to_seiler(cd)
    assert bbox_err(host(bz.eval_seiler(sc, td)), ref, extents(ctrl), nt) <= TOL_F32
    # shared parameters, and an output that starts off a cache line
    flat = torch.full((dim * n * nt + 5,), float("nan"), device=cd.device)
    got = bz.eval_bezier(cd, td[0].contiguous(), "bernstein", out=flat[5:].view(dim, n * nt))
    ref = orc.bezier_decasteljau(ctrl, t[0])
    assert bbox_err(host(got), ref, extents(ctrl), nt) <= TOL_F32
    assert torch.isnan(flat[:5]).all()


@pytest.mark.parametrize("n,nt", [(3, 64), (31, 33), (1000, 9), (5242, 100), (524, 1001)])
@pytest.mark.parametrize("dtype", [torch.float32, torch.float16, torch.bfloat16])
def test_rational(orc, n, nt, dtype):
    ctrl, w, t = bz_synth.rational_curves(n, 5, 3, nt, seed=n + nt)
    cd, wd, td = to_dev(ctrl).to(dtype), to_dev(w).to(dtype), to_dev(t)
    c, wr = cd.float().cpu().numpy(), wd.float().cpu().numpy()
    ref = orc.rational_eval(c, wr, t, per_object=True)
    for m in ("decasteljau", "bernstein", "seiler"):
        assert bbox_err(host(bz.eval_rational(cd, wd, td, m)), ref, extents(c), nt) <= TOL_F32, m


@pytest.mark.parametrize("n,nt", [(40, 33), (5242, 100), (16400, 33)])
def test_recomputed_points_are_counted_once(n, nt):
    """Weights w, -w, w cancel at t = 1/2 exactly: each such query is
    recomputed, and counted by one workgroup only."""
    ctrl = torch.rand((n, 3, 3), device="cuda")
    w = torch.tensor([1.0, -1.0, 1.0], device="cuda").repeat(n, 1)
    t = torch.full((n, nt), 0.125, device="cuda")
    t[:, ::3] = 0.5  # 1/4 - 1/2 + 1/4 = 0: conditioning number infinite
    cnt = torch.zeros(1, dtype=torch.int32, device="cuda")
    bz.eval_rational(ctrl, w, t, "bernstein", n_fixed=cnt)
    assert int(cnt) == n * len(range(0, nt, 3))


def test_division_ranges(orc):
    """The shared reciprocal and its fallback: weight sums and products from
    the denormals to near overflow, zero and negative zero coordinates."""
    n, nt = 64, 33
    rng = np.random.default_rng(5)
    ctrl = rng.uniform(-1, 1, (n, 3, 2)).astype(np.float32)
    ctrl[:, 2] = 0.0
    ctrl[::2, 1] = -0.0
    ctrl *= np.exp2(rng.integers(-30, 31, (n, 1, 1))).astype(np.float32)
    w = np.exp2(rng.integers(-90, 91, (n, 1)) + rng.uniform(-1, 1, (n, 2))).astype(np.float32)
    t = rng.random((n, nt)).astype(np.float32)
    got = host(bz.eval_rational(to_dev(ctrl), to_dev(w), to_dev(t), "bernstein"))
    assert bbox_err(got, orc.rational_eval(ctrl, w, t, per_object=True), extents(ctrl), nt) <= TOL_F32


@pytest.mark.parametrize("n,nt", [(40, 33), (31, 65), (4039, 65), (15932, 33)])
@pytest.mark.parametrize("rational", [False, True])
def test_planes_that_end_before_the_last_part(orc, n, nt, rational):
    """Planes that don't lie alike and end up to 31 queries before the last
    workgroup's part of them begins: that part is empty, in the plane's
    neighbour nothing is written."""
    if rational:
        ctrl, w, t = bz_synth.rational_curves(n, 3, 3, nt, seed=n)
        ref = orc.rational_eval(ctrl, w, t, per_object=True)
    else:
        ctrl, t = bz_synth.random_curves(n, 3, 3, nt, seed=n)
        ref = orc.bezier_decasteljau(ctrl, t, per_object=True)
    cd, td, m = to_dev(ctrl), to_dev(t), 3 * n * nt
    for shift in (0, 7):
        flat = torch.full((m + 2048,), -7.0, device="cuda")
        out = flat[shift:shift + m].view(3, n * nt)
        if rational:
            bz.eval_rational(cd, to_dev(w), td, "bernstein", out=out)
        else:
            bz.eval_bezier(cd, td, "bernstein", out=out)
        assert bbox_err(host(out), ref, extents(ctrl), nt) <= TOL_F32, shift
        assert bool((flat[:shift] == -7.0).all()) and bool((flat[shift + m:] == -7.0).all()), shift


@pytest.mark.parametrize("nt", [9, 64, 100])
def test_seiler_terms_of_weighted_points_are_rounded_once(nt):
    """Quadratics whose end points a, -3 a cancel at t = 1/4 and whose inner
    product p w = -a + r rounds to -a: the point there is (3/8) r over the weight
    sum, if the product enters the terms unrounded, and else zero.  All steps
    before the weight sum's four roundings and the quotient's are exact but one."""
    rng = np.random.default_rng(nt)
    n = 500
    p, w1 = (rng.uniform(0.5, 2.0, n).astype(np.float32) for _ in range(2))
    a = -(p * w1)
    r = p.astype(np.float64) * w1 + a.astype(np.float64)
    ctrl = np.stack([a, p, -3.0 * a], axis=1)[:, None].repeat(3, axis=1)
    ctrl[:, :, 1] = p[:, None]
    w = np.stack([np.ones(n), w1, np.ones(n)], axis=1).astype(np.float32)
    exact = -3.0 * a.astype(np.float64) == (np.float32(-3.0) * a).astype(np.float64)  # (3 a needs at most 24 bits)
    t = np.full((n, nt), 0.25, np.float32)
    got = host(bz.eval_rational(to_dev(ctrl.astype(np.float32)), to_dev(w), to_dev(t), "seiler")).reshape(3, n, nt)
    ref = 0.375 * r / (1.0 + 0.375 * (w1.astype(np.float64) - 1.0))
    assert exact.sum() > n // 4 and (r[exact] != 0).sum() > n // 8
    assert np.abs(got - ref[:, None])[:, exact].max() <= 8 * 2.0 ** -24 * np.abs(ref).max()
