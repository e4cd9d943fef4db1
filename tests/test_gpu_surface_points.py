"""GPU: scattered points of surfaces, staged for runs of queries that cover
whole objects, parts of them or many -- every pair of degrees, points per
object around the runs' and wavefronts' edges, planes that lie alike and not,
16-bit storage, parameters outside [0, 1] and not finite -- against the FP64
oracle."""
import numpy as np
import pytest
import torch

import paper_2603_15447_amd as bz
from tests._gpu import TOL_F32, bbox_err, extents, host, to_dev

pytestmark = pytest.mark.gpu


def _problem(n, n_per, du, dv, dim, seed, lo=0.0, hi=1.0):
    rng = np.random.default_rng(seed)
    P = rng.uniform(-1, 1, size=(n, dim, (du + 1) * (dv + 1))).astype(np.float32)
    return P, rng.uniform(lo, hi, size=(n, n_per, 2)).astype(np.float32)


def _check(orc, n, n_per, du, dv, dim, seed):
    """The points, into a buffer at an odd place whose neighbours stay as they were."""
    P, uv = _problem(n, n_per, du, dv, dim, seed)
    m = dim * n * n_per
    for shift in (0, 5):
        flat = torch.full((m + 64,), -7.0, device="cuda")
        out = flat[shift:shift + m].view(dim, n * n_per)
        bz.eval_tensor_patch(to_dev(P), du, dv, uvw=to_dev(uv), out=out)
        got = host(out)
        assert bbox_err(got, orc.tensor_points(P, du, dv, 0, uv), extents(P), n_per) <= TOL_F32, shift
        assert bool((flat[:shift] == -7.0).all()) and bool((flat[shift + m:] == -7.0).all()), shift


@pytest.mark.parametrize("du", [1, 2, 3, 4])
@pytest.mark.parametrize("dv", [1, 2, 3, 4])
@pytest.mark.parametrize("n,n_per,dim", [(300, 1, 4), (77, 9, 3), (64, 16, 2), (3, 257, 1)])
def test_degrees(orc, du, dv, n, n_per, dim):
    _check(orc, n, n_per, du, dv, dim, seed=10 * du + dv + n)


@pytest.mark.parametrize("n,n_per", [(1, 1), (1, 255), (1, 256), (1, 257), (2, 224), (5, 225), (40, 31), (40, 32), (40, 33),
                                     (20000, 1), (9000, 2), (4001, 65), (1300, 250), (1100, 512), (601, 1000), (2, 300001)])
def test_points_per_object(orc, n, n_per):
    _check(orc, n, n_per, 3, 3, 3, seed=n + n_per)


@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16])
def test_storage_widens_exactly(dtype):
    P, uv = _problem(137, 13, 3, 2, 3, seed=8)
    h, u = to_dev(P).to(dtype), to_dev(uv)
    assert torch.equal(bz.eval_tensor_patch(h, 3, 2, uvw=u), bz.eval_tensor_patch(h.float(), 3, 2, uvw=u))


@pytest.mark.parametrize("n_per", [40, 64])
def test_outside_and_not_finite(orc, n_per):
    P, uv = _problem(19, n_per, 3, 2, 3, seed=9, lo=-1.0, hi=2.0)
    got = host(bz.eval_tensor_patch(to_dev(P), 3, 2, uvw=to_dev(uv)))
    # outside [0, 1] the basis grows: |1-t| + |t| <= 3 per factor, five factors
    assert np.abs(got - orc.tensor_points(P, 3, 2, 0, uv)).max() <= 40 * 2.0 ** -24 * 3 ** 5
    bad = uv.copy()
    bad[::2, 3, 0], bad[1::2, 7, 1], bad[4, 39, 1] = np.nan, np.inf, -np.inf
    hit = ~np.isfinite(bad).all(axis=2).reshape(-1)
    out = host(bz.eval_tensor_patch(to_dev(P), 3, 2, uvw=to_dev(bad)))
    assert not np.isfinite(out[:, hit]).any()
    np.testing.assert_array_equal(out[:, ~hit], got[:, ~hit])
