"""GPU: scattered points of volumes on the matrix cores -- degrees 2 and 3,
objects of fewer than, exactly and just over 64 points, several wavefronts per object and several steps per wavefront, 16-bit storage,
parameters outside [0, 1] and not finite -- against the FP64 oracle; and
surfaces' points over several wavefronts per object."""
import numpy as np
import pytest
import torch

import paper_2603_15447_amd as bz
from tests._gpu import TOL_F32, bbox_err, extents, host, to_dev

pytestmark = pytest.mark.gpu


def _problem(n, n_per, du, dv, dw, dim, seed, lo=0.0, hi=1.0):
    rng = np.random.default_rng(seed)
    P = rng.uniform(-1, 1, size=(n, dim, (du + 1) * (dv + 1) * (dw + 1))).astype(np.float32)
    return P, rng.uniform(lo, hi, size=(n, n_per, 3 if dw else 2)).astype(np.float32)


@pytest.mark.parametrize("du,dv,dw", [(2, 2, 2), (3, 3, 2), (2, 3, 3), (3, 2, 3), (2, 2, 3), (3, 3, 3), (2, 3, 2)])
@pytest.mark.parametrize("n,n_per,dim", [(1, 1, 3), (5, 63, 2), (3, 64, 3), (7, 65, 4), (2, 257, 1), (3, 1500, 3),
                                         (3000, 200, 3), (1100, 500, 3)])
def test_points(orc, du, dv, dw, n, n_per, dim):
    P, uvw = _problem(n, n_per, du, dv, dw, dim, seed=n + n_per + 10 * du + dw)
    got = host(bz.eval_tensor_patch(to_dev(P), du, dv, dw, uvw=to_dev(uvw)))
    assert bbox_err(got, orc.tensor_points(P, du, dv, dw, uvw), extents(P), n_per) <= TOL_F32


@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16])
def test_storage_widens_exactly(dtype):
    P, uvw = _problem(37, 130, 3, 3, 3, 3, seed=8)
    h, u = to_dev(P).to(dtype), to_dev(uvw)
    assert torch.equal(bz.eval_tensor_patch(h, 3, 3, 3, uvw=u), bz.eval_tensor_patch(h.float(), 3, 3, 3, uvw=u))


def test_outside_and_not_finite(orc):
    P, uvw = _problem(9, 100, 2, 3, 3, 3, seed=9, lo=-1.0, hi=2.0)
    ref = orc.tensor_points(P, 2, 3, 3, uvw)
    # outside [0, 1] the basis grows: sum |B| is at most 3^8 there (|1-t| + |t| <= 3 per factor)
    got = host(bz.eval_tensor_patch(to_dev(P), 2, 3, 3, uvw=to_dev(uvw)))
    assert np.abs(got - ref).max() <= 40 * 2.0 ** -24 * 3 ** 8
    bad = uvw.copy()
    bad[::2, 3, 0], bad[1::2, 7, 2], bad[4, 64, 1] = np.nan, np.inf, -np.inf
    hit = ~np.isfinite(bad).all(axis=2).reshape(-1)
    out = host(bz.eval_tensor_patch(to_dev(P), 2, 3, 3, uvw=to_dev(bad)))
    assert not np.isfinite(out[:, hit]).any()
    np.testing.assert_array_equal(out[:, ~hit], got[:, ~hit])


@pytest.mark.parametrize("n,n_per", [(3, 2000), (200, 600), (5000, 257)])
def test_surface_points(orc, n, n_per):
    P, uv = _problem(n, n_per, 3, 3, 0, 3, seed=n)
    got = host(bz.eval_tensor_patch(to_dev(P), 3, 3, uvw=to_dev(uv)))
    assert bbox_err(got, orc.tensor_points(P, 3, 3, 0, uv), extents(P), n_per) <= TOL_F32
