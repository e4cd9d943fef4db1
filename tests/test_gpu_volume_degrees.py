"""GPU: scattered points of volumes on the matrix cores in the degrees whose rows
or columns of the 16 x 16 x 4 tile are half empty -- a linear axis in u or v, w of
degree 2 under a cubic u -- against the FP64 oracle; and parameters without a
limit, where the basis is infinite with alternating signs."""
import numpy as np
import pytest
import torch

import paper_2603_15447_amd as bz
from tests._gpu import TOL_F32, bbox_err, extents, host, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("du,dv,dw", [(1, 3, 3), (3, 1, 3), (3, 2, 2)])
@pytest.mark.parametrize("n,n_per,dim", [(1, 1, 3), (5, 63, 2), (3, 64, 3), (7, 65, 4), (2, 257, 1), (1100, 300, 3)])
def test_points(orc, du, dv, dw, n, n_per, dim):
    rng = np.random.default_rng(n + n_per)
    P = rng.uniform(-1, 1, (n, dim, (du + 1) * (dv + 1) * (dw + 1))).astype(np.float32)
    uvw = rng.uniform(0, 1, (n, n_per, 3)).astype(np.float32)
    got = host(bz.eval_tensor_patch(to_dev(P), du, dv, dw, uvw=to_dev(uvw)))
    assert bbox_err(got, orc.tensor_points(P, du, dv, dw, uvw), extents(P), n_per) <= TOL_F32
    bad = uvw.copy()
    bad[:, 0, 0], bad[:, -1, 2] = np.nan, np.inf
    hit = ~np.isfinite(bad).all(axis=2).reshape(-1)
    out = host(bz.eval_tensor_patch(to_dev(P), du, dv, dw, uvw=to_dev(bad)))
    assert not np.isfinite(out[:, hit]).any()
    np.testing.assert_array_equal(out[:, ~hit], got[:, ~hit])


@pytest.mark.parametrize("degrees", [(1, 3, 3), (3, 1, 3), (3, 2, 2), (2, 2, 2), (2, 3, 3), (3, 3, 3)])
@pytest.mark.parametrize("axis", [0, 1, 2])
@pytest.mark.parametrize("value", [np.inf, 3e38, -3e38, -np.inf])
def test_infinite_basis(degrees, axis, value):
    """Along the axis the control points' signs are those of the basis at the
    value: every term is +infinity (a linear basis is finite at 3e38)."""
    d = degrees[axis]
    t = np.float64(value)
    sign = np.array([np.sign(t) ** i * np.sign(1 - t) ** (d - i) for i in range(d + 1)])
    shape = [1, 1, 1]
    shape[axis] = d + 1
    P = np.ones([k + 1 for k in degrees]) * sign.reshape(shape)
    P = np.broadcast_to(P.reshape(1, 1, -1), (3, 2, P.size)).astype(np.float32)
    uvw = np.full((3, 70, 3), 0.25, np.float32)
    uvw[:, 5, axis] = value
    out = host(bz.eval_tensor_patch(to_dev(np.ascontiguousarray(P)), *degrees, uvw=to_dev(uvw))).reshape(2, 3, 70)
    if d == 1 and np.isfinite(value):
        assert (out[:, :, 5] > 1e38).all()
    else:
        assert (out[:, :, 5] == np.inf).all()
    assert np.isfinite(np.delete(out, 5, axis=2)).all()
