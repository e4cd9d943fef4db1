"""GPU: grids of many patches give the points of the same patches in calls of a
few, bit for bit -- patches of one row or column, sizes that divide a workgroup
and that don't, of few and of many points, each storage type -- and those are the
FP64 oracle's."""
import numpy as np
import pytest
import torch

import paper_2603_15447_amd as bz
from tests._gpu import TOL_F32, bbox_err, extents, host

pytestmark = pytest.mark.gpu

SIZES = [(1, 1), (1, 40), (1, 70), (2, 130), (3, 90), (40, 1), (5, 8), (16, 16), (17, 17), (24, 32), (40, 32), (32, 32), (33, 33),
         (9, 256), (64, 64), (70, 31), (300, 2), (2, 300), (260, 260)]


@pytest.mark.parametrize("nu,nv", SIZES)
@pytest.mark.parametrize("du,dv,dim,dtype", [(3, 3, 3, torch.float32), (1, 4, 4, torch.float16), (4, 2, 1, torch.bfloat16),
                                             (2, 2, 2, torch.float32)])
def test_many_and_few(orc, nu, nv, du, dv, dim, dtype):
    n = max(300, min(5000, (3 << 20) // (nu * nv)))
    g = torch.Generator(device="cuda").manual_seed(nu + nv + du)
    P = (torch.rand((n, dim, (du + 1) * (dv + 1)), generator=g, device="cuda") * 2 - 1).to(dtype)
    for f in (lambda p: bz.eval_tensor_patch(p, du, dv, nu=nu, nv=nv),
              lambda p: bz.eval_tensor_seiler(p.float(), du, dv, nu=nu, nv=nv)):
        whole = f(P).view(dim, n, nu * nv)
        for a in [*range(0, n, max(1, n // 7)), n - 3]:
            assert torch.equal(whole[:, a:a + 3], f(P[a:a + 3]).view(dim, -1, nu * nv))
    u, v = (np.linspace(0.0, 1.0, k) if k > 1 else np.zeros(1) for k in (nu, nv))
    uv = np.stack(np.meshgrid(u, v, indexing="ij"), axis=-1).reshape(1, nu * nv, 2)
    few = P[:2].float().cpu().numpy()
    got = host(bz.eval_tensor_patch(P[:2], du, dv, nu=nu, nv=nv))
    ref = orc.tensor_points(few, du, dv, 0, np.repeat(uv, 2, axis=0).astype(np.float32))
    # (the parameters a / (nu - 1) are rounded once on either side)
    assert bbox_err(got, ref, extents(few), nu * nv) <= TOL_F32


# calls on either side of the output sizes up to which a workgroup takes a patch
@pytest.mark.parametrize("nu,nv,dim,n", [(32, 32, 3, 5461), (32, 32, 3, 5462), (32, 32, 1, 20000), (64, 64, 2, 1023), (64, 64, 2, 1024),
                                         (40, 32, 2, 6553), (40, 32, 2, 6554), (12, 256, 2, 1500), (16, 256, 2, 1500),
                                         (4, 128, 3, 1500), (3, 128, 1, 1500), (33, 33, 3, 95), (33, 33, 3, 96)])
@pytest.mark.parametrize("du,dv,dtype", [(3, 3, torch.float32), (4, 4, torch.float16), (2, 1, torch.bfloat16)])
def test_large_and_few(nu, nv, dim, n, du, dv, dtype):
    g = torch.Generator(device="cuda").manual_seed(n + du)
    P = (torch.rand((n, dim, (du + 1) * (dv + 1)), generator=g, device="cuda") * 2 - 1).to(dtype)
    whole = bz.eval_tensor_patch(P, du, dv, nu=nu, nv=nv).view(dim, n, nu * nv)
    for a in [*range(0, n, max(1, n // 7)), n - 3]:
        assert torch.equal(whole[:, a:a + 3], bz.eval_tensor_patch(P[a:a + 3], du, dv, nu=nu, nv=nv).view(dim, -1, nu * nv))
