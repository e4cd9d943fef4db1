"""GPU: uniform patch grids at the edges of the tile rule -- whole patches in
groups (the last one partly filled), one patch per workgroup, patches cut into
rows, and rows cut into columns (more than 256 of either) -- against the FP64
oracle."""
import pytest

import bz_synth
import paper_2603_15447_amd as bz
import torch
from tests._gpu import TOL_F32, bbox_err, extents, host, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_obj,nu,nv,du,dv,dim", [
    (5003, 2, 2, 3, 3, 3), (4099, 1, 7, 2, 4, 4), (2051, 32, 32, 3, 3, 3), (2050, 33, 31, 4, 3, 2), (1000, 45, 45, 3, 3, 3),
    (997, 46, 46, 3, 2, 3), (3, 256, 8, 3, 3, 3), (2, 257, 3, 1, 1, 4), (2, 3, 257, 4, 4, 4), (1, 600, 1, 3, 3, 3),
    (1, 1, 600, 2, 2, 1), (1, 301, 517, 3, 3, 3)])
def test_tile_edges(orc, n_obj, nu, nv, du, dv, dim):
    P = bz_synth.patches(n_obj=n_obj, du=du, dv=dv, dim=dim, seed=n_obj + nu)
    ref = orc.tensor_grid(P, du, dv, nu, nv)
    got = bz.eval_tensor_patch(to_dev(P), du, dv, nu=nu, nv=nv)
    assert bbox_err(host(got), ref, extents(P), nu * nv) <= TOL_F32
    sc = bz.tensor_to_seiler(to_dev(P), du, dv)
    assert bbox_err(host(bz.eval_tensor_seiler(sc, du, dv, nu=nu, nv=nv)), ref, extents(P), nu * nv) <= TOL_F32
    h = to_dev(P).half()
    same = bz.eval_tensor_patch(h.float(), du, dv, nu=nu, nv=nv)
    assert torch.equal(bz.eval_tensor_patch(h, du, dv, nu=nu, nv=nv), same)  # widening is exact
