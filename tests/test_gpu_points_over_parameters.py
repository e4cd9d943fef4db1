"""GPU: curves evaluated over their own parameters -- t the memory of a plane of
out -- give the points of separate buffers, bit for bit, also where the planes'
lines don't begin alike (a number of queries that is no multiple of 16)."""
import pytest
import torch

import paper_2603_15447_amd as bz

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,n_t", [(40009, 100), (30001, 51), (70001, 16), (20011, 64), (3001, 33), (100003, 7)])
@pytest.mark.parametrize("dim,plane", [(3, 0), (3, 2), (2, 1), (1, 0)])
@pytest.mark.parametrize("kind", ["bernstein", "seiler", "rational", "terms"])
def test_points_over_parameters(n, n_t, dim, plane, kind):
    g = torch.Generator(device="cuda").manual_seed(n + dim)
    ctrl = torch.rand((n, dim, 6), generator=g, device="cuda") * 2 - 1
    w = torch.rand((n, 6), generator=g, device="cuda") + 0.5
    t = torch.rand((n, n_t), generator=g, device="cuda")
    call = {"bernstein": lambda t, **o: bz.eval_bezier(ctrl, t, "bernstein", **o),
            "seiler": lambda t, **o: bz.eval_bezier(ctrl, t, "seiler", **o),
            "rational": lambda t, **o: bz.eval_rational(ctrl, w, t, "bernstein", **o),
            "terms": lambda t, **o: bz.eval_seiler(ctrl, t, **o)}[kind]
    ref = call(t)
    out = torch.empty_like(ref)
    out[plane] = t.view(-1)
    call(out[plane].view(n, n_t), out=out)
    assert torch.equal(out, ref)
