"""GPU: calls large enough to be staged give the points of the same curves in
calls too small for it, bit for bit -- every form, integral and rational, signed
weights, each storage type, planes that lie alike and that don't, shared and own
parameters, curves of 64 queries and of under 12."""
import pytest
import torch

import paper_2603_15447_amd as bz

pytestmark = pytest.mark.gpu


# (curves, queries each, degree, dim): from each form's line on, and just below
SIZES = [(21011, 50, 9, 3), (20971, 50, 9, 3), (90001, 47, 3, 4), (4099, 64, 12, 2), (2048, 64, 12, 3), (31337, 101, 14, 2),
         (200003, 22, 11, 3), (50021, 11, 13, 3), (400009, 11, 7, 2), (40961, 130, 2, 1), (70001, 130, 5, 2)]


@pytest.mark.parametrize("n,n_t,degree,dim", SIZES)
@pytest.mark.parametrize("form", ["decasteljau", "bernstein", "seiler", "terms"])
@pytest.mark.parametrize("weights", ["none", "positive", "signed"])
def test_large_and_small_calls(n, n_t, degree, dim, form, weights):
    if form == "terms" and weights != "none":
        pytest.skip("terms have no weights")
    g = torch.Generator(device="cuda").manual_seed(n + degree)
    dtype = [torch.float32, torch.float16, torch.bfloat16][(n + len(form) + len(weights)) % 3]
    shared = (n + dim) % 2 == 0
    ctrl = torch.rand((n, dim, degree + 1), generator=g, device="cuda") * 2 - 1
    ctrl = ctrl if form == "terms" else ctrl.to(dtype)
    w = torch.rand((n, degree + 1), generator=g, device="cuda") + 0.25
    if weights == "signed":
        w[::3, 1] *= -1.5
    w = w.to(dtype)
    t = torch.rand(n_t if shared else (n, n_t), generator=g, device="cuda")
    fixed = torch.zeros(2, dtype=torch.int32, device="cuda")

    def call(a, b, count):
        tt = t if shared else t[a:b]
        if form == "terms":
            return bz.eval_seiler(ctrl[a:b], tt)
        if weights == "none":
            return bz.eval_bezier(ctrl[a:b], tt, form)
        return bz.eval_rational(ctrl[a:b], w[a:b], tt, form, n_fixed=count)

    whole = call(0, n, fixed[:1])
    piece = max(1, (1 << 15) // n_t)  # pieces of 2^15 queries: one thread per query
    for a in [*range(0, n, 16 * piece), max(0, n - piece)]:  # every 16th, and the last
        b = min(n, a + piece)
        assert torch.equal(whole[:, a * n_t:b * n_t], call(a, b, fixed[1:]))
    if weights == "signed":
        assert int(fixed[0]) > 0
