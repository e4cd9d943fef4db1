"""GPU: the many-step fit at the edges of its launch rule -- samples per lane
1, 2, 4 and 8, one to four wavefronts per curve, a last wavefront with few or
no full lanes, odd curve counts, and runs longer than one launch's 128 steps:
bit-identical to single steps, which follow the FP64 oracle."""
import numpy as np
import pytest
import torch

import bz_synth
import paper_2603_15447_amd as bz
from tests._gpu import host, to_dev

pytestmark = pytest.mark.gpu

KEYS = ("ctrl", "t", "m_ctrl", "v_ctrl", "m_t", "v_t", "loss")


def _state(y, c0, t0):
    s = {"ctrl": to_dev(c0), "t": to_dev(t0), "y": to_dev(y)}
    for k in ("ctrl", "t"):
        s["m_" + k], s["v_" + k] = torch.zeros_like(s[k]), torch.zeros_like(s[k])
    s["loss"] = torch.zeros(s["ctrl"].shape[0], device=s["t"].device)
    return s


def _args(s):
    return (s["ctrl"], s["t"], s["y"], s["m_ctrl"], s["v_ctrl"], s["m_t"], s["v_t"])


@pytest.mark.parametrize("n,nt,degree,dim,steps", [
    (5, 1, 3, 3, 4), (3, 32, 3, 3, 4), (7, 33, 3, 2, 4), (5, 129, 3, 3, 10), (33, 200, 3, 3, 10), (6, 256, 5, 3, 5),
    (7, 257, 3, 3, 10), (4, 300, 2, 2, 5), (5, 512, 3, 1, 5), (3, 513, 3, 3, 5), (9, 769, 4, 3, 5), (3, 1024, 3, 3, 5),
    (3, 256, 9, 4, 4), (2, 512, 15, 3, 4), (3, 513, 8, 4, 4), (2, 1024, 15, 4, 4), (17, 40, 3, 3, 300), (3, 300, 3, 3, 130)])
def test_run_equals_steps(orc, n, nt, degree, dim, steps):
    gt, tau, eps = bz_synth.fit_problem(n_curves=n, n_samples=nt, dim=dim, degree=degree, seed=n + nt)
    y = (orc.bezier_decasteljau(gt, tau, per_object=True) + eps).astype(np.float32)
    y3 = y.reshape(dim, n, nt)
    f = np.linspace(0.0, 1.0, degree + 1)
    c0 = (y3[:, :, 0].T[:, :, None] * (1 - f) + y3[:, :, -1].T[:, :, None] * f).astype(np.float32)
    t0 = np.tile(np.linspace(0.0, 1.0, nt), (n, 1)).astype(np.float32)
    a, b = _state(y, c0, t0), _state(y, c0, t0)
    for step in range(1, steps + 1):
        bz.fit_adam_step(*_args(a), step, loss_part=a["loss"])
    bz.fit_adam_run(*_args(b), 1, steps, loss_part=b["loss"])
    for k in KEYS:
        assert torch.equal(a[k], b[k]), k
    if steps <= 10:  # and both follow the oracle (the single steps' own tolerances)
        rc, rt = np.array(c0, np.float64, order="C"), np.array(t0, np.float64, order="C")
        losses = orc.fit_steps(y.astype(np.float64), rc, rt, steps)
        assert np.abs(host(b["ctrl"]) - rc).max() < 2e-3 and np.abs(host(b["t"]) - rt).max() < 2e-3
        assert abs(host(b["loss"]).sum() - losses[-1]) <= 1e-2 * losses[-1] + 1e-9
