"""Chain evaluators at query counts around their workgroups' edges: the first
n_q results are the ones of a long call bit for bit, that call's are the
oracle's, and nothing behind a plane's n_q results is written."""
import numpy as np
import pytest
import torch

import bz_synth
import paper_2603_15447_amd as bz
from tests._gpu import TOL_F32, host, to_dev

pytestmark = pytest.mark.gpu

N_SEG = 700
COUNTS = (1, 63, 64, 65, 255, 256, 257, 511, 512, 513, 767, 768, 769, 1023, 1024, 1025)


def _evaluators(dim, seed):
    chain, T = bz_synth.chain_walk(n_seg=N_SEG, dim=dim, n_q=3001, seed=seed)
    cubic, _ = bz_synth.cubic_chain_walk(n_seg=N_SEG, dim=dim, n_q=1, seed=seed)
    grid = bz.encode_piecewise(to_dev(chain))
    tiles, half = bz.tile_piecewise(grid), bz.tile_piecewise16(grid, torch.float16)
    grid3 = bz.encode_piecewise_cubic(to_dev(cubic))
    tiles3 = bz.tile_piecewise_cubic(grid3)
    return chain, cubic, T, {
        "grid": lambda t, o: bz.eval_piecewise(grid, t, out=o),
        "tiles": lambda t, o: bz.eval_piecewise_tiled(tiles, N_SEG, dim, t, out=o),
        "tiles16": lambda t, o: bz.eval_piecewise_tiled16(half, N_SEG, dim, t, out=o),
        "cubic": lambda t, o: bz.eval_piecewise_cubic(grid3, t, out=o),
        "cubic_tiles": lambda t, o: bz.eval_piecewise_cubic_tiled(tiles3, N_SEG, dim, t, out=o),
        "texemu": lambda t, o: bz.eval_piecewise_texemu_tiled(tiles, N_SEG, dim, t, out=o),
    }


@pytest.mark.parametrize("dim", [1, 2, 3, 4])
def test_query_counts(orc, dim):
    chain, cubic, T, evaluators = _evaluators(dim, 31 + dim)
    t = to_dev(T)
    for name, f in evaluators.items():
        full = torch.empty(dim, T.size, device="cuda")
        f(t, full)
        if name in ("grid", "tiles", "cubic", "cubic_tiles"):
            c = cubic if name.startswith("cubic") else chain
            ref = (orc.cubic_chain_eval if name.startswith("cubic") else orc.chain_eval)(c, T)
            c = np.asarray(c, np.float64)
            assert np.abs(host(full) - ref).max() <= TOL_F32 * (c.max(axis=0) - c.min(axis=0)).max(), name
        for n in COUNTS:
            flat = torch.full((dim * n + 1024,), -7.0, device="cuda")
            f(t[:n], flat[:dim * n].view(dim, n))
            assert torch.equal(flat[:dim * n].view(dim, n), full[:, :n]), (name, n)
            assert bool((flat[dim * n:] == -7.0).all()), (name, n)


@pytest.mark.parametrize("n_q", [(1 << 18) - 1, 1 << 18, (1 << 19) + 5, (1 << 21) - 1, 1 << 21])
@pytest.mark.parametrize("n_seg", [N_SEG, 1 << 13, 1 << 15])
def test_queries_per_thread(n_q, n_seg):
    """On both sides of the rule for four queries per thread: the results of
    calls far below it, bit for bit."""
    chain, T = bz_synth.chain_walk(n_seg=n_seg, dim=3, n_q=n_q, seed=n_seg)
    cubic, _ = bz_synth.cubic_chain_walk(n_seg=n_seg, dim=3, n_q=1, seed=n_seg)
    grid, grid3 = bz.encode_piecewise(to_dev(chain)), bz.encode_piecewise_cubic(to_dev(cubic))
    tiles, half, tiles3 = bz.tile_piecewise(grid), bz.tile_piecewise16(grid, torch.float16), bz.tile_piecewise_cubic(grid3)
    t = to_dev(T)
    for f in (lambda x: bz.eval_piecewise(grid, x), lambda x: bz.eval_piecewise_tiled(tiles, n_seg, 3, x),
              lambda x: bz.eval_piecewise_tiled16(half, n_seg, 3, x),
              lambda x: bz.eval_piecewise_cubic_tiled(tiles3, n_seg, 3, x)):
        parts = [f(x) for x in torch.split(t, 100000)]
        assert torch.equal(f(t), torch.cat(parts, dim=1))
