"""GPU: chains of few segments evaluated at many queries, on both sides of the
rules for four queries per thread: the results of calls far below them, bit for
bit, for every evaluator and dimension."""
import pytest
import torch

import bz_synth
import paper_2603_15447_amd as bz
from tests._gpu import to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_q", [(1 << 20) - 1, 1 << 20, (1 << 21) - 1, 1 << 21, (1 << 22) + 3])
@pytest.mark.parametrize("n_seg,dim", [(1, 3), (64, 4), (65, 4), (113, 3), (114, 3), (151, 3), (152, 3), (256, 2), (257, 2),
                                       (512, 2), (513, 2), (512, 4), (910, 3), (911, 3), (1023, 2), (1024, 1), (1025, 1), (2048, 1), (2048, 2),
                                       (2049, 2), (4096, 1), (4097, 1), (8192, 1), (8193, 1)])
def test_queries_per_thread(n_q, n_seg, dim):
    chain, T = bz_synth.chain_walk(n_seg=n_seg, dim=dim, n_q=1 << 16, seed=n_seg)
    cubic, _ = bz_synth.cubic_chain_walk(n_seg=n_seg, dim=dim, n_q=1, seed=n_seg)
    grid, grid3 = bz.encode_piecewise(to_dev(chain)), bz.encode_piecewise_cubic(to_dev(cubic))
    tiles, half, tiles3 = bz.tile_piecewise(grid), bz.tile_piecewise16(grid, torch.float16), bz.tile_piecewise_cubic(grid3)
    short = to_dev(T)
    t = short.repeat(n_q // short.numel() + 1)[:n_q].contiguous()
    for f in (lambda x: bz.eval_piecewise(grid, x), lambda x: bz.eval_piecewise_tiled(tiles, n_seg, dim, x),
              lambda x: bz.eval_piecewise_tiled16(half, n_seg, dim, x), lambda x: bz.eval_piecewise_cubic(grid3, x),
              lambda x: bz.eval_piecewise_cubic_tiled(tiles3, n_seg, dim, x), lambda x: bz.eval_piecewise_texemu(grid, x),
              lambda x: bz.eval_piecewise_texemu_tiled(tiles, n_seg, dim, x)):
        once = f(short)
        assert torch.equal(f(t), once.repeat(1, n_q // short.numel() + 1)[:, :n_q])


@pytest.mark.parametrize("n_q", [(6 << 20) - 1, 6 << 20])
@pytest.mark.parametrize("n_seg,dim", [(2048, 1), (2049, 1), (1023, 2), (1024, 2), (1, 3)])
def test_filter_queries_per_thread(n_q, n_seg, dim):
    chain, T = bz_synth.chain_walk(n_seg=n_seg, dim=dim, n_q=1 << 16, seed=n_seg)
    grid = bz.encode_piecewise(to_dev(chain))
    tiles, short = bz.tile_piecewise(grid), to_dev(T)
    t = short.repeat(n_q // short.numel() + 1)[:n_q].contiguous()
    for f in (lambda x: bz.eval_piecewise_texemu(grid, x), lambda x: bz.eval_piecewise_texemu_tiled(tiles, n_seg, dim, x)):
        assert torch.equal(f(t), f(short).repeat(1, n_q // short.numel() + 1)[:, :n_q])
