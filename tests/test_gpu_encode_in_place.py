"""GPU: a quadratic chain encoded in place -- the grid over the chain it comes
from, one row longer -- with and without an allocation, in one block and in
many, in a captured graph: the values of the encoding into another buffer."""
import numpy as np
import pytest
import torch

import bz_synth
import paper_2603_15447_amd as bz
from tests._gpu import to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_seg,dim", [(1, 3), (2, 1), (2047, 3), (2048, 3), (5000, 4), (32767, 2), (32768, 3), (40001, 1),
                                       (1 << 18, 3), ((1 << 20) + 5, 3), (3 << 20, 4)])
@pytest.mark.parametrize("noalloc", [False, True])
def test_in_place(n_seg, dim, noalloc):
    chain = to_dev(bz_synth.chain_walk(n_seg=n_seg, dim=dim, n_q=1, seed=n_seg + dim)[0])
    ref = bz.encode_piecewise(chain)
    buf = torch.full((2 * n_seg + 2 + 64, dim), -7.0, device="cuda")
    buf[:2 * n_seg + 1] = chain
    grid = buf[:2 * n_seg + 2].view(n_seg + 1, 2, dim)
    (bz.encode_piecewise_noalloc if noalloc else bz.encode_piecewise)(buf[:2 * n_seg + 1], out=grid)
    # (shorter chains are scanned in other blocks: last bits of an FP64 sum, rounded once to FP32)
    tol = 0.0 if n_seg + 1 > 1 << 18 else 2.0 ** -23 * float(ref.abs().max())
    assert float((grid - ref).abs().max()) <= tol
    assert bool((buf[2 * n_seg + 2:] == -7.0).all())


def test_in_place_captured():
    n_seg, dim = 70001, 3
    chain = to_dev(bz_synth.chain_walk(n_seg=n_seg, dim=dim, n_q=1, seed=4)[0])
    ref = bz.encode_piecewise(chain)
    buf = torch.zeros((2 * n_seg + 2, dim), device="cuda")
    grid = buf.view(n_seg + 1, 2, dim)
    stream = torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(stream):
        bz.encode_piecewise_noalloc(buf[:-1], grid)
        with torch.cuda.graph(graph, stream=stream):
            bz.encode_piecewise_noalloc(buf[:-1], grid)
    torch.cuda.synchronize()
    for scale in (1.0, 0.5, 2.0):
        buf[:-1] = chain * scale
        graph.replay()
        torch.cuda.synchronize()
        np.testing.assert_allclose(grid.cpu().numpy(), (ref * scale).cpu().numpy(), rtol=0,
                                   atol=2.0 ** -23 * scale * float(ref.abs().max()))
