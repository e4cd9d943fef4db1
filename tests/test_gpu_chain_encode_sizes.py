"""GPU: the chain encoder at sizes on both sides of its blocks and launches -- the
columns of a thread (4) and of a block (512 or 2048), chains of one block and of
several in one launch (up to 2^15 columns), the change of block size (2^18
columns), and more blocks than the scan takes at once -- against the FP64
oracle's encoding."""
import numpy as np
import pytest

import bz_synth
import paper_2603_15447_amd as bz
from tests._gpu import host, to_dev

pytestmark = pytest.mark.gpu


def _close(got, ref, n_seg):
    """One FP32 rounding of an FP64 sum of n_seg terms, on both sides of which
    the partial sums stay within the largest |texel|: half an FP32 ulp, plus
    an FP64 rounding per term."""
    scale = np.abs(ref).max()
    tol = 2.0 ** -24 * np.abs(ref) * (1 + 2.0 ** -20) + 2 * n_seg * 2.0 ** -53 * scale
    assert (np.abs(got - ref) <= tol).all()


@pytest.mark.parametrize("n_seg,dim", [(2, 3), (3, 1), (4, 4), (5, 2), (2046, 3), (2047, 3), (2048, 2), (8190, 3),
                                       (8191, 1), (8191, 4), (8192, 3), (8703, 2), (8704, 4), ((1 << 18) - 1, 3),
                                       (1 << 18, 3), ((1 << 18) + 2049, 1), (4096 * 2048 + 5, 1)])
def test_quadratic_sizes(orc, n_seg, dim):
    chain, _ = bz_synth.chain_walk(n_seg=n_seg, dim=dim, n_q=1, seed=n_seg + dim)
    c = to_dev(chain)
    grid = bz.encode_piecewise(c)
    _close(host(grid), orc.piecewise_encode(chain), n_seg)
    again = bz.encode_piecewise_noalloc(c, grid.clone().fill_(float("nan")))
    np.testing.assert_array_equal(host(again), host(grid))


@pytest.mark.parametrize("n_seg,dim", [(1, 4), (2, 1), (4, 3), (2047, 3), (2048, 4), (8191, 2), (8192, 3),
                                       ((1 << 18) - 1, 2), (1 << 18, 3), ((1 << 18) + 3, 4)])
def test_cubic_sizes(orc, n_seg, dim):
    chain, _ = bz_synth.cubic_chain_walk(n_seg=n_seg, dim=dim, n_q=1, seed=n_seg + dim)
    _close(host(bz.encode_piecewise_cubic(to_dev(chain))), orc.cubic_chain_encode(chain), n_seg)
