"""GPU: the chain encoder around 2^15 columns, the longest chain that goes in one
launch (its last block adds up all columns before it) and the first that goes in
three, and beyond, where blocks of 512 columns are scanned -- quadratic and cubic,
in every dimension -- against the FP64 oracle's encoding."""
import numpy as np
import pytest

import bz_synth
import paper_2603_15447_amd as bz
from tests._gpu import host, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_seg", [32766, 32767, 32768, 33000, 40000])
@pytest.mark.parametrize("dim", [1, 2, 3, 4])
@pytest.mark.parametrize("cubic", [False, True])
def test_sizes(orc, n_seg, dim, cubic):
    walk, encode, ref = ((bz_synth.cubic_chain_walk, bz.encode_piecewise_cubic, orc.cubic_chain_encode) if cubic else
                         (bz_synth.chain_walk, bz.encode_piecewise, orc.piecewise_encode))
    chain, _ = walk(n_seg=n_seg, dim=dim, n_q=1, seed=n_seg + dim)
    want = ref(chain)
    # one FP32 rounding of an FP64 sum of n_seg terms, on both sides of which the
    # partial sums stay within the largest |texel|
    tol = 2.0 ** -24 * np.abs(want) * (1 + 2.0 ** -20) + 2 * n_seg * 2.0 ** -53 * np.abs(want).max()
    assert (np.abs(host(encode(to_dev(chain))) - want) <= tol).all()
