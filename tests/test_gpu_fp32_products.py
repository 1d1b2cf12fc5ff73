"""The latency-bound fp32 product (32 x 32 tiles, K split over waves, rows
gathered by token id) at its edges, through the fp32 codec calls: remainders
in every dimension, both anchor spaces, K shorter than one batch, outputs on
either side of the rule that chooses it, and the accumulating weight
gradient.  Gate: 1e-5 relative Frobenius error against float64 (fp32 sums of
a few thousand terms)."""
import numpy as np
import pytest

from paper_2606_05484_amd import synth
from _helpers import chain, check_chain

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("space", ["ambient", "coord"])
@pytest.mark.parametrize("T,d,r,k", [(1, 64, 32, 16), (31, 64, 64, 48), (33, 320, 96, 64), (257, 192, 32, 0),
                                     (1025, 576, 160, 112), (15400, 128, 128, 16), (300, 7808, 160, 32),
                                     (4500, 512, 96, 48), (18001, 128, 128, 16), (26001, 192, 160, 112)])
def test_fp32_chain(T, d, r, k, space):
    """(d = 7808, r = 160): dU takes the large kernel and the anchor term is
    added to it.  The last three: the large kernel with a k-contiguous B and
    gathered rows (lift, dX), the second also with gathered rows alone (the
    coordinate anchor of 18001 x 128) and in the projection."""
    print("fp32", T, d, r, k, space, flush=True)
    x = synth.codec_inputs(None, seed=41, T=T, d=d, r=r, V=200, k=k, L=0, K=0, dtype="f32", alpha=0.8, n_out=4,
                           cb_sigma=None, gscale=1.0, anchor_space=space, rotate=d <= 1024)
    check_chain(x, chain(x))
