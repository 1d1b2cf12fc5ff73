"""The bf16 token products over the kernel rule and at the edges of their
tiles: 64- and 128-token tiles of the deep-ring kernel, the 128-token kernel
and the short-K kernel, with gathered widths that end inside a 64-column
stage and token counts around the tiles."""
import pytest

from paper_2606_05484_amd import synth
from _helpers import chain, check_chain, stress_codebooks

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,d,r,k,L,K", [
    (1, 64, 64, 16, 0, 0), (63, 128, 64, 48, 0, 0), (65, 320, 192, 80, 0, 0), (129, 576, 128, 0, 0, 0),  # 64-token tiles
    (9001, 256, 256, 16, 0, 0), (12200, 192, 64, 112, 0, 0),   # more than 512 of them: 128-token tiles
    (25000, 320, 128, 48, 0, 0),                               # the 128-token kernel
    (16421, 1024, 64, 48, 2, 64), (17000, 1024, 128, 96, 1, 96), (33000, 512, 256, 112, 2, 32),  # short K, codes gathered
])
def test_chain(T, d, r, k, L, K):
    print("token products", T, d, r, k, L, K, flush=True)
    x = synth.codec_inputs(None, seed=51, T=T, d=d, r=r, V=300, k=k, L=L, K=K, dtype="bf16", alpha=0.8, n_out=4,
                           cb_sigma=None, gscale=1.0)
    C = stress_codebooks(x, 9) if L else None
    check_chain(x, chain(x, C=C), C=C)
