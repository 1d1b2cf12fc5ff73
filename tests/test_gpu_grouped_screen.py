"""The grouped quantiser's screen against an exact search in the kernel's own
arithmetic: |X| is chosen so that the projection is exact (X's leading
columns are the residuals, U an identity block), and every code has to equal
the lowest index with the smallest fp32 distance fma(dy, dy, dx dx).  The
fp32 fma is formed in float64: dy dy and its sum with the rounded dx dx need
at most 54 bits for the small integers and powers of two used here, so one
rounding to fp32 is left."""
import numpy as np
import pytest

from paper_2606_05484_amd import mapl
from _helpers import dev, torch

pytestmark = pytest.mark.gpu


def exact_codes(Z, C):
    """[T, L, G]: first index of the smallest distance per round and group."""
    T, r = Z.shape
    L, K, _ = C.shape
    R = Z.reshape(T, r // 2, 2).astype(np.float32).copy()
    out = np.zeros((T, L, r // 2), dtype=np.int64)
    with np.errstate(all="ignore"):
        for l in range(L):
            c = C[l].reshape(K, r // 2, 2)
            for g in range(r // 2):
                d = R[:, None, g, :] - c[None, :, g, :]  # fp32
                x2 = d[..., 0] * d[..., 0]
                dd = (d[..., 1].astype(np.float64) ** 2 + x2.astype(np.float64)).astype(np.float32)
                dd = np.where(np.isnan(dd), np.inf, dd)
                j = dd.argmin(axis=1)
                out[:, l, g] = j
                R[:, g, :] = R[:, g, :] - c[j, g, :]
    return out


@pytest.mark.parametrize("T,r,L,K", [(1, 64, 1, 32), (31, 64, 2, 64), (33, 128, 1, 96), (127, 64, 8, 128),
                                     (129, 96, 3, 160), (300, 64, 2, 256), (257, 32, 1, 224), (257, 64, 3, 32)])
@pytest.mark.parametrize("kind", ["ties", "spread", "far"])
def test_codes_are_the_first_nearest(T, r, L, K, kind):
    """ties: small integer coordinates, so most searches have several
    nearest codewords and every distance is exact; spread: codewords of very
    different sizes; far: a codeword beyond fp32's square range, infinite
    and undefined ones, in single groups (those groups' thresholds are not
    finite, and they are searched in full)."""
    print("grouped screen", T, r, L, K, kind, flush=True)
    rng = np.random.default_rng(T + K)
    Z = rng.integers(-8, 9, (T, r)).astype(np.float32)
    C = rng.integers(-6, 7, (L, K, r)).astype(np.float32)
    if kind == "spread":
        C *= np.exp2(rng.integers(-6, 7, (L, K, 1))).astype(np.float32)
    if kind == "far":
        C[:, 5, 0], C[:, 6, 3], C[0, 7, 4], C[0, 8, 7] = 1e30, np.inf, np.nan, -np.inf
    t = torch()
    d = 512
    U = np.eye(d, r, dtype=np.float32)
    X = np.zeros((T, d), dtype=np.float32)
    X[:, :r] = Z
    D = mapl.desc(T=T, d=d, r=r, V=4, k=0, L=L, K=K, group_dim=2, x_dtype="f32")
    payload = t.full((T, L, r // 2), 255, dtype=t.uint8, device="cuda")
    ws = mapl.workspace(mapl.workspace_bytes(D, mapl.CALL_ENCODE))
    mapl.encode(D, dev(X, "f32"), dev(np.zeros(T, np.int32), "i32"), dev(U, "f32"), None, None, dev(C, "f32"),
                payload, ws)
    assert np.array_equal(payload.cpu().numpy(), exact_codes(Z, C))
