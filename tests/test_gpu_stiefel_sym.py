"""The symmetric r x r products of the SPEL step over the tile rule: 32 x 32
tiles with K split four and two ways, 64 x 64 tiles, ranks that leave partial
64-row blocks, and more projectors than the eight XCDs divide evenly.  Gates as
in the other SPEL tests (iteration-matched float64 oracle)."""
import numpy as np
import pytest

from oracle import spel
from paper_2606_05484_amd import mapl, synth
from _helpers import rel_fro, torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("P,d,r,check", [(1, 64, 64, [0]), (2, 128, 96, [0, 1]), (13, 192, 192, [0, 6, 12]),
                                         (43, 160, 128, [0, 21, 42]), (9, 512, 512, [0, 8]), (16, 544, 512, [5])])
def test_step(P, d, r, check):
    print("spel", P, d, r, flush=True)
    st = synth.stiefel_inputs(None, seed=70 + r, P=P, d=d, r=r, gscale=1.0, lr=1e-2, beta=0.95, steps=1)
    t = torch()
    U, G, M = (t.from_numpy(np.ascontiguousarray(a)).cuda() for a in (st["U"], st["G"][0] if st["G"].ndim == 4 else st["G"], st["M"]))
    ws = mapl.workspace(mapl.workspace_bytes(None, mapl.CALL_STIEFEL, P, d, r))
    mapl.stiefel_step(P, d, r, U, G, M, st["lr"], st["beta"], 5, 7, ws)
    t.cuda.synchronize()
    sel = np.asarray(check)
    Ur, Mr = spel.stiefel_step_batched(st["U"][sel], st["G"][sel], st["M"][sel], st["lr"], st["beta"], mode="pe")
    Un, Mn = U.cpu().numpy().astype(np.float64)[sel], M.cpu().numpy().astype(np.float64)[sel]
    e_u, e_m, du = rel_fro(Un, Ur), rel_fro(Mn, Mr), rel_fro(Un - st["U"][sel], Ur - st["U"][sel])
    orth = max(np.abs(u.T @ u - np.eye(r)).max() for u in Un)
    print("U", e_u, "M", e_m, "dU", du, "orth", orth)
    assert e_u <= 1e-5 and e_m <= 1e-5 and du <= 2e-4 and orth <= 1e-5
