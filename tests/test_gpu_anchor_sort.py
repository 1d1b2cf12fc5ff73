"""The binned sort of the anchor-table gradient at its edges: token
counts around each instance and beyond the largest (the multi-launch sort),
one id for every token or for most, ids at both ends of the table, tables of one bin
and beyond the most, and companions with padded rows.  dY rows are small
integers and B is a scaled identity block, so every sum is exact and the
comparison is equality."""
import numpy as np
import pytest

from paper_2606_05484_amd import mapl
from _helpers import dev, torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,V,k,ids", [
    (1, 300, 16, "zipf"), (63, 300, 48, "rand"), (2048, 5, 64, "rand"), (2049, 32000, 64, "zipf"), (8192, 256, 80, "one"),
    (8193, 65534, 64, "ends"), (16385, 40000, 128, "rand"), (32767, 65534, 16, "zipf"), (32768, 1000, 144, "one"),
    (32769, 1000, 64, "zipf"), (3000, 131072, 32, "ends"), (5000, 131073, 64, "rand"), (10240, 256, 16, "rand"),
    (10241, 256, 48, "zipf"), (30001, 40000, 32, "most")])
@pytest.mark.parametrize("accumulate", [0, 1])
def test_receiver_table_exact(T, V, k, ids, accumulate):
    print("anchor sort", T, V, k, ids, accumulate, flush=True)
    rng = np.random.default_rng(T + V)
    d = 192
    if ids == "zipf":
        p = np.arange(1, V + 1) ** -1.1
        tid = rng.choice(V, T, p=p / p.sum())
    elif ids == "one":
        tid = np.full(T, V - 1)
    elif ids == "most":
        tid = np.where(rng.uniform(size=T) < 0.9, 5, rng.integers(0, V, T))
    elif ids == "ends":
        tid = rng.choice([0, 1, V - 2, V - 1], T)
    else:
        tid = rng.integers(0, V, T)
    tid = tid.astype(np.int32)
    dY = rng.integers(-3, 4, (T, d)).astype(np.float32)
    B = np.zeros((k, d), dtype=np.float32)
    B[np.arange(k), np.arange(k)] = 2.0
    t = torch()
    D = mapl.desc(T=T, d=d, r=64, V=V, k=k)
    gY, gB = (t.from_numpy(a).cuda().to(t.bfloat16) for a in (dY, B))
    dA = t.full((V, k), 1.0 if accumulate else float("nan"), device="cuda")
    ws = mapl.workspace(mapl.anchor_bwd_workspace_bytes(D, mapl.RECEIVER))
    mapl.anchor_bwd(D, mapl.RECEIVER, gY, dev(tid, "i32"), None, gB, dA, accumulate, ws)
    ref = np.full((V, k), float(accumulate))
    np.add.at(ref, tid, 2.0 * dY[:, :k].astype(np.float64))
    assert np.array_equal(dA.cpu().numpy().astype(np.float64), ref)


@pytest.mark.parametrize("T,k,r,d", [(50, 16, 64, 128), (2500, 80, 192, 1088), (9000, 64, 256, 512)])
def test_sender_projected_companion(T, k, r, d):
    """W = bf16(B U~): unit-vector rows of U pick columns of B, so W is exact."""
    print("anchor sender", T, k, r, d, flush=True)
    rng = np.random.default_rng(T)
    V = 700
    tid = rng.integers(0, V, T).astype(np.int32)
    U = np.zeros((d, r), dtype=np.float32)
    cols = rng.permutation(d)[:r]
    U[cols, np.arange(r)] = 1.0
    B = rng.integers(-2, 3, (k, d)).astype(np.float32)
    dZ = rng.integers(-2, 3, (T, r)).astype(np.float32)
    t = torch()
    D = mapl.desc(T=T, d=d, r=r, V=V, k=k)
    gZ, gB = (t.from_numpy(a).cuda().to(t.bfloat16) for a in (dZ, B))
    dA = t.full((V, k), float("nan"), device="cuda")
    ws = mapl.workspace(mapl.anchor_bwd_workspace_bytes(D, mapl.SENDER))
    mapl.anchor_bwd(D, mapl.SENDER, gZ, dev(tid, "i32"), dev(U, "f32"), gB, dA, 0, ws)
    ref = np.zeros((V, k))
    np.add.at(ref, tid, -(dZ.astype(np.float64) @ B[:, cols].T))
    assert np.array_equal(dA.cpu().numpy().astype(np.float64), ref)
