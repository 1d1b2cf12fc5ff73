"""The fp16 screen of the RVQ encoder at the edges of its range and of its
candidate lists.

The screen runs in units of a power of two per round (from a sample of the
codebook's coordinates) and decides a token only where its certified bounds
do; every code is still the exact fp32 argmin.  Checked here: the bound
itself in float64 (CPU), and on the GPU codebooks of extreme scale, codewords
and tokens far outside fp16's range, and near ties that fall on the two
lane halves and their first, second and third keys."""
import numpy as np
import pytest

from oracle import codec as ocodec
from paper_2606_05484_amd import mapl, synth
from _helpers import Dev, codes_np, compare_codes, descr, f64, run_encode, stress_codebooks

SMALL = dict(T=300, d=512, r=64, V=300, k=16, L=2, K=64, dtype="bf16", alpha=0.8, n_out=4, cb_sigma=None, gscale=1.0)


def _flush16(x):
    """fp16 rounding, saturated, subnormals taken as zero (the worst a matrix unit may do)."""
    y = np.clip(x, -65504.0, 65504.0).astype(np.float16).astype(np.float64)
    return np.where(np.abs(y) < 2.0 ** -14, 0.0, y)


@pytest.mark.parametrize("r", [64, 128, 256])
@pytest.mark.parametrize("spread", [0.0, 3.0, 30.0])
def test_margin_bounds_the_screen_error(r, spread):
    """|s~_j - s_j| <= Delta_j with the kernel's formula, the kernel's error
    norms taken with subnormals kept and the per-coordinate allowance added."""
    rng = np.random.default_rng(r + int(spread))
    mag = np.exp(-spread * rng.uniform(0, 1, (2, r)))  # coordinates over e^30 of magnitudes
    R = 2.0 ** rng.uniform(-4, 9, (200, 1)) * mag[0] * rng.standard_normal((200, r))
    C = 40.0 * mag[1] * rng.standard_normal((100, r))
    C[0] *= 1e4  # saturates
    C[1] = 0.0
    Rq, Cq = _flush16(-2 * R) / -2, _flush16(C)
    ka = (8 * r / 2 ** 24 + 2.0 ** -20 + 2.0 ** -16) * 1.0078125
    k2 = 4 * (r + 4) / 2 ** 24 + 2.0 ** -17
    flush = 2.0 ** -14 * np.sqrt(r)
    eR = np.linalg.norm(R - (-2 * R).astype(np.float16).astype(np.float64) / -2, axis=1) + flush
    with np.errstate(over="ignore"):
        Ck = np.clip(C, -65504, 65504).astype(np.float16).astype(np.float64)
    ej = np.linalg.norm(C - Ck, axis=1) + flush
    nR, nC = np.linalg.norm(R, axis=1), np.linalg.norm(C, axis=1)
    err = np.abs(2 * R @ C.T - 2 * Rq @ Cq.T)
    delta = 2 * nR[:, None] * ej + 2 * eR[:, None] * (1 + 2.0 ** -8) * nC + ka * nR[:, None] * nC + k2 * nC ** 2
    assert (err <= delta).all()


def _encode(x, C):
    D = descr(x)
    print("encode", x["T"], x["r"], x["K"], flush=True)
    return codes_np(run_encode(x, D, Dev(x, C)), D)


@pytest.mark.gpu
@pytest.mark.parametrize("r", [64, 128, 256])
@pytest.mark.parametrize("q", [-60, 0, 40])
def test_codebook_scale(r, q):
    """Projector and codebooks times 2^q: the same codes at any scale (the
    squared norms stay inside fp32)."""
    x = synth.codec_inputs(None, seed=31, **dict(SMALL, r=r))
    C = stress_codebooks(x, 7)
    x["U"] = (x["U"] * np.float32(2.0 ** q)).astype(np.float32)
    C = (C * np.float32(2.0 ** q)).astype(np.float32)
    Z0 = ocodec.project(f64(x, "X"), x["ids"], x["U"], f64(x, "A"), f64(x, "B"), "ambient", "bf16")
    ref, gap, _ = ocodec.rvq_encode(Z0, C)
    bad, ex = compare_codes(_encode(x, C), ref, gap)
    print("mismatched", bad, "exempt", ex)
    assert bad == 0


@pytest.mark.gpu
@pytest.mark.parametrize("r", [64, 128, 256])
@pytest.mark.parametrize("q", [-149, -125, -121])
def test_sampled_coordinates_near_zero(r, q):
    """The codewords' coordinates that the round's scale is taken from (four of
    each, see rvq_round_scale) at 2^q, the others ordinary, and every token
    with an exactly zero coordinate: the scale ends at its largest power of
    two, the bounds are not finite, and the codes are the exact ones."""
    x = synth.codec_inputs(None, seed=34, **dict(SMALL, r=r, L=1))
    x["U"] = x["U"].copy()
    x["U"][:, 3] = 0.0
    C = stress_codebooks(x, 11)
    for j in range(C.shape[1]):
        c0 = 4 * ((j * 17) % (r // 4))
        C[0, j, c0:c0 + 4] = np.float32(2.0 ** q)
    Z0 = ocodec.project(f64(x, "X"), x["ids"], x["U"], f64(x, "A"), f64(x, "B"), "ambient", "bf16")
    assert (Z0[:, 3] == 0).all()
    ref, gap, _ = ocodec.rvq_encode(Z0, C)
    assert (ref != 0).mean() > 0.5
    bad, ex = compare_codes(_encode(x, C), ref, gap)
    print("mismatched", bad, "exempt", ex)
    assert bad == 0


@pytest.mark.gpu
@pytest.mark.parametrize("r", [64, 128, 256])
def test_out_of_range_token_and_codeword(r):
    """A token 2^13 times the others and a codeword on it whose sampled
    coordinates are zero, so the round's scale does not see it: the codeword
    saturates, the token leaves fp16, and both are decided exactly."""
    x = synth.codec_inputs(None, seed=32, **dict(SMALL, r=r, k=0))
    C = stress_codebooks(x, 8)
    X = x["X"].copy()
    X[7] = np.where(X[7] & 0x7F80, X[7] + (13 << 7), X[7])  # bf16 bits: the exponent up by 13
    x["X"] = X
    Z0 = ocodec.project(f64(x, "X"), x["ids"], x["U"], f64(x, "A"), f64(x, "B"), "ambient", "bf16")
    C[0, 5] = Z0[7]
    c0 = 4 * ((5 * 17) % (r // 4))
    C[0, 5, c0:c0 + 4] = 0.0
    ref, gap, _ = ocodec.rvq_encode(Z0, C)
    assert ref[7, 0] == 5 and gap[7, 0] > 1e-2
    got = _encode(x, C)
    bad, ex = compare_codes(got, ref, gap)
    print("mismatched", bad, "exempt", ex, "token 7", got[7], ref[7])
    assert got[7, 0] == 5 and bad == 0


@pytest.mark.gpu
@pytest.mark.parametrize("r", [64, 128, 256])
@pytest.mark.parametrize("q,part", [(-10, 1.0), (-12, 1.0), (-12, 0.3), (-30, 1.0)])
def test_tokens_far_above_the_codebook(r, q, part):
    """Codebooks 2^q of the residuals (part of the tokens; the others' X is
    scaled down to match): fp16(-2R) overflows in the round's units, the
    tokens take a power of two of their own, and are screened like others: no
    list overflows.  Codes count where the distances differ by more than fp32
    resolves (2e-6 of ||R||^2; at 2^-30 none does, and the first codeword of
    the equal fp32 distances is not determined by the float64 oracle)."""
    x = synth.codec_inputs(None, seed=35, **dict(SMALL, r=r, k=0))
    C = (stress_codebooks(x, 12) * np.float32(2.0 ** q)).astype(np.float32)
    C[:, 0] = C[:, 1] * np.float32(0.5)  # no zero codeword: the screen's scale is that of the others
    near = np.random.default_rng(5).uniform(size=x["T"]) >= part
    X = x["X"].copy()
    X[near] = np.where((X[near] & 0x7F80) > (-q << 7), X[near] - (-q << 7), 0)  # bf16 bits: the exponent down by -q
    x["X"] = X
    Z0 = ocodec.project(f64(x, "X"), x["ids"], x["U"], f64(x, "A"), f64(x, "B"), "ambient", "bf16")
    ref, gap, _ = ocodec.rvq_encode(Z0, C)
    mapl.profile(2)
    try:
        got = _encode(x, C)
        stats = mapl.profile_report()
    finally:
        mapl.profile(0)
    exempt = (gap < 2e-6).any(1)
    bad = int(((got != ref).any(1) & ~exempt).sum())
    print("mismatched", bad, "exempt", int(exempt.sum()), {k: v[0] for k, v in stats.items() if k.startswith("rvq:")})
    assert bad == 0 and (q < -20 or exempt.mean() < 0.5)
    assert stats["rvq:list_overflows"][0] == 0


@pytest.mark.gpu
@pytest.mark.parametrize("r", [64, 128, 256])
@pytest.mark.parametrize("rows", [(0, 1), (0, 4), (0, 1, 2), (3, 8, 40), (0, 1, 4, 5), (0, 1, 4, 5, 8, 12),
                                  tuple(range(40, 60))])
def test_near_ties_by_lane_half(r, rows):
    """Codewords at squared distances (1e-3 + 4e-5 i) ||Z0||^2 around one
    token, the nearest at the last of the given rows.  Rows 0-3, 8-11, ... of
    a 32-row tile belong to one lane half, 4-7, 12-15, ... to the other: up
    to two per half are decided from the kept keys, more by the listing pass,
    and twenty overflow the list."""
    x = synth.codec_inputs(None, seed=33, **dict(SMALL, r=r, k=16))
    Z0 = ocodec.project(f64(x, "X"), x["ids"], x["U"], f64(x, "A"), f64(x, "B"), "ambient", "bf16")
    rng = np.random.default_rng(3)
    sig = float(np.sqrt(np.mean(Z0 ** 2)))
    C = (sig * (5 + rng.standard_normal((2, 64, r)))).astype(np.float32)
    z, n2 = Z0[5], float(Z0[5] @ Z0[5])
    for i, j in enumerate(reversed(rows)):
        u = rng.standard_normal(r)
        C[0, j] = (z + np.sqrt((1e-3 + 4e-5 * i) * n2) * u / np.linalg.norm(u)).astype(np.float32)
    ref, gap, _ = ocodec.rvq_encode(Z0, C)
    assert ref[5, 0] == rows[-1] and gap[5, 0] > 2e-5  # fp32 distances resolve 1e-6 ||Z0||^2 here
    got = _encode(x, C)
    bad, ex = compare_codes(got, ref, gap)
    print("token 5", got[5], "mismatched", bad, "exempt", ex)
    assert got[5, 0] == rows[-1] and bad == 0


@pytest.mark.gpu
@pytest.mark.parametrize("r", [64, 128, 256])
@pytest.mark.parametrize("K", [32, 96, 160, 256])
def test_equal_codewords_over_tiles(r, K):
    """Every codeword two or three times, at places of the same and of
    different slots, lane halves and 32-row tiles (K % 64 == 32 among them,
    whose last chunk has one tile): equal keys meet in every merge, and the
    lowest index is the code."""
    x = synth.codec_inputs(None, seed=36, **dict(SMALL, r=r, K=K))
    C = stress_codebooks(x, 13)
    rng = np.random.default_rng(K)
    base = {s: rng.permutation(K)[:K // 3 + 1] for s in range(2)}
    for l in range(2):
        src = base[l][np.arange(K) % len(base[l])]
        C[l] = C[l][src[rng.permutation(K)]]
        for j in range(0, K - 32, 7):  # the same slot of the next tile
            C[l, j + 32] = C[l, j]
    Z0 = ocodec.project(f64(x, "X"), x["ids"], x["U"], f64(x, "A"), f64(x, "B"), "ambient", "bf16")
    got = _encode(x, C).astype(np.int64)
    R = Z0.copy()
    open_ = np.ones(len(R), bool)  # no near tie between different codewords so far
    bad = 0
    for l in range(2):
        d = ((R[:, None, :] - C[l].astype(np.float64)[None]) ** 2).sum(-1)
        first = np.array([np.flatnonzero((C[l] == C[l, j]).all(1))[0] for j in range(K)])
        best = first[d.argmin(1)]
        others = np.where(first[None] == best[:, None], np.inf, d).min(1)
        open_ &= others - d.min(1) > 1e-4 * (R ** 2).sum(1)
        bad += int((open_ & (got[:, l] != best)).sum())
        R = R - C[l].astype(np.float64)[best]
    print("mismatched", bad, "compared", int(open_.sum()))
    assert bad == 0 and open_.mean() > 0.5
