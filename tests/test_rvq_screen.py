"""The fp16 screen of the RVQ encoder at the edges of its range and of its
candidate lists.

The screen runs in units of a power of two per round (from a sample of the
codebook's coordinates) and decides a token only where its certified bounds
do; every code is still the exact fp32 argmin.  Checked here: the bounds
themselves, in the kernels' arithmetic and with their constants (CPU), and on the GPU codebooks of extreme scale, codewords
and tokens far outside fp16's range, and near ties that fall on the two
lane halves and their first, second and third keys."""
import os
import shutil
import subprocess

import numpy as np
import pytest

from oracle import codec as ocodec
from paper_2606_05484_amd import mapl, synth
from _helpers import Dev, codes_np, compare_codes, descr, f64, run_encode, stress_codebooks

SMALL = dict(T=300, d=512, r=64, V=300, k=16, L=2, K=64, dtype="bf16", alpha=0.8, n_out=4, cb_sigma=None, gscale=1.0)


CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2606_05484_amd", "csrc")
PROG = r"""
#include <cstdio>
#include <initializer_list>
#include "rvq_margin.hpp"
int main() {
  using namespace mapl;
  for (int R : {64, 128, 256}) std::printf("%d %.9g %.9g\n", R, rvq_margin_ka(R), rvq_margin_k2(R));
  std::printf("0 %.9g %.9g %.9g %.9g %d %.9g\n", RVQ_K1_SLACK, RVQ_K2_SLACK, RVQ_SUB_FACTOR, RVQ_TINY, RVQ_CB_EXP,
              RVQ_TOK_SCALE);
  return 0;
}
"""


@pytest.fixture(scope="module")
def bounds(tmp_path_factory):
    """The kernels' constants, from their header."""
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no host C++ compiler")
    d = tmp_path_factory.mktemp("rvq_margin")
    (d / "m.cpp").write_text(PROG)
    subprocess.run([cxx, "-std=c++17", "-I", CSRC, str(d / "m.cpp"), "-o", str(d / "m")], check=True)
    rows = [l.split() for l in subprocess.run([str(d / "m")], check=True, capture_output=True, text=True).stdout.splitlines()]
    out = {int(r[0]): (float(r[1]), float(r[2])) for r in rows[:3]}
    return out, [float(v) for v in rows[3][1:]]


f32 = np.float32


def _bf(v):
    b = np.asarray(v, f32).view(np.uint32).astype(np.uint64)
    return (((b + 0x7FFF + ((b >> 16) & 1)) >> 16) << 16).astype(np.uint32).view(f32)


def _bf_up(v):  # of non-negative values
    b = np.asarray(v, f32).view(np.uint32)
    return (((b >> 16) + ((b & 0xFFFF) != 0)) << 16).astype(np.uint32).view(f32)


def _bf_trunc(v):
    return (np.asarray(v, f32).view(np.uint32) & np.uint32(0xFFFF0000)).view(f32)


def _f16(v):
    with np.errstate(over="ignore"):
        return v.astype(np.float16).astype(f32)


@pytest.mark.parametrize("r", [64, 128, 256])
@pytest.mark.parametrize("grid", [False, True])
@pytest.mark.parametrize("spread,size", [(0.0, 0), (3.0, 0), (30.0, 0), (0.0, -18), (0.0, 14), (0.0, -30), (3.0, 30)])
def test_margin_bounds_the_screen(bounds, r, spread, size, grid):
    """L_j <= s_j <= L_j + (RVQ_SUB_FACTOR + 1) Delta_j for the screen's score
    L_j as the kernels form it (fp16 coordinates, reduced norm and bound
    columns in bf16 pieces, fp32 sums in any order, a 4-bit tag), with the
    bounds from its own rounding errors and the header's constants; tokens
    within and 2^size outside the codebook's scale, coordinates over e^spread
    of magnitudes, codewords saturated, subnormal and zero.  grid: coordinates
    that fp16 holds exactly, so that only ka and k2 (sums, norms, tag) are
    left in the bounds; one token is its codeword, one opposite to it."""
    per_r, (k1s, k2s, sub, tiny, cbexp, tok) = bounds
    ka, k2 = per_r[r]
    rng = np.random.default_rng(r + int(spread) + 100 * (size + 40))
    NT, NC = 24, 40
    mag = np.exp(-spread * rng.uniform(0, 1, (2, r)))
    C = 2.0 ** (cbexp - 1) * mag[1] * rng.standard_normal((NC, r))
    C[0] *= 1e4   # saturates
    C[1] = 0.0
    C[2:6] *= 2.0 ** np.array([[-12], [-20], [-34], [-37]])  # into fp16's subnormals and below
    R = 2.0 ** (cbexp - 1 + size + rng.uniform(-4, 4, (NT, 1))) * mag[0] * rng.standard_normal((NT, r))
    R[:8] = C[rng.integers(2, NC, 8)] * 2.0 ** size * rng.uniform(0.9, 1.1, (8, r))
    C, R = C.astype(f32), R.astype(f32)
    if grid:
        C = _f16(np.clip(C, f32(-60000), f32(60000)))
        up = f32(2.0 ** (9 - size))
        R = _f16(np.clip(R * up, f32(-60000), f32(60000))) / up
        R[8:16], R[16:] = C[2:10] * f32(2.0 ** size), -C[10:18] * f32(2.0 ** size)
    # codebook side (prep_codebook_block)
    Cq = _f16(np.clip(C, f32(-65504), f32(65504)))
    n2 = (C * C).sum(1, dtype=f32)
    eu = (np.sqrt(((C - Cq) ** 2).sum(1, dtype=f32)) * f32(1 + 2.0 ** -15) + f32(tiny)).astype(f32)
    red = (n2 - n2 * f32(k2s * k2)).astype(f32)
    hi = _bf(red)
    mid = _bf(red - hi)
    lo = _bf(red - hi - mid)
    cu = (np.sqrt(n2) * f32(1 + 2.0 ** -15)).astype(f32)
    chi = _bf(cu)
    rem = cu - chi
    clo = np.where(rem > 0, _bf_up(np.abs(rem)), _bf_trunc(rem))
    assert (hi.astype(np.float64) + mid + lo == red).all() and (chi.astype(np.float64) + clo >= cu).all()
    # token side (rvq_rounds)
    x = -2 * R
    mx = np.abs(x).max(1)
    far = ((mx * tok >= 65504) | (mx < 2.0 ** -3)) & (mx >= 2.0 ** -60) & (mx < 2.0 ** 49)
    tsc = np.where(far, 2.0 ** (14 - np.floor(np.log2(np.maximum(mx, 2.0 ** -60)))), tok).astype(f32)[:, None]
    x = x * tsc
    xq = _f16(x)
    rn = (f32(0.5) * np.sqrt((x * x).sum(1, dtype=f32)) * f32(1 + 2.0 ** -15) + f32(tiny)).astype(f32)[:, None]
    en = (f32(0.5) * np.sqrt(((x - xq) ** 2).sum(1, dtype=f32)) * f32(1 + 2.0 ** -15) + f32(tiny)).astype(f32)[:, None]
    assert np.isfinite(en).all()
    bco = (2 * en * f32(1.0078125) + f32(ka) * rn).astype(f32)
    cco = (2 * (rn + en)).astype(f32)
    b, c = -_bf_up(bco * f32(k1s)), -_bf_up(cco * f32(k1s))
    delta = (cco * eu + bco * cu + f32(k2) * (tsc * n2)).astype(np.float64) * 1.0002 + 1e-30
    terms = [tsc * hi, tsc * mid, tsc * lo, b * chi, b * clo, c * _bf_up(eu)]
    terms += [xq[:, i:i + 1] * Cq[None, :, i] for i in range(r)]
    exact = tsc.astype(np.float64) * (C.astype(np.float64) ** 2).sum(1) + x.astype(np.float64) @ C.astype(np.float64).T
    for _ in range(3):
        L = np.zeros((NT, NC), f32)
        for i in [0, 1, 2, 3, 4, 5] + list(6 + rng.permutation(r)):
            L = (L + terms[i]).astype(f32)
        tagged = ((L.view(np.uint32) & ~np.uint32(15)) | rng.integers(0, 16, L.shape, dtype=np.uint32)).view(f32)
        for k in (L, tagged):
            assert (k <= exact + 1e-30).all()
            assert (exact <= k + (sub + 1) * delta).all()


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
@pytest.mark.parametrize("kind", ["outlier", "tokens", "alternate"])
def test_wide_ranges_are_screened(r, kind):
    """Sizes over many powers of two, which the screen has to decide without
    scoring tokens against the whole codebook: one codeword 10^6 times the
    others, tokens (and the codewords drawn from them) over 2^20, and every
    second codeword 2^-20 of the others (K = 512: the scale's sample takes one
    codeword in two)."""
    K = 512 if kind == "alternate" else 64
    x = synth.codec_inputs(None, seed=37, **dict(SMALL, T=700, r=r, k=0, L=1, K=K))
    if kind == "tokens":
        X = x["X"].copy()
        e = np.random.default_rng(6).integers(-10, 11, (len(X), 1))
        x["X"] = np.where((X & 0x7F80) > (11 << 7), X + (e << 7), 0).astype(X.dtype)  # bf16 bits: the exponent
    C = stress_codebooks(x, 14)
    C[0, 0] = C[0, 1]  # no zero codeword
    if kind == "outlier":
        C[0, 5] *= np.float32(1e6)
    if kind == "alternate":
        C[0, ::2] *= np.float32(2.0 ** -20)
    Z0 = ocodec.project(f64(x, "X"), x["ids"], x["U"], f64(x, "A"), f64(x, "B"), "ambient", "bf16")
    ref, gap, _ = ocodec.rvq_encode(Z0, C)
    mapl.profile(2)
    try:
        got = _encode(x, C)
        stats = mapl.profile_report()
    finally:
        mapl.profile(0)
    bad, ex = compare_codes(got, ref, gap)
    print("mismatched", bad, "exempt", ex, {k: v[0] for k, v in stats.items() if k.startswith("rvq:")})
    assert bad == 0
    # a token whose nearest is among the 256 tiny ones may list more than fit
    assert stats["rvq:list_overflows"][0] <= (3 if kind == "alternate" else 0)


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
