"""The margin of the grouped quantiser's screen, on the CPU: the scores in the
kernel's arithmetic (three bf16 pieces per value, the kept products summed in
fp32 in any order), the exact distances as the kernel rounds them, and the
threshold of the codeword blocks that are searched.  The lowest codeword of
the smallest fp32 distance has to lie below the threshold for residuals and
codewords of equal, very different and nearly equal sizes."""
import numpy as np
import pytest

f32 = np.float32


def _bf(v):
    b = v.astype(f32).view(np.uint32).astype(np.uint64)
    return (((b + 0x7FFF + ((b >> 16) & 1)) >> 16) << 16).astype(np.uint32).view(f32)


def _pieces(v):
    h = _bf(v)
    m = _bf((v - h).astype(f32))
    return h, m, _bf((v - h - m).astype(f32))


def _fma(a, b, c):  # fp32 result of a fused multiply-add (float64 holds the product exactly)
    return (a.astype(np.float64) * b + c).astype(f32)


@pytest.mark.parametrize("kind", ["equal", "outlier", "spread", "tiny", "near", "integers"])
def test_nearest_codeword_is_below_the_threshold(kind):
    rng = np.random.default_rng(len(kind))
    for _ in range(200):
        K = 64
        R = rng.standard_normal(2).astype(f32)
        C = rng.standard_normal((K, 2))
        if kind == "outlier":
            C[::3] *= 3e4
        if kind == "spread":
            C *= np.exp2(rng.uniform(-20, 12, (K, 1)))
        if kind == "tiny":
            C *= 2e-4
        if kind == "near":
            C = R + 1e-4 * C
        if kind == "integers":
            R, C = np.rint(4 * R).astype(f32), np.rint(3 * C)
        C = C.astype(f32)
        terms = []
        for c in range(2):
            ch, cm, cl = _pieces(C[:, c])
            rh, rm, rl = _pieces(np.array([-2 * R[c]], f32))
            terms += [ch * rh, ch * rm, cm * rh, cm * rm, ch * rl, cl * rh]
        n2 = _fma(C[:, 1], C[:, 1], (C[:, 0] * C[:, 0]).astype(f32))
        terms += list(_pieces(n2))
        s = np.zeros(K, f32)
        for i in rng.permutation(len(terms)):
            s = (s + terms[i]).astype(f32)
        d = (R - C).astype(f32)
        dist = _fma(d[:, 1], d[:, 1], (d[:, 0] * d[:, 0]).astype(f32))
        rr = _fma(R[1:], R[1:], (R[:1] * R[:1]).astype(f32))[0]
        v = s.min()
        thr = f32(v + 2.0 ** -15 * float(rr + max(v + rr, f32(0)) + f32(2.0 ** -17) * rr)) + f32(1e-35)
        assert s[dist.argmin()] < thr
