"""The generator's short division and square root, which start from the hardware's reciprocal and
reciprocal square root estimates: over all 2^24 uniforms, which of them depend on more than an
estimate within one unit of the last place (CPU), and those against the oracle (GPU)."""
import numpy as np
import pytest

from oracle import rng as orng

F = np.float32
# w >> 8 of the uniforms for which an estimate one ulp off gives another bit, and arena indices at
# which seed 1, step 1, query 0 draws them
DRAWN = {
    6267533: (3228324, 1034602, 81787716, 132254044),
    8388606: (23405198, 34654768, 42593238, 56846796),
    10528154: (30446182, 65260234, 74788372, 93633178),
    11239982: (61482946, 79967474, 87051464, 96925820),
    15076673: (753074, 45967040, 67285684, 75078412),
    16777213: (49287684, 101100652, 131388170, 167304076),
}


def _fma(a, b, c):
    """fp32 fused multiply-add: the exact product in fp64, its sum with c rounded to odd, then to fp32."""
    p, c = np.asarray(a, np.float64) * np.asarray(b, np.float64), np.asarray(c, np.float64)
    s = p + c
    t = s - p
    err = (p - (s - t)) + (c - t)
    bits = s.view(np.int64)
    step = np.where((err > 0) == (s > 0), 1, -1)
    return np.where((err != 0) & ((bits & 1) == 0), bits + step, bits).view(np.float64).astype(F)


def _ulps(a, k):
    return (a.view(np.int32) + k).view(F)


def _near_tie(v):
    """fp64 values within 2^-16 ulp of the middle between two fp32 values."""
    u = np.spacing(np.abs(v).astype(F)).astype(np.float64)
    return np.abs(np.abs(v / u - np.floor(v / u)) - 0.5) < 2.0 ** -16


def test_which_uniforms_need_more_than_one_ulp():
    # before its last rounding either result is within 2^-43 of the exact one for any estimate
    # within an ulp (an error of 2^-22 squared, and the residual's rounding times 2^-22), so only
    # values that near to a tie can round another way: 2^-19 ulp and less
    n = np.arange(1, 2 ** 24 + 1).astype(F)
    bits = n.view(np.uint32)
    e = (bits >> np.uint32(23)).astype(np.int32) - 127
    m = ((bits & np.uint32(0x007FFFFF)) | np.uint32(0x3F800000)).view(F)
    big = m >= orng.SQRT2
    m, e = np.where(big, m * F(0.5), m).astype(F), e + big
    num, den = m - F(1.0), m + F(1.0)
    assert np.abs(num).max() < 0.42 and den.min() >= 1.7 and den.max() < 2.5
    i = np.nonzero(_near_tie(num.astype(np.float64) / den))[0]
    a, d, want = num[i], den[i], num[i] / den[i]
    est = (1.0 / d.astype(np.float64)).astype(F)
    off = set()
    for k in (-1, 0, 1):
        r = _ulps(est, k)
        r = _fma(_fma(-d, r, F(1.0)), r, r)
        q = a * r
        off |= set(i[_fma(_fma(-d, q, a), r, q) != want].tolist())
    del num, den, m, n, bits
    x = np.empty(2 ** 24, F)
    for c in range(0, 2 ** 24, 2 ** 22):   # (the oracle's logarithm: rounded divisions)
        x[c:c + 2 ** 22] = F(-2.0) * orng._ln_u1((np.arange(c, c + 2 ** 22, dtype=np.uint32) << np.uint32(8)))
    assert x[-1] == 0 and x[:-1].min() >= 1e-7 and x.max() < 34
    i = np.nonzero(_near_tie(np.sqrt(x[:-1].astype(np.float64))))[0]
    v, want = x[i], np.sqrt(x[i])
    est = (1.0 / np.sqrt(v.astype(np.float64))).astype(F)
    for k in (-1, 0, 1):
        y = _ulps(est, k)
        g = v * y
        off |= set(i[_fma(_fma(-g, g, v), F(0.5) * y, g) != want].tolist())
    assert off == set(DRAWN)


def test_drawn_indices():
    for u, es in DRAWN.items():
        for idx in es:
            w = orng.philox4x32_10(np.uint32([idx >> 2]), np.uint32([0]), np.uint32([1]), np.uint32([0]), 1, 0)
            assert int(w[idx & 2][0] >> np.uint32(8)) == u


@pytest.mark.gpu
@pytest.mark.parametrize("u", sorted(DRAWN))
def test_gen_z_at_those_uniforms(u):
    import torch

    from gpu_helpers import announce, dev
    from paper_2607_01125_amd import zoact as Z
    announce("gen_z at uniform", u)
    for e in DRAWN[u]:
        out = torch.full((2,), float("nan"), device=dev())
        Z.gen_z(1, 1, 0, e, 2, out)
        assert np.array_equal(out.cpu().numpy().view(np.uint32), orng.gauss_range(1, 1, 0, e, 2).view(np.uint32))
