"""The fp32 kernels of small models (GPU): the adapted linear on fp32 MFMA and the attention, at
the edges of their tiles, against float64."""
import math

import numpy as np
import pytest
import torch

from gpu_helpers import announce, dev, host
from oracle import linear as olin
from paper_2607_01125_amd import zoact as Z

pytestmark = pytest.mark.gpu


def _r(seed, *shape, std=1.0):
    return (np.random.default_rng(seed).standard_normal(shape) * std).astype(np.float32)


def _dev(a, shift=0):
    """Device copy, `shift` floats into its allocation (off 16-byte alignment when not 0)."""
    buf = torch.zeros(a.size + 4, device=dev())
    v = buf[shift:shift + a.size].view(a.shape)
    v.copy_(torch.from_numpy(a))
    return v


# tokens and features off the 16 / 32 / 64 tiles, depths off 16 and off 4 (element loads), a
# misaligned x, ranks off 4 and 16, and one shape of the large-tile form (512 tiles of 64 x 64)
@pytest.mark.parametrize("T,K,N,r,flags,bias,resid,shift", [
    (1, 4, 1, 1, 0, False, False, 0),
    (15, 20, 33, 3, 0, True, True, 0),
    (65, 130, 40, 8, Z.EPI_RELU, True, False, 0),
    (64, 128, 96, 17, Z.EPI_SWIGLU, True, False, 0),
    (17, 64, 128, 8, 0, False, True, 1),
    (1030, 96, 1000, 8, 0, True, True, 0),
    (1030, 131, 1000, 8, 0, False, False, 1),
    (40, 6, 48, 2, 0, False, False, 3),
])
def test_linear_f32(T, K, N, r, flags, bias, resid, shift):
    announce("fp32 linear", T, K, N, r, flags, shift)
    x, w, ut = _r(1, 2, T, K), _r(2, N, K, std=0.1), _r(3, r, K, std=1 / math.sqrt(K))
    c, off = _r(4, 3 + N * r, std=0.1), 3
    b = _r(5, N) if bias else None
    nout = N // 2 if flags == Z.EPI_SWIGLU else N
    res = _r(6, 2, T, nout) if resid else None
    seed, step, eps = 7, 3, 1e-2
    ct = _dev(c)
    arena = Z.Arena(ct, torch.zeros_like(ct), torch.zeros_like(ct))
    xt = _dev(x.reshape(2 * T, K), shift)
    p = torch.full((2 * T, r), float("nan"), device=dev())
    Z.project(xt, _dev(ut), p)
    p64 = x.reshape(2 * T, K).astype(np.float64) @ ut.astype(np.float64).T
    # fp32 chains of K products: rounding errors of at most K ulp, in practice sqrt(K)
    assert np.max(np.abs(host(p) - p64)) <= 2.0 ** -23 * K * np.sqrt(np.mean(p64 ** 2) + 1e-30) + 1e-6
    y = torch.full((2 * T, nout), float("nan"), device=dev())
    Z.linear_fwd_pm(Z.Linear(_dev(w), K, N, r, _dev(ut), off, _dev(b) if bias else None), arena, xt, T, p, y,
                    Z.Pert(seed, step, 0, eps), residual=_dev(res.reshape(2 * T, nout)) if resid else None, flags=flags)
    ref = olin.adapted_linear_pm(x, w, b, ut, c[off:].reshape(N, r), eps, seed, step, 0, off, "fp32",
                                 p_pm=host(p).reshape(2, T, r))
    if flags == Z.EPI_SWIGLU:
        v = ref.reshape(2, T, N // 32, 2, 16)
        ref = (v[..., 0, :] / (1 + np.exp(-v[..., 0, :])) * v[..., 1, :]).reshape(2, T, nout)
    if resid:
        ref = ref + res
    if flags == Z.EPI_RELU:
        ref = np.maximum(ref, 0)
    err = np.max(np.abs(host(y).reshape(2, T, nout) - ref))
    assert err <= 2.0 ** -23 * (K + r) * np.sqrt(np.mean(ref ** 2)) + 1e-5, err


def test_linear_f32_many_features():
    """More 64-feature tiles than one grid dimension holds (65,535)."""
    K, N = 4, 65535 * 64 + 33
    announce("fp32 linear, many features", N)
    g = torch.Generator(device=dev())
    g.manual_seed(8)
    x, w = torch.randn(2, K, generator=g, device=dev()), torch.randn(N, K, generator=g, device=dev())
    y = torch.full((2, N), float("nan"), device=dev())
    Z.linear_fwd_pm(Z.Linear(w, K, N), None, x, 1, None, y, Z.Pert(1, 1, 0, 0.0))
    want = x.double() @ w.double().T
    # a chain of four products: four roundings of at most half an ulp of sums below 4 x 36
    assert float((y.double() - want).abs().max()) <= 4 * 2.0 ** -24 * 144


# one query, a query group short of 8, keys across the 64-key steps, grouped heads, head sizes
# below and above one column per lane, the longest sequence a head size allows
@pytest.mark.parametrize("n_seq,seq,H,Hkv,hd", [(1, 1, 1, 1, 4), (3, 9, 4, 2, 32), (2, 65, 4, 4, 32), (2, 130, 2, 1, 30),
                                                (1, 32, 2, 2, 128), (2, 45, 3, 1, 90), (1, 512, 1, 1, 8)])
def test_attention_f32(n_seq, seq, H, Hkv, hd):
    announce("fp32 attention", n_seq, seq, H, Hkv, hd)
    n = n_seq * seq
    qkv = _r(1, n, (H + 2 * Hkv) * hd)
    t = _dev(qkv)
    out = torch.full((n, H * hd), float("nan"), device=dev())
    a, b = H * hd, (H + Hkv) * hd
    scale = 1 / math.sqrt(hd)
    Z.attention(t[:, :a], t[:, a:b], t[:, b:], out, n_seq, seq, H, Hkv, hd, scale)
    x = qkv.astype(np.float64).reshape(n_seq, seq, H + 2 * Hkv, hd)
    want = np.zeros((n_seq, seq, H, hd))
    for h in range(H):
        k, v = x[:, :, H + h // (H // Hkv)], x[:, :, H + Hkv + h // (H // Hkv)]
        s = np.einsum("bqe,bke->bqk", x[:, :, h], k) * scale
        s = np.where(np.tril(np.ones((seq, seq), bool)), s, -np.inf)
        pr = np.exp(s - s.max(axis=2, keepdims=True))
        want[:, :, h] = np.einsum("bqk,bke->bqe", pr / pr.sum(axis=2, keepdims=True), v)
    # scores of |s| <= ~6 in fp32: their rounding (hd ulp) enters the exponentials
    assert np.max(np.abs(host(out) - want.reshape(n, -1))) <= 2.0 ** -22 * hd + 2.0 ** -22 * math.sqrt(seq) + 2e-6
