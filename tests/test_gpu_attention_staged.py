"""The staged bf16 attention (GPU) against float64, at the edges of its tiles: one token, sequences
off the 64-key blocks, one, two and four query heads per key/value head, workgroup counts on and off
multiples of the chip's eight XCDs, and q, k, v as strided views of one projection."""
import math

import pytest
import torch

from gpu_helpers import announce, assert_bf16_close, dev, host
from paper_2607_01125_amd import zoact as Z

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_seq,seq,H,Hkv,hd", [
    (1, 1, 8, 8, 128), (3, 63, 5, 5, 64), (2, 64, 8, 8, 128), (2, 65, 6, 3, 64), (1, 127, 8, 4, 128),
    (2, 129, 12, 3, 128), (1, 300, 16, 2, 64), (2, 511, 3, 3, 128), (1, 513, 8, 8, 64),
])
def test_attention_staged(n_seq, seq, H, Hkv, hd):
    _check(n_seq, seq, H, Hkv, hd, 0)


@pytest.mark.parametrize("n_seq,seq,H,Hkv,hd", [(1, 1, 8, 8, 128), (2, 65, 6, 3, 64), (1, 300, 40, 40, 128),
                                                (1, 497, 16, 4, 128)])
def test_attention_staged_rows_behind(n_seq, seq, H, Hkv, hd):
    """Rows behind the last sequence, up to the end of its 64-key block, hold NaN: they count as
    zeros with probability 0."""
    _check(n_seq, seq, H, Hkv, hd, 64)


def _check(n_seq, seq, H, Hkv, hd, behind):
    announce("attention staged", n_seq, seq, H, Hkv, hd, behind)
    g = torch.Generator(device=dev())
    g.manual_seed(seq)
    n, a, b = n_seq * seq, H * hd, (H + Hkv) * hd
    buf = torch.full((n + behind, (H + 2 * Hkv) * hd), float("nan"), dtype=torch.bfloat16, device=dev())
    qkv = buf[:n]
    qkv.copy_(torch.randn(n, (H + 2 * Hkv) * hd, generator=g, device=dev()))
    out = torch.full((n, a), float("nan"), dtype=torch.bfloat16, device=dev())
    scale = 1.0 / math.sqrt(hd)
    Z.attention(qkv[:, :a], qkv[:, a:b], qkv[:, b:], out, n_seq, seq, H, Hkv, hd, scale)
    d = qkv.double().cpu()
    q = d[:, :a].reshape(n_seq, seq, H, hd).transpose(1, 2)
    k = d[:, a:b].reshape(n_seq, seq, Hkv, hd).transpose(1, 2).repeat_interleave(H // Hkv, 1)
    v = d[:, b:].reshape(n_seq, seq, Hkv, hd).transpose(1, 2).repeat_interleave(H // Hkv, 1)
    s = torch.matmul(q, k.transpose(2, 3).contiguous()) * scale
    s = s.masked_fill(torch.ones(seq, seq).triu(1).bool(), -math.inf)
    p = torch.exp(s - s.amax(3, keepdim=True))
    o = torch.matmul(p.to(torch.bfloat16).double(), v) / p.sum(3, keepdim=True)   # probabilities rounded as defined
    want = o.transpose(1, 2).reshape(n, a).numpy()
    # a probability whose fp32 value crosses a bf16 rounding boundary moves the output by 2^-9 of it
    assert_bf16_close(host(out), want, atol_rel_rms=4e-3, what="staged attention vs float64")
