"""The adapted linear at few tokens, where the depth is split over workgroups (GPU): against a
float64 evaluation of the same bf16 operands, and the forms whose bits must agree."""
import math

import numpy as np
import pytest
import torch

from gpu_helpers import announce, assert_bf16_close, dev, host
from paper_2607_01125_amd import zoact as Z

pytestmark = pytest.mark.gpu


def _g(seed, *shape, std=1.0):
    g = torch.Generator(device=dev())
    g.manual_seed(seed)
    return (torch.randn(shape, generator=g, device=dev()) * std).to(torch.bfloat16)


def _int4(N, K, seed):
    """Random packed INT4 weights with values in [-7, 7] and bf16 scales near 0.02 / 4."""
    g = torch.Generator(device=dev())
    g.manual_seed(seed)
    q = torch.randint(-7, 8, (N, K), generator=g, device=dev()) & 0xF
    packed = (q[:, 0::2] | (q[:, 1::2] << 4)).to(torch.uint8).contiguous()
    return packed, (0.005 * (1 + torch.rand(N, K // 128, generator=g, device=dev()))).to(torch.bfloat16)


def _want(x, w, b, p, ch, r, T, plain, flags, res):
    """The call in float64 from the operands it reads (P and C_h as stored)."""
    y = x.double() @ w.double().T
    if r:
        c = ch.double().reshape(2, -1, r)
        full = torch.zeros(2, w.shape[0], r, dtype=torch.float64, device=dev())
        full[:, :plain[0]] = c[:, :plain[0]]
        full[:, plain[1]:] = c[:, plain[0]:]
        for h in range(2):
            y[h * T:(h + 1) * T] += p[h * T:(h + 1) * T].double() @ full[h].T
    if b is not None:
        y += b.double()
    if flags == Z.EPI_SWIGLU:
        y = y.reshape(2 * T, -1, 2, 16)
        y = (torch.nn.functional.silu(y[:, :, 0]) * y[:, :, 1]).reshape(2 * T, -1)
    if res is not None:
        y = y + res.double()
    if flags == Z.EPI_RELU:
        y = y.clamp(min=0)
    return y.cpu().numpy()


# T at the edges of 16-token blocks and of tiles holding both halves, N off the 128-feature
# tiles, the smallest depth, ranks in one and several 32-deep steps and off multiples of 8
@pytest.mark.parametrize("T,K,N,r,flags,bias,resid,plain,out_f32", [
    (1, 128, 144, 8, 0, True, True, (0, 0), False),          # one token, two stages
    (20, 192, 272, 16, Z.EPI_RELU, True, False, (0, 0), False),   # three stages
    (200, 128, 1552, 8, 0, True, True, (0, 0), False),       # two stages, larger tiles
    (300, 192, 4096, 32, Z.EPI_SWIGLU, False, False, (0, 0), False),
    (16, 512, 128, 32, 0, False, False, (0, 0), False),      # whole blocks: one 32-row tile
    (17, 1024, 4096, 64, Z.EPI_RELU, True, False, (0, 0), False),
    (33, 2048, 1040, 5, 0, True, True, (0, 0), False),       # odd rank: element-wise correction
    (31, 4096, 768, 32, 0, True, False, (256, 512), False),  # plain range
    (65, 1024, 2080, 40, Z.EPI_SWIGLU, True, True, (0, 0), False),
    (100, 4096, 512, 0, 0, False, False, (0, 0), True),      # no adaptation, fp32 output
    (200, 8192, 1552, 32, 0, False, True, (0, 0), False),    # several token tiles
    (129, 14336, 4096, 32, 0, False, True, (0, 0), False),   # 256-token tiles, many slices
])
@pytest.mark.parametrize("int4", [False, True])
def test_few_tokens(T, K, N, r, flags, bias, resid, plain, out_f32, int4):
    announce("few tokens", T, K, N, r, flags, bias, resid, plain, out_f32, int4)
    if int4 and K < 256:
        pytest.skip("the INT4 schedules need whole scale groups and a depth of 256")
    rows = N - (plain[1] - plain[0])
    nout = N // 2 if flags == Z.EPI_SWIGLU else N
    x = _g(1, 2 * T, K)
    if int4:
        packed, scales = _int4(N, K, 2)
        w = torch.empty(N, K, dtype=torch.bfloat16, device=dev())
        Z.dequant_int4(packed, scales, w)
    else:
        w = _g(2, N, K, std=0.02)
    b = _g(3, N, std=0.1) if bias else None
    res = _g(4, 2 * T, nout) if resid else None
    ut = p = ch = arena = None
    if r:
        ut = _g(5, r, K, std=1.0 / math.sqrt(K))
        p = (x.float() @ ut.float().T).to(torch.bfloat16)
        ch = _g(6, 2, rows * r, std=0.02)
        c = torch.zeros(rows * r, device=dev())
        arena = Z.Arena(c, c, c)
    ws = torch.empty(Z.linear_workspace_bytes(), dtype=torch.uint8, device=dev())

    def call(weight, sc, use_ws, xx=x, pp=p, cc=ch, fl=flags):
        lay = Z.Linear(weight, K, N, r, ut, 0, b, sc, ch=cc, ch_stride=rows * r if r else 0, plain=plain,
                       ws=ws if use_ws else None)
        y = torch.full((2 * T, nout), float("nan"), dtype=torch.float32 if out_f32 else torch.bfloat16, device=dev())
        Z.linear_fwd_pm(lay, arena, xx, T, pp, y, Z.Pert(1, 1, 0, 1e-3), residual=res, flags=fl)
        return y

    ref = _want(x, w, b, p, ch, r, T, plain, flags, res)
    bits = torch.int32 if out_f32 else torch.int16
    got = call(w, None, True)
    # fp32 sums of bf16 products in another order: 1e-3 of the rms covers K = 14336 terms;
    # SwiGLU's hardware exponential and reciprocal are a few ulp of fp32
    assert_bf16_close(host(got), ref, what="split depth vs float64")
    assert torch.equal(got.view(bits), call(w, None, True).view(bits)), "two runs differ"
    assert_bf16_close(host(call(w, None, False)), ref, what="whole depth vs float64")
    if int4:   # the packed weights give the bits of the dequantised ones, with and without ws
        assert torch.equal(call(packed, scales, True).view(bits), got.view(bits))
        assert torch.equal(call(packed, scales, False).view(bits), call(w, None, False).view(bits))
    # equal halves (x, p and C_h) give equal bits
    if resid:
        return
    x2 = torch.cat([x[:T], x[:T]])
    p2 = torch.cat([p[:T], p[:T]]) if r else None
    c2 = torch.stack([ch[0], ch[0]]) if r else None
    y2 = call(w, None, True, x2, p2, c2)
    assert torch.equal(y2[:T].view(bits), y2[T:].view(bits)), "the pair's halves differ"
    # one shared copy of x and p: the bits of the stacked form
    if r in (8, 16, 24, 32) and flags != Z.EPI_SWIGLU and plain == (0, 0):
        y1 = call(w, None, True, x[:T].contiguous(), p[:T].contiguous(), ch, flags | Z.SHARED_X)
        assert torch.equal(y1.view(bits), call(w, None, True, x2, p2, ch).view(bits)), "shared x differs"


@pytest.mark.parametrize("ws_kb", [0, 64, 1024, 8192])
def test_few_tokens_small_workspace(ws_kb):
    """A workspace smaller than zoact_linear_workspace_bytes() is used as far as it goes."""
    T, K, N = 40, 8192, 640
    announce("few tokens, workspace", ws_kb)
    x, w = _g(1, 2 * T, K), _g(2, N, K, std=0.02)
    guard = torch.full((ws_kb * 1024 + 4096,), 0x5A, dtype=torch.uint8, device=dev())
    lay = Z.Linear(w, K, N, ws=guard[:ws_kb * 1024] if ws_kb else None)
    y = torch.full((2 * T, N), float("nan"), dtype=torch.bfloat16, device=dev())
    Z.linear_fwd_pm(lay, None, x, T, None, y, Z.Pert(1, 1, 0, 1e-3))
    assert_bf16_close(host(y), (x.double() @ w.double().T).cpu().numpy(), what=f"ws {ws_kb} KB")
    assert np.all(guard[ws_kb * 1024:].cpu().numpy() == 0x5A), "written past the workspace"


# token counts at the edges of 16- and 32-token tiles and on both sides of each tile choice
# (one round of 256 workgroups), depths below one wave's unit, off the 1024-deep rounds and in
# four chunks with a ragged last one, ranks off the 16-column tiles
@pytest.mark.parametrize("n,d,r", [(1, 32, 1), (17, 96, 16), (33, 1056, 5), (512, 4096, 32), (1025, 4096, 33),
                                   (2048, 4096, 32), (700, 8224, 64), (2047, 14336, 32), (100, 5120, 100),
                                   (2049, 1024, 8), (2560, 3072, 16), (2560, 5120, 32), (4098, 4096, 32)])
@pytest.mark.parametrize("use_ws", [False, True])
def test_project_few_tokens(n, d, r, use_ws):
    announce("project few tokens", n, d, r, use_ws)
    x, ut = _g(1, n, d), _g(2, r, d, std=1.0 / math.sqrt(d))
    ws = torch.empty(max(Z.project_workspace_bytes(n, d, r), 16), dtype=torch.uint8, device=dev()) if use_ws else None
    guard = torch.full((n + 2, r), 3.0, dtype=torch.bfloat16, device=dev())
    p = guard[1:n + 1] if r % 8 == 0 else torch.empty(n, r, dtype=torch.bfloat16, device=dev())
    Z.project(x, ut, p, ws)
    assert_bf16_close(host(p), (x.double() @ ut.double().T).cpu().numpy(), what="project, few tokens")
    assert torch.all(guard[0] == 3.0) and torch.all(guard[n + 1] == 3.0)
    # a row's bits do not depend on the rows beside it: one half computed as part of the whole
    for n2 in {n // 2, (n + 1) // 2} - {0}:
        part = torch.full((n2, r), float("nan"), dtype=torch.bfloat16, device=dev())
        Z.project(x[:n2], ut, part, ws, n_all=n)
        assert torch.equal(part.view(torch.int16), p[:n2].contiguous().view(torch.int16))
    # nor while both calls are of this form
    if 1 < n <= 1024 and r <= 64:
        half = torch.empty(n // 2, r, dtype=torch.bfloat16, device=dev())
        Z.project(x[:n // 2], ut, half, ws)
        assert torch.equal(half.view(torch.int16), p[:n // 2].contiguous().view(torch.int16))
