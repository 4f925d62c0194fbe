"""The last, partly idle round of the 256 x 256 schedule spread over the workgroups by depth (GPU):
against float64, the call without a workspace, and the pair's halves against each other."""
import math

import pytest
import torch

from gpu_helpers import announce, assert_bf16_close, dev, host
from paper_2607_01125_amd import zoact as Z
from test_gpu_few_tokens import _g, _want

pytestmark = pytest.mark.gpu


# on 256 compute units: 268 tiles (12 cut into 60 shares, 5 each), 272 (16 into 64), 288 (32 into
# 128), 400 (144 into 256 shares that cross tiles), 160 (no whole round, all of them cut), 524 (12
# into 60 after two whole rounds: past every line of the few-token schedule); odd numbers of
# stages, ragged T and N
@pytest.mark.parametrize("T,K,N,r,flags,bias,resid,out_f32", [
    (500, 1088, 16912, 32, 0, True, True, True),
    (500, 1088, 17184, 8, Z.EPI_SWIGLU, True, True, False),
    (1000, 1088, 8464, 64, Z.EPI_RELU, True, True, False),
    (1000, 1600, 9216, 0, 0, False, False, True),
    (512, 8128, 25600, 32, 0, False, False, True),
    (1000, 20480, 5120, 64, 0, True, True, True),
    (2200, 8192, 2304, 8, 0, False, True, True),   # nine token tiles per half: groups of five and four
    (500, 1088, 33328, 32, 0, True, True, False),
    (500, 1088, 33312, 8, Z.EPI_SWIGLU, True, False, False),
    (500, 1088, 33328, 16, Z.EPI_RELU, True, True, False),
])
def test_split_tail(T, K, N, r, flags, bias, resid, out_f32):
    announce("split tail", T, K, N, r, flags, bias, resid, out_f32)
    nout = N // 2 if flags == Z.EPI_SWIGLU else N
    x, w = _g(1, 2 * T, K), _g(2, N, K, std=0.02)
    b = _g(3, N, std=0.1) if bias else None
    res = _g(4, 2 * T, nout) if resid else None
    ut = p = ch = arena = None
    if r:
        ut = _g(5, r, K, std=1.0 / math.sqrt(K))
        p = (x.float() @ ut.float().T).to(torch.bfloat16)
        ch = _g(6, 2, N * r, std=0.02)
        c = torch.zeros(N * r, device=dev())
        arena = Z.Arena(c, c, c)
    # (filled with NaN: a slot that is read and was not written shows)
    ws = torch.full((Z.linear_workspace_bytes() // 4,), float("nan"), device=dev()).view(torch.uint8)

    def call(use_ws, xx=x, pp=p, cc=ch, rr=res):
        lay = Z.Linear(w, K, N, r, ut, 0, b, ch=cc, ch_stride=N * r if r else 0, ws=ws if use_ws else None)
        y = torch.full((2 * T, nout), float("nan"), dtype=torch.float32 if out_f32 else torch.bfloat16, device=dev())
        Z.linear_fwd_pm(lay, arena, xx, T, pp, y, Z.Pert(1, 1, 0, 1e-3), residual=rr, flags=flags)
        return y

    got, whole = call(True), call(False)
    assert bool(torch.isfinite(ws.view(torch.float32)).any()), "no partial sum was stored"
    ref = _want(x, w, b, p, ch, r, T, (0, 0), flags, res)
    # fp32 sums of bf16 products in another order: as for the depth-split schedule of few tokens
    assert_bf16_close(host(got), ref, what="split tail vs float64")
    assert_bf16_close(host(whole), ref, what="whole tiles vs float64")
    if out_f32:
        assert not torch.equal(got, whole), "no tile was split"
    y2 = call(True, torch.cat([x[:T], x[:T]]), torch.cat([p[:T], p[:T]]) if r else None,
              torch.stack([ch[0], ch[0]]) if r else None, torch.cat([res[:T], res[:T]]) if resid else None)
    assert torch.equal(y2[:T], y2[T:]), "the pair's halves differ"
    assert torch.equal(call(True), got), "two runs differ"


@pytest.mark.parametrize("B,S,K,V", [(3, 100, 1024, 16656), (4, 128, 2048, 50272)])
def test_split_tail_cross_entropy(B, S, K, V):
    """264 tiles, and 788 (20 in the tail, the last column half empty)."""
    announce("split tail, cross entropy", B, S, K, V)
    T = B * S
    x, w = _g(1, 2 * T, K), _g(2, V, K, std=0.02)
    tok = torch.randint(0, V, (B, S), device=dev(), dtype=torch.int32)
    tok[0, 1], tok[0, 2], tok[0, 3] = V - 1, V - 256, V   # in the tail's columns; past the end: clamped
    full = Z.linear_xent_workspace_bytes(T, V)
    # the tail's part: a 256 KB slot per compute unit and per tile of the last round
    ncu = torch.cuda.get_device_properties(0).multi_processor_count
    own = full - (ncu + 2 * ((T + 255) // 256) * ((V + 255) // 256) % ncu) * 256 * 1024
    out = []
    for cut in (0, 512 * 1024 * 256):   # with and without the tail's part of the workspace
        loss = torch.full((2,), float("nan"), device=dev())
        ws = torch.full((max(full - cut, 2 * T * ((V + 127) // 128) * 8 + 64 * 1024) // 4,), float("nan"),
                        device=dev()).view(torch.uint8)
        Z.linear_xent(Z.Linear(w, K, V), None, x, tok, None, Z.Pert(1, 1, 0, 0.0), loss, ws)
        out.append(loss)
        tail = ws.view(torch.float32)[own // 4:]
        assert bool(torch.isfinite(tail).any()) == (cut == 0), "the tail's slots"
    logits = (x.double() @ w.double().T).reshape(2, B, S, V)
    tgt = tok.long().clamp(0, V - 1)[:, 1:].reshape(-1)
    for h in range(2):
        want = torch.nn.functional.cross_entropy(logits[h, :, :-1].reshape(-1, V), tgt)
        for loss in out:   # fp32 logits and exponentials of a mean over hundreds of rows
            assert abs(float(loss[h]) - float(want)) <= 1e-5 * float(want)


def _i(seed, *shape, scale=1.0):
    g = torch.Generator(device=dev())
    g.manual_seed(seed)
    return (torch.randint(-2, 3, shape, generator=g, device=dev()) * scale).to(torch.bfloat16)


# the tail's shapes of 524 tiles, and a few-token one (depth slices)
@pytest.mark.parametrize("T,K,N", [(500, 1088, 33312), (40, 4096, 1056)])
@pytest.mark.parametrize("flags,out_f32", [(0, False), (0, True), (Z.EPI_RELU, False), (Z.EPI_SWIGLU, False)])
def test_epilogues_agree(T, K, N, flags, out_f32):
    """Operands whose sums are exact in fp32 (small integers times powers of two): the depth's split
    changes no sum, so the epilogue behind stored partial sums gives the bits of the one that runs
    from the accumulators."""
    announce("epilogues agree", T, K, N, flags, out_f32)
    nout, r = N // 2 if flags == Z.EPI_SWIGLU else N, 8
    x, w = _i(1, 2 * T, K), _i(2, N, K, scale=2.0 ** -6)
    b, res = _i(3, N, scale=0.5), _i(4, 2 * T, nout)
    ut, p, ch = _i(5, r, K), _i(6, 2 * T, r), _i(7, 2, N * r, scale=2.0 ** -4)
    c = torch.zeros(N * r, device=dev())
    ws = torch.full((Z.linear_workspace_bytes() // 4,), float("nan"), device=dev()).view(torch.uint8)
    y = []
    for use in (True, False):
        y.append(torch.full((2 * T, nout), float("nan"), dtype=torch.float32 if out_f32 else torch.bfloat16, device=dev()))
        lay = Z.Linear(w, K, N, r, ut, 0, b, ch=ch, ch_stride=N * r, ws=ws if use else None)
        Z.linear_fwd_pm(lay, Z.Arena(c, c, c), x, T, p, y[-1], Z.Pert(1, 1, 0, 1e-3), residual=res, flags=flags)
    assert bool(torch.isfinite(ws.view(torch.float32)).any()), "no partial sum was stored"
    assert torch.equal(y[0], y[1]) and bool(torch.isfinite(y[0]).all())


def test_cross_entropy_epilogues_agree():
    """The same for the cross entropy: its row partials, and so the loss, to the last bit."""
    B, S, K, V = 3, 100, 1024, 16656
    announce("cross entropy epilogues agree")
    T = B * S
    x, w, b = _i(1, 2 * T, K), _i(2, V, K, scale=2.0 ** -6), _i(3, V, scale=0.5)
    tok = torch.randint(0, V, (B, S), device=dev(), dtype=torch.int32)
    full, losses = Z.linear_xent_workspace_bytes(T, V), []
    for nbytes in (full, full - 264 * 256 * 1024):
        losses.append(torch.full((2,), float("nan"), device=dev()))
        ws = torch.empty(nbytes, dtype=torch.uint8, device=dev())
        Z.linear_xent(Z.Linear(w, K, V, bias=b), None, x, tok, None, Z.Pert(1, 1, 0, 0.0), losses[-1], ws)
    assert torch.equal(losses[0].view(torch.int32), losses[1].view(torch.int32))
