"""Performance cases of the forward-only ZO step: what a fine-tuning program has the library do.

A program fine-tunes a frozen Llama- or OPT-shaped decoder in bf16 or on an INT4 backbone (or a
tiny fp32 model).  It computes each site's basis once (Algorithm 1), then per step runs both
perturbation halves forward through adapted linears, attention and the fused head loss, and
updates the coefficients.  Batches run from one short sequence (tens of tokens per half) to 16
sequences of 256 or 8 of 512; ranks from 8 to 64.  Layer shapes are those of the decoders in
synth and bench.py; sequence and token counts are spread over their range, ragged ones among them.

Each case is one public entry point (or the two calls of one adapted layer), besides one whole
decoder forward and one whole step of the tiny model.  `exact` recomputes a case in float64 with
plain torch, from the same seeded inputs.
"""
import math

import torch

from paper_2607_01125_amd import model as M
from paper_2607_01125_amd import zoact as Z

DEV = "cuda"
EPS = 1e-3          # perturbation scale of the steps
LR = 5e-5

# fused projections of the two model shapes: name -> (d_in, d_out, epilogue, bias, residual, plain range)
LAYERS = {
    "llama_qkv": (4096, 6144, "none", False, False, (0, 0)),
    "llama_o": (4096, 4096, "none", False, True, (0, 0)),
    "llama_gate_up": (4096, 28672, "swiglu", False, False, (0, 0)),
    "llama_down": (14336, 4096, "none", False, True, (0, 0)),
    "opt_qkv": (5120, 15360, "none", True, False, (5120, 10240)),
    "opt_out": (5120, 5120, "none", True, True, (0, 0)),
    "opt_fc1": (5120, 20480, "relu", True, False, (0, 0)),
    "opt_fc2": (20480, 5120, "none", True, True, (0, 0)),
}
FLAGS = {"none": 0, "swiglu": Z.EPI_SWIGLU, "relu": Z.EPI_RELU}


def listed():
    return [
        # the tiny fp32 model's whole step (4 x 64 tokens): launches and latency only
        {"name": "tiny_step_fp32", "kind": "tiny_step", "n_seq": 4, "seq": 64},
        # one adapted q|k|v on a micro-batch of one short sequence
        {"name": "linear_qkv_t64", "kind": "linear", "layer": "llama_qkv", "dtype": "bf16", "T": 64, "r": 32},
        # an adapted o projection on the INT4 backbone, one sequence of 256 tokens, through the INT4 call
        {"name": "linear_o_int4_t256", "kind": "linear", "layer": "llama_o", "dtype": "int4", "T": 256, "r": 32},
        # gate|up with SwiGLU on a ragged batch (2 x 250 tokens)
        {"name": "linear_gate_up_t500", "kind": "linear", "layer": "llama_gate_up", "dtype": "bf16", "T": 500, "r": 32},
        # OPT's fc2 (bias, residual, rank 64) on a quarter of its usual batch
        {"name": "linear_fc2_t1024", "kind": "linear", "layer": "opt_fc2", "dtype": "bf16", "T": 1024, "r": 64},
        # down with its residual at the headline batch (16 x 256 tokens per half)
        {"name": "linear_down_t4096", "kind": "linear", "layer": "llama_down", "dtype": "bf16", "T": 4096, "r": 32},
        # OPT's causal attention, both halves of 8 x 512 tokens
        {"name": "attention_opt_16x512", "kind": "attention", "n_seq": 16, "seq": 512, "H": 40, "Hkv": 40, "hd": 128},
        # OPT's head with the cross entropy, 4 x 128 tokens per half
        {"name": "head_loss_opt_4x128", "kind": "head", "d": 5120, "vocab": 50272, "B": 4, "S": 128},
        # the update that also writes the next perturbation, eight Llama layers' coefficients
        {"name": "update_11m", "kind": "update", "k": 11010048, "c_bf16": False},
        # the one-sided update over q = 8 queries
        {"name": "update_q8_11m", "kind": "update_q", "k": 11010048, "q": 8, "c_bf16": False},
        # Algorithm 1 for one 4096-wide site from 16 x 256 calibration tokens
        {"name": "basis_4096", "kind": "basis", "n": 4096, "d": 4096, "r": 32},
        # a whole forward of both halves: two Llama-width INT4 layers and a head, 2 x 128 tokens per half
        {"name": "forward_int4_2x128", "kind": "forward", "mode": "int4", "n_seq": 2, "seq": 128, "layers": 2,
         "vocab": 8192},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["linear", "linear", "linear", "attention", "head", "update", "update_q", "basis", "forward",
                       "tiny_step"])
    if kind == "linear":
        layer = rng.choice(sorted(LAYERS))
        wide = LAYERS[layer][0] * LAYERS[layer][1] > 14336 * 4096
        # INT4 weights need whole scale groups, which every listed layer has; the plain
        # feature range and rank 64 belong to the OPT layers
        return {"kind": kind, "layer": layer, "dtype": rng.choice(["bf16", "bf16", "int4"]),
                "T": _log_int(rng, 16, 2048 if wide else 4096),
                "r": rng.choice([16, 32, 32, 64]) if layer.startswith("llama") else 64}
    if kind == "attention":
        hd = rng.choice([64, 128, 128])
        hkv = rng.choice([4, 8, 16])
        return {"kind": kind, "n_seq": 2 * rng.randint(1, 8), "seq": _log_int(rng, 17, 512), "H": hkv * rng.choice([1, 4]),
                "Hkv": hkv, "hd": hd}
    if kind == "head":
        return {"kind": kind, "d": rng.choice([1024, 2048, 4096, 5120]), "vocab": 16 * _log_int(rng, 500, 3142),
                "B": rng.randint(1, 4), "S": _log_int(rng, 20, 256)}
    if kind == "update":
        return {"kind": kind, "k": _log_int(rng, 4096, 11010048), "c_bf16": rng.random() < 0.5}
    if kind == "update_q":
        return {"kind": kind, "k": _log_int(rng, 4096, 11010048), "q": rng.randint(2, 8), "c_bf16": rng.random() < 0.5}
    if kind == "basis":
        return {"kind": kind, "n": rng.choice([1024, 2048, 3000, 4096]), "d": 64 * rng.randint(16, 64),
                "r": rng.choice([16, 32])}
    if kind == "forward":
        return {"kind": kind, "mode": rng.choice(["bf16", "int4"]), "n_seq": rng.randint(1, 4),
                "seq": _log_int(rng, 16, 256), "layers": 1, "vocab": 8192}
    return {"kind": "tiny_step", "n_seq": rng.randint(1, 8), "seq": rng.randint(9, 64)}


# ------------------------------------------------------------------ seeded inputs
class _Gen:
    def __init__(self, seed):
        self.g = torch.Generator(device=DEV)
        self.g.manual_seed(int(seed) * 7919 + 17)

    def normal(self, shape, std=1.0, dtype=torch.float32):
        return torch.randn(shape, generator=self.g, device=DEV, dtype=torch.float32).mul_(std).to(dtype)

    def tokens(self, shape, vocab):
        return torch.randint(0, vocab, shape, generator=self.g, device=DEV, dtype=torch.int64).to(torch.int32)


def _basis(g, r, d, dtype):
    """Random U^T [r][d] with rows of unit length (nearly orthogonal at these widths)."""
    return g.normal((r, d), 1.0 / math.sqrt(d)).to(dtype)


def _quantize(w):
    """Symmetric INT4, one bf16 scale per row and 128 columns: (packed uint8 [N][K/2], scales bf16)."""
    n, k = w.shape
    grp = w.float().reshape(n, k // 128, 128)
    s = (grp.abs().amax(dim=2) / 7.0).to(torch.bfloat16)
    sf = s.float()[:, :, None]
    q = torch.where(sf == 0, torch.zeros_like(grp), torch.round(grp / torch.where(sf == 0, torch.ones_like(sf), sf)))
    nib = (q.clamp_(-7, 7).to(torch.int16).reshape(n, k) & 0xF).to(torch.uint8)
    return (nib[:, 0::2] | (nib[:, 1::2] << 4)).contiguous(), s.contiguous()


def _dequantize(packed, scales):
    """The stored weight values, bf16(q s), in float64."""
    n, kb = packed.shape
    q = torch.stack([packed & 0xF, packed >> 4], dim=2).reshape(n, 2 * kb).to(torch.int32)
    q = torch.where(q >= 8, q - 16, q).float()
    return (q * scales.float().repeat_interleave(128, dim=1)).to(torch.bfloat16).double()


def _linear_inputs(case, seed):
    K, N, epi, bias, resid, plain = LAYERS[case["layer"]]
    T, r, g = case["T"], case["r"], _Gen(seed)
    rows = N - (plain[1] - plain[0])
    x = g.normal((2 * T, K), 1.0, torch.bfloat16)
    w = g.normal((N, K), 0.02, torch.bfloat16)
    ut = _basis(g, r, K, torch.bfloat16)
    c = g.normal((rows * r,), 0.01)
    z = g.normal((rows * r,), 1.0)
    ch = torch.stack([c + EPS * z, c - EPS * z]).to(torch.bfloat16).contiguous()
    b = g.normal((N,), 0.1, torch.bfloat16) if bias else None
    res = g.normal((2 * T, N), 1.0, torch.bfloat16) if resid else None
    packed = scales = None
    if case["dtype"] == "int4":
        packed, scales = _quantize(w)
        w = None
    return x, w, packed, scales, ut, c, ch, b, res


def _qkv(case, seed):
    g = _Gen(seed)
    n = case["n_seq"] * case["seq"]
    return g.normal((n, (case["H"] + 2 * case["Hkv"]) * case["hd"]), 1.0, torch.bfloat16)


def _head_inputs(case, seed):
    g = _Gen(seed)
    x = g.normal((2 * case["B"] * case["S"], case["d"]), 1.0, torch.bfloat16)
    w = g.normal((case["vocab"], case["d"]), 0.02, torch.bfloat16)
    return x, w, g.tokens((case["B"], case["S"]), case["vocab"])


def _arena_inputs(case, seed):
    """C, m, v in mid-training and the losses of one step (a directional derivative of order one)."""
    g, k = _Gen(seed), case["k"]
    c = g.normal((k,), 0.01, torch.bfloat16 if case["c_bf16"] else torch.float32)
    m = g.normal((k,), 0.1)
    v = g.normal((k,), 0.3).square_().add_(1e-4)
    loss = 2.0 + EPS * g.normal((case.get("q", 1) + 1,), 1.0)
    return c, m, v, loss


def _calibration(case, seed):
    """Activations with 64 planted directions carrying 90% of the variance (squared scales
    falling by 0.95 each), the rest isotropic: bf16 [n][d]."""
    g, n, d = _Gen(seed), case["n"], case["d"]
    q = torch.linalg.qr(g.normal((d, 64)))[0]
    s2 = 0.95 ** torch.arange(64, device=DEV, dtype=torch.float32)
    s2 *= 0.9 * d / s2.sum()
    return ((g.normal((n, 64)) * s2.sqrt()) @ q.T + math.sqrt(0.1) * g.normal((n, d))).to(torch.bfloat16)


class _Shape:
    """A decoder shape (the attributes the framework's Decoder reads)."""

    def __init__(self, **kw):
        self.__dict__.update(kw)
        self.head_dim = self.d_model // self.n_heads


def _shape(case):
    if case["kind"] == "tiny_step":
        return _Shape(name="tiny", n_layers=2, d_model=128, n_heads=4, n_kv_heads=4, d_ff=512, vocab=512, family="llama",
                      rope_theta=1.0e4, norm_eps=1e-5, max_pos=2048, adapted=("q", "v"), rank=8)
    return _Shape(name="llama-width", n_layers=case["layers"], d_model=4096, n_heads=32, n_kv_heads=8, d_ff=14336,
                  vocab=case["vocab"], family="llama", rope_theta=5.0e5, norm_eps=1e-5, max_pos=2048,
                  adapted=("q", "k", "v", "o", "gate", "up", "down"), rank=32)


def _model_inputs(case, seed):
    """Weights (wq .. wd as stored), bases, coefficients and tokens of a decoder."""
    s, g = _shape(case), _Gen(seed)
    dt = torch.float32 if case["kind"] == "tiny_step" else torch.bfloat16
    int4 = case.get("mode") == "int4"
    d, dkv, ff = s.d_model, s.n_kv_heads * s.head_dim, s.d_ff
    W = {"emb": g.normal((s.vocab, d), 0.02, dt),
         "head": g.normal((s.vocab, d), 0.02, dt), "nf": torch.ones(d, dtype=dt, device=DEV)}
    for l in range(s.n_layers):
        L = {"n1": torch.ones(d, dtype=dt, device=DEV), "n2": torch.ones(d, dtype=dt, device=DEV)}
        for name, n, k in (("wq", d, d), ("wk", dkv, d), ("wv", dkv, d), ("wo", d, d), ("wg", ff, d), ("wu", ff, d),
                           ("wd", d, ff)):
            w = g.normal((n, k), 0.02, dt)
            L[name] = _quantize(w) if int4 else w
        W[l] = L
    blocks = M.arena_layout(s)
    dims = {"attn": d, "o": d, "mlp": d, "down": ff}
    ut = {}
    for b in blocks:
        if (b.layer, b.site) not in ut:
            ut[(b.layer, b.site)] = _basis(g, s.rank, dims[b.site], dt)
    k = sum(b.rows * b.r for b in blocks)
    c = g.normal((k,), 0.01).to(torch.bfloat16 if int4 else torch.float32)
    return s, W, ut, c, g.tokens((case["n_seq"], case["seq"]), s.vocab)


# ------------------------------------------------------------------ what a program holds before the call
def prepare(case, seed):
    kind = case["kind"]
    if kind == "linear":
        K, N, epi, _, _, plain = LAYERS[case["layer"]]
        T, r = case["T"], case["r"]
        x, w, packed, scales, ut, c, ch, b, res = _linear_inputs(case, seed)
        lin_ws = torch.empty(Z.linear_workspace_bytes(), dtype=torch.uint8, device=DEV)
        layer = Z.Linear(w if w is not None else packed, K, N, r, ut, 0, bias=b, w_scales=scales, ch=ch,
                         ch_stride=ch.shape[1], plain=plain, ws=lin_ws)
        arena = Z.Arena(c, torch.zeros_like(c), torch.zeros_like(c))
        return {"kind": kind, "layer": layer, "arena": arena, "x": x, "T": T, "res": res, "flags": FLAGS[epi],
                "p": torch.empty(2 * T, r, dtype=torch.bfloat16, device=DEV),
                "y": torch.empty(2 * T, N // 2 if epi == "swiglu" else N, dtype=torch.bfloat16, device=DEV),
                "pws": torch.empty(Z.project_workspace_bytes(2 * T, K, r), dtype=torch.uint8, device=DEV),
                "pert": Z.Pert(seed, 1, 0, EPS)}
    if kind == "attention":
        qkv = _qkv(case, seed)
        a, b = case["H"] * case["hd"], (case["H"] + case["Hkv"]) * case["hd"]
        return {"kind": kind, "case": case, "q": qkv[:, :a], "k": qkv[:, a:b], "v": qkv[:, b:],
                "out": torch.empty(qkv.shape[0], a, dtype=torch.bfloat16, device=DEV),
                "scale": 1.0 / math.sqrt(case["hd"])}
    if kind == "head":
        x, w, tok = _head_inputs(case, seed)
        T = case["B"] * case["S"]
        return {"kind": kind, "layer": Z.Linear(w, case["d"], case["vocab"]), "x": x, "tok": tok,
                "pert": Z.Pert(seed, 1, 0, EPS), "loss": torch.empty(2, dtype=torch.float32, device=DEV),
                "ws": torch.empty(Z.linear_xent_workspace_bytes(T, case["vocab"]), dtype=torch.uint8, device=DEV)}
    if kind in ("update", "update_q"):
        c, m, v, loss = _arena_inputs(case, seed)
        st = {"kind": kind, "arena": Z.Arena(c, m, v), "loss": loss, "seed": seed, "q": case.get("q", 1), "t": 100,
              "status": torch.zeros(1, dtype=torch.int32, device=DEV)}
        if kind == "update":
            st["ch"] = torch.empty(2, case["k"], dtype=torch.bfloat16, device=DEV)
        return st
    if kind == "basis":
        x = _calibration(case, seed)
        opts = Z.EigOpts(0, 64, 0x5EED, 1e-4, 1, 8)   # adaptive to 1e-4, as the models run it
        d, r = case["d"], case["r"]
        return {"kind": kind, "x": x, "r": r, "opts": opts,
                "ws": torch.empty(Z.basis_init_workspace_bytes(d, r, opts), dtype=torch.uint8, device=DEV),
                "ut": torch.empty(r, d, dtype=torch.float32, device=DEV),
                "ev": torch.empty(r, dtype=torch.float32, device=DEV)}
    s, W, ut, c, tok = _model_inputs(case, seed)
    dec = M.Decoder(s, W, "fp32" if kind == "tiny_step" else case["mode"], device=DEV)
    dec.set_basis(ut)
    dec.arena.c.copy_(c)
    return {"kind": kind, "dec": dec, "tok": tok, "seed": seed, "pert": Z.Pert(seed, 1, 0, EPS)}


def run(st):
    kind = st["kind"]
    if kind == "linear":
        Z.project(st["x"], st["layer"].ut, st["p"], st["pws"])
        Z.linear_fwd_pm(st["layer"], st["arena"], st["x"], st["T"], st["p"], st["y"], st["pert"], st["res"], st["flags"])
        return st["p"], st["y"]
    if kind == "attention":
        k = st["case"]
        Z.attention(st["q"], st["k"], st["v"], st["out"], k["n_seq"], k["seq"], k["H"], k["Hkv"], k["hd"], st["scale"])
        return st["out"]
    if kind == "head":
        Z.linear_xent(st["layer"], None, st["x"], st["tok"], None, st["pert"], st["loss"], st["ws"])
        return st["loss"]
    if kind == "update":
        st["t"] += 1
        t, a = st["t"], st["arena"]
        Z.step_perturb(a, st["loss"], Z.Pert(st["seed"], t, 0, EPS), Z.adam_desc(LR, t), Z.Pert(st["seed"], t + 1, 0, EPS),
                       st["ch"], st["status"])
        return a.c, a.m, a.v, st["ch"]
    if kind == "update_q":
        st["t"] += 1
        t, a = st["t"], st["arena"]
        Z.step_q(a, st["loss"], st["q"], st["seed"], t, EPS, Z.adam_desc(LR, t), st["status"])
        return a.c, a.m, a.v
    if kind == "basis":
        Z.basis_init(st["x"], st["r"], st["ut"], st["ws"], st["opts"], eigvals=st["ev"])
        return st["ut"], st["ev"]
    dec = st["dec"]
    if kind == "tiny_step":
        loss = dec.step(st["tok"], st["seed"], EPS, LR)
        return loss, dec.arena.m, dec.arena.v, dec.arena.c
    return dec.forward(st["tok"], st["pert"])


# ------------------------------------------------------------------ what a pass cannot do without
def _attention_flops(n_seq, seq, H, hd):
    return 4.0 * hd * H * n_seq * seq * (seq + 1) / 2      # causal: q k^T and p v


def _linear_work(K, N, T, r, wbytes, n_out, bias, resid, rows):
    M2 = 2 * T
    flops = 2.0 * M2 * N * K + 2.0 * M2 * K * r + 2.0 * M2 * rows * r
    nbytes = 2.0 * M2 * K + wbytes * N * K + 2.0 * r * K + 2 * 2.0 * rows * r + 2.0 * M2 * (n_out + r)
    return nbytes + (2.0 * N if bias else 0) + (2.0 * M2 * N if resid else 0), flops


def work(case):
    kind = case["kind"]
    if kind == "linear":
        K, N, epi, bias, resid, plain = LAYERS[case["layer"]]
        wb = 2.0 if case["dtype"] == "bf16" else 0.5 + 2.0 / 128
        b, f = _linear_work(K, N, case["T"], case["r"], wb, N // 2 if epi == "swiglu" else N, bias, resid,
                            N - (plain[1] - plain[0]))
    elif kind == "attention":
        n = case["n_seq"] * case["seq"]
        b = 2.0 * n * case["hd"] * (2 * case["H"] + 2 * case["Hkv"])
        f = _attention_flops(case["n_seq"], case["seq"], case["H"], case["hd"])
    elif kind == "head":
        T2 = 2 * case["B"] * case["S"]
        b = 2.0 * case["d"] * (case["vocab"] + T2) + 2.0 * T2 + 8
        f = 2.0 * T2 * case["d"] * case["vocab"]
    elif kind == "update":
        cb = 2 if case["c_bf16"] else 4
        b, f = case["k"] * (16.0 + 2 * cb + 4), 100.0 * case["k"]
    elif kind == "update_q":
        cb = 2 if case["c_bf16"] else 4
        b, f = case["k"] * (16.0 + 2 * cb), 50.0 * case["q"] * case["k"]
    elif kind == "basis":
        n, d, r = case["n"], case["d"], case["r"]
        # the smaller Gram's triangle, and one pass of products with a 2r block
        side = min(n, d)
        b, f = 2.0 * n * d + 4.0 * r * d, float(max(n, d)) * side * side + 2.0 * side * side * 2 * r
    else:
        s = _shape(case)
        T = case["n_seq"] * case["seq"]
        d, dkv, ff, r = s.d_model, s.n_kv_heads * s.head_dim, s.d_ff, s.rank
        tiny = kind == "tiny_step"
        wb = 4.0 if tiny else (2.0 if case["mode"] == "bf16" else 0.5 + 2.0 / 128)
        ab = 4.0 if tiny else 2.0
        b = f = 0.0
        for n, k, ad in ((d + 2 * dkv, d, True), (d, d, not tiny), (2 * ff, d, not tiny), (d, ff, not tiny)):
            b += wb * n * k + (2 * ab * n * r + ab * r * k if ad else 0)
            f += 4.0 * T * n * k + (4.0 * T * r * (n + k) if ad else 0)
        f += _attention_flops(2 * case["n_seq"], case["seq"], s.n_heads, s.head_dim)
        b, f = b * s.n_layers, f * s.n_layers
        b += ab * d * (s.vocab + T)
        f += 4.0 * T * d * s.vocab
        b += 8.0 if tiny else 8.0 * T * s.vocab
        if tiny:
            b += 24.0 * 2 * s.n_layers * d * r
    return {"bytes": b, "flops": f}


def tolerance(case):
    kind = case["kind"]
    if kind in ("update", "update_q"):
        return "exact"       # the generator and the update are defined operation by operation in fp32
    # measured against float64 on an MI355X, stated at about four times that
    if kind == "tiny_step":
        return {"rel": 1e-3}     # the moments carry (L+ - L-) / 2 eps of fp32 losses: 1.7e-4 (m), 3.5e-4 (v)
    if kind == "head":
        return {"rel": 1e-6}     # fp32 log-sum-exp, fp64 mean: 4e-8
    if kind == "basis":
        return {"rel": 2e-3}     # the residual bound 1e-4 over eigenvalue gaps of 5%
    if kind == "forward":
        return {"rel": 4e-2}     # bf16 between kernels, through the layers to the logits: 1.2e-2
    return {"rel": 8e-3}         # one rounding to bf16: 1.7e-3 (linears), 2.0e-3 (attention)


# ------------------------------------------------------------------ the same in float64
def _philox(seed, step, query, k):
    """Z at arena indices 0 .. k - 1 in float64: Philox4x32-10 words, Box-Muller in quarter turns."""
    mask = 0xFFFFFFFF
    nb = (k + 3) // 4

    def mulhilo(a, x):       # the 64-bit product of two 32-bit values as (high, low) words
        lo16, hi16 = x & 0xFFFF, x >> 16
        p0, p1 = a * lo16, a * hi16
        low = (p0 + ((p1 & 0xFFFF) << 16))
        return (p1 >> 16) + (low >> 32), low & mask

    c0 = torch.arange(nb, dtype=torch.int64, device=DEV)
    c1 = torch.zeros_like(c0)
    c2, c3 = torch.full_like(c0, step), torch.full_like(c0, query)
    k0, k1 = seed & mask, (seed >> 32) & mask
    for _ in range(10):
        h0, l0 = mulhilo(0xD2511F53, c0)
        h1, l1 = mulhilo(0xCD9E8D57, c2)
        c0, c1, c2, c3 = h1 ^ c1 ^ k0, l1, h0 ^ c3 ^ k1, l0
        k0, k1 = (k0 + 0x9E3779B9) & mask, (k1 + 0xBB67AE85) & mask
    out = torch.empty(nb, 4, dtype=torch.float64, device=DEV)
    for i, (wa, wb) in enumerate(((c0, c1), (c2, c3))):
        rad = torch.sqrt(-2.0 * torch.log(((wa >> 8) + 1).double() * 2.0 ** -24))
        ang = ((wb >> 30).double() + ((wb >> 8) & 0x3FFFFF).double() * 2.0 ** -22) * (math.pi / 2)
        out[:, 2 * i], out[:, 2 * i + 1] = rad * torch.cos(ang), rad * torch.sin(ang)
    return out.reshape(-1)[:k]


def _f32(x):
    return float(torch.tensor(x, dtype=torch.float32))


def _attend(q, k, v, n_seq, seq, H, Hkv, hd, scale):
    """Causal attention of [n_seq seq][heads hd] float64 rows."""
    out = torch.empty(n_seq * seq, H * hd, dtype=torch.float64, device=q.device)
    mask = torch.ones(seq, seq, dtype=torch.bool, device=q.device).triu(1)
    for b in range(n_seq):
        rows = slice(b * seq, (b + 1) * seq)
        qq = q[rows].reshape(seq, H, hd).transpose(0, 1)
        kk = k[rows].reshape(seq, Hkv, hd).transpose(0, 1).repeat_interleave(H // Hkv, dim=0)
        vv = v[rows].reshape(seq, Hkv, hd).transpose(0, 1).repeat_interleave(H // Hkv, dim=0)
        s = torch.matmul(qq, kk.transpose(1, 2).contiguous()).mul_(scale).masked_fill_(mask, -math.inf)
        out[rows] = torch.matmul(torch.softmax(s, dim=-1), vv.contiguous()).transpose(0, 1).reshape(seq, H * hd)
    return out


def _adam(c, m, v, gh, t):
    b1, b2 = _f32(0.9), _f32(0.999)
    m = b1 * m + _f32(1.0 - 0.9) * gh
    v = b2 * v + _f32(1.0 - 0.999) * gh * gh
    d = v.sqrt() * _f32(1.0 / math.sqrt(1.0 - 0.999 ** t)) + _f32(1e-8)
    return c - _f32(LR / (1.0 - 0.9 ** t)) * (m / d), m, v


def _decoder_logits(s, W, ut, c, z, tok):
    """Logits [2][n_seq][seq][V] of both halves in float64 (Llama family)."""
    n_seq, seq = tok.shape
    d, H, Hkv, hd = s.d_model, s.n_heads, s.n_kv_heads, s.head_dim
    half = hd // 2
    ang = (torch.arange(seq, dtype=torch.float64, device=DEV)[:, None]
           * (s.rope_theta ** (-2.0 * torch.arange(half, dtype=torch.float64, device=DEV) / hd))[None, :])
    cos, sin = ang.cos().repeat(n_seq, 1)[:, None, :], ang.sin().repeat(n_seq, 1)[:, None, :]

    def weight(w):
        return _dequantize(*w) if isinstance(w, tuple) else w.double()

    def rms(x, w):
        return x * torch.rsqrt(x.square().mean(dim=1, keepdim=True) + s.norm_eps) * w.double()

    def rope(x, n):
        x = x.reshape(-1, n, hd)
        lo, hi = x[..., :half], x[..., half:]
        return torch.cat([lo * cos - hi * sin, hi * cos + lo * sin], dim=-1).reshape(-1, n * hd)

    blocks = {(b.layer, b.name): b for b in M.arena_layout(s)}
    hs = [W["emb"].double()[tok.reshape(-1).long()] for _ in range(2)]
    for l in range(s.n_layers):
        L = W[l]

        def adapted(name, site, x, w, h):
            y = x @ w.T
            b = blocks.get((l, name))
            if b is not None:
                co = slice(b.offset, b.offset + b.rows * b.r)
                cc = (c[co] + (EPS if h == 0 else -EPS) * z[co]).reshape(b.rows, b.r)
                y = y + (x @ ut[(l, site)].double().T) @ cc.T
            return y

        wq, wk, wv = weight(L["wq"]), weight(L["wk"]), weight(L["wv"])
        fused = (l, "qkv") in blocks
        att = []
        for h in range(2):
            a = rms(hs[h], L["n1"])
            if fused:
                y = adapted("qkv", "attn", a, torch.cat([wq, wk, wv]), h)
                q, k, v = y[:, :d], y[:, d:d + wk.shape[0]], y[:, d + wk.shape[0]:]
            else:
                y = adapted("qv", "attn", a, torch.cat([wq, wv]), h)
                q, k, v = y[:, :d], a @ wk.T, y[:, d:]
            att.append(_attend(rope(q, H), rope(k, Hkv), v, n_seq, seq, H, Hkv, hd, 1.0 / math.sqrt(hd)))
        w = weight(L["wo"])
        hs = [hs[h] + adapted("o", "o", att[h], w, h) for h in range(2)]
        wg = M.interleave_gate_up(weight(L["wg"]), weight(L["wu"]))
        ffs = []
        for h in range(2):
            y = adapted("gu", "mlp", rms(hs[h], L["n2"]), wg, h).reshape(-1, s.d_ff // 16, 2, 16)
            ffs.append((torch.nn.functional.silu(y[:, :, 0]) * y[:, :, 1]).reshape(-1, s.d_ff))
        del wg
        w = weight(L["wd"])
        hs = [hs[h] + adapted("down", "down", ffs[h], w, h) for h in range(2)]
    head = W["head"].double()
    return torch.stack([rms(hs[h], W["nf"]) @ head.T for h in range(2)]).reshape(2, n_seq, seq, s.vocab)


def _xent(logits, tok):
    lp = torch.log_softmax(logits[:, :-1], dim=-1)
    return -lp.gather(2, tok[:, 1:, None].long()).mean()


def exact(case, seed):
    kind = case["kind"]
    if kind == "linear":
        K, N, epi, _, _, plain = LAYERS[case["layer"]]
        T, r = case["T"], case["r"]
        x, w, packed, scales, ut, c, ch, b, res = _linear_inputs(case, seed)
        wd = w.double() if w is not None else _dequantize(packed, scales)
        p = x.double() @ ut.double().T
        y = x.double() @ wd.T
        del wd
        cd = ch.double().reshape(2, -1, r)
        cols = [i for i in ((0, plain[0]), (plain[1], N)) if i[1] > i[0]] if plain[1] > plain[0] else [(0, N)]
        for h in range(2):
            rows, at = slice(h * T, (h + 1) * T), 0
            for lo, hi in cols:
                y[rows, lo:hi] += p[rows] @ cd[h, at:at + hi - lo].T
                at += hi - lo
        if b is not None:
            y += b.double()
        if epi == "swiglu":
            y = y.reshape(2 * T, N // 32, 2, 16)
            y = (torch.nn.functional.silu(y[:, :, 0]) * y[:, :, 1]).reshape(2 * T, N // 2)
        elif epi == "relu":
            y = y.clamp_(min=0)
        return p, (y + res.double() if res is not None else y)
    if kind == "attention":
        qkv = _qkv(case, seed).double()
        a, b = case["H"] * case["hd"], (case["H"] + case["Hkv"]) * case["hd"]
        return _attend(qkv[:, :a], qkv[:, a:b], qkv[:, b:], case["n_seq"], case["seq"], case["H"], case["Hkv"],
                       case["hd"], 1.0 / math.sqrt(case["hd"]))
    if kind == "head":
        x, w, tok = _head_inputs(case, seed)
        wd = w.double()
        T = case["B"] * case["S"]
        return torch.stack([_xent((x[h * T:(h + 1) * T].double() @ wd.T).reshape(case["B"], case["S"], -1), tok)
                            for h in range(2)])
    if kind in ("update", "update_q"):
        c, m, v, loss = _arena_inputs(case, seed)
        c, m, v, l, t, k = c.double(), m.double(), v.double(), loss.double(), 101, case["k"]
        if kind == "update":
            gh = (l[0] - l[1]) / (2 * _f32(EPS)) * _philox(seed, t, 0, k)
            c, m, v = _adam(c, m, v, gh, t)
            ez = _f32(EPS) * _philox(seed, t + 1, 0, k)
            return c, m, v, torch.stack([c + ez, c - ez])
        gh = torch.zeros(k, dtype=torch.float64, device=DEV)
        for j in range(1, case["q"] + 1):
            gh += (l[j] - l[0]) / _f32(EPS) * _philox(seed, t, j, k)
        return _adam(c, m, v, gh / case["q"], t)
    if kind == "basis":
        x, r = _calibration(case, seed).double(), case["r"]
        q = torch.linalg.qr(torch.randn(case["d"], 2 * r + 64, dtype=torch.float64, device=DEV))[0]
        g = x.T @ x
        for _ in range(60):
            q = torch.linalg.qr(g @ q)[0]
        w, s = torch.linalg.eigh(q.T @ (g @ q))
        u = (q @ s).flip(1)[:, :r]
        top = u.abs().argmax(dim=0)
        return (u * u.gather(0, top[None, :]).sign()).T.contiguous(), w.flip(0)[:r].contiguous()
    s, W, ut, c, tok = _model_inputs(case, seed)
    z = _philox(seed, 1, 0, c.numel())
    logits = _decoder_logits(s, W, ut, c.double(), z, tok)
    if kind == "forward":
        return logits
    loss = torch.stack([_xent(logits[h], tok) for h in range(2)])
    zero = torch.zeros_like(z)
    c1, m, v = _adam(c.double(), zero, zero, (loss[0] - loss[1]) / (2 * _f32(EPS)) * z, 1)
    return loss, m, v, c1
