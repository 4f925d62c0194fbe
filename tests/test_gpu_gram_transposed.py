"""Algorithm 1's Gram through X^T and the GEMM (GPU): the same basis as from the triangle kernel's
Gram, at the edges of the transpose's tiles, with strided rows, and where the triangle kernel stays."""
import pytest
import torch

from gpu_helpers import announce, dev
from paper_2607_01125_amd import zoact as Z

pytestmark = pytest.mark.gpu


# one tile, several with ragged edges, strided rows; token counts off the 64-deep stages, odd, and
# below the GEMM's least depth (X^T padded with zeros); a workspace too small for X^T (65536 x 64):
# the triangle kernel
@pytest.mark.parametrize("n,d,ld,r", [
    (128, 64, 64, 4), (192, 128, 136, 8), (320, 320, 320, 8), (1024, 576, 640, 16), (4096, 192, 192, 8),
    (200, 128, 128, 8), (100, 64, 64, 4), (1029, 1024, 1024, 16), (65536, 64, 64, 4),
])
def test_basis_init_matches_gram(n, d, ld, r):
    _check(n, d, ld, r, 0)


# both sides of the line to the triangle kernel (512 tokens below 256 features), ragged edges of the
# transpose's tiles past it; fewer tokens than the block, X^T padded to the GEMM's least depth
@pytest.mark.parametrize("n,d,ld,r,p", [(511, 64, 64, 4, 0), (512, 64, 72, 4, 0), (577, 192, 200, 8, 0),
                                        (300, 256, 256, 8, 0), (100, 256, 264, 4, 100)])
def test_basis_init_matches_gram_at_the_line(n, d, ld, r, p):
    _check(n, d, ld, r, p)


def _check(n, d, ld, r, p):
    announce("gram transposed", n, d, ld, r, p)
    g = torch.Generator(device=dev())
    g.manual_seed(n + d)
    k = min(2 * r, d)
    q = torch.linalg.qr(torch.randn(d, k, generator=g, device=dev()))[0]
    s = 0.7 ** torch.arange(k, device=dev(), dtype=torch.float32)   # well separated
    wide = torch.full((n, ld), float("nan"), dtype=torch.bfloat16, device=dev())
    wide[:, :d] = ((torch.randn(n, k, generator=g, device=dev()) * s * 8) @ q.T
                   + 0.01 * torch.randn(n, d, generator=g, device=dev())).to(torch.bfloat16)
    x = wide[:, :d]
    opts = Z.EigOpts(p, 40, 0x5EED, 0.0, 0, 0)
    out = []
    for one in (True, False):
        ut = torch.full((r, d), float("nan"), device=dev())
        ev = torch.full((r,), float("nan"), device=dev())
        ws = torch.empty(Z.basis_init_workspace_bytes(d, r, opts), dtype=torch.uint8, device=dev())
        if one:
            Z.basis_init(x, r, ut, ws, opts, eigvals=ev)
        else:
            gram = torch.empty(d, d, device=dev())
            Z.gram(x, gram)
            Z.basis_from_gram(gram, r, ut, ws, opts, eigvals=ev)
        out.append((ut.double(), ev.double()))
    (u0, e0), (u1, e1) = out
    want = torch.linalg.eigvalsh(x.double().T @ x.double()).flip(0)[:r]
    # fp32 Grams of n bf16 products in two orders: 1e-5 of the largest eigenvalue
    assert float((e0 - want).abs().max() / want[0]) < 1e-5
    assert float((e0 - e1).abs().max() / want[0]) < 1e-5
    # neighbours 0.7^2 apart: the vectors move by about the Gram's error over their gap
    assert float(((u0 * u1).sum(1) - 1).abs().max()) < 1e-4
