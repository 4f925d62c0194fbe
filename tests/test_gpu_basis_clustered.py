"""Algorithm 1's small eigenproblem (GPU) where many eigenvalues agree to about the ratio at which
its Jacobi sweeps stop: the block spans the whole space, so the reported residual is the
eigenproblem's alone."""
import pytest
import torch

from gpu_helpers import announce, dev
from paper_2607_01125_amd import zoact as Z

pytestmark = pytest.mark.gpu


# d = r + oversample (= 2 r): blocks of 32, 64 and 128 columns; all eigenvalues equal, agreeing to
# 1e-10 .. 1e-7, and a quarter of them a cluster beside separated ones
@pytest.mark.parametrize("d", [32, 64, 128])
@pytest.mark.parametrize("delta", [0.0, 1e-10, 1e-9, 1e-8, 1e-7])
@pytest.mark.parametrize("spread", [False, True])
def test_clustered_eigenvalues(d, delta, spread):
    announce("clustered eigenvalues", d, delta, spread)
    g = torch.Generator()
    g.manual_seed(1)
    s = torch.randn(d, d, generator=g)
    s = (s + s.T).fill_diagonal_(0) * (delta / d ** 0.5)
    diag = torch.ones(d)
    if spread:
        diag[d // 4:] = 0.9 ** torch.arange(1, d - d // 4 + 1)
    gram = (s + torch.diag(diag)).to(dev()).contiguous()   # (fp32 holds the small off-diagonal entries)
    r = d // 2
    ut = torch.empty(r, d, device=dev())
    ws = torch.empty(Z.basis_workspace_bytes(d, r), dtype=torch.uint8, device=dev())
    rep = Z.eig_report_tensor(dev())
    assert Z.basis_from_gram(gram, r, ut, ws, report=rep)
    # fp64 sums over d terms and the sweeps' rotations: a few d ulp (measured: 1.2e-14 at d = 128)
    assert Z.read_eig_report(rep)["resid"] <= 8 * d * 2.0 ** -52
    u = ut.double()   # rounded to fp32: each entry off by half an ulp
    assert float((u @ u.T - torch.eye(r, device=dev(), dtype=torch.float64)).abs().max()) <= 2.0 ** -23
