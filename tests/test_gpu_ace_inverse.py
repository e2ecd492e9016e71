"""The triangular inverse of the ACE build at the edges of its forms (64, 256, 512
and 1024 orbitals): xi = L^-1 W against a triangular solve in FP64.

Bar: both are backward stable, with an error of at most n 2^-53 cond(L) each (a dot
product of n terms a row), doubled for the product with W.
"""
import pytest

from paper_2208_06097_amd import sea

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("n", [64, 65, 256, 257, 512, 513, 1024, 1025])
def test_xi_against_triangular_solve(n):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"case ace inverse {n}", flush=True)
    g = torch.Generator().manual_seed(n)
    phi = (torch.randn(n, 8 * n + 5, generator=g, dtype=torch.float64) / (8 * n) ** 0.5).cuda()
    ctx = sea.Context(ace_dtype=sea.SEA_F64)
    out = ctx.ace_build(phi, phi, 1.0)
    ctx.close()
    xi = next(t for t in out if torch.is_tensor(t) and t.shape == phi.shape)
    L = torch.linalg.cholesky((phi @ phi.T).cpu())
    ref = torch.linalg.solve_triangular(L, phi.cpu(), upper=False)
    rel = float((xi.cpu() - ref).norm() / ref.norm())
    bar = 4 * n * 2.0 ** -53 * float(torch.linalg.cond(L))
    print(f"|dxi|/|xi| {rel:.2e} bar {bar:.2e}", flush=True)
    assert rel < bar
