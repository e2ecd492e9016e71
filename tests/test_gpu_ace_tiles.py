"""The ACE products at the edges of their tiles: orbital and vector counts
around each block height (32, 64, 96, 128 rows, one block and several), grid
lengths that leave partial stages, slices and column tiles and rows aligned to
one element only; resident and staged coefficients; the triangular product.

Bars, elementwise, from the standard bound of a product of K terms, |error| <=
K u |A||B| in any order of the sum (u = 2^-53; 2^-24 for FP32 operands), plus
the operands' rounding (BF16, eight significant bits: 2^-8 each).
"""
import numpy as np
import pytest

from paper_2208_06097_amd import sea

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

KINDS = {"f64": (2.0 ** -53, 0.0), "f32": (2.0 ** -24, 0.0), "bf16": (2.0 ** -24, 2.0 ** -8)}
DTYPES = {"f64": (torch.float64, sea.SEA_F64), "f32": (torch.float32, sea.SEA_F32), "bf16": (torch.bfloat16, sea.SEA_BF16)}


def _ctx(kind):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return sea.Context(ace_dtype=DTYPES[kind][1])


@pytest.mark.parametrize("kind", list(KINDS))
@pytest.mark.parametrize("n_occ,n_vec,ng", [(1, 1, 7), (31, 33, 2049), (32, 64, 4099), (65, 96, 2500), (97, 129, 8193),
                                            (128, 160, 5001), (161, 20, 2048), (257, 300, 2177)])
def test_apply_at_tile_edges(kind, n_occ, n_vec, ng):
    u, ru = KINDS[kind]
    ctx = _ctx(kind)
    print(f"case ace apply {kind} {n_occ} x {n_vec} x {ng}", flush=True)
    g = torch.Generator().manual_seed(n_occ + n_vec)
    xi = torch.randn(n_occ, ng, generator=g, dtype=torch.float64).to(DTYPES[kind][0])
    psi = torch.randn(n_vec, ng, generator=g, dtype=torch.float64).to(DTYPES[kind][0])
    dV = 0.37
    got = ctx.ace_apply(xi.cuda(), psi.cuda(), dV).double().cpu()
    x, p = xi.double(), psi.double()
    want = -dV * (p @ x.T) @ x
    scale = dV * (p.abs() @ x.abs().T) @ x.abs()
    tol = (ng + n_occ + 8) * u + 2 * ru
    err = ((got - want).abs() / scale).max().item()
    ctx.close()
    assert err <= tol, (err, tol)


@pytest.mark.parametrize("kind", list(KINDS))
@pytest.mark.parametrize("n,ng", [(1, 9), (33, 517), (64, 1000), (97, 640), (128, 1153), (161, 2051), (257, 1931)])
def test_build_at_tile_edges(kind, n, ng):
    u, ru = KINDS[kind]
    ctx = _ctx(kind)
    print(f"case ace build {kind} {n} x {ng}", flush=True)
    g = torch.Generator().manual_seed(n)
    phi = torch.randn(n, ng, generator=g, dtype=torch.float64)
    W = phi + 0.01 * torch.randn(n, ng, generator=g, dtype=torch.float64)
    dV = 0.37
    M, L, xi, fp = ctx.ace_build(phi.cuda(), W.cuda(), dV)
    assert fp == 0
    M, L, xi = M.cpu(), L.cpu(), xi.double().cpu()
    err_m = ((M - dV * phi @ W.T).abs() / (dV * phi.abs() @ W.abs().T)).max().item()
    assert err_m <= (ng + 4) * 2.0 ** -53, err_m
    scale = L.abs() @ torch.linalg.inv(L).abs() @ W.abs()
    # the inverse's own residual is n 2^-53 |L||L^-1|; xi is stored in its kind
    tol = 4 * n * 2.0 ** -53 + (n + 4) * u + 4 * ru
    err = ((L @ xi - W).abs() / scale).max().item()
    ctx.close()
    assert err <= tol, (err, tol)
