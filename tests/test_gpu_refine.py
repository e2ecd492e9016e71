"""The exact correction after the spectral start (x += A^-1 (b - A x) by the
stencil matrix's own eigenvectors) on domains at the edges of its tiles: axes
shorter than the stencil, one below, at and above the 16- and 32-point blocks,
and the longest, odd and even, square and not.

Bars: the corrections end at the rounding of b - A x, whose terms are the
stencil's (|A| |x| <= 12.9 / h^2 |x|, and |b| >= lambda_min |x|): a relative
residual of 2^-53 x cond(A) < 1e-12 for 64 points (cond < 5300), so a tolerance
of 1e-12 is met.  The oracle's CG at 1e-12 is within cond(A) x 1e-12 of the
solution: potentials to 1e-8.
"""
import numpy as np
import pytest

import oracle
from paper_2208_06097_amd import sea, synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

BOXES = [(3, 5, 4), (1, 7, 12), (15, 16, 17), (31, 32, 33), (32, 32, 31), (47, 48, 49), (64, 10, 63), (63, 63, 16),
         (20, 64, 64)]


@pytest.mark.parametrize("state", ["f64", "f32"])
def test_corrected_potentials_on_tile_edges(state):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    cell = synth.mini(seed=7)
    n_pairs = len(BOXES)
    pairs = np.zeros(n_pairs, dtype=sea.PAIR_DTYPE)
    for k, n in enumerate(BOXES):
        lo = np.floor(cell.centres[k % 3] / cell.h).astype(int) - np.array(n) // 2
        pairs[k] = (k % 3, 3 + k % 3, lo, n, (lo + (np.array(n) - 1) / 2 + 0.25) * cell.h)
    print(f"case refine boxes {state}", flush=True)
    ctx = sea.Context(rel_tol=1e-12, stencil_dtype=sea.SEA_F64 if state == "f64" else sea.SEA_F32,
                      start=sea.SEA_START_SPECTRAL)
    v, _, e, stats, st = ctx.pair_solve(torch.from_numpy(cell.phi).cuda(), cell.N, cell.L, pairs)
    ctx.close()
    assert st == sea.SEA_OK and np.all(stats["converged"] == 1)
    assert stats["iters"].max() >= 1
    assert np.all(stats["rel_res"] <= 1e-12)
    pl = oracle.PairList(np.stack([pairs["i"], pairs["j"]], 1).astype(np.int32), pairs["lo"].astype(np.int32),
                         pairs["n"].astype(np.int32), pairs["origin"].copy())
    v = v.cpu().numpy()
    for k, n in enumerate(BOXES):
        ref, _, info = oracle.pair_potential(cell.phi, cell.N, cell.L, pl, k, tol=1e-12)
        got = v[k, :n[0] * n[1] * n[2]].reshape(ref.shape)
        rel = np.linalg.norm(got - ref) / np.linalg.norm(ref)
        print(f"box {n}: |dv|/|v| {rel:.2e} iters {stats['iters'][k]} rel_res {stats['rel_res'][k]:.2e}", flush=True)
        assert rel < 1e-8
