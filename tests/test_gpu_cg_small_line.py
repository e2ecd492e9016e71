"""The FP64 CG on either side of the line between the small form and the row tiles
that its planes draw: 64 x 44 points with at most 48 rows, 33 x 64 with more; all in
one call and each by itself.

Bars: the CG stops at 0.9 x rel_tol of |b|, so a potential is within cond(A)
rel_tol of the oracle's (1e-12 of its own): cond < 6000 for 65 points an axis.  A
pair's result does not depend on its batch: bitwise equal.
"""
import numpy as np
import pytest

import oracle
from paper_2208_06097_amd import sea, synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

BOXES = [(64, 44, 46), (64, 45, 17), (58, 48, 16), (59, 48, 16), (43, 49, 15), (44, 49, 15), (33, 64, 62), (34, 64, 9),
         (47, 47, 47), (49, 49, 49)]


def test_line_of_the_small_fp64_form():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print("case cg small line", flush=True)
    cell = synth.mini(seed=5)
    rel_tol = 1e-10
    pairs = np.zeros(len(BOXES), dtype=sea.PAIR_DTYPE)
    for k, n in enumerate(BOXES):
        lo = np.floor(cell.centres[k % 3] / cell.h).astype(int) - np.array(n) // 2
        pairs[k] = (k % 3, 3 + k % 3, lo, n, (lo + (np.array(n) - 1) / 2 + 0.25) * cell.h)
    ctx = sea.Context(rel_tol=rel_tol, stencil_dtype=sea.SEA_F64)
    phi = torch.from_numpy(cell.phi).cuda()
    v, _, e, stats, st = ctx.pair_solve(phi, cell.N, cell.L, pairs)
    assert st == sea.SEA_OK and np.all(stats["converged"] == 1)
    v = v.cpu().numpy()
    pl = oracle.PairList(np.stack([pairs["i"], pairs["j"]], 1).astype(np.int32), pairs["lo"].astype(np.int32),
                         pairs["n"].astype(np.int32), pairs["origin"].copy())
    for k, n in enumerate(BOXES):
        ref, _, _ = oracle.pair_potential(cell.phi, cell.N, cell.L, pl, k, tol=1e-12)
        m = n[0] * n[1] * n[2]
        rel = np.linalg.norm(v[k, :m].reshape(ref.shape) - ref) / np.linalg.norm(ref)
        print(f"box {n}: |dv|/|v| {rel:.2e} iters {stats['iters'][k]}", flush=True)
        assert rel < 6000 * rel_tol
        v1, _, e1, s1, _ = ctx.pair_solve(phi, cell.N, cell.L, pairs[k:k + 1])
        assert np.array_equal(v1.cpu().numpy()[0, :m], v[k, :m]) and s1[0] == stats[k]
    ctx.close()
