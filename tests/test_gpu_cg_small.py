"""The FP64 CG on domains at the edges of the small form's workgroups (16 rows,
8 planes, blocks of 2048 points, rows of 29 points two to a wavefront) and of its
range (131072 points, 128 planes; the first sizes beyond it go the other way), all
in one call and each by itself.

Bars: the CG stops at 0.9 x rel_tol of |b|, so a potential is within cond(A)
rel_tol of the oracle's (1e-12 of its own): cond < 24000 for 129 points an axis.
A pair's result does not depend on its batch: bitwise equal.
"""
import numpy as np
import pytest

import oracle
from paper_2208_06097_amd import sea, synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

BOXES = [(1, 1, 1), (3, 5, 4), (16, 16, 8), (17, 15, 9), (29, 31, 16), (30, 33, 7), (64, 64, 32), (64, 64, 33),
         (10, 12, 128), (10, 12, 129), (29, 29, 29), (16, 16, 8), (64, 17, 60)]


@pytest.mark.parametrize("start", [sea.SEA_START_ZERO, sea.SEA_START_MULTIPOLE])
def test_small_domains_of_the_fp64_cg(start):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    cell = synth.mini(seed=5)
    rel_tol = 1e-10
    pairs = np.zeros(len(BOXES), dtype=sea.PAIR_DTYPE)
    for k, n in enumerate(BOXES):
        lo = np.floor(cell.centres[k % 3] / cell.h).astype(int) - np.array(n) // 2
        pairs[k] = (k % 3, 3 + k % 3, lo, n, (lo + (np.array(n) - 1) / 2 + 0.25) * cell.h)
    print(f"case cg small domains start {start}", flush=True)
    ctx = sea.Context(rel_tol=rel_tol, stencil_dtype=sea.SEA_F64, start=start)
    phi = torch.from_numpy(cell.phi).cuda()
    v, _, e, stats, st = ctx.pair_solve(phi, cell.N, cell.L, pairs)
    assert st == sea.SEA_OK and np.all(stats["converged"] == 1)
    v = v.cpu().numpy()
    pl = oracle.PairList(np.stack([pairs["i"], pairs["j"]], 1).astype(np.int32), pairs["lo"].astype(np.int32),
                         pairs["n"].astype(np.int32), pairs["origin"].copy())
    for k, n in enumerate(BOXES):
        ref, _, _ = oracle.pair_potential(cell.phi, cell.N, cell.L, pl, k, tol=1e-12)
        m = n[0] * n[1] * n[2]
        got = v[k, :m].reshape(ref.shape)
        rel = np.linalg.norm(got - ref) / np.linalg.norm(ref)
        print(f"box {n}: |dv|/|v| {rel:.2e} iters {stats['iters'][k]} rel_res {stats['rel_res'][k]:.2e}", flush=True)
        assert rel < 24000 * rel_tol
        v1, _, e1, s1, _ = ctx.pair_solve(phi, cell.N, cell.L, pairs[k:k + 1])
        assert np.array_equal(v1.cpu().numpy()[0, :m], v[k, :m]) and s1["iters"][0] == stats["iters"][k]
    ctx.close()
