"""Which pairs the FP32 CG gives to teams: by their domain alone, so that a pair's
result is the same bit for bit in a list of any length.  The two forms add their FP64
sums in another order, which the residual history shows at some iteration.
"""
import numpy as np
import pytest

from paper_2208_06097_amd import sea, synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

# on either side of the line, and a domain with many points and few planes
BOXES = {(44, 44, 45): False, (45, 45, 45): True, (64, 64, 51): False, (64, 64, 52): True, (64, 64, 31): False,
         (48, 48, 45): False, (64, 22, 64): True, (64, 21, 64): False}


def _pairs(cell, boxes):
    pairs = np.zeros(len(boxes), dtype=sea.PAIR_DTYPE)
    for k, n in enumerate(boxes):
        lo = np.floor(cell.centres[k % 3] / cell.h).astype(int) - np.array(n) // 2
        pairs[k] = (k % 3, 3 + k % 3, lo, n, (lo + (np.array(n) - 1) / 2 + 0.25) * cell.h)
    return pairs


def test_line_between_teams_and_one_workgroup():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print("case cg team rule", flush=True)
    cell = synth.mini(seed=5)
    phi = torch.from_numpy(cell.phi).cuda()
    m, reps = len(BOXES), 36                     # 36 x 8 pairs: a multiple of the three orbital pairs
    pairs = _pairs(cell, list(BOXES) * reps)
    hist, stats = {}, {}
    for v, n in ((-1, m), (-1, m * reps), (0, m)):
        ctx = sea.Context(rel_tol=1e-6, stencil_dtype=sea.SEA_F32, cg_variant=v)
        h = ctx.residual_history(n, 500)
        _, _, s, st = ctx.exx_action(phi, cell.N, cell.L, pairs[:n])
        assert st == sea.SEA_OK and np.all(s["converged"] == 1)
        hist[v, n], stats[v, n] = h.cpu().numpy(), s
        ctx.close()
    for k, (box, team) in enumerate(BOXES.items()):
        assert np.array_equal(hist[-1, m][k], hist[0, m][k], equal_nan=True) != team, box
    assert np.array_equal(hist[-1, m * reps][:m], hist[-1, m], equal_nan=True)
    assert np.array_equal(stats[-1, m * reps][:m], stats[-1, m])
    for q in range(0, m * reps, 3 * m):          # and in every place of the list
        assert np.array_equal(stats[-1, m * reps][q:q + m], stats[-1, m])
