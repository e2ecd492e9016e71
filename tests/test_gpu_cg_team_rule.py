"""Which pairs the FP32 CG gives to teams: by their planes and the length of the
list.  The two forms add their FP64 sums in another order, so the reported residual
says which one solved a pair: the one-workgroup form's is reproduced bit for bit,
and over a dozen pairs a team's is not.
"""
import numpy as np
import pytest

from paper_2208_06097_amd import sea, synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _pairs(cell, boxes):
    pairs = np.zeros(len(boxes), dtype=sea.PAIR_DTYPE)
    for k, n in enumerate(boxes):
        lo = np.floor(cell.centres[k % 3] / cell.h).astype(int) - np.array(n) // 2
        pairs[k] = (k % 3, 3 + k % 3, lo, n, (lo + (np.array(n) - 1) / 2 + 0.25) * cell.h)
    return pairs


# planes taken by teams at each length: 12 pairs from 5 on, 270 from 37, 600 from 47
@pytest.mark.parametrize("n_pairs,planes", [(12, {22: True, 48: True, 64: True}),
                                            (270, {31: False, 40: True, 64: True}),
                                            (600, {22: False, 44: False, 53: True})])
def test_line_between_teams_and_one_workgroup(n_pairs, planes):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"case cg team rule {n_pairs}", flush=True)
    cell = synth.mini(seed=5)
    phi = torch.from_numpy(cell.phi).cuda()
    nzs = list(planes)
    boxes = [(64, 64, nzs[k % len(nzs)]) for k in range(n_pairs)]
    pairs = _pairs(cell, boxes)
    rel = {}
    for v in (-1, 0):
        ctx = sea.Context(rel_tol=1e-6, stencil_dtype=sea.SEA_F32, cg_variant=v)
        _, _, stats, st = ctx.exx_action(phi, cell.N, cell.L, pairs)
        assert st == sea.SEA_OK and np.all(stats["converged"] == 1)
        rel[v] = stats["rel_res"]
        ctx.close()
    for q, nz in enumerate(nzs):
        same = np.array_equal(rel[-1][q::len(nzs)], rel[0][q::len(nzs)])
        assert same != planes[nz], (n_pairs, nz)
