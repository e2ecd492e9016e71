"""The FP32 CG by teams of workgroups: domains at the edges of its range (90000
points; up to 64 an axis; planes that fill the last workgroup's share or not),
next to domains that the one-workgroup form takes, more pairs than teams, each
pair by itself, and in a plan.

Bars: the FP64 residual is below 0.3 x rel_tol, so a potential is within cond(A)
rel_tol of the oracle's: cond < 6000 for 65 points an axis; the two forms (0.3 x
that each) are within the same of each other.  A pair's result does not depend on
its batch: bitwise equal.
"""
import numpy as np
import pytest

import oracle
from paper_2208_06097_amd import sea, synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

BOXES = [(64, 64, 22), (64, 64, 21), (45, 45, 45), (63, 63, 63), (64, 22, 64), (50, 61, 33), (64, 64, 65), (29, 29, 29)]


def _pairs(cell, boxes):
    pairs = np.zeros(len(boxes), dtype=sea.PAIR_DTYPE)
    for k, n in enumerate(boxes):
        lo = np.floor(cell.centres[k % 3] / cell.h).astype(int) - np.array(n) // 2
        pairs[k] = (k % 3, 3 + k % 3, lo, n, (lo + (np.array(n) - 1) / 2 + 0.25) * cell.h)
    return pairs


@pytest.mark.parametrize("start", [sea.SEA_START_ZERO, sea.SEA_START_MULTIPOLE])
def test_team_domains(start):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    cell = synth.mini(seed=5)
    rel_tol = 1e-9
    pairs = _pairs(cell, BOXES)
    print(f"case cg team domains start {start}", flush=True)
    phi = torch.from_numpy(cell.phi).cuda()
    ctx = sea.Context(rel_tol=rel_tol, stencil_dtype=sea.SEA_F32, start=start)
    v, _, e, stats, st = ctx.pair_solve(phi, cell.N, cell.L, pairs)
    assert st == sea.SEA_OK and np.all(stats["converged"] == 1)
    v = v.cpu().numpy()
    one = sea.Context(rel_tol=rel_tol, stencil_dtype=sea.SEA_F32, start=start, cg_variant=0)
    vo, _, eo, so, _ = one.pair_solve(phi, cell.N, cell.L, pairs)
    vo = vo.cpu().numpy()
    one.close()
    pl = oracle.PairList(np.stack([pairs["i"], pairs["j"]], 1).astype(np.int32), pairs["lo"].astype(np.int32),
                         pairs["n"].astype(np.int32), pairs["origin"].copy())
    for k, n in enumerate(BOXES):
        m = n[0] * n[1] * n[2]
        ref, _, _ = oracle.pair_potential(cell.phi, cell.N, cell.L, pl, k, tol=1e-11)
        got = v[k, :m].reshape(ref.shape)
        rel = np.linalg.norm(got - ref) / np.linalg.norm(ref)
        forms = np.linalg.norm(v[k, :m] - vo[k, :m]) / np.linalg.norm(ref)
        print(f"box {n}: |dv|/|v| {rel:.2e} forms {forms:.2e} iters {stats['iters'][k]}", flush=True)
        assert rel < 6000 * rel_tol
        assert forms < 6000 * rel_tol
        v1, _, e1, s1, _ = ctx.pair_solve(phi, cell.N, cell.L, pairs[k:k + 1])
        assert np.array_equal(v1.cpu().numpy()[0, :m], v[k, :m]) and s1[0] == stats[k]
    ctx.close()


def test_more_pairs_than_teams_and_plan():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    cell = synth.mini(seed=5)
    boxes = [((63, 63, 63), (50, 61, 33), (29, 29, 29), (64, 64, 22), (45, 45, 45))[k % 5] for k in range(75)]
    pairs = _pairs(cell, boxes)
    print("case cg team queue and plan", flush=True)
    phi = torch.from_numpy(cell.phi).cuda()
    ctx = sea.Context(rel_tol=1e-8, stencil_dtype=sea.SEA_F32)
    W, E, stats, st = ctx.exx_action(phi, cell.N, cell.L, pairs)
    assert st == sea.SEA_OK and np.all(stats["converged"] == 1)
    W = W.clone()
    for k in (0, 16, 44, 73):   # pairs of the same kind give the same result wherever they stand
        same = [q for q in range(75) if q % 15 == k % 15]
        assert all(stats[q]["iters"] == stats[same[0]]["iters"] for q in same)
        assert all(stats[q]["e_ij"] == stats[same[0]]["e_ij"] for q in same)
    plan = ctx.exx_plan([(phi, cell.N, cell.L, pairs)])
    for rep in range(3):
        plan.W[0].fill_(float("nan"))
        plan.launch()
        Ep, sp, st = plan.results()
        assert st == sea.SEA_OK and Ep[0] == E and np.array_equal(sp, stats), rep
        assert torch.equal(plan.W[0], W), rep
        W2, E2, s2, _ = ctx.exx_action(phi, cell.N, cell.L, pairs)   # eager work between the replays
        assert E2 == E and torch.equal(W2, W)
    plan.close()
    ctx.close()
