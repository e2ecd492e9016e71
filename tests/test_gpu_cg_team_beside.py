"""FP32 CG calls with few pairs for teams, which run beside the z-march of the others:
every pair's result is the one it has in a call by itself, and the plan's (where the
z-march goes behind the teams), bit for bit; at the numbers of pairs where the room
beside the teams ends, on a stream of the caller's, call after call on one workspace.
"""
import numpy as np
import pytest

from paper_2208_06097_amd import sea, synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

LARGE, SMALL = [(63, 63, 63), (64, 64, 52), (47, 50, 48)], [(29, 29, 29), (44, 44, 44), (11, 64, 64), (64, 64, 20)]


# 256 CUs: beside 1 to 8 teams 192 others have a CU each, beside 9 to 16 teams 128,
# beside 17 to 24 teams 64, beside more none
@pytest.mark.parametrize("large,small", [(1, 1), (3, 40), (8, 192), (8, 193), (9, 128), (9, 129), (24, 64), (25, 4)])
def test_teams_beside_the_others(large, small):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"case cg teams beside {large} {small}", flush=True)
    cell = synth.mini(seed=5)
    phi = torch.from_numpy(cell.phi).cuda()
    boxes = [SMALL[k % 4] for k in range(small)]
    for k in range(large):   # in between
        boxes.insert(min(3 * k, len(boxes)), LARGE[k % 3])
    pairs = np.zeros(len(boxes), dtype=sea.PAIR_DTYPE)
    seen = {}
    for k, n in enumerate(boxes):
        q = seen.setdefault(n, len(seen)) % 3
        lo = np.floor(cell.centres[q] / cell.h).astype(int) - np.array(n) // 2
        pairs[k] = (q, 3 + q, lo, n, (lo + (np.array(n) - 1) / 2 + 0.25) * cell.h)
    stream = torch.cuda.Stream()
    stream.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(stream):
        ctx = sea.Context(rel_tol=1e-7, stencil_dtype=sea.SEA_F32)
        alone = {}
        for n in seen:
            k = boxes.index(n)
            _, _, s1, _ = ctx.exx_action(phi, cell.N, cell.L, pairs[k:k + 1])
            alone[n] = s1[0]
        ws = ctx.workspace(ctx.exx_workspace_bytes(cell.N, cell.L, cell.phi.shape[0], pairs))
        ref = None
        for rep in range(2):
            W, E, stats, st = ctx.exx_action(phi, cell.N, cell.L, pairs, ws=ws)
            total = W.sum()   # on the call's stream, right behind it
            assert st == sea.SEA_OK and np.all(stats["converged"] == 1)
            for k, n in enumerate(boxes):
                assert stats[k] == alone[n], (rep, k, n)
            if ref is not None:
                assert torch.equal(W, ref[0]) and E == ref[1]
            assert float(total) == float(W.sum())
            ref = (W.clone(), E)
        plan = ctx.exx_plan([(phi, cell.N, cell.L, pairs)])
        plan.launch(stream)
        Ep, sp, st = plan.results()
        assert st == sea.SEA_OK and Ep[0] == ref[1] and np.array_equal(sp, stats) and torch.equal(plan.W[0], ref[0])
        plan.close()
        torch.cuda.synchronize()
        ctx.close()
