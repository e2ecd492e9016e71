"""The autotuned FP32 CG and teams of workgroups: a tuned context keeps teams where
they are faster than the fastest variant alone, whichever that is; a choice restored
from the cache does the same as the one just made.

Eight pairs of 63^3 leave most of the chip idle in any one-workgroup variant (11 ms
for 40 iterations against 2), so teams are kept; their residuals, summed in another
order, differ from those of a variant by itself at some iteration.
"""
import numpy as np
import pytest

from paper_2208_06097_amd import sea, synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def test_tuned_context_keeps_teams(tmp_path):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print("case cg teams tuned", flush=True)
    cell = synth.mini(seed=5)
    phi = torch.from_numpy(cell.phi).cuda()
    pairs = np.zeros(8, dtype=sea.PAIR_DTYPE)
    n = np.array((63, 63, 63))
    for k in range(8):
        lo = np.floor(cell.centres[k % 4] / cell.h).astype(int) - n // 2
        pairs[k] = (k % 4, 4 + k % 3, lo, n, (lo + (n - 1) / 2 + 0.25) * cell.h)
    opts = dict(rel_tol=1e-8, stencil_dtype=sea.SEA_F32)
    cache = str(tmp_path / "tune.json")

    def solve(ctx):
        hist = ctx.residual_history(8, 600)
        _, E, stats, st = ctx.exx_action(phi, cell.N, cell.L, pairs)
        assert st == sea.SEA_OK and np.all(stats["converged"] == 1)
        return E, stats.copy(), hist.cpu().numpy()

    def same(a, b):
        return a[0] == b[0] and np.array_equal(a[1], b[1]) and np.array_equal(a[2], b[2], equal_nan=True)

    ctx = sea.Context(**opts)
    names = ctx.cg_variants()
    untuned = solve(ctx)
    for rep in range(2):
        c = sea.Context(**opts)
        res = c.autotune([(phi, cell.N, cell.L, pairs)], sample_pairs=8, iters=10, cache=cache)
        assert res["cached"] == (rep == 1) and res["teams"]
        assert same(solve(c), untuned)
        c.close()
    for variant in (res["variant"], next(v for v in names if v.endswith("-xc"))):
        ctx.set_opts(cg_variant=names.index(variant))
        alone = solve(ctx)
        assert not same(alone, untuned)
        ctx.cg_choice(variant, True)
        assert same(solve(ctx), untuned)
        ctx.cg_choice(variant, False)
        assert same(solve(ctx), alone)
    for variant, teams in ((-2, 1), (len(names), 1), (0, 2), (0, -1)):
        with pytest.raises(sea.SeaError):
            ctx._check(ctx.lib.sea_set_cg_choice(ctx.h, variant, teams))
    ctx.close()
