"""The autotuned FP32 CG and teams of workgroups: a tuned context keeps teams where
they are faster than the tuned variant, whichever that is; a choice restored from
the cache does the same as the one just made.

Eight pairs of 63^3 leave most of the chip idle in any one-workgroup variant (11 ms
for 40 iterations against 2), so teams solve them; their reported residuals, summed
in another order, differ from those of the variant by itself.
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
    cells = [(phi, cell.N, cell.L, pairs)]
    opts = dict(rel_tol=1e-8, stencil_dtype=sea.SEA_F32)
    cache = str(tmp_path / "tune.json")
    runs = []
    ctx = sea.Context(**opts)
    names = ctx.cg_variants()
    for rep in range(2):
        c = sea.Context(**opts)
        res = c.autotune(cells, sample_pairs=8, iters=10, cache=cache)
        assert res["cached"] == (rep == 1)
        _, E, stats, st = c.exx_action(phi, cell.N, cell.L, pairs)
        assert st == sea.SEA_OK and np.all(stats["converged"] == 1)
        runs.append((E, stats.copy()))
        c.close()
    assert runs[0][0] == runs[1][0] and np.array_equal(runs[0][1], runs[1][1])
    for variant in (res["variant"], next(v for v in names if v.endswith("-xc"))):
        ctx.set_opts(cg_variant=names.index(variant))
        _, _, alone, st = ctx.exx_action(phi, cell.N, cell.L, pairs)
        assert st == sea.SEA_OK
        ctx.cg_choice(variant, {names[0]: 1.0, variant: 0.8})
        _, E, stats, st = ctx.exx_action(phi, cell.N, cell.L, pairs)
        assert st == sea.SEA_OK
        assert np.array_equal(stats, runs[0][1]) and E == runs[0][0], variant
        assert not np.array_equal(stats["rel_res"], alone["rel_res"]), variant
    for variant, cost in ((0, 0.0), (0, 1.5), (0, float("nan")), (-1, 1.0), (len(names), 1.0)):
        with pytest.raises(sea.SeaError):
            ctx._check(ctx.lib.sea_set_cg_choice(ctx.h, variant, cost))
    ctx.close()
