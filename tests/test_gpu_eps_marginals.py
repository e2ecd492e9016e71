"""Boxes of the epsilon rule on grids where the marginal pass ends raggedly
(rows longer than one sweep of 128 points, planes not a multiple of its groups
of eight, rows fewer than its wavefronts), against the oracle's boxes: the
self pairs' unpadded boxes are the orbital boxes, integers equal."""
import numpy as np
import pytest
import torch

import oracle
from paper_2208_06097_amd import sea

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N", [(130, 7, 9), (64, 33, 8), (257, 3, 17), (5, 12, 1)])
@pytest.mark.parametrize("dtype", [np.float64, np.float32])
def test_self_boxes_on_ragged_grids(N, dtype):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    rng = np.random.default_rng(sum(N))
    n_occ = 3
    phi = np.empty((n_occ, N[2], N[1], N[0]))
    for i in range(n_occ):
        ax = []
        for n in N:
            d = np.arange(n) - rng.uniform(0, n)
            d -= n * np.round(d / n)
            ax.append(np.exp(-d * d / (2 * (0.06 * n + 0.4) ** 2)))
        phi[i] = ax[2][:, None, None] * ax[1][None, :, None] * ax[0] * (1 + 0.1 * rng.standard_normal(phi.shape[1:]))
    phi = phi.astype(dtype)
    print(f"case eps marginals N={N} {dtype.__name__}", flush=True)
    lo, ln = oracle.eps_boxes(phi.astype(np.float64), N, 1e-3)
    ctx = sea.Context()
    p, _ = ctx.build_pairs_eps(torch.from_numpy(phi).cuda(), N, [0.2 * n for n in N], 1e-3, 0.0)
    ctx.close()
    own = p[p["i"] == p["j"]]
    assert len(own) == n_occ
    assert np.array_equal(own["n"], ln)
    assert np.array_equal(own["lo"] % np.array(N), lo % np.array(N))
