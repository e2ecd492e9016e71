"""W on boxes at the edges of the scatter's branches: domains wider than the
cell (one and two images, on one axis and on all, odd and even), boxes beyond
their domain (multipole values outside it) up to the whole cell, and tiles that
more pairs reach than one load of the coefficient table holds (12), against the
oracle.

Bars: both sides solve to a relative residual of 1e-12, so potentials agree to
cond(A) 1e-12 <= 1e-8 (64 points an axis: cond < 5300), and W and E with them.
"""
import numpy as np
import pytest

import oracle
from paper_2208_06097_amd import sea, synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

CASES = {
    "wide by one": dict(n=(31, 31, 31)),
    "two images of one axis": dict(n=(20, 62, 9)),
    "three images of two axes": dict(n=(64, 16, 63)),
    "as wide as the cell": dict(n=(30, 30, 30)),
    "reaching": dict(n=(10, 12, 9), grow=(5, 6, 3)),
    "reaching the cell": dict(n=(10, 11, 12), grow=(20, 19, 18)),
    "reaching on one axis": dict(n=(16, 16, 17), grow=(0, 0, 13)),
}


@pytest.mark.parametrize("state", ["f64", "f32"])
@pytest.mark.parametrize("name", list(CASES))
def test_w_on_box_edges(name, state):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    n = np.array(CASES[name]["n"])
    grow = CASES[name].get("grow")
    cell = synth.mini(seed=11)
    no = cell.phi.shape[0]
    pairs = np.zeros(no * (no + 1) // 2, dtype=sea.PAIR_DTYPE)
    dbox = np.zeros((len(pairs), 12), np.int32)
    k = 0
    for i in range(no):
        for j in range(i, no):
            lo = np.floor(cell.centres[i] / cell.h).astype(int) - n // 2 + (j - i) % 3
            pairs[k] = (i, j, lo, n, (lo + (n - 1) / 2) * cell.h)
            if grow is not None:   # W_i: before the domain, W_j: behind it
                g = np.array(grow)
                dbox[k] = np.concatenate([lo - g, n + g, lo, n + g])
            k += 1
    print(f"case scatter {name} {state}", flush=True)
    ctx = sea.Context(rel_tol=1e-12, stencil_dtype=sea.SEA_F64 if state == "f64" else sea.SEA_F32,
                      start=sea.SEA_START_SPECTRAL)
    db = None if grow is None else dbox
    W, E, stats, st = ctx.exx_action(torch.from_numpy(cell.phi).cuda(), cell.N, cell.L, pairs, dbox=db)
    W = W.cpu().numpy()
    ctx.close()
    assert st == sea.SEA_OK and np.all(stats["converged"] == 1)
    pl = oracle.PairList(np.stack([pairs["i"], pairs["j"]], 1).astype(np.int32), pairs["lo"].astype(np.int32),
                         pairs["n"].astype(np.int32), pairs["origin"].copy())
    ref = oracle.exx(cell.phi, cell.N, cell.L, pl, tol=1e-12, dbox=db)
    rel = np.linalg.norm(W - ref.W) / np.linalg.norm(ref.W)
    worst = np.abs(W - ref.W).max() / np.abs(ref.W).max()
    print(f"{name} {state}: |dW|/|W| {rel:.2e} worst {worst:.2e} dE {abs(E - ref.E) / abs(ref.E):.2e}", flush=True)
    assert rel < 1e-8 and worst < 1e-8
    assert abs(E - ref.E) < 1e-8 * abs(ref.E)
