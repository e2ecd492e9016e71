"""FP64 CG calls that mix small domains with larger ones, whose loops run side by
side: every pair's result is the one it has in a call by itself, bit for bit, also
where the iterations run out, on a stream of the caller's, call after call on one
workspace, and from two threads at once.
"""
import threading

import numpy as np
import pytest

from paper_2208_06097_amd import sea, synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

BOXES = [(63, 63, 63), (29, 29, 29), (21, 33, 40), (64, 50, 48), (9, 60, 30), (50, 50, 50), (31, 31, 31)]


def _case():
    cell = synth.mini(seed=5)
    pairs = np.zeros(len(BOXES), dtype=sea.PAIR_DTYPE)
    for k, n in enumerate(BOXES):
        lo = np.floor(cell.centres[k % 3] / cell.h).astype(int) - np.array(n) // 2
        pairs[k] = (k % 3, 3 + k % 3, lo, n, (lo + (np.array(n) - 1) / 2 + 0.25) * cell.h)
    return cell, torch.from_numpy(cell.phi).cuda(), pairs


@pytest.mark.parametrize("max_iter", [0, 1, 15, 16, 17, 2000])
def test_mixed_calls_match_single_pairs(max_iter):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"case cg mixed max_iter {max_iter}", flush=True)
    cell, phi, pairs = _case()
    stream = torch.cuda.Stream()
    stream.wait_stream(torch.cuda.current_stream())
    for s in (None, stream):
        ctx = sea.Context(rel_tol=1e-9, stencil_dtype=sea.SEA_F64, max_iter=max_iter, stream=s)
        with torch.cuda.stream(s if s is not None else torch.cuda.current_stream()):
            v, _, _, stats, st = ctx.pair_solve(phi, cell.N, cell.L, pairs)
            total = v.double().sum()      # on the call's stream, right behind it
            assert np.all(stats["converged"] == (1 if max_iter == 2000 else 0))
            for k, n in enumerate(BOXES):
                m = n[0] * n[1] * n[2]
                v1, _, _, s1, _ = ctx.pair_solve(phi, cell.N, cell.L, pairs[k:k + 1])
                assert torch.equal(v1[0, :m], v[k, :m]) and s1[0] == stats[k], (s is None, n)
            assert float(total) == float(v.double().sum())
        torch.cuda.synchronize()
        ctx.close()


def test_mixed_calls_from_two_threads():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print("case cg mixed, two threads", flush=True)
    cell, phi, pairs = _case()
    ref = sea.Context(rel_tol=1e-9, stencil_dtype=sea.SEA_F64)
    W0, E0, s0, _ = ref.exx_action(phi, cell.N, cell.L, pairs)
    torch.cuda.synchronize()
    ref.close()
    streams = [torch.cuda.Stream() for _ in range(2)]
    ctxs = [sea.Context(rel_tol=1e-9, stencil_dtype=sea.SEA_F64, stream=s) for s in streams]
    wss = [c.workspace(c.exx_workspace_bytes(cell.N, cell.L, cell.phi.shape[0], pairs)) for c in ctxs]
    Ws = [torch.empty_like(W0) for _ in range(2)]
    torch.cuda.synchronize()
    out = [[], []]

    def work(q):
        for _ in range(3):
            _, E, stats, _ = ctxs[q].exx_action(phi, cell.N, cell.L, pairs, ws=wss[q], W=Ws[q])
            out[q].append((E, stats.copy()))

    th = [threading.Thread(target=work, args=(q,)) for q in range(2)]
    for t in th:
        t.start()
    for t in th:
        t.join()
    torch.cuda.synchronize()
    for q in range(2):
        assert len(out[q]) == 3
        for E, stats in out[q]:
            assert E == E0 and np.array_equal(stats, s0)
        assert torch.equal(Ws[q], W0)
        ctxs[q].close()
