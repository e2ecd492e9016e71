"""The FP32 network's tiled kernels (forward, input and weight gradients) at
the grid sizes where their tiles end raggedly, against the FP64 oracle.

Biases of +-4 on small weights keep every activation far from the ReLU's
kink, so the oracle and the GPU agree on every mask and the bar is rounding
alone: a layer sums at most 864 products in FP32, a relative error of at most
864 x 2^-24 = 5e-5.
"""
import numpy as np
import pytest
import torch

from oracle import nn
from paper_2208_06097_amd import sea

pytestmark = pytest.mark.gpu
BAR = 864 * 2.0 ** -24


def _rel(a, b):
    return float(np.linalg.norm(np.ravel(a - b)) / max(np.linalg.norm(np.ravel(b)), 1e-300))


# 8: levels of 8, 4, 2 and 1 voxels; 24: rows of 24, 12, 6, 3 (not a multiple
# of four); 40: rows split in two tiles of 20
@pytest.mark.parametrize("D,batch", [(8, 1), (8, 3), (24, 2), (40, 1)])
def test_forward_and_gradient_on_ragged_tiles(D, batch):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    rng = np.random.default_rng(100 + D + batch)
    p = nn.init_params(D)
    for name, _, co, _ in nn.LAYERS:
        p[name + ".w"] *= 0.1
        p[name + ".b"] = np.where(np.arange(co) % 4 == 1, -4.0, 4.0)
    p = {k: v.astype(np.float32).astype(np.float64) for k, v in p.items()}
    x = np.clip(rng.standard_normal((batch, 1, D, D, D)), -3, 3).astype(np.float32).astype(np.float64)
    t = rng.standard_normal(x.shape).astype(np.float32).astype(np.float64)
    yo, act = nn.forward(p, x)
    for name, _, _, relu in nn.LAYERS:
        if relu:
            z = nn.conv3d(act[name + ".in"], p[name + ".w"], p[name + ".b"])
            assert np.min(np.abs(z)) > 0.05, name   # no mask within rounding of its kink
    Lo, gy = nn.mse(yo, t)
    go = nn.backward(p, act, gy)
    print(f"case nn tiles D={D} batch={batch}", flush=True)
    ctx = sea.Context(nn_weight_dtype=sea.SEA_F32)
    st = ctx.nn_state(sea.nn_pack(p))
    xd = torch.from_numpy(x[:, 0].astype(np.float32)).cuda()
    td = torch.from_numpy(t[:, 0].astype(np.float32)).cuda()
    y = ctx.nn_forward(st, xd).cpu().numpy()
    grad = torch.full((ctx.nn_param_count(),), float("nan"), dtype=torch.float32, device="cuda")
    loss = ctx.nn_train_step(st, xd, td, 1e-3, 1, grad=grad)
    ctx.close()
    assert _rel(y, yo[:, 0]) < BAR
    assert abs(loss / Lo - 1) < BAR
    gg = sea.nn_unpack(grad.cpu().numpy())
    for name, _, _, _ in nn.LAYERS:
        for sfx in (".w", ".b"):
            g, w = gg[name + sfx], go[name + sfx]
            assert np.all(g[w == 0.0] == 0.0), (name, sfx)
            assert _rel(g, w) < BAR, (name, sfx)
