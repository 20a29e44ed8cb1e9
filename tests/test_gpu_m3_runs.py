"""The M3 backward's units per wave (k_m3_bwd) follow the pack's size: 16 for
small packs, then 32, 64, 128 and, for batches of up to 64 samples, 256.  One
gradient step at a size of each, with runs that split models and models inside
one run, against the fp64 oracle on a sample of the models (they are
independent)."""
import numpy as np
import pytest

import pmlp_workloads as wl
from parity import dw2_terms, err_dw2, err_losses, err_rows

pytestmark = pytest.mark.gpu

TOL_STEP = 1e-5


@pytest.fixture(scope="module")
def torch():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    torch.cuda.set_device(0)
    return torch


@pytest.fixture(scope="module")
def pm(torch):
    import paper_2206_08369_amd as pm
    pm.load_library()
    return pm


# (units wanted, O, B): 16, 64, 128, 32, 64, 128, 256 and 256 units per wave; one
# and two passes over the batch, three to sixteen outputs (at sixteen, 256 units
# take all of the 64 KB of LDS that a launch has without asking)
@pytest.mark.parametrize("units,O,B", [(3000, 3, 260), (550000, 3, 270), (1100000, 4, 290),
                                       (130000, 3, 33), (250000, 10, 20), (500000, 16, 40),
                                       (1000000, 16, 9), (1000000, 3, 64)])
def test_units_per_wave(pm, orc, torch, units, O, B):
    F = 6 if O == 3 else 200   # (other outputs: past the fused backward's columns)
    rng = np.random.default_rng(units)
    hs = rng.integers(1, 300, units // 150).astype(np.int32)
    acts = rng.integers(0, 10, len(hs)).astype(np.int32)
    X, y = wl.make_dataset(F, O, B, seed=5)
    Xd, yd = torch.from_numpy(X).cuda(), torch.from_numpy(y).cuda()
    net = pm.PackedMLP(F, O, hs, acts, seed=3)
    W1, W2 = net.get_params()
    dW1, dW2 = (t.cpu().numpy() for t in net.gradients(Xd, yd))
    loss = net.losses()
    assert net.kernel_variants()["m3_bwd"][0] == "k_m3_bwd"
    off = np.concatenate([[0], np.cumsum(hs)])
    models = np.unique(np.linspace(0, len(hs) - 1, 20).astype(int))
    rows = np.concatenate([np.arange(off[m], off[m + 1]) for m in models])
    h, a, w1, w2 = hs[models], acts[models], W1[rows], W2[:, rows]
    r1, r2, rl, allow = orc.gradients(h, a, w1, w2, X, y)
    assert err_rows(dW1[rows], r1, h, allow).max() <= TOL_STEP
    assert err_dw2(dW2[:, rows], r2, h, dw2_terms(orc, h, a, w1, w2, X, y)).max() <= TOL_STEP
    assert err_losses(loss[models], rl).max() <= TOL_STEP
    net.close()
