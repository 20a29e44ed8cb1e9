"""The hidden-to-hidden kernels of two-layer packs (k_seg_fwd, k_seg_grad,
k_seg_back) at the edges of their tiles: widths of 1, just below, at and
above 16 rows, 16-unit passes and 64 columns, in batches of one, two and four
16-sample blocks per wave and one whose last wave is partly past the batch;
gradients of every model against the fp64 oracle (per-model normwise 1e-5,
the oracle's allowances for kink ties as in the other two-layer tests)."""
import numpy as np
import pytest

import pmlp_workloads as wl
from parity import err_dw2, err_logits, err_losses, err_rows
from test_gpu_deep import dev, err_blocks, pm, torch  # noqa: F401

pytestmark = pytest.mark.gpu

TOL_STEP = 1e-5
WIDTHS = [1, 2, 15, 16, 17, 31, 32, 33, 48, 63, 64, 65, 100, 130]


@pytest.mark.parametrize("B", [9, 25, 64, 300])
def test_tile_edges(pm, orc, torch, B):  # noqa: F811
    h1 = np.array([w for w in WIDTHS for _ in range(3)], np.int32)
    h2 = np.array([WIDTHS[(5 * i + 3 * k) % len(WIDTHS)] for i in range(len(WIDTHS))
                   for k in range(3)], np.int32)
    acts = (np.arange(len(h1)) % 10).astype(np.int32)
    F, O = 7, 2
    X, y = wl.make_dataset(F, O, B, seed=31 + B)
    net = pm.DeepPackedMLP(F, O, h1, h2, acts, seed=6)
    W1, W12, W2 = net.get_params()
    Xd, yd = dev(torch, X), dev(torch, y)
    got = net.forward(Xd).cpu().numpy()
    assert err_logits(got, orc.deep_forward(h1, h2, acts, W1, W12, W2, X)).max() <= TOL_STEP
    g1, g12, g2 = (t.cpu().numpy() for t in net.gradients(Xd, yd))
    r1, r12, r2, rl, a1, a12 = orc.deep_gradients(h1, h2, acts, W1, W12, W2, X, y)[:6]
    assert err_rows(g1, r1, h1, a1).max() <= TOL_STEP
    assert err_blocks(g12, r12, h1, h2, a12).max() <= TOL_STEP
    # dW2 = G^T H2 cancels across samples, so its error is taken relative to
    # sum_b |G| |H2|, as for one hidden layer
    L = orc.deep_forward(h1, h2, acts, W1, W12, W2, X)
    P = np.exp(L - L.max(axis=2, keepdims=True))
    P /= P.sum(axis=2, keepdims=True)
    P[np.arange(B), :, y] -= 1.0
    _, H1 = orc.hidden(h1, acts, W1, X)
    o1, o2 = np.concatenate([[0], np.cumsum(h1)]), np.concatenate([[0], np.cumsum(h2)])
    ko = np.concatenate([[0], np.cumsum(h1 * h2)])
    terms = np.empty_like(r2)
    for m in range(len(h1)):
        W = W12[ko[m]:ko[m + 1]].reshape(h2[m], h1[m])
        _, H2 = orc.hidden(h2[m:m + 1], acts[m:m + 1], W, H1[:, o1[m]:o1[m + 1]])
        terms[:, o2[m]:o2[m + 1]] = np.abs(P[:, m]).T @ np.abs(H2) / B
    assert err_dw2(g2, r2, h2, terms).max() <= TOL_STEP
    assert err_losses(net.losses(), rl).max() <= TOL_STEP
    net.close()
