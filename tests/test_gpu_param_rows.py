"""Parameters to and from the host: packed rows through the staging buffer
(rows narrower than their stride, in one piece and in several), contiguous
rows, wide rows, and the one-column bias rows.  Values written come back bit
for bit, and the padding between rows stays what training needs it to be: a
forward pass and a gradient step after parameters were set equal the oracle's."""
import numpy as np
import pytest

import pmlp_workloads as wl
from parity import err_logits, err_losses, err_rows

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pm():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    torch.cuda.set_device(0)
    import paper_2206_08369_amd as pm
    pm.load_library()
    return pm


# (F, units, biases): 4-byte and 200-byte rows in one piece, rows of 50
# floats in two pieces (4.6 million floats), rows without padding, and W2 rows
# above 64 KiB
@pytest.mark.parametrize("F,units,biases", [(1, 77, False), (50, 300, True), (50, 92000, False),
                                            (8, 500, False), (3, 20000, True)])
def test_round_trip(pm, F, units, biases):
    rng = np.random.default_rng(F * units)
    hs = np.full(max(units // 20, 1), 20, np.int32)
    N, O = int(hs.sum()), 3
    W1 = rng.standard_normal((N, F)).astype(np.float32)
    W2 = rng.standard_normal((O, N)).astype(np.float32)
    net = pm.PackedMLP(F, O, hs, np.zeros(len(hs), np.int32), seed=1, biases=biases)
    if biases:
        b1, b2 = net.get_biases()
        n1 = rng.standard_normal(N).astype(np.float32)
        net.set_biases(n1, b2)
    net.set_params(W1, W2)
    g1, g2 = net.get_params()
    assert np.array_equal(g1, W1) and np.array_equal(g2, W2)
    if biases:
        c1, c2 = net.get_biases()
        assert np.array_equal(c1, n1) and np.array_equal(c2, b2)
    m1, m2 = net.get_models([len(hs) - 1, 0])
    assert np.array_equal(m1[:20], W1[-20:]) and np.array_equal(m2[:, 20:], W2[:, :20])
    net.close()


def test_two_layer_round_trip(pm):
    rng = np.random.default_rng(7)
    h1, h2 = rng.integers(1, 40, 60).astype(np.int32), rng.integers(1, 40, 60).astype(np.int32)
    net = pm.DeepPackedMLP(5, 2, h1, h2, np.arange(60, dtype=np.int32) % 10, seed=1)
    W = [rng.standard_normal(a.shape).astype(np.float32) for a in net.get_params()]
    net.set_params(*W)
    for a, b in zip(net.get_params(), W):
        assert np.array_equal(a, b)
    net.close()


@pytest.mark.parametrize("F,biases", [(1, False), (3, True), (50, False), (50, True), (150, False)])
def test_padding_between_rows(pm, orc, F, biases):
    import torch
    rng = np.random.default_rng(F)
    hs = rng.integers(1, 60, 50).astype(np.int32)
    acts = (np.arange(50) % 10).astype(np.int32)
    N, O, B = int(hs.sum()), 3, 140
    X, y = wl.make_dataset(F, O, B, seed=F)
    net = pm.PackedMLP(F, O, hs, acts, seed=2, biases=biases)
    for _ in range(2):                      # the second time over used rows
        W1 = rng.uniform(-0.5, 0.5, (N, F)).astype(np.float32)
        W2 = rng.uniform(-0.5, 0.5, (O, N)).astype(np.float32)
        kw = {}
        net.set_params(W1, W2)
        if biases:
            kw = dict(b1=rng.uniform(-0.5, 0.5, N).astype(np.float32),
                      b2=rng.uniform(-0.5, 0.5, (50, O)).astype(np.float32))
            net.set_biases(kw["b1"], kw["b2"])
        Xd, yd = torch.from_numpy(X).cuda(), torch.from_numpy(y).cuda()
        got = net.forward(Xd).cpu().numpy()
        assert err_logits(got, orc.forward(hs, acts, W1, W2, X, **kw)).max() <= 1e-5
        g1 = net.gradients(Xd, yd)[0].cpu().numpy()
        ref = orc.gradients(hs, acts, W1, W2, X, y, **kw)
        assert err_rows(g1, ref[0], hs, ref[3]).max() <= 1e-5
        assert err_losses(net.losses(), ref[2]).max() <= 1e-5
    net.close()
