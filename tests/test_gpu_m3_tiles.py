"""The M3 forward's tiles: a small pack of up to 1,024 models has one model a
tile, a larger one several.  A model's sums do not depend on it: the same
models alone and in front of others give the same losses and gradients, bit
for bit (two to sixteen outputs, whole models and split ones)."""
import numpy as np
import pytest

from test_gpu_m3_runs import pm, torch  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("O,B", [(2, 32), (4, 9), (10, 32), (2, 260)])
def test_sums_do_not_depend_on_the_tiles(pm, torch, O, B):  # noqa: F811
    rng = np.random.default_rng(B + O)
    M, F = 1024, 9
    hs = rng.integers(1, 40, M + 1).astype(np.int32)
    hs[-1] = 7
    acts = rng.integers(0, 10, M + 1).astype(np.int32)
    n = int(hs.sum())
    W1 = rng.uniform(-0.3, 0.3, (n, F)).astype(np.float32)
    W2 = rng.uniform(-0.3, 0.3, (O, n)).astype(np.float32)
    X = torch.from_numpy(rng.standard_normal((B, F)).astype(np.float32)).cuda()
    y = torch.from_numpy(rng.integers(0, O, B).astype(np.int32)).cuda()
    got = []
    for m in (M, M + 1):
        k = int(hs[:m].sum())
        net = pm.PackedMLP(F, O, hs[:m], acts[:m], seed=1)
        net.set_params(W1[:k], np.ascontiguousarray(W2[:, :k]))
        dW1, dW2 = net.gradients(X, y)
        got.append((net.losses()[:M], dW1.cpu().numpy(), dW2.cpu().numpy()))
        net.close()
    k = int(hs[:M].sum())
    assert np.array_equal(got[0][0], got[1][0])
    assert np.array_equal(got[0][1], got[1][1][:k])
    assert np.array_equal(got[0][2], got[1][2][:, :k])


@pytest.mark.parametrize("deep", [False, True])
def test_tiles_of_large_forward_passes(pm, torch, deep):  # noqa: F811
    """Logits above 512 MiB of 8 to 15 outputs are stored by tiles of several
    models; the same samples in two halves, below, by tiles of one."""
    rng = np.random.default_rng(3)
    M, F, O, B = 1000, 9, 10, 14000
    hs = rng.integers(1, 5, M).astype(np.int32)
    acts = rng.integers(0, 10, M).astype(np.int32)
    X = torch.from_numpy(rng.standard_normal((B, F)).astype(np.float32)).cuda()
    net = (pm.DeepPackedMLP(F, O, hs, hs[::-1].copy(), acts, seed=4) if deep
           else pm.PackedMLP(F, O, hs, acts, seed=4))
    whole = net.forward(X)
    parts = torch.cat([net.forward(X[:B // 2]), net.forward(X[B // 2:])])
    assert torch.equal(whole, parts)
    net.close()
