"""The sample-split forward (k_fwd_s: product, activation and M3 forward in
one kernel) against the fp64 oracle at the edges of its instances: every
column-block count (F rounded to 4 a multiple of 16, of 32, and with 4, 8 and
12 columns past it), every batch class (16 to 256 samples, full and ragged),
two to four outputs, models narrower than a 16-unit tile and several in one
tile, models that end on and off tile edges or take many stages, and packs of
one to many groups per workgroup; the training step of the same packs, whose
logits are cleared by its batch copy.  Bars as in the other parity tests (per-model normwise 1e-5)."""
import zlib

import numpy as np
import pytest

import pmlp_workloads as wl
from parity import dw2_terms, err_cols, err_dw2, err_logits, err_losses, err_rows

pytestmark = pytest.mark.gpu

TOL_STEP = 1e-5
EDGES = [3, 1, 1, 17, 16, 15, 70, 2, 1, 33, 65, 5, 48, 1, 16, 64]


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


@pytest.fixture(autouse=True)
def default_path(monkeypatch):
    monkeypatch.delenv("PMLP_GENERIC_KERNELS", raising=False)
    monkeypatch.delenv("PMLP_FUSED_FORWARD", raising=False)


def dev(torch, a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


# (F, O, B, models)
SHAPES = [
    (3, 2, 40, "mixed"), (12, 4, 64, "mixed"), (16, 3, 100, "mixed"), (30, 2, 128, "narrow"),
    (33, 4, 200, "mixed"), (48, 2, 250, "mixed"), (64, 3, 64, "narrow"), (76, 2, 129, "mixed"),
    (80, 4, 256, "narrow"), (96, 2, 100, "mixed"), (100, 2, 256, "mixed"), (104, 3, 130, "narrow"),
    (100, 4, 33, "mixed"), (50, 2, 128, "narrow"), (100, 2, 250, "many"), (100, 2, 256, "wide"),
    (104, 4, 16, "few"), (100, 2, 20, "few"), (9, 3, 1, "few"), (68, 2, 32, "mixed"),
    (10, 2, 200, "few"), (100, 4, 64, "few"), (20, 3, 300, "few"),
]


def inputs(F, O, B, kind):
    rng = np.random.default_rng(zlib.crc32(repr((F, O, B, kind)).encode()))
    if kind == "mixed":       # widths on and off tile edges, and random models
        hs = np.concatenate([EDGES, rng.integers(1, 71, 60)])
    elif kind == "narrow":    # widths of 1 to 12: several models per tile
        hs = rng.integers(1, 13, 900)
    elif kind == "many":      # several groups per workgroup
        hs = rng.integers(1, 60, 9000)
    elif kind == "wide":      # models of many stages, one activation to a tile
        hs = np.tile(np.arange(1, 401), 1)
    else:
        hs = np.array([1, 20, 3, 16, 7, 40, 1])
    hs = hs.astype(np.int32)
    acts = rng.integers(0, 10, len(hs)).astype(np.int32)
    X, y = wl.make_dataset(F, O, B, seed=int(rng.integers(1 << 30)))
    return hs, acts, X, y


def sampled(hs, acts, W1, W2, kind):
    """Models and units the oracle looks at (the models are independent)."""
    step = {"many": 97, "wide": 13}.get(kind, 1)
    off = np.concatenate([[0], np.cumsum(hs)])
    models = np.arange(0, len(hs), step)
    rows = np.concatenate([np.arange(off[m], off[m + 1]) for m in models])
    return models, rows, hs[models], acts[models], W1[rows], W2[:, rows]


@pytest.mark.parametrize("F,O,B,kind", SHAPES)
def test_logits_and_hidden(pm, orc, torch, F, O, B, kind):
    hs, acts, X, _ = inputs(F, O, B, kind)
    net = pm.PackedMLP(F, O, hs, acts, seed=21)
    W1, W2 = net.get_params()
    models, rows, hs_s, ac_s, W1_s, W2_s = sampled(hs, acts, W1, W2, kind)
    Xd = dev(torch, X)
    got = net.forward(Xd).cpu().numpy()
    assert net.kernel_variants()["fwd_m3"] == ("k_fwd_s", pm.PMLP_ARITH_X3)
    assert err_logits(got[:, models], orc.forward(hs_s, ac_s, W1_s, W2_s, X)).max() <= TOL_STEP
    Z, _ = net.hidden(Xd)
    RZ, _ = orc.hidden(hs_s, ac_s, W1_s, X)
    assert err_cols(Z.cpu().numpy()[:, rows], RZ, hs_s).max() <= TOL_STEP
    net.close()


@pytest.mark.parametrize("F,O,B", [(100, 2, 256), (36, 4, 140)])
def test_step_of_wide_models(pm, orc, torch, F, O, B):
    hs, acts, X, y = inputs(F, O, B, "wide")
    net = pm.PackedMLP(F, O, hs, acts, seed=26)
    W1, W2 = net.get_params()
    models, rows, hs_s, ac_s, W1_s, W2_s = sampled(hs, acts, W1, W2, "wide")
    dW1, dW2 = (t.cpu().numpy() for t in net.gradients(dev(torch, X), dev(torch, y)))
    assert net.kernel_variants()["bwd_fused"][0] == "k_bwd_x3"
    r1, r2, rl, allow = orc.gradients(hs_s, ac_s, W1_s, W2_s, X, y)
    assert err_rows(dW1[rows], r1, hs_s, allow).max() <= TOL_STEP
    terms = dw2_terms(orc, hs_s, ac_s, W1_s, W2_s, X, y)
    assert err_dw2(dW2[:, rows], r2, hs_s, terms).max() <= TOL_STEP
    assert err_losses(net.losses()[models], rl).max() <= TOL_STEP
    net.close()


@pytest.mark.parametrize("F,O,B,part", [(50, 2, 1000, 64), (20, 3, 300, 100), (100, 2, 513, 100),
                                        (36, 2, 380, 64)])
def test_forward_of_large_batches_equals_its_parts(pm, torch, F, O, B, part):
    """A forward pass over more than 256 samples runs them in batches of one
    class (256, 64, 64 and 128 samples here); the parts alone, in batches of
    another, sum each model's units in another order only."""
    hs, acts, X, _ = inputs(F, O, B, "mixed")
    net = pm.PackedMLP(F, O, hs, acts, seed=24)
    Xd = dev(torch, X)
    whole = net.forward(Xd)
    assert net.kernel_variants()["fwd_m3"][0] == "k_fwd_s"
    parts = torch.cat([net.forward(Xd[s:s + part]) for s in range(0, B, part)])
    assert err_logits(whole.cpu().numpy(), parts.cpu().numpy()).max() <= TOL_STEP
    net.close()


@pytest.mark.parametrize("F,O,B,kind", [(12, 2, 16, "few"), (100, 3, 128, "narrow"),
                                        (33, 2, 200, "mixed")])
def test_overflow_stays_infinite(pm, torch, F, O, B, kind):
    """Pre-activations of finite operands that overflow to infinity, positive
    output weights: every logit is infinite, also of the models whose last tile
    has rows past them (those add nothing, not 0 times infinity)."""
    hs, _, _, _ = inputs(F, O, B, kind)
    net = pm.PackedMLP(F, O, hs, np.arange(len(hs), dtype=np.int32) % 2, seed=5)
    n = int(hs.sum())
    net.set_params(np.full((n, F), 3e38, np.float32), np.ones((O, n), np.float32))
    got = net.forward(torch.full((B, F), 10.0, device="cuda"))
    assert net.kernel_variants()["fwd_m3"][0] == "k_fwd_s"
    assert bool((got == float("inf")).all())
    net.close()


# products of one column whose fp32 value a sum of bf16 pieces loses: pieces
# that overflow with the other sign, an operand above the largest bf16,
# infinite operands, and ordinary values between them
WILD = [(1.1e20, 1.1e21), (1300.0, 3e38), (1.3e20, -1.7e25), (1.0000001, 3.4e38),
        (20.07, 3e38), (float("inf"), -2.0), (0.5, float("inf")), (-3e38, 0.25), (0.37, 1.3),
        (float("nan"), 0.7)]


def saturated(z):
    with np.errstate(over="ignore"):
        return z.astype(np.float32).astype(np.float64)


@pytest.mark.parametrize("F,O,B,biases", [
    (40, 2, 16, False), (100, 4, 30, True), (64, 2, 64, False), (50, 2, 128, False),
    (33, 3, 200, True), (16, 2, 256, False), (100, 2, 250, False), (70, 4, 300, False),
    (50, 2, 1000, True), (99, 2, 380, False)])
def test_values_out_of_the_pieces_range(pm, torch, F, O, B, biases):
    """Each logit is finite, infinite or NaN as the fp32 products of its sample
    and weights are, and right where it is finite: large and infinite entries
    in some samples and some models, on ordinary ones beside them."""
    rng = np.random.default_rng(F * B)
    hs, _, _, _ = inputs(F, O, B, "mixed")
    n = int(hs.sum())
    acts = np.resize([0, 1, 2, 3], len(hs)).astype(np.int32)
    mid = np.repeat(np.arange(len(hs)), hs)
    W1 = (rng.uniform(0.1, 1.0, (n, F)) * np.where(mid % 8 < 4, 1, -1)[:, None]).astype(np.float32)
    W2 = rng.uniform(0.1, 1.0, (O, n)).astype(np.float32)
    col = F // 2 if F < 64 else 3                  # within the first 32 columns
    X = np.zeros((B, F), np.float32)
    X[::3] = rng.standard_normal((len(X[::3]), F))  # ordinary samples
    for b in range(B):
        if b % 3:
            X[b, col] = WILD[b % len(WILD)][0]
    for m in range(0, len(hs), 7):                  # one model in seven
        W1[mid == m] = 0.0
        W1[mid == m, col] = WILD[(m // 7) % len(WILD)][1]
    net = pm.PackedMLP(F, O, hs, acts, seed=2, biases=biases)
    net.set_params(W1, W2)
    b1, b2 = np.zeros(n, np.float32), np.zeros((len(hs), O), np.float32)
    if biases:
        b1 = rng.standard_normal(n).astype(np.float32)
        b2 = rng.standard_normal(b2.shape).astype(np.float32)
        net.set_biases(b1, b2)
    got = net.forward(dev(torch, X)).cpu().numpy().astype(np.float64)
    assert net.kernel_variants()["fwd_m3"][0] == "k_fwd_s"
    net.close()
    with np.errstate(all="ignore"):
        A, C = X.astype(np.float64), W1.T.astype(np.float64)
        Z, T = np.zeros((B, n)), np.zeros((B, n))
        for f in range(F):                          # (as written: 0 times infinity is NaN)
            Z += A[:, f:f + 1] * C[f]
            T += np.abs(A[:, f:f + 1] * C[f])
        Z = saturated(Z + b1)
        a = acts[mid]
        H = np.where(a == 0, Z, np.where(a == 1, np.where(Z > 0, Z, 0.0),
                     np.where(a == 2, np.tanh(Z), 1.0 / (1.0 + np.exp(-Z)))))
        # the size of what a logit sums: an error of Z enters with slope at most 1
        size = np.where(np.isfinite(T), T, 0.0) + np.abs(b1) + np.abs(H)
        off = np.concatenate([[0], np.cumsum(hs)])[:-1]
        for o in range(O):
            want = saturated(np.add.reduceat(H * W2[o], off, axis=1) + b2[:, o])
            scale = np.add.reduceat(size * W2[o], off, axis=1) + np.abs(b2[:, o])
            g = got[:, :, o]
            assert np.array_equal(np.isnan(g), np.isnan(want))
            assert np.array_equal(g[np.isinf(g)], want[np.isinf(g)])
            ok = np.isfinite(want) & np.isfinite(g)
            assert np.array_equal(ok, np.isfinite(want))
            assert (np.abs(g - want)[ok] <= TOL_STEP * scale[ok]).all()


def test_handles_of_one_kernel_and_two_shapes(pm, orc, torch):
    """Two live handles whose forward passes are the same kernel with different
    amounts of LDS (159 KB for 108 columns, 151 KB for 100): the later and
    smaller one leaves the earlier one its own."""
    nets = []
    for F in (108, 100):
        hs, acts, X, _ = inputs(F, 2, 256, "mixed")
        nets.append((pm.PackedMLP(F, 2, hs, acts, seed=F), hs, acts, X))
    for _ in range(2):
        for net, hs, acts, X in nets:
            got = net.forward(dev(torch, X)).cpu().numpy()
            assert net.kernel_variants()["fwd_m3"][0] == "k_fwd_s"
            W1, W2 = net.get_params()
            assert err_logits(got, orc.forward(hs, acts, W1, W2, X)).max() <= TOL_STEP
    for net, *_ in nets:
        net.close()


def test_a_handle_that_does_not_forward_has_no_plan(pm, torch):
    """The forward pass's per-unit words (4 bytes a unit) are made by the first
    forward pass, not with the handle."""
    hs = np.full(16000, 1000, np.int32)
    n = int(hs.sum())
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    net = pm.PackedMLP(4, 2, hs, np.zeros(len(hs), np.int32), seed=1)
    used = before - torch.cuda.mem_get_info()[0]
    weights, index = 4 * n * (4 + 2), 2 * 4 * n    # W1, W2; model and activation of each unit
    assert used < weights + index + 4 * n // 2
    net.close()


@pytest.mark.parametrize("mode", ["global", "relaxed"])
def test_first_forward_may_be_captured(pm, torch, mode):
    """A first forward pass makes its plan beside the capture it is part of, and
    replays equal the eager pass."""
    hs, acts, X, _ = inputs(50, 2, 256, "mixed")
    e_net = pm.PackedMLP(50, 2, hs, acts, seed=8)
    g_net = pm.PackedMLP(50, 2, hs, acts, seed=8)
    xs = [dev(torch, X), dev(torch, X[::-1].copy())]
    Xd, out = torch.empty_like(xs[0]), torch.empty(256, len(hs), 2, device="cuda")
    want = [e_net.forward(x) for x in xs]
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, capture_error_mode=mode):
        g_net.forward(Xd, out)
    assert g_net.kernel_variants()["fwd_m3"][0] == "k_fwd_s"
    for rep in range(4):
        Xd.copy_(xs[rep % 2])
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, want[rep % 2]), rep
        assert torch.equal(e_net.forward(xs[0]), want[0])
    for net in (g_net, e_net):
        net.close()


@pytest.mark.parametrize("F,O,B,kind", [(50, 2, 200, "mixed"), (104, 4, 16, "few"),
                                        (150, 2, 300, "wide"), (50, 2, 1000, "mixed")])
def test_logits_may_lie_over_the_samples(pm, torch, F, O, B, kind):
    """Logits written over the samples they come from (before, across the end
    of and exactly on them) equal those written elsewhere to the order of their
    sums."""
    hs, acts, X, _ = inputs(F, O, B, kind)
    net = pm.PackedMLP(F, O, hs, acts, seed=11)
    M = len(hs)
    want = net.forward(dev(torch, X)).cpu().numpy()
    for at in (0, B * F // 2, B * M * O - 1):       # the samples' place in the buffer
        buf = torch.zeros(max(B * M * O, at + B * F), device="cuda")
        buf[at:at + B * F] = dev(torch, X).reshape(-1)
        net._stream()
        pm.pmlp_forward(net.handle, buf.data_ptr() + 4 * at, B, buf.data_ptr())
        got = buf[:B * M * O].reshape(B, M, O).cpu().numpy()
        assert err_logits(got, want).max() <= TOL_STEP
    net.close()


@pytest.mark.parametrize("M,w,F,O,B", [(900, 2, 100, 4, 5000), (300, 4, 50, 2, 10000),
                                       (40, 3, 20, 3, 1000), (2000, 1, 36, 2, 3000),
                                       (550, 2, 100, 2, 33100), (300, 4, 70, 2, 16500)])
def test_many_batches_of_narrow_models(pm, orc, torch, M, w, F, O, B):
    """Passes of many batches take runs of several models (whose logits of a
    sample fill lines) where the pack has enough of them, and several rounds of
    workgroups where one leaves many idle (130 batches of 256 or of 128 here);
    against the oracle, on every model and a part of the samples."""
    rng = np.random.default_rng(M + w)
    hs = np.maximum(rng.integers(w - 1, w + 2, max(M, 1100 // w)), 1).astype(np.int32)
    acts = rng.integers(0, 10, len(hs)).astype(np.int32)
    X, _ = wl.make_dataset(F, O, B, seed=M)
    net = pm.PackedMLP(F, O, hs, acts, seed=13)
    W1, W2 = net.get_params()
    got = net.forward(dev(torch, X))
    assert net.kernel_variants()["fwd_m3"][0] == "k_fwd_s"
    rows = np.unique(np.concatenate([np.arange(0, B, max(61, B // 60)), np.arange(B - 70, B)]))
    want = orc.forward(hs, acts, W1, W2, X[rows])
    assert err_logits(got[torch.from_numpy(rows).cuda()].cpu().numpy(), want).max() <= TOL_STEP
    one = net.forward(dev(torch, X[:200]))      # and one batch, by its own groups
    assert err_logits(one.cpu().numpy(), got[:200].cpu().numpy()).max() <= TOL_STEP
    net.close()


@pytest.mark.parametrize("F,biases,one", [(108, False, True), (109, False, False),
                                          (112, False, False), (104, True, True),
                                          (105, True, False)])
def test_the_widest_input(pm, orc, torch, F, biases, one):
    """The kernel takes rows of up to 108 floats (the bias has four of its own);
    wider ones take the other kernels, with the same logits."""
    hs, acts, X, _ = inputs(F, 2, 100, "mixed")
    net = pm.PackedMLP(F, 2, hs, acts, seed=6, biases=biases)
    W1, W2 = net.get_params()
    if biases:
        net.set_biases(np.zeros(int(hs.sum()), np.float32), np.zeros((len(hs), 2), np.float32))
    got = net.forward(dev(torch, X)).cpu().numpy()
    assert (net.kernel_variants()["fwd_m3"][0] == "k_fwd_s") == one
    assert err_logits(got, orc.forward(hs, acts, W1, W2, X)).max() <= TOL_STEP
    net.close()


def test_large_narrow_packs_at_one_wave_per_simd(pm, orc, torch):
    """108 columns, four outputs and 128 samples leave one workgroup to a CU: a
    large pack of narrow models takes the other kernels there, and the one kernel
    at 64 samples; both against the oracle on a sample of the models."""
    hs, acts, X, _ = inputs(108, 4, 100, "many")
    assert hs.sum() > 100000 and hs.mean() < 32
    net = pm.PackedMLP(108, 4, hs, acts, seed=9)
    W1, W2 = net.get_params()
    models, _, hs_s, ac_s, W1_s, W2_s = sampled(hs, acts, W1, W2, "many")
    for B, one in ((100, False), (64, True)):
        got = net.forward(dev(torch, X[:B])).cpu().numpy()
        assert (net.kernel_variants()["fwd_m3"][0] == "k_fwd_s") == one
        want = orc.forward(hs_s, ac_s, W1_s, W2_s, X[:B])
        assert err_logits(got[:, models], want).max() <= TOL_STEP
    net.close()
