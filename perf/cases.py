"""Performance cases of the packed-MLP training framework.

Each case is one thing a user of ``paper_2206_08369_amd`` does with a pool of
independent MLPs, through ``PackedMLP`` / ``DeepPackedMLP``:

* kind "train": SGD steps over consecutive batches of a data set that is
  resident on the GPU.  With ``ends = "params"`` the pass is a whole epoch and
  ends as a training script does, with the losses and the parameters read back
  to the host; with ``ends = "gradients"`` it ends with the gradients of the
  next batch at the updated weights (a caller that monitors them, or applies
  an update rule of its own), which stay on the GPU.
* kind "deep": the same for a pool of MLPs with two hidden layers.
* kind "forward": the logits of every model of the pool on a set of samples
  (prediction, validation).

The pools are those of the paper's grid (hidden widths times activation
functions, Section 4.2) or random ones; the sizes are those of this
repository's workloads and tests.

Nothing but ``prepare`` and ``run`` uses the framework: ``exact`` computes
what ``run`` returns in float64 with torch alone.
"""
import math

import numpy as np
import torch

LR = 0.01

BASE = dict(kind="train", grid="paper", models=0, wmin=1, wmax=10, acts=10, repeats=1, F=10, O=2,
            B=32, S=0, steps=1, ends="gradients", precision="fp32", biases=False, head="ce",
            rates=False, masks=False)


def _case(**kw):
    c = dict(BASE)
    c.update(kw)
    if not c["S"]:
        c["S"] = c["B"] * (c["steps"] + 1)
    return c


def listed():
    return [
        # one sample through a pool of 60 small models: the latency of a prediction
        _case(name="predict_one", kind="forward", acts=6, B=1, S=1),
        # an epoch of the smallest pool: 60 models of 1..10 units, 1,000 samples in
        # batches of 32 (the last one of 8); launches and latency count
        _case(name="small_epoch", acts=6, S=1000, steps=32, ends="params"),
        # an epoch of 1,000 models of 1..100 units, 50 features, 10,000 samples in
        # batches of 128 (the last one of 16)
        _case(name="thousand_epoch", wmax=100, F=50, B=128, S=10000, steps=79, ends="params"),
        # validation: the same pool on all its 10,000 samples in one call
        _case(name="thousand_validate", kind="forward", wmax=100, F=50, B=10000, S=10000),
        # the paper's grid: 10,000 models, 1..100 units, ten activations, ten repeats
        _case(name="paper_pool", wmax=100, repeats=10, F=100, B=256, steps=8),
        # the flagship: 10,000 models of 1..1000 units (5 million hidden units)
        _case(name="wide_pool", wmax=1000, F=100, B=256, steps=4),
        # the same models on 32 features, ten classes and batches of 32: weight traffic
        # and the output layer's reductions count
        _case(name="ten_class_pool", wmax=1000, F=32, O=10, B=32, steps=4),
        # 1,000 features and batches of 1,024: the input-layer products count
        _case(name="wide_input_fp32", wmax=200, F=1000, B=1024, steps=2),
        # the same with bfloat16 operands and Z kept in bfloat16
        _case(name="wide_input_bf16", wmax=200, F=1000, B=1024, steps=2, precision="bf16_store"),
        # a random pool with biases: odd feature count, three classes, a ragged batch
        _case(name="ragged_biased", grid="random", models=700, wmax=250, acts=13, F=37, O=3, B=200,
              steps=4, biases=True),
        # regression with two targets in batches of 1,000
        _case(name="regression_b1000", wmax=50, repeats=4, F=100, B=1000, steps=4, head="mse"),
        # 1,000 models with two hidden layers each (Section 7)
        _case(name="two_layers", kind="deep", wmax=100, F=50, B=128, steps=4),
    ]


def _log(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi + 1)))))))


def draw(rng):
    kind = rng.choice(["train"] * 7 + ["forward"] * 2 + ["deep"])
    c = _case(kind=kind, grid="random", models=_log(rng, 10, 10000), acts=rng.choice([1, 6, 10, 13]))
    c["wmax"] = _log(rng, 2, 1000 if kind != "deep" else 150)
    c["F"] = _log(rng, 2, 1000)
    c["O"] = rng.choice([2, 2, 2, 3, 4, 5, 10, 16])
    c["B"] = _log(rng, 1, 1024 if kind != "forward" else 10000)
    c["steps"] = rng.choice([1, 2, 3]) if kind != "forward" else 1
    if kind != "deep":
        c["precision"] = rng.choice(["fp32"] * 7 + ["bf16"] + ["bf16_store"])
        c["biases"] = rng.random() < 0.3
    if kind == "train":
        c["head"] = "mse" if rng.random() < 0.15 else "ce"
        if c["head"] == "mse":
            c["biases"] = False
        else:
            c["rates"] = rng.random() < 0.2
        c["masks"] = rng.random() < 0.15
    # no dearer than the flagship: products, activations and memory
    while True:
        n = c["models"] * (c["wmax"] + 1) / 2 * (1 if kind != "deep" else 1 + c["wmax"] / 30)
        if (n * c["F"] * c["B"] * (c["steps"] + 1) <= 1.5e11 and n * c["B"] * c["O"] <= 1e9
                and n * c["F"] <= 4e8):
            break
        c["models"] = max(1, c["models"] * 2 // 3)
    c["S"] = c["B"] * (c["steps"] + 1) if kind != "forward" else c["B"]
    return c


# --- inputs ---------------------------------------------------------------

def _models(c):
    """(hidden widths, activation ids) and, for two layers, the second widths."""
    if c["grid"] == "paper":  # activation-major, width-ascending
        w = np.arange(c["wmin"], c["wmax"] + 1)
        hs = np.tile(np.repeat(w, c["repeats"]), c["acts"]).astype(np.int32)
        ac = np.repeat(np.arange(c["acts"]), len(w) * c["repeats"]).astype(np.int32)
    else:
        r = np.random.default_rng([c["models"], c["wmax"], c["acts"]])
        hs = r.integers(c["wmin"], c["wmax"] + 1, c["models"]).astype(np.int32)
        ac = r.integers(0, c["acts"], c["models"]).astype(np.int32)
    return hs, ac, np.ascontiguousarray(hs[::-1])


def _data(c, seed):
    """Samples, targets (a noisy linear teacher's), per-model rates and masks."""
    g = torch.Generator(device="cuda").manual_seed(1000003 * seed + 17)
    rand = lambda *s: torch.randn(*s, generator=g, device="cuda", dtype=torch.float32)  # noqa: E731
    X = rand(c["S"], c["F"])
    score = X.double() @ rand(c["F"], c["O"]).double() + 0.1 * rand(c["S"], c["O"]).double()
    if c["head"] == "mse":
        y = (score / math.sqrt(c["F"])).float().contiguous()
    else:
        y = score.argmax(1).to(torch.int32)
    M = len(_models(c)[0])
    rates = LR * (0.5 + torch.rand(M, generator=g, device="cuda")) if c["rates"] else None
    mask = None
    if c["masks"]:
        mask = torch.rand(M, c["F"], generator=g, device="cuda") < 0.7
        mask[:, 0] = True
    return X, y, rates, mask


def _batches(c):
    k = c["steps"] if c["kind"] != "forward" else 0
    return [(min(i * c["B"], c["S"]), min((i + 1) * c["B"], c["S"])) for i in range(k)]


def _final(c):
    s = c["steps"] * c["B"] if c["kind"] != "forward" else 0
    return s, min(s + c["B"], c["S"])


def prepare(case, seed):
    import paper_2206_08369_amd as pm
    c = dict(BASE, **case)
    hs, ac, h2 = _models(c)
    X, y, rates, mask = _data(c, seed)
    if c["kind"] == "deep":
        net = pm.DeepPackedMLP(c["F"], c["O"], hs, h2, ac, seed=seed)
    else:
        prec = {"fp32": pm.PMLP_FP32, "bf16": pm.PMLP_BF16_GEMM, "bf16_store": pm.PMLP_BF16_STORE}
        net = pm.PackedMLP(c["F"], c["O"], hs, ac, seed=seed, precision=prec[c["precision"]],
                           biases=c["biases"], head=c["head"])
        if mask is not None:
            net.set_feature_mask(mask.cpu().numpy())
    s, e = _final(c)
    return {"net": net, "lr": LR if rates is None else rates, "ends": c["ends"], "kind": c["kind"],
            "deep": c["kind"] == "deep", "steps": [(X[a:b], y[a:b]) for a, b in _batches(c)],
            "last": (X[s:e], y[s:e])}


def run(state):
    net = state["net"]
    if state["kind"] == "forward":
        return net.forward(state["last"][0])
    for X, y in state["steps"]:
        net.train_step(X, y, state["lr"])
    if state["ends"] == "params":
        W1, W2 = net.get_params()
        return {"losses": net.losses(), "W1": W1, "W2": W2}
    return tuple(net.gradients(*state["last"]))


# --- the work of a pass -----------------------------------------------------

def work(case):
    """Per step: the parameters read and (in a training step) written, the
    batch read, the two input-layer products and the output layer's three.
    The final gradients read the parameters and write as many values."""
    c = dict(BASE, **case)
    hs, _, h2 = _models(c)
    N, M, F, O = int(hs.sum()), len(hs), c["F"], c["O"]
    params = N * F + N * O + ((N + M * O) if c["biases"] else 0)
    per_sample = 2 * N * (F + O)
    if c["kind"] == "deep":
        K, N2 = int((hs.astype(np.int64) * h2).sum()), int(h2.sum())
        params = N * F + K + N2 * O
        per_sample = 2 * (N * F + K + N2 * O)
    if c["kind"] == "forward":
        b = c["S"]
        return {"bytes": 4.0 * (params + b * F + b * M * O), "flops": float(per_sample * b)}
    samples = sum(e - s for s, e in _batches(c))
    passes = c["steps"]
    if c["ends"] == "gradients":
        s, e = _final(c)
        samples += e - s
        passes += 1
    # forward once; backward: the weights' gradients, and the hidden gradient of
    # every layer above the first
    back = per_sample + 2 * N * O if c["kind"] != "deep" else 2 * per_sample - 2 * N * F
    return {"bytes": 4.0 * (2 * params * passes + samples * (F + (O if c["head"] == "mse" else 1))),
            "flops": float((per_sample + back) * samples)}


def tolerance(case):
    """fp32 logits, losses and weights: sums of up to 1,000 float32 terms in
    another order (measured against float64: 1e-7 to 9e-7).  fp32 gradients:
    also the few samples whose pre-activation lies within a rounding of the
    kink of ReLU or LeakyReLU and gets the other slope (measured 2e-7 to 5e-5
    over 1e5 to 1e9 pre-activations), or,
    with thirteen activations, on the other side of Hardshrink's jump.
    bfloat16 operands: the rounding of two operands per product, 2^-9 each
    (measured 8e-4 to 1.4e-2 against float64)."""
    c = dict(BASE, **case)
    if c["precision"] != "fp32":
        return {"rel": 1e-2}
    if c["kind"] == "forward" or c["ends"] == "params":
        return {"rel": 1e-5}
    return {"rel": 1e-5 if c["acts"] == 1 else 2e-4 if c["acts"] <= 10 else 1e-3}


# --- the same in float64, without the framework ------------------------------

_MASK = (1 << 64) - 1


def _i64(v):
    v &= _MASK
    return v - (1 << 64) if v >> 63 else v


def _shr(x, k):
    return (x >> k) & ((1 << (64 - k)) - 1)


def _splitmix(x):
    z = x + _i64(0x9E3779B97F4A7C15)
    z = (z ^ _shr(z, 30)) * _i64(0xBF58476D1CE4E5B9)
    z = (z ^ _shr(z, 27)) * _i64(0x94D049BB133111EB)
    return z ^ _shr(z, 31)


def _uniform(seed, tag, idx, bound):
    """The documented initial weights: uniform in (-bound, bound) from the
    counter-based splitmix64 stream, rounded as float32 values."""
    key = int(_splitmix(torch.tensor(_i64(seed)))) & _MASK
    r = _splitmix(idx ^ _i64(key ^ (tag << 60)))
    u = ((_shr(r, 40) * 2 - (1 << 24)).float() * 2.0 ** -24)
    return (u * bound).double()


def _act(a, z):
    """Value and derivative of activation id a."""
    one = torch.ones_like(z)
    pos = z > 0
    sig = torch.sigmoid
    if a == 0:
        return z, one
    if a == 1:
        return torch.where(pos, z, 0 * z), pos.double()
    if a == 2:
        t = torch.tanh(z)
        return t, 1 - t * t
    if a == 3:
        s = sig(z)
        return s, s * (1 - s)
    if a == 4:
        e = torch.exp(torch.clamp(z, max=0.0))
        return torch.where(pos, z, e - 1), torch.where(pos, one, e)
    if a == 5:
        return torch.where(pos, z, 0.01 * z), torch.where(pos, one, 0.01 * one)
    if a == 6:
        cdf = 0.5 * torch.erfc(-z / math.sqrt(2.0))
        return z * cdf, cdf + z * torch.exp(-0.5 * z * z) / math.sqrt(2 * math.pi)
    if a == 7:
        s = sig(z)
        return z * s, s + z * s * (1 - s)
    if a == 8:
        return torch.logaddexp(z, 0 * z), sig(z)
    if a == 9:
        s = sig(2 * z)
        return z * s, s + 2 * z * s * (1 - s)
    if a == 10:
        al, la = 1.6732632423543772, 1.0507009873554805
        e = torch.exp(torch.clamp(z, max=0.0))
        return torch.where(pos, la * z, la * al * (e - 1)), torch.where(pos, la * one, la * al * e)
    if a == 11:
        on = z.abs() > 0.5
        return torch.where(on, z, 0 * z), on.double()
    sp = torch.logaddexp(z, 0 * z)
    t = torch.tanh(sp)
    return z * t, t + z * (1 - t * t) * sig(z)


def _acts(ids, z):
    """Activation of [n, B] pre-activations, row by row; rows with equal ids are adjacent runs."""
    h, d = torch.empty_like(z), torch.empty_like(z)
    edges = [0] + (np.flatnonzero(np.diff(ids)) + 1).tolist() + [len(ids)]
    if len(edges) > 200:
        for a in np.unique(ids).tolist():
            rows = torch.from_numpy(np.flatnonzero(ids == a)).cuda()
            h[rows], d[rows] = _act(a, z[rows])
    else:
        for s, e in zip(edges[:-1], edges[1:]):
            h[s:e], d[s:e] = _act(int(ids[s]), z[s:e])
    return h, d


def _loss_grad(c, L, y):
    """Per-model loss [m] and dLoss/dlogits [m, B, O]."""
    B = L.shape[1]
    if c["head"] == "mse":
        D = L - y.double()[None]
        return (D * D).mean((1, 2)), 2 * D / (B * c["O"])
    lp = torch.log_softmax(L, 2)
    t = y.long()[None, :, None].expand(L.shape[0], -1, 1)
    G = torch.exp(lp)
    G.scatter_add_(2, t, -torch.ones_like(t, dtype=torch.double))
    return -lp.gather(2, t)[..., 0].mean(1), G / B


def _chunks(cost, most):
    """Runs of whole models of a summed cost up to `most`."""
    s, tot = 0, 0.0
    for m, w in enumerate(cost):
        if m > s and tot + w > most:
            yield s, m
            s, tot = m, 0.0
        tot += w
    yield s, len(cost)


def exact(case, seed):
    c = dict(BASE, **case)
    hs, ac, h2 = _models(c)
    F, O, B, N, M = c["F"], c["O"], c["B"], int(hs.sum()), len(hs)
    if c["kind"] == "deep":
        if M > 3000:  # a loop over the models
            return None
        return _exact_deep(c, seed, hs, h2, ac)
    X, y, rates, mask = _data(c, seed)
    X = X.double()
    off = np.concatenate([[0], np.cumsum(hs.astype(np.int64))])
    s, e = _final(c)
    W1s, W2s, Ls, b1s, b2s, loss_s = [], [], [], [], [], []
    for m0, m1 in _chunks(hs, max(1, 4e7 / max(B * O, F))):
        n0, n1 = int(off[m0]), int(off[m1])
        n, m = n1 - n0, m1 - m0
        cnt = torch.from_numpy(hs[m0:m1].astype(np.int64)).cuda()
        mid = torch.repeat_interleave(torch.arange(m, device="cuda"), cnt)
        ids = np.repeat(ac[m0:m1], hs[m0:m1])
        rows = torch.arange(n0, n1, device="cuda")
        bound2 = (1.0 / torch.sqrt(cnt.double())).float()
        bound1 = np.float32(1.0 / math.sqrt(F)).item()
        W1 = _uniform(seed, 1, rows[:, None] * F + torch.arange(F, device="cuda")[None], bound1)
        W2 = _uniform(seed, 2, torch.arange(O, device="cuda")[:, None] * N + rows[None],
                      bound2[mid][None])
        b1 = torch.zeros(n, dtype=torch.double, device="cuda")
        b2 = torch.zeros(m, O, dtype=torch.double, device="cuda")
        if c["biases"]:
            b1 = _uniform(seed, 3, rows, bound1)
            b2 = _uniform(seed, 4, torch.arange(m0 * O, m1 * O, device="cuda").reshape(m, O),
                          bound2[:, None])
        seen = 1.0 if mask is None else mask[m0:m1][mid].double()
        W1 = W1 * seen
        lr = LR if rates is None else rates[m0:m1].double()
        lru = LR if rates is None else lr[mid]
        at = lambda v, axes: v if isinstance(v, float) else v.reshape(axes)  # noqa: E731

        def forward(Xb):
            Z = W1 @ Xb.t() + b1[:, None]
            H, D = _acts(ids, Z)
            L = torch.stack([torch.zeros(m, Xb.shape[0], dtype=torch.double, device="cuda")
                             .index_add_(0, mid, H * W2[o][:, None]) for o in range(O)], 2)
            return H, D, L + b2[:, None, :]

        def backward(Xb, yb):
            H, D, L = forward(Xb)
            loss, G = _loss_grad(c, L, yb)
            dH, dW2 = torch.zeros_like(H), torch.empty_like(W2)
            for o in range(O):
                Go = G[:, :, o][mid]
                dH.add_(Go * W2[o][:, None])
                dW2[o] = (Go * H).sum(1)
            dZ = dH.mul_(D)
            return loss, (dZ @ Xb) * seen, dW2, dZ.sum(1), G.sum(1)

        if c["kind"] == "forward":
            Ls.append(torch.cat([forward(X[a:min(a + 4096, e)])[2].transpose(0, 1)
                                 for a in range(s, e, 4096)]))
            continue
        loss = None
        for a, b in _batches(c):
            loss, g1, g2, gb1, gb2 = backward(X[a:b], y[a:b])
            W1 = W1 - at(lru, (-1, 1)) * g1
            W2 = W2 - at(lru, (1, -1)) * g2
            if c["biases"]:
                b1 = b1 - at(lru, (-1,)) * gb1
                b2 = b2 - at(lr, (-1, 1)) * gb2
        if c["ends"] == "params":
            W1s.append(W1)
            W2s.append(W2)
            loss_s.append(loss)
        else:
            _, g1, g2, gb1, gb2 = backward(X[s:e], y[s:e])
            W1s.append(g1)
            W2s.append(g2)
            b1s.append(gb1)
            b2s.append(gb2)
    if c["kind"] == "forward":
        return torch.cat(Ls, 1)
    W1, W2 = torch.cat(W1s), torch.cat(W2s, 1)
    if c["ends"] == "params":
        return {"losses": torch.cat(loss_s), "W1": W1, "W2": W2}
    return (W1, W2, torch.cat(b1s), torch.cat(b2s)) if c["biases"] else (W1, W2)


def _exact_deep(c, seed, hs, h2, ac):
    X, y, _, _ = _data(c, seed)
    X = X.double()
    F, O, N, N2 = c["F"], c["O"], int(hs.sum()), int(h2.sum())
    o1 = np.concatenate([[0], np.cumsum(hs.astype(np.int64))])
    o2 = np.concatenate([[0], np.cumsum(h2.astype(np.int64))])
    ko = np.concatenate([[0], np.cumsum(hs.astype(np.int64) * h2)])
    f32 = lambda k: np.float32(1.0 / math.sqrt(float(k))).item()  # noqa: E731
    V1 = _uniform(seed, 1, torch.arange(N * F, device="cuda").reshape(N, F), f32(F))
    s, e = _final(c)
    out1 = torch.empty(N, F, dtype=torch.double, device="cuda")
    out12 = torch.empty(int(ko[-1]), dtype=torch.double, device="cuda")
    out2 = torch.empty(O, N2, dtype=torch.double, device="cuda")
    for m in range(len(hs)):
        a, b, k = int(o1[m]), int(o2[m]), int(ko[m])
        n1, n2, act = int(hs[m]), int(h2[m]), int(ac[m])
        W1 = V1[a:a + n1]
        W12 = _uniform(seed, 5, torch.arange(k, k + n1 * n2, device="cuda"), f32(n1)).reshape(n2, n1)
        idx = torch.arange(O, device="cuda")[:, None] * N2 + torch.arange(b, b + n2, device="cuda")
        W2 = _uniform(seed, 2, idx, f32(n2))

        def backward(Xb, yb):
            H1, D1 = _act(act, Xb @ W1.t())
            H2, D2 = _act(act, H1 @ W12.t())
            G = _loss_grad(c, (H2 @ W2.t())[None], yb)[1][0]
            dZ2 = (G @ W2) * D2
            dZ1 = (dZ2 @ W12) * D1
            return dZ1.t() @ Xb, dZ2.t() @ H1, G.t() @ H2

        for p, q in _batches(c):
            g1, g12, g2 = backward(X[p:q], y[p:q])
            W1, W12, W2 = W1 - LR * g1, W12 - LR * g12, W2 - LR * g2
        g1, g12, g2 = backward(X[s:e], y[s:e])
        out1[a:a + n1] = g1
        out12[k:k + n1 * n2] = g12.reshape(-1)
        out2[:, b:b + n2] = g2
    return out1, out12, out2
