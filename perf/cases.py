"""Performance cases of the DBW parameter-server simulation on one GPU.

Every case is one call (or one whole iteration) through the public binding,
``paper_2004_14696_amd.Context``: the worker gradients of the three model
families, the full DBW step, and the parameter server's aggregation and
statistics calls.  Sizes are those of the workloads in ``dbw_inputs`` plus
generic ones: an odd feature count, class counts off the tile sizes, a large
class count, a wide hidden layer.

A case is a dict of plain values:
  call      "step" (dbw_step), "grads" (dbw_worker_grads), "aggregate", "stats"
  model     "softmax", "mlp", "cnn"
  n B d C H workers, minibatch rows, features, classes, hidden units
  S         rows of the resident dataset the minibatches index (0: the
            minibatches are passed materialised, X [n][B][d])
  features  "uniform" [0, 1) or "normal"; sparsity: share of zeroed entries
  policy, k, g_rows  how a step chooses k_t, and which G rows it writes
"""
from __future__ import annotations

import math

import torch
import torch.nn.functional as F

from paper_2004_14696_amd import Context, make_config

BATCHES = 4           # minibatches (and arrival times) a training loop goes through
CONV1, CONV2 = (20, 1, 5, 5), (50, 20, 5, 5)


def _case(name, call, model, n, B, d, C, H=0, S=0, features="uniform", sparsity=0.0, policy="dbw", k=0,
          g_rows="all", eta=0.1):
    case = {"call": call, "model": model, "n": n, "B": B, "d": d, "C": C, "H": H, "S": S, "features": features,
            "sparsity": sparsity, "policy": policy, "k": k, "g_rows": g_rows, "eta": eta}
    return {"name": name, **case} if name else case


def listed():
    return [
        # the smallest training loop (4 workers on 28x28 images, 80% zeros):
        # an iteration is launches and latencies
        _case("step softmax 4x32x784x10", "step", "softmax", 4, 32, 784, 10, S=60000, sparsity=0.8),
        # the paper's cluster size with a fixed number of backup workers
        _case("step softmax 16x128x784x10", "step", "softmax", 16, 128, 784, 10, S=60000, policy="static", k=12),
        # images with a constant-one column as the bias: an odd feature count
        # and a ragged minibatch
        _case("step softmax 16x100x785x10", "step", "softmax", 16, 100, 785, 10, S=60000, policy="static", k=12),
        # the bandwidth-bound workload: 32x32x3 inputs, ten classes
        _case("step softmax 64x256x3072x10", "step", "softmax", 64, 256, 3072, 10, S=50000, features="normal",
              policy="static", k=48, g_rows="none"),
        # the largest workload: 256 workers, 100 classes
        _case("step softmax 256x512x3072x100", "step", "softmax", 256, 512, 3072, 100, S=50000, features="normal",
              g_rows="none"),
        # a class count that is no multiple of four, minibatches passed
        # materialised by the user's own data pipeline
        _case("grads softmax 24x200x1000x37", "grads", "softmax", 24, 200, 1000, 37, features="normal"),
        # a thousand classes on 2048 features (a linear probe)
        _case("grads softmax 32x128x2048x1000", "grads", "softmax", 32, 128, 2048, 1000, S=20000, features="normal"),
        # the two-layer network workload
        _case("grads mlp 32x64x784x512x10", "grads", "mlp", 32, 64, 784, 10, H=512, S=60000),
        # a wide hidden layer on 32x32x3 inputs with larger minibatches
        _case("grads mlp 16x256x3072x1024x10", "grads", "mlp", 16, 256, 3072, 10, H=1024, S=50000, features="normal"),
        # the paper's MNIST network at its setting, 16 workers x 500 images
        _case("grads cnn 16x500x784x500x10", "grads", "cnn", 16, 500, 784, 10, H=500, S=60000, sparsity=0.8,
              eta=0.01),
        # the parameter server's calls by themselves, on gradients a caller
        # holds: the mean of the fastest three quarters of 256 workers
        _case("aggregate 256x307200 k=192", "aggregate", "softmax", 256, 1, 3072, 100, k=192),
        # and the statistics of the received gradients
        _case("stats 256x307200 k=192", "stats", "softmax", 256, 1, 3072, 100, k=192),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step narrow", "step narrow", "step mid", "step mid", "grads wide", "mlp", "mlp", "cnn",
                       "aggregate", "stats"])
    features = rng.choice(["uniform", "normal"])
    sparsity = rng.choice([0.0, 0.0, 0.8]) if features == "uniform" else 0.0
    n = _log(rng, 4, 256)
    if kind in ("aggregate", "stats"):
        d, C = _log(rng, 64, 3072), rng.randint(2, 100)
        return _case(None, kind, "softmax", n, 1, d, C, k=rng.randint(2, n))
    if kind == "cnn":
        n = _log(rng, 2, 16)
        return _case(None, "grads", "cnn", n, _log(rng, 16, 500), 784, 10, H=rng.randint(64, 512),
                     S=rng.choice([60000, 60000, 0]), features=features, sparsity=sparsity, eta=0.01)
    d = _log(rng, 64, 3072)
    if rng.random() < 0.6:
        d = (d + 3) // 4 * 4
    C = {"step narrow": rng.randint(2, 16), "step mid": rng.randint(17, 112), "grads wide": rng.randint(113, 1000),
         "mlp": rng.randint(2, 10)}[kind]
    if kind != "step narrow" and rng.random() < 0.6:
        C = (C + 3) // 4 * 4 if kind != "mlp" else C
    H = rng.randint(32, 1024) if kind == "mlp" else 0
    if H and rng.random() < 0.6:
        H = (H + 3) // 4 * 4
    B = _log(rng, 16, 512)
    # no more work than the largest listed cases
    P = d * H + H + H * C + C if H else d * C
    n = max(4, min(n, 131072 // B, 4 * 10**10 // (B * P), 100_000_000 // P))
    S = rng.choice([20000, 50000, 0]) if n * B * d < 2 * 10**8 else 50000
    if kind.startswith("step"):
        policy = rng.choice(["dbw", "static"])
        return _case(None, "step", "softmax", n, B, d, C, S=S or 20000, features=features, sparsity=sparsity,
                     policy=policy, k=rng.randint(1, n) if policy == "static" else 0,
                     g_rows=rng.choice(["all", "selected", "none"]))
    return _case(None, "grads", "mlp" if H else "softmax", n, B, d, C, H=H, S=S, features=features,
                 sparsity=sparsity)


# -- inputs ------------------------------------------------------------------


def _cnn_hidden(Wc1, bc1, Wc2, bc2, X):
    """The 800 features of each image (valid 5x5 convolutions, 2x2 max
    pooling, ReLU) in X's precision."""
    def conv(h, W, b):
        m, side = h.shape[0], h.shape[2] - 4
        z = W.reshape(W.shape[0], -1) @ F.unfold(h, 5) + b[:, None]
        return F.relu(F.max_pool2d(z.reshape(m, W.shape[0], side, side), 2))
    return conv(conv(X.reshape(-1, 1, 28, 28), Wc1, bc1), Wc2, bc2).reshape(X.shape[0], 800)


def _split(case, w):
    """The blocks of a flat MLP or CNN parameter vector."""
    d, H, C = (800 if case["model"] == "cnn" else case["d"]), case["H"], case["C"]
    shapes = [(d, H), (H,), (H, C), (C,)]
    if case["model"] == "cnn":
        shapes += [CONV1, (20,), CONV2, (50,)]
    out, at = [], 0
    for s in shapes:
        out.append(w[at:at + math.prod(s)].reshape(s))
        at += math.prod(s)
    return out


def _clear_bias(A):
    """Per hidden unit, the offset (out of 65 small ones) that keeps the
    unit's pre-activations A [rows][H] farthest from the ReLU's kink: a
    pre-activation within rounding of zero could go either way in a correct
    implementation, and the gradients would differ by a whole row."""
    best = torch.full((A.shape[1],), -1.0, device=A.device, dtype=A.dtype)
    bias = torch.zeros_like(best)
    for c in torch.linspace(-0.1, 0.1, 65).tolist():
        gap = (A + c).abs().amin(dim=0)
        bias = torch.where(gap > best, torch.full_like(bias, c), bias)
        best = torch.maximum(gap, best)
    return bias


def _inputs(case, seed):
    """w, dataset or minibatches X and y, row indices and arrival ticks."""
    dev = "cuda"
    gen = torch.Generator(device=dev).manual_seed(1_000_003 * int(seed) + 7)
    n, B, d, C, H, S = (case[k] for k in ("n", "B", "d", "C", "H", "S"))
    batches = BATCHES if case["call"] == "step" else 1
    if case["call"] in ("aggregate", "stats"):
        # gradients of workers that share a mean, as near the start of training
        P = d * C
        mean = torch.randn(P, generator=gen, device=dev) * 0.01
        G = torch.randn((n, P), generator=gen, device=dev).mul_(0.03).add_(mean)
        loss = math.log(C) + 0.1 * torch.rand(n, generator=gen, device=dev)
        ticks = ((1.0 - torch.log1p(-torch.rand(n, generator=gen, device=dev, dtype=torch.float64))) * 2**20).long()
        return {"G": G, "loss": loss, "ticks": ticks}
    shape = (S, d) if S else (n, B, d)
    X = torch.rand(shape, generator=gen, device=dev) if case["features"] == "uniform" \
        else torch.randn(shape, generator=gen, device=dev)
    if case["sparsity"]:
        X *= torch.rand(shape, generator=gen, device=dev) >= case["sparsity"]
    y = torch.randint(0, C, shape[:-1], generator=gen, device=dev, dtype=torch.int32)
    rows = [torch.randint(0, S, (n, B), generator=gen, device=dev, dtype=torch.int32) if S else None
            for _ in range(batches)]
    # round trips 1 + Exp(1), in ticks of 2^-20
    ticks = [((1.0 - torch.log1p(-torch.rand(n, generator=gen, device=dev, dtype=torch.float64))) * 2**20).long()
             .cpu().numpy() for _ in range(batches)]
    if case["model"] == "softmax":
        w = 0.01 * torch.randn(d * C, generator=gen, device=dev)
    elif case["model"] == "mlp":
        W1 = torch.randn((d, H), generator=gen, device=dev) * math.sqrt(2.0 / d)
        W2 = torch.randn((H, C), generator=gen, device=dev) * math.sqrt(2.0 / H)
        Xr = (X[rows[0].reshape(-1).long()] if S else X.reshape(-1, d)).double()
        b1 = _clear_bias(Xr @ W1.double()).float()
        w = torch.cat([W1.reshape(-1), b1, W2.reshape(-1), torch.zeros(C, device=dev)])
    else:
        def uniform(shape, fan_in):
            return (2 * torch.rand(shape, generator=gen, device=dev) - 1) / math.sqrt(fan_in)
        W1, W2, b2 = uniform((800, H), 800), uniform((H, C), H), uniform((C,), H)
        conv = [uniform(CONV1, 25), uniform((20,), 25), uniform(CONV2, 500), uniform((50,), 500)]
        Xr = X[rows[0].reshape(-1).long()] if S else X.reshape(-1, d)
        feat = torch.cat([_cnn_hidden(*conv, x) for x in Xr.split(1000)]).double()
        b1 = _clear_bias(feat @ W1.double()).float()
        w = torch.cat([t.reshape(-1) for t in (W1, b1, W2, b2, *conv)])
    return {"w": w, "X": X, "y": y, "rows": rows, "ticks": ticks}


def prepare(case, seed):
    s = _inputs(case, seed)
    cfg = make_config(case["model"], case["n"], case["B"], case["d"], case["C"], case["H"], eta=case["eta"],
                      S=case["S"], policy=case["policy"] if case["call"] == "step" else "dbw",
                      k_static=case["k"] if case["policy"] == "static" else 0, g_rows=case["g_rows"])
    s["case"], s["ctx"], s["t"] = case, Context(cfg), 0
    n, dev = case["n"], "cuda"
    if case["call"] == "aggregate":
        s["g"] = torch.empty(s["ctx"].P, device=dev)
        s["mask"] = torch.empty(n, dtype=torch.uint8, device=dev)
    elif case["call"] == "stats":
        # the received gradients and their mean, as the aggregation left them
        s["g"], s["mask"] = s["ctx"].aggregate_fastest(s["G"], s["ticks"], case["k"])
        s["sqnorm"] = torch.empty(n, device=dev)
        s["stats"] = torch.empty(4, dtype=torch.float64, device=dev)
    elif case["call"] == "grads":
        s["G"] = torch.empty((n, s["ctx"].P), device=dev)
        s["loss"] = torch.empty(n, device=dev)
    return s


def run(s):
    case, ctx = s["case"], s["ctx"]
    if case["call"] == "step":
        t = s["t"] % BATCHES
        s["t"] += 1
        ctx.step(s["w"], s["X"], s["y"], s["ticks"][t], rows=s["rows"][t])
        return {"w": s["w"]}
    if case["call"] == "aggregate":
        g, mask = ctx.aggregate_fastest(s["G"], s["ticks"], case["k"], g=s["g"], mask=s["mask"])
        return {"g": g, "mask": mask}
    if case["call"] == "stats":
        sqnorm, stats = ctx.grad_stats(s["G"], s["mask"], case["k"], s["g"], s["loss"], sqnorm=s["sqnorm"],
                                       stats=s["stats"])
        return {"sqnorm": sqnorm, "stats": stats}
    G, loss = ctx.worker_grads(s["w"], s["X"], s["y"], rows=s["rows"][0], G=s["G"], loss=s["loss"])
    if case["model"] == "cnn":
        fc = ctx.P - 25570   # the fully connected block, then the convolutions'
        return {"G_fc": G[:, :fc], "G_conv": G[:, fc:], "loss": loss}
    return {"G": G, "loss": loss}


def work(case):
    n, B, d, C, H, S = (case[k] for k in ("n", "B", "d", "C", "H", "S"))
    if case["call"] == "aggregate":
        return {"bytes": 4 * (case["k"] + 1) * d * C + 9 * n, "flops": case["k"] * d * C}
    if case["call"] == "stats":
        # ||G_j||^2 and ||G_j - g||^2 over the received rows, ||g||^2
        return {"bytes": 4 * (case["k"] + 1) * d * C + 9 * n + 32, "flops": 5 * case["k"] * d * C}
    # different dataset rows among n B draws out of S
    m = n * B
    rows = S * -math.expm1(m * math.log1p(-1.0 / S)) if S else m
    if case["model"] == "softmax":
        P, flops = d * C, 4 * m * d * C
    elif case["model"] == "mlp":
        P, flops = d * H + H + H * C + C, 4 * m * d * H + 6 * m * H * C
    else:
        P = 800 * H + H + H * C + C + 25570
        # per image: both convolutions forward; backward over the entries the
        # pooling passed on (one in four): conv2's input and filter gradients,
        # conv1's filter gradient; the fully connected layers three times
        conv1, conv2 = 2 * 576 * 20 * 25, 2 * 64 * 50 * 500
        flops = m * (conv1 + conv2 + conv1 / 4 + 2 * conv2 / 4 + 6 * (800 * H + H * C))
    out = P if case["call"] == "step" else n * P + n
    return {"bytes": 4 * (rows * (d + 1) + (m if S else 0) + P + out), "flops": flops}


def tolerance(case):
    # about four times what the calls are off their 64-bit results by
    if case["call"] in ("aggregate", "stats"):
        return {"rel": 8e-7, "max": 2e-5}
    if case["call"] == "step":
        # the updated parameters: their own rounding and that of eta times the
        # gradient
        return {"rel": 2e-7, "max": 4e-6}
    if case["model"] == "cnn":
        # pooling windows whose entries tie within rounding pass their
        # gradient through another entry
        return {"rel": 4e-3, "max": 0.4}
    return {"rel": 2.5e-6, "max": 2e-4}


# -- 64-bit results ------------------------------------------------------------


def _grads64(case, s):
    """Per-worker gradients [n][P] and losses of the first minibatch in
    float64 (one worker at a time)."""
    n, B, d, C = (case[k] for k in ("n", "B", "d", "C"))
    w = s["w"].double()
    for i in range(n):
        if s["rows"][0] is None:
            X, y = s["X"][i].double(), s["y"][i].long()
        else:
            r = s["rows"][0][i].long()
            X, y = s["X"][r].double(), s["y"][r].long()
        if case["model"] == "softmax":
            z = X @ w.reshape(d, C)
            p = torch.softmax(z, 1)
            p[torch.arange(B, device=p.device), y] -= 1.0
            yield (X.t() @ (p / B)).reshape(-1), F.cross_entropy(z, y)
            continue
        v = w.clone().requires_grad_()
        b = _split(case, v)
        h = _cnn_hidden(*b[4:], X) if case["model"] == "cnn" else X
        loss = F.cross_entropy(torch.relu(h @ b[0] + b[1]) @ b[2] + b[3], y)
        yield torch.autograd.grad(loss, v)[0], loss.detach()


def exact(case, seed):
    s = _inputs(case, seed)
    n, k = case["n"], case["k"]
    if case["call"] in ("aggregate", "stats"):
        first = torch.sort(s["ticks"], stable=True).indices[:k]
        g = sum(s["G"][i].double() for i in first.tolist()) / k
        mask = torch.zeros(n, dtype=torch.uint8, device="cuda")
        mask[first] = 1
        if case["call"] == "aggregate":
            return {"g": g, "mask": mask}
        sq = torch.zeros(n, dtype=torch.float64, device="cuda")
        dev = 0.0
        for i in first.tolist():
            row = s["G"][i].double()
            sq[i] = row.square().sum()
            dev += (row - g).square().sum()
        g2, V = g.square().sum(), dev / (k - 1)
        stats = torch.stack([g2, V, torch.clamp(g2 - V / k, min=0.0), s["loss"].double()[first].mean()])
        return {"sqnorm": sq, "stats": stats}
    if case["call"] == "step":
        # before its first estimates DBW waits for all n workers
        k = k if case["policy"] == "static" else n
        order = sorted(range(n), key=lambda i: (int(s["ticks"][0][i]), i))
        chosen, g = set(order[:k]), 0.0
        for i, (gi, _) in enumerate(_grads64(case, s)):
            if i in chosen:
                g = g + gi / k
        return {"w": s["w"].double() - case["eta"] * g}
    got = list(_grads64(case, s))
    loss = torch.stack([v for _, v in got])
    if case["model"] == "cnn":
        # which entry of a pooling window passes the gradient is a matter of
        # rounding where two tie: no 64-bit value for the filters' gradients
        return {"G_fc": torch.stack([g[:-25570] for g, _ in got]), "G_conv": None, "loss": loss}
    return {"G": torch.stack([g for g, _ in got]), "loss": loss}
