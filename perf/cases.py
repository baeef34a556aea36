"""What a program does with this library, as cases that can be timed and whose results can be compared.

Kinds of cases
    train     iterations of all workers: `NetMax.run` (one call enqueues several iterations, as a training loop between two
              visits of the monitor does) or `NetMax.step` (the three calls of one iteration).  Perceptrons train on their
              own data, flat parameter vectors on the synthetic gradient.
    async     global steps of the asynchronous schedule, one active worker each.
    snapshot  what a loop does now and then: the consensus distance and the row-major copies of parameters and momentum
              that a checkpoint is written from.

Ranges: worker counts 2 .. 128; softmax regression and perceptrons with one or two hidden layers on 64 .. 3072 features,
hidden widths 32 .. 1024, 2 .. 32 classes, batches 8 .. 256, float32 and bfloat16 operands; flat vectors of ten thousand to
twenty million parameters; momentum and plain SGD, weight decay, the policy's mix weights and plain averaging.
"""
import math

import numpy as np
import torch

import paper_2009_05766_amd as nm

SIGMA = float(np.float32(1e-3 ** 0.5))      # standard deviation of the synthetic gradient
MOST_BYTES, MOST_FLOPS = 14.4e9, 3.2e11     # no drawn case needs more than the largest listed one


def _perceptron(name, dims, M, batch, dtype, iters, **more):
    return dict({"name": name, "kind": "train", "call": "run", "model": "perceptron", "dims": dims, "M": M, "batch": batch,
                 "dtype": dtype, "rows": 4096, "iters": iters, "lr": 0.01, "momentum": 0.9, "decay": 0.0, "averaging": False,
                 "fused": False}, **more)


def _flat(name, D, M, call, **more):
    return dict({"name": name, "kind": "train", "call": call, "model": "flat", "D": D, "M": M, "iters": 1, "lr": 0.1,
                 "momentum": 0.9, "decay": 0.0, "averaging": False, "fused": False}, **more)


def listed():
    return [
        # the smallest model: softmax regression on 256 features, two groups of four workers; latency is everything
        _perceptron("softmax_256", "256-10", 8, 32, "f32", 16, rows=1024, lr=0.05, momentum=0.0),
        # softmax regression on 28 x 28 images
        _perceptron("softmax_784", "784-10", 16, 64, "f32", 8),
        # the small perceptron on 28 x 28 images
        _perceptron("mlp_784", "784-512-10", 16, 64, "f32", 4),
        # a perceptron on 32 x 32 x 3 images in float32, the batch of the CIFAR experiments, weight decay
        _perceptron("mlp_3072_f32", "3072-1024-10", 32, 128, "f32", 1, decay=1e-4),
        # widths and a batch that are multiples of nothing, bfloat16 operands
        _perceptron("mlp_odd_bf16", "784-500-300-10", 16, 100, "bf16", 2),
        # the large perceptron: 128 workers, bfloat16 operands
        _perceptron("mlp_3072_bf16", "3072-1024-1024-10", 128, 128, "bf16", 1),
        # the same network on fewer workers with the update applied by the weight-gradient kernels
        _perceptron("mlp_3072_bf16_fused", "3072-1024-1024-10", 48, 128, "bf16", 1, fused=True),
        # a MobileNet-sized vector on few workers
        _flat("flat_4m", 4_231_976, 8, "step"),
        # a ResNet18-sized vector on 64 workers: the headline workload
        _flat("flat_11m", 11_200_000, 64, "step"),
        # a VGG19-sized vector, gradient generated by the update kernel, plain averaging
        _flat("flat_20m_fused", 20_000_000, 32, "run", fused=True, averaging=True),
        # the paper's own schedule on the small perceptron
        dict(_perceptron("async_mlp_784", "784-512-10", 16, 64, "f32", 64), kind="async"),
        # consensus distance and checkpoint copies of ResNet18-sized vectors
        dict(_flat("snapshot_11m", 11_200_000, 32, "step"), kind="snapshot"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    while True:
        c = _drawn(rng)
        w = work(c)
        # the state (four matrices) and what exact() keeps of it have to fit the card several times
        if w["bytes"] <= MOST_BYTES and w["flops"] <= MOST_FLOPS and c["M"] * _size(c) <= 720e6:
            return c


def _drawn(rng):
    pick = rng.random()
    M = _log(rng, 2, 128)
    common = {"momentum": rng.choice([0.9, 0.9, 0.0]), "decay": rng.choice([0.0, 0.0, 1e-4]), "averaging": rng.random() < 0.2}
    if pick < 0.28 or pick >= 0.90:                  # flat vectors and their snapshots
        fused = rng.random() < 0.3
        c = _flat("", _log(rng, 10_000, 20_000_000), M, "run" if fused or rng.random() < 0.5 else "step", **common)
        if pick >= 0.90:
            c["kind"] = "snapshot"
        else:
            c["fused"] = fused
            if rng.random() < 0.25:
                c["kind"], c["fused"], c["iters"] = "async", False, rng.choice([8, 16, 32])
        c["M"] = max(2, min(c["M"], int(700e6 // c["D"])))
    else:
        bf16 = rng.random() < 0.4
        features = rng.choice([784, 3072, _log(rng, 64, 1024), _log(rng, 64, 3072), 256 * rng.randint(1, 4)])
        classes = rng.choice([10, 10, rng.randint(2, 32)])
        layers = rng.choice([0, 1, 1, 2]) if not bf16 else rng.choice([1, 1, 2])
        hidden = [rng.choice([_log(rng, 32, 1024), 64 * rng.randint(1, 16), 128 * rng.randint(1, 8)]) for _ in range(layers)]
        batch = rng.choice([32, 64, 128, _log(rng, 8, 256)])
        fused = bf16 and rng.random() < 0.35
        if fused:                                    # only networks with a matrix-core layer have the fused variant
            features, hidden, batch = 128 * rng.randint(1, 24), [128 * rng.randint(1, 8) for _ in range(layers)], 32 * rng.randint(1, 4)
        c = _perceptron("", "-".join(str(d) for d in [features] + hidden + [classes]), M, batch, "bf16" if bf16 else "f32",
                        rng.choice([1, 2, 4]), rows=rng.choice([500, 1024, 2000]), fused=fused, **common)
        if not fused and rng.random() < 0.2:
            c["kind"], c["iters"] = "async", rng.choice([16, 32, 64])
    del c["name"]
    return c


# ---- sizes ---------------------------------------------------------------------------------------------------------

def _dims(case):
    return [int(d) for d in case["dims"].split("-")] if case["model"] == "perceptron" else []


def _size(case):
    d = _dims(case)
    return sum(d[k] * d[k + 1] + d[k + 1] for k in range(len(d) - 1)) if d else case["D"]


def _padded(D):
    return -(-D // nm.NETMAX_TILE) * nm.NETMAX_TILE


def work(case):
    D, M, n, dims = _size(case), case["M"], case["iters"], _dims(case)
    if case["kind"] == "snapshot":                   # x once for the distance and the copy, v once; both copies written
        return {"bytes": 16.0 * M * D, "flops": 6.0 * M * D}
    rows = (1 if case["kind"] == "async" else M) * n             # worker-iterations
    flops = 8.0 * D * rows
    features = 0.0
    if dims:
        flops += rows * case["batch"] * (6.0 * sum(dims[k] * dims[k + 1] for k in range(len(dims) - 1)) - 2.0 * dims[0] * dims[1])
        features = float(rows) * case["batch"] * dims[0] * (2 if case["dtype"] == "bf16" else 4)
    # per worker-iteration: x, v in, x', v' out; flat models and unfused perceptrons also leave the gradient
    state = 16 if case["fused"] and dims else 20
    passes = rows
    if case["kind"] == "async":
        state += 4                                   # the peer's row
    elif state * D * M <= 64e6:
        passes = M                                   # a state that fits on the chip has to come in and go out once per call
    return {"bytes": float(state) * D * passes + features, "flops": flops}


# ---- inputs --------------------------------------------------------------------------------------------------------

def _policy(case, seed):
    """Lognormal link speeds, normalised row by row with a floor, and the weight that makes the largest mix weight 1/4;
    iteration times are the inverse speeds."""
    M = case["M"]
    rng = np.random.default_rng([seed, 1])
    s = np.exp(np.triu(rng.standard_normal((M, M)), 1))
    s = np.triu(s, 1) + np.triu(s, 1).T
    P = s / s.sum(axis=1, keepdims=True)
    off = ~np.eye(M, dtype=bool)
    P[off] = np.maximum(P[off], 1.0 / (4.0 * M))
    P /= P.sum(axis=1, keepdims=True)
    lr = float(np.float32(case["lr"]))
    rho = float(np.float32(P[off].min() / (4.0 * lr)))
    t = np.zeros((M, M))
    t[off] = s.max() / s[off]
    return P, rho, t


def _rows(case, seed):
    """Initial parameters (a shared draw and a tenth of it per worker) and a momentum as training has it: [M, D] each."""
    D, M, dims = _size(case), case["M"], _dims(case)
    gen = torch.Generator(device="cuda").manual_seed(seed * 7 + 3)
    x = torch.randn((M, D), generator=gen, device="cuda")
    x *= 0.1
    x += torch.randn((1, D), generator=gen, device="cuda")
    if dims:
        scale, o = torch.zeros(D, device="cuda"), 0
        for k in range(len(dims) - 1):
            scale[o:o + dims[k] * dims[k + 1]] = 1.0 / math.sqrt(dims[k])
            o += dims[k] * dims[k + 1] + dims[k + 1]
        x *= scale
        v = torch.randn((M, D), generator=gen, device="cuda") * 1e-3
    else:
        x *= 0.1
        v = torch.randn((M, D), generator=gen, device="cuda") * 0.05
    if case["momentum"] == 0.0:
        v.zero_()
    return x, v


def _data(case, seed):
    """Shards of unequal sizes; every class a cluster.  float32: normal features; bfloat16: pixels in (0, 1)."""
    dims, M, n = _dims(case), case["M"], case["rows"]
    off = np.concatenate([[0], np.cumsum([n - (37 * i) % 101 for i in range(M)])]).astype(np.int64)
    total = int(off[-1])
    gen = torch.Generator(device="cuda").manual_seed(seed * 7 + 4)
    labels = torch.randint(0, dims[-1], (total,), generator=gen, device="cuda", dtype=torch.int32)
    bf16 = case["dtype"] == "bf16"
    make = torch.rand if bf16 else torch.randn
    means = make((dims[-1], dims[0]), generator=gen, device="cuda")
    feats = torch.empty((total, dims[0]), device="cuda", dtype=torch.bfloat16 if bf16 else torch.float32)
    for r in range(0, total, 65536):
        some = feats[r:r + 65536]
        some.copy_(0.7 * make(some.shape, generator=gen, device="cuda") + 0.3 * means[labels[r:r + 65536].long()])
    return feats, labels, off


def _draw_seed(seed):
    return 20090576 + 1000003 * seed


def prepare(case, seed):
    P, rho, t = _policy(case, seed)
    dims, D, M = _dims(case), _size(case), case["M"]
    more = {}
    if dims:
        feats, labels, off = _data(case, seed)
        more = dict(dims=dims, batch=case["batch"], gemm_in=nm.NETMAX_BF16 if case["dtype"] == "bf16" else nm.NETMAX_F32, feats=feats, labels=labels, shard_off=off)
    if case["averaging"]:
        more.update(mix_mode=nm.NETMAX_MIX_FIXED, fixed_weight=0.5)
    net = nm.NetMax(M=M, D=D, ld=_padded(D), model=nm.NETMAX_MLP if dims else nm.NETMAX_FLAT, lr=case["lr"], momentum=case["momentum"],
                    weight_decay=case["decay"], rho=rho, grad_sigma=0.0 if dims else SIGMA, seed=_draw_seed(seed), P=P, **more)
    x, v = _rows(case, seed)
    net.set("x", x)
    net.set("v", v)
    state = {"case": case, "net": net, "at": 0}
    if case["fused"]:
        nm.netmax_set_fusion(net.ctx, True)
    if case["kind"] == "async":
        nm.netmax_set_activity(net.ctx, nm.netmax_activity(t, P))
        state["active"] = torch.zeros(case["iters"], dtype=torch.int32, device="cuda")
        state["peers"] = torch.zeros(case["iters"], dtype=torch.int32, device="cuda")
    return state


# ---- one pass ------------------------------------------------------------------------------------------------------

def run(state):
    case, net, at = state["case"], state["net"], state["at"]
    state["at"] = at + case["iters"]
    if case["kind"] == "snapshot":
        return {"distance": net.consensus_dist(), "x": net.get("x"), "v": net.get("v")}
    if case["kind"] == "async":
        nm.netmax_async_run(net.ctx, at, case["iters"], state["active"], state["peers"])
        out = {"active": state["active"], "peers": state["peers"]}
    else:
        if case["call"] == "run":
            net.run(at, case["iters"])
        else:
            net.step(at)
        out = {"peers": net.peers}
    out["x"], out["v"] = net.params(), net.v
    if case["model"] == "flat":
        out["g"] = net.g
    elif case["kind"] == "train":                    # the asynchronous schedule leaves the losses of idle workers alone
        out["loss"] = net.losses()
    return out


# ---- the same in 64 bits -------------------------------------------------------------------------------------------

_MASK = 0xFFFFFFFF


def _philox(c0, c1, c2, c3, k0, k1):
    """Philox4x32-10 on int64 tensors (or broadcastable integers) that hold 32-bit words."""
    for _ in range(10):
        a, b = c0 * 0xD2511F53, c2 * 0xCD9E8D57      # the low 64 bits: products of int64 tensors wrap
        c0, c1, c2, c3 = ((b >> 32) & _MASK) ^ c1 ^ k0, b & _MASK, ((a >> 32) & _MASK) ^ c3 ^ k1, a & _MASK
        k0, k1 = (k0 + 0x9E3779B9) & _MASK, (k1 + 0xBB67AE85) & _MASK
    return c0, c1, c2, c3


def _words(seed, stream, block, worker, it):
    t = lambda a: a if isinstance(a, torch.Tensor) else torch.tensor(a, dtype=torch.int64)  # noqa: E731
    return _philox(t(block), t(worker), t(it & _MASK), t(it >> 32), seed & _MASK, (seed >> 32) ^ stream)


def _thresholds(p):
    last = int(np.nonzero(p > 0)[0][-1])
    c = np.floor(np.ldexp(np.cumsum(p), 32) + 0.5)
    c[last:] = 2.0 ** 32
    return c, last


def _pick(table, u):
    c, last = table
    return min(int(np.searchsorted(c, float(u), side="right")), last)


def _noise(case, seed, it, workers, j0, j1):
    """The synthetic gradient of the listed workers, columns j0 .. j1 - 1 (both multiples of four), float64 on the GPU."""
    block = torch.arange(j0 // 4, j1 // 4, device="cuda", dtype=torch.int64)[None, :]
    w = _words(_draw_seed(seed), 2, block, torch.tensor(workers, device="cuda", dtype=torch.int64)[:, None], it)
    u = [((q >> 9).double() + 0.5) * 2.0 ** -23 for q in w]
    z = []
    for a, b in ((u[0], u[1]), (u[2], u[3])):
        r = torch.sqrt(-2.0 * torch.log(a))
        z += [r * torch.cos(2.0 * math.pi * b), r * torch.sin(2.0 * math.pi * b)]
    return SIGMA * torch.stack(z, dim=2).reshape(len(workers), j1 - j0)


def _gradient(dims, x, feats, labels):
    """Mean cross-entropy and its gradient of one worker's ReLU perceptron; all float64."""
    at, o, acts = [], 0, [feats]
    for k in range(len(dims) - 1):
        at.append((o, o + dims[k] * dims[k + 1], o + dims[k] * dims[k + 1] + dims[k + 1]))
        o = at[-1][2]
    for k, (a, b, c) in enumerate(at):
        z = acts[-1] @ x[a:b].view(dims[k], dims[k + 1]) + x[b:c]
        acts.append(z if k + 2 == len(dims) else z.clamp(min=0.0))
    n = feats.shape[0]
    logp = torch.log_softmax(acts[-1], dim=1)
    loss = -logp.gather(1, labels[:, None].long()).mean()
    dz = torch.exp(logp)
    dz[torch.arange(n, device="cuda"), labels.long()] -= 1.0
    dz /= n
    g = torch.empty_like(x)
    for k in range(len(at) - 1, -1, -1):
        a, b, c = at[k]
        g[a:b] = (acts[k].T @ dz).reshape(-1)
        g[b:c] = dz.sum(dim=0)
        if k:
            dz = (dz @ x[a:b].view(dims[k], dims[k + 1]).T) * (acts[k] > 0)
    return loss, g


def _tiles(rows):
    """[M, D] in the layout of the library's buffers."""
    M, D = rows.shape
    out = torch.zeros((_padded(D) // nm.NETMAX_TILE, M, nm.NETMAX_TILE), device="cuda", dtype=torch.float64)
    full = D // nm.NETMAX_TILE
    if full:
        out[:full] = rows[:, :full * nm.NETMAX_TILE].reshape(M, full, nm.NETMAX_TILE).permute(1, 0, 2)
    if D % nm.NETMAX_TILE:
        out[full, :, :D % nm.NETMAX_TILE] = rows[:, full * nm.NETMAX_TILE:]
    return out.reshape(-1)


def exact(case, seed):
    P, rho, t = _policy(case, seed)
    dims, D, M = _dims(case), _size(case), case["M"]
    x, v = _rows(case, seed)
    if case["kind"] == "snapshot":
        far = 0.0
        for j in range(0, D, 1 << 18):
            some = x[:, j:j + (1 << 18)].double()
            far += float((some - some.mean(dim=0)).square().sum())
        pad = lambda a: torch.nn.functional.pad(a, (0, _padded(D) - D))  # noqa: E731
        return {"distance": far, "x": pad(x), "v": pad(v)}
    lr, mu, wd = (float(np.float32(case[k])) for k in ("lr", "momentum", "decay"))
    tables = [_thresholds(P[i]) for i in range(M)]
    weight = lambda i, m: 0.0 if m == i else 0.5 if case["averaging"] else lr * rho / P[i, m]  # noqa: E731
    key = _draw_seed(seed)
    peer_of = lambda i, it: _pick(tables[i], int(_words(key, 0, 0, i, it)[0]))  # noqa: E731
    if dims:
        feats, labels, off = _data(case, seed)
        blocks = torch.arange((case["batch"] + 3) // 4, dtype=torch.int64)

        def gradient(i, row, it):
            u = torch.stack(_words(key, 1, blocks, i, it), dim=1).reshape(-1)[:case["batch"]]
            at = (int(off[i]) + ((u * int(off[i + 1] - off[i])) >> 32)).cuda()
            return _gradient(dims, row, feats[at].double(), labels[at])
    x, v = x.double(), v.double()
    g = torch.empty_like(x) if not dims else None
    loss = torch.zeros(M, device="cuda", dtype=torch.float64)
    if case["kind"] == "async":
        speed = np.array([1.0 / sum(t[i, m] * P[i, m] for m in range(M) if m != i) for i in range(M)])
        act = _thresholds(speed / speed.sum())
        g = torch.zeros_like(x) if not dims else None
        for k in range(case["iters"]):
            i = _pick(act, int(_words(key, 3, 0, 0, k)[0]))
            m = peer_of(i, k)
            if dims:
                loss[i], gi = gradient(i, x[i], k)
            else:
                gi = g[i] = _noise(case, seed, k, [i], 0, -(-D // 4) * 4)[0, :D]
            v[i] = mu * v[i] + gi + wd * x[i]
            h = x[i] - lr * v[i]
            x[i] = h - weight(i, m) * (h - x[m])
    else:
        for it in range(case["iters"]):
            peers = [peer_of(i, it) for i in range(M)]
            w = torch.tensor([weight(i, m) for i, m in enumerate(peers)], device="cuda", dtype=torch.float64)[:, None]
            if dims:
                for i in range(M):
                    loss[i], gi = gradient(i, x[i], it)
                    v[i] = mu * v[i] + gi + wd * x[i]
                h = x - lr * v
                x = h - w * (h - x[peers])
            else:
                step = max(4, (1 << 24) // M // 4 * 4)
                for j in range(0, D, step):
                    end = min(D, j + step)
                    g[:, j:end] = _noise(case, seed, it, list(range(M)), j, j + -(-(end - j) // 4) * 4)[:, :end - j]
                    v[:, j:end] = mu * v[:, j:end] + g[:, j:end] + wd * x[:, j:end]
                    h = x[:, j:end] - lr * v[:, j:end]
                    x[:, j:end] = h - w * (h - x[peers, j:end])
    out = {"peers": None, "x": _tiles(x), "v": _tiles(v)}
    if case["kind"] == "async":
        out["active"] = None
    if dims:
        if case["kind"] == "train":
            out["loss"] = loss
        # A hidden unit whose input is zero within float32 rounding passes its error back or not, whichever way the sum was
        # rounded; the gradient jumps there by _jump(), far more than a float32 sum is off, so its value in 64 bits says
        # nothing about the sums.  (With bfloat16 operands there are such units in every pass, on both sides of a comparison.)
        if len(dims) > 2 and case["dtype"] == "f32":
            out["v"] = None
    else:
        out["g"] = _tiles(g)
    return out


# ---- how far another correct implementation may be off ----------------------------------------------------------------

def _jump(case):
    """Relative change of the gradient of all workers when one ReLU decision of one worker flips: one of the batch x (active
    half of the units) terms of that worker's gradient."""
    hidden = min(_dims(case)[1:-1], default=case["batch"])
    return 1.0 / math.sqrt(case["batch"] * hidden / 2.0 * case["M"])


def tolerance(case):
    if case["kind"] == "snapshot":
        return {"rel": 1e-9, "max": 1e-9}
    if case["model"] == "flat":                      # against float64: 6.6e-8 and 6e-7 at the most
        return {"rel": 1e-6, "max": 4e-6}
    if len(_dims(case)) == 2 and case["dtype"] == "f32":         # 1.5e-7 and 1.1e-6
        return {"rel": 2e-6, "max": 2e-5}
    if case["dtype"] == "f32":                       # 4e-7, or 9e-4 where a ReLU decision flipped
        return {"rel": min(0.03, 4.0 * _jump(case)), "max": 0.99}
    # the same operands rounded to bfloat16, all sums in float64: up to 1.4e-3, by flipped decisions and by activations that
    # round to the other neighbour
    return {"rel": min(0.03, 0.006 + _jump(case)), "max": 0.99}
