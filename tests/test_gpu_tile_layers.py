"""The tiled layer kernels at the edges of their blocks, steps and load widths: gradients against the oracle."""
import numpy as np
import pytest

from harness import inputs_of, make_gpu, make_oracle, rel_err_rows
from kernel_cases import ERRORS, FEW_CLASSES, FORWARD, SAME_BITS
from netmax_inputs import workload

pytestmark = pytest.mark.gpu

# A sum of n fp32 products in any order is off by at most n 2^-24 sum |a b|; with the cancellation of these sums 1e-5 of the
# gradient's norm (3072 terms).  bfloat16 operands against the oracle with the same operands: an activation on a rounding
# boundary moves by 2^-8 of itself, one of hundreds in a sum.
TOL = {"f32": 1e-5, "bf16": 1e-3}


@pytest.mark.parametrize("dtype,M,batch,dims", [
    # one block and its remainder in every direction: batches around 32, 64 and 128, widths around 32, 64 and 128,
    # contractions around one step (64 and 128) and of a single element more
    ("f32", 3, 31, (63, 33, 65, 10)), ("f32", 2, 33, (64, 64, 64, 40)), ("f32", 3, 65, (65, 127, 129, 10)),
    ("f32", 2, 128, (128, 96, 34, 33)), ("f32", 2, 129, (130, 68, 36, 10)), ("f32", 2, 257, (40, 44, 36, 5)),
    ("bf16", 3, 31, (63, 33, 65, 10)), ("bf16", 2, 33, (64, 64, 64, 40)), ("bf16", 3, 65, (65, 127, 129, 10)),
    ("bf16", 2, 127, (127, 130, 36, 33)), ("bf16", 2, 129, (130, 68, 36, 10)), ("bf16", 2, 257, (40, 44, 36, 5)),
    # load widths: features a multiple of four, outputs not (and the other way round), a weight offset that is not
    ("f32", 2, 100, (100, 50, 40, 10)), ("f32", 2, 100, (101, 52, 38, 10)), ("bf16", 2, 100, (100, 50, 40, 10)),
    ("bf16", 2, 100, (101, 52, 38, 10)),
    # enough blocks for the short-step form (512 blocks of 128 x 64)
    ("f32", 64, 128, (36, 513, 10)), ("bf16", 64, 128, (36, 513, 10)),
    # a batch of 64 in two workgroups for each group of 32 columns: few, the most (256), and one worker more
    ("f32", 2, 64, (8, 32, 10)), ("f32", 8, 64, (72, 512, 32, 10)), ("f32", 9, 64, (72, 512, 32, 10)),
    # general layers under and over matrix-core layers (bfloat16 copies in both orientations are wanted)
    ("bf16", 3, 64, (100, 128, 256, 10)), ("bf16", 3, 32, (128, 128, 100, 128, 10)), ("bf16", 2, 96, (60, 128, 40)),
])
def test_gradient_of_odd_layers(ora, dtype, M, batch, dims):
    w = workload("cfg5" if dtype == "bf16" else "cfg2", M=M, batch=batch, n_per_worker=batch + 7, dims=dims)
    inp = inputs_of(w)
    gpu, o = make_gpu(w, inp), make_oracle(w, inp, operands_bf16=dtype == "bf16")
    ora.set_threads(8)
    for it in (0, 3):
        gpu.local_step(it)
        o.local_step(it)
        G = gpu.get("g").cpu().numpy()
        assert np.all(G[:, w.D:] == 0)
        assert rel_err_rows(G, o.G) < TOL[dtype]
        np.testing.assert_allclose(gpu.losses().cpu().numpy(), o.loss, rtol=1e-4 if dtype == "bf16" else 1e-5)
    ora.set_threads(1)
    gpu.close()


@pytest.mark.parametrize("M,batch,dims,kernel", FEW_CLASSES)
def test_last_layer_of_few_classes(ora, M, batch, dims, kernel):
    test_gradient_of_odd_layers(ora, "bf16", M, batch, dims)


@pytest.mark.parametrize("dtype,M,batch,dims,kernel", FORWARD)
def test_gradient_of_long_contractions(ora, dtype, M, batch, dims, kernel):
    """The forward kernels for few blocks in every form, and either side of the lines to the others."""
    test_gradient_of_odd_layers(ora, dtype, M, batch, dims)


@pytest.mark.parametrize("dtype,M,batch,dims,kernel", ERRORS)
def test_errors_of_few_blocks(ora, dtype, M, batch, dims, kernel):
    """Their error kernels."""
    test_gradient_of_odd_layers(ora, dtype, M, batch, dims)


@pytest.mark.parametrize("few,many,batch,dims,among_few,among_many,sums", SAME_BITS)
def test_few_blocks_bit_for_bit(few, many, batch, dims, among_few, among_many, sums):
    """bfloat16 layers in few blocks have kernels of their own, which add in the order of those for many: a worker's gradient is the same among few
    workers and among many.  sums: the first layer's bias gradient, too."""
    runs = []
    for M in (few, many):
        w = workload("cfg5", M=M, batch=batch, n_per_worker=batch + 7, dims=dims)
        gpu = make_gpu(w, inputs_of(w))
        for it in (0, 3):
            gpu.local_step(it)
        g = gpu.get("g")[:few].cpu().numpy()
        if not sums:
            g[:, dims[0] * dims[1]:(dims[0] + 1) * dims[1]] = 0
        runs.append([gpu.hidden(l)[:few].cpu().numpy() for l in range(1, len(dims) - 1)] + [g])
        gpu.close()
    for a, b in zip(*runs):
        assert np.array_equal(a, b)


@pytest.mark.parametrize("M,batch,dims", [(7, 96, (640, 128)), (3, 64, (256, 128, 128)), (40, 32, (256, 512))])
def test_last_layer_of_aligned_width_adds_as_any_other(M, batch, dims):
    """A last layer on bfloat16 operands adds in the same order whether its classes are a multiple of 128 or four more that never win: the same losses bit
    for bit."""
    C, more = dims[-1], 4
    w = workload("cfg5", M=M, batch=batch, n_per_worker=batch + 7, dims=dims)
    inp = inputs_of(w)
    wide = workload("cfg5", M=M, batch=batch, n_per_worker=batch + 7, dims=(*dims[:-1], C + more))
    at = w.D - (dims[-2] + 1) * C                                    # the last layer's first parameter
    W = inp["X0"][:, at:at + dims[-2] * C].reshape(M, dims[-2], C)
    b = inp["X0"][:, at + dims[-2] * C:w.D]
    X = np.zeros((M, inputs_of(wide)["X0"].shape[1]), np.float32)
    X[:, :at] = inp["X0"][:, :at]
    X[:, at:wide.D] = np.concatenate([np.pad(W, ((0, 0), (0, 0), (0, more))).reshape(M, -1), np.pad(b, ((0, 0), (0, more)), constant_values=-1e30)], axis=1)
    losses = []
    for v, i in ((w, inp), (wide, dict(inp, X0=X))):
        gpu = make_gpu(v, i)
        gpu.local_step(1)
        losses.append(gpu.losses().cpu().numpy())
        gpu.close()
    assert np.isfinite(losses[0]).all() and np.array_equal(losses[0], losses[1])


def test_wide_fp32_layers_keep_what_is_not_finite():
    """Large fp32 layers multiply bfloat16 planes of their operands, which an infinity, or a number that rounds to one, does not
    survive: such blocks are computed again in fp32.  Activations against float64, block edges included."""
    import oracle
    w = workload("cfg2", M=64, batch=128, n_per_worker=130, dims=(36, 513, 10))
    inp = inputs_of(w)
    X = inp["X0"].copy()
    inf, big = np.float32(np.inf), np.float32(3.4e38)          # the latter lies above the largest bfloat16
    X[1, 3 * 513 + 7] = inf
    X[5, 35 * 513 + 512] = -inf
    X[9, 20 * 513 + 64] = np.float32(np.nan)
    X[13, 0] = big
    gpu = make_gpu(w, dict(inp, X0=X))
    gpu.local_step(2)
    h = gpu.hidden(1).cpu().numpy()
    idx = oracle.sample_batch(w.M, w.batch, inp["shard_off"], w.seed, 2)
    for i in range(w.M):
        a = inp["feats"][inp["shard_off"][i] + idx[i]].astype(np.float64)
        with np.errstate(invalid="ignore", over="ignore"):
            W = X[i, :36 * 513].reshape(36, 513).astype(np.float64)
            z = a @ W + X[i, 36 * 513:37 * 513]
            # 36 products and the bias, each addition off by at most 2^-24 of the sum of the magnitudes
            bound = 38 * 2.0**-24 * (np.abs(a) @ np.abs(W) + np.abs(X[i, 36 * 513:37 * 513]))
            want = np.where(z > 0, z, 0.0).astype(np.float32)
        assert np.array_equal(np.isinf(h[i]), np.isinf(want)) and not np.isnan(h[i]).any()
        fine = np.isfinite(want) & np.isfinite(bound)
        assert np.all(np.abs(h[i][fine].astype(np.float64) - np.where(z > 0, z, 0.0)[fine]) <= bound[fine])
    assert np.isinf(h).any() and h[13].max() > 1e37
    gpu.close()


@pytest.mark.parametrize("batch,dims", [
    # one step of 32 and its remainder, whole steps, steps and a remainder; features a multiple of four and not, outputs likewise
    (128, (36, 516, 10)), (128, (64, 513, 10)), (128, (96, 516, 10)), (128, (100, 516, 10)), (100, (101, 513, 10)), (65, (163, 516, 10)),
])
def test_wide_fp32_layers_against_64_bits(batch, dims):
    """Large fp32 layers multiply bfloat16 planes of their operands.  Every activation against float64, of ordinary operands (a lost
    product of planes is 2^-16 of a term, the bound some 2^-22 of the sum) and of operands near and below the smallest normal
    number, which planes do not hold: such blocks are computed again in fp32."""
    import oracle
    w = workload("cfg2", M=64, batch=batch, n_per_worker=130, dims=dims)
    inp = inputs_of(w)
    K, N = dims[0], dims[1]
    X, feats, off = inp["X0"].copy(), inp["feats"].copy(), inp["shard_off"]
    X[3, :K * N] *= np.float32(1e-37)                            # weights of which planes keep a part
    feats[off[5]:off[6]] *= np.float32(3e-37)                    # data rows likewise
    X[8, :K * N] *= np.float32(1e-20)                            # operands that planes hold, products that are subnormal numbers
    feats[off[8]:off[9]] *= np.float32(1e-20)
    X[11, 7:K * N:N] *= np.float32(1e-37)                        # one column of them
    X[14, :K * N] *= np.float32(1e-41)                           # subnormal weights
    gpu = make_gpu(w, dict(inp, X0=X, feats=feats))
    gpu.local_step(2)
    h = gpu.hidden(1).cpu().numpy().astype(np.float64)
    idx = oracle.sample_batch(w.M, w.batch, off, w.seed, 2)
    for i in range(w.M):
        a = feats[off[i] + idx[i]].astype(np.float64)
        W, b = X[i, :K * N].reshape(K, N).astype(np.float64), X[i, K * N:K * N + N].astype(np.float64)
        z = np.maximum(a @ W + b, 0.0)
        # K products and the bias: each addition off by at most 2^-24 of the sum of the magnitudes, or half the smallest number
        bound = (K + 2) * (2.0**-24 * (np.abs(a) @ np.abs(W) + np.abs(b)) + 2.0**-150)
        assert np.all(np.abs(h[i] - z) <= bound), (i, float((np.abs(h[i] - z) / bound).max()))
    assert 0 < h[3].max() < 1e-34 and 0 < h[14].max() < 1e-38
    gpu.close()


@pytest.mark.parametrize("hidden,call", [(2, "local_step"), (4, "run")])
def test_more_workgroups_than_one_direction_holds(hidden, call):
    """A wide first layer of few outputs with many workers: more than 2^32 work-items in the weight gradient's launch.  Every worker
    owns one data row, so its weight gradient is the product of that row and the bias gradient."""
    import torch
    import paper_2009_05766_amd as nm
    M, K, T = 130, 64 * 65535, nm.NETMAX_TILE
    dims = (K, hidden, 10)
    D = K * hidden + hidden + hidden * 10 + 10
    gen = torch.Generator(device="cuda").manual_seed(5)
    feats = torch.randn((M, K), generator=gen, device="cuda")
    labels = torch.arange(M, device="cuda", dtype=torch.int32) % 10
    net = nm.NetMax(M=M, D=D, ld=-(-D // T) * T, model=nm.NETMAX_MLP, dims=dims, batch=4, lr=0.01, momentum=0.9, rho=0.001, seed=3,
                    P=(np.ones((M, M)) - np.eye(M)) / (M - 1), feats=feats, labels=labels, shard_off=np.arange(M + 1))
    net.x_a.normal_(generator=gen).mul_(1e-3)
    net.x_a.view(-1, M, T)[-1, :, D % T:] = 0.0                      # the padding
    for buffer in (net.x_b, net.g):
        buffer.fill_(7.0)
    net.run(0, 1) if call == "run" else net.local_step(0)
    torch.cuda.synchronize()
    g = net.get("g", D)
    slope = g[:, K * hidden:K * hidden + hidden]
    assert int((slope != 0).any(dim=1).sum()) > M // 2               # some workers' units may all be off
    for i in range(M):
        want = feats[i][:, None] * slope[i][None, :]
        # four products of four equal rows and their sums, each rounded, on either side
        assert bool((g[i, :K * hidden].view(K, hidden) - want).abs().le(want.abs() * 2.0**-20 + 1e-30).all()), i
    if call == "run":                                                # v was 0: it is g now; every parameter has been written
        assert torch.equal(net.get("v", D), g)
        x = net.get("x", D)
        assert not bool((x == 7.0).any()) and bool(x.isfinite().all())
    net.close()


@pytest.mark.parametrize("dtype,M,batch,dims", [
    # steps shared by four waves: contractions around its step of 128 and of one to four elements, rows of data and of weights at
    # every alignment
    *[(t, 2, b, d) for t in ("f32", "bf16") for b, d in (
        (33, (127, 35, 33, 10)), (20, (129, 64, 10)), (128, (257, 51, 66, 10)), (31, (1, 40, 10)), (45, (2, 37, 9)), (32, (3, 36, 10)), (7, (4, 33, 10)),
        (64, (5, 2050, 10)), (100, (1023, 46, 10)))],
])
def test_gradient_where_waves_share_the_steps(ora, dtype, M, batch, dims):
    test_gradient_of_odd_layers(ora, dtype, M, batch, dims)


@pytest.mark.parametrize("dtype,M,batch,dims", [(t, 2, b, d) for t in ("f32", "bf16") for b, d in (
    # weight gradients: blocks of 64 and of 128 columns and their remainders, rows aligned or not, one to seven features or outputs,
    # batches around a step of 64
    (63, (65, 64, 10)), (65, (66, 65, 10)), (64, (130, 128, 192, 10)), (40, (5, 129, 193, 10)), (129, (6, 188, 7, 10)), (33, (7, 132, 5, 10)),
    (17, (2, 60, 3, 40)), (70, (90, 2, 61, 33)), (50, (64, 1, 130, 10)),
    # few blocks and batches from 128 on: four waves share the rows of 32 x 32 blocks
    (128, (31, 33, 10)), (130, (65, 97, 32, 10)), (255, (3, 40, 35, 10)), (161, (200, 2, 30)), (300, (34, 64, 66, 7)), (513, (5, 36, 10)))])
def test_weight_gradients_of_every_width(ora, dtype, M, batch, dims):
    test_gradient_of_odd_layers(ora, dtype, M, batch, dims)


@pytest.mark.parametrize("dtype,M,batch,dims", [
    # enough blocks for the larger forms: batches up to 32, 64 and more, weights in pieces and not, rows of any length
    ("f32", 128, 20, (149, 515, 10)), ("f32", 128, 32, (132, 516, 10)), ("bf16", 64, 20, (131, 515, 10)), ("bf16", 64, 32, (66, 516, 10)),
    ("f32", 40, 50, (130, 515, 10)), ("f32", 40, 64, (67, 516, 10)), ("bf16", 32, 50, (131, 515, 10)), ("bf16", 32, 64, (260, 516, 10)),
    ("bf16", 20, 100, (150, 515, 10)), ("bf16", 20, 128, (129, 516, 10)), ("bf16", 64, 100, (133, 513, 10)), ("bf16", 64, 128, (196, 516, 10)),
    # and one block less than the lines between them (in blocks of 32 x 64: 512 and 641, 1025; 256 of 128 x 64)
    ("f32", 114, 20, (149, 515, 10)), ("f32", 35, 50, (130, 515, 10)), ("f32", 28, 128, (130, 515, 10)), ("bf16", 28, 50, (131, 515, 10)),
    ("bf16", 28, 128, (129, 515, 10)), ("bf16", 29, 128, (129, 515, 10)),
    # more workers than 32-bit offsets reach over
    ("f32", 2049, 3, (3, 36, 3)), ("bf16", 2049, 3, (3, 36, 3)),
])
def test_activations_of_the_larger_forms(dtype, M, batch, dims):
    """Every activation of the first layer against float64 with the same operands."""
    import oracle
    w = workload("cfg5" if dtype == "bf16" else "cfg2", M=M, batch=batch, n_per_worker=batch + 7, dims=dims)
    inp = inputs_of(w)
    K, N, off = dims[0], dims[1], inp["shard_off"]
    gpu = make_gpu(w, inp)
    gpu.local_step(2)
    h = gpu.hidden(1).cpu().numpy().astype(np.float64)
    idx = oracle.sample_batch(w.M, w.batch, off, w.seed, 2)

    def operand(x):                                                  # to the nearest bfloat16, ties to even
        u = x.view(np.uint32)
        return (((u + 0x7FFF + ((u >> 16) & 1)) >> 16) << 16).view(np.float32)
    for i in range(M):
        a, W = inp["feats"][off[i] + idx[i]], inp["X0"][i, :K * N]
        if dtype == "bf16":
            a, W = (a.astype(np.uint32) << 16).view(np.float32), operand(W)
        a, W, b = a.astype(np.float64), W.reshape(K, N).astype(np.float64), inp["X0"][i, K * N:K * N + N].astype(np.float64)
        z = np.maximum(a @ W + b, 0.0)
        # K products and the bias, each addition off by at most 2^-24 of the sum of the magnitudes; stored as bfloat16 2^-8 more
        bound = (K + 2) * 2.0**-24 * (np.abs(a) @ np.abs(W) + np.abs(b)) + (2.0**-8 * z if dtype == "bf16" else 0.0)
        assert np.all(np.abs(h[i] - z) <= bound), i
    gpu.close()


@pytest.mark.parametrize("dtype,M,batch,dims", [
    # error kernel: blocks of 128 x 64 and 128 x 32 on either side of the line between them (128 and 256 of the former), weights in
    # pieces and not, one and two blocks of rows
    ("f32", 64, 128, (36, 516, 68, 10)), ("f32", 64, 100, (36, 513, 67, 10)), ("f32", 15, 128, (20, 516, 40, 10)), ("f32", 14, 127, (20, 515, 130, 10)),
    ("f32", 9, 200, (20, 516, 260, 10)),
    ("bf16", 64, 128, (36, 516, 68, 10)), ("bf16", 64, 100, (36, 513, 67, 10)), ("bf16", 29, 128, (20, 516, 40, 10)), ("bf16", 28, 127, (20, 515, 130, 10)),
    ("bf16", 16, 200, (20, 516, 260, 10)),
])
def test_errors_of_wide_layers(dtype, M, batch, dims):
    """The gradient of two hidden layers in float64 from the library's own activations: the same ReLU decisions, so what is left is
    the rounding of the sums (and of bfloat16 errors that lie between two numbers)."""
    import oracle
    w = workload("cfg5" if dtype == "bf16" else "cfg2", M=M, batch=batch, n_per_worker=batch + 7, dims=dims)
    inp = inputs_of(w)
    off = inp["shard_off"]
    gpu = make_gpu(w, inp)
    gpu.local_step(1)
    h1, h2, G = (t.cpu().numpy() for t in (gpu.hidden(1), gpu.hidden(2), gpu.get("g")))
    idx = oracle.sample_batch(w.M, w.batch, off, w.seed, 1)

    def operand(x):
        if dtype == "f32":
            return np.asarray(x, np.float64)
        u = np.ascontiguousarray(x, np.float32).view(np.uint32)
        return (((u + 0x7FFF + ((u >> 16) & 1)) >> 16) << 16).view(np.float32).astype(np.float64)
    want = np.zeros_like(G, dtype=np.float64)
    for i in range(M):
        rows = off[i] + idx[i]
        a, o, W, b = inp["feats"][rows], 0, [], []
        a = (a.astype(np.uint32) << 16).view(np.float32).astype(np.float64) if dtype == "bf16" else a.astype(np.float64)
        for k in range(3):
            n = dims[k] * dims[k + 1]
            W.append(operand(inp["X0"][i, o:o + n]).reshape(dims[k], dims[k + 1]))
            b.append(inp["X0"][i, o + n:o + n + dims[k + 1]].astype(np.float64))
            o += n + dims[k + 1]
        acts = [a, h1[i].astype(np.float64), h2[i].astype(np.float64)]
        z = acts[2] @ W[2] + b[2]
        e = np.exp(z - z.max(axis=1, keepdims=True))
        dz = (e / e.sum(axis=1, keepdims=True) - np.eye(dims[3])[inp["labels"][rows]]) / batch
        parts = []
        for k in (2, 1, 0):
            parts = [(acts[k].T @ operand(dz)).ravel(), dz.sum(axis=0)] + parts
            if k:
                dz = (operand(dz) @ W[k].T) * (acts[k] > 0)
        want[i, :o] = np.concatenate(parts)
    assert np.all(G[:, w.D:] == 0)
    assert rel_err_rows(G, want) < TOL[dtype]
    # and each layer's part by itself: the first one, which the error kernel's results make, is a fraction of the whole
    first = dims[0] * dims[1] + dims[1]
    assert rel_err_rows(G[:, :first], want[:, :first]) < 3 * TOL[dtype]
    gpu.close()
