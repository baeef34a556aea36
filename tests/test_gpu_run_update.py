"""netmax_run lets weight gradients apply the update to their columns (and the first layer's to those that are left); the separate
calls do it with the mix kernel.  Parameters, momentum, gradient and losses have to be the same bits, padding included, whichever kernels a shape takes."""
import numpy as np
import pytest
import torch

import paper_2009_05766_amd as nm
from harness import inputs_of, make_gpu
from kernel_cases import RUNS
from netmax_inputs import workload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name,M,batch,dims", [
    ("cfg2", 9, 64, (784, 10)), ("cfg2", 3, 200, (900, 17)), ("cfg5", 4, 33, (130, 32)),     # softmax regression
    ("cfg2", 5, 64, (70, 96, 10)), ("cfg2", 3, 32, (33, 64, 32, 7)),                            # batches of 32 and 64, fp32
    ("cfg2", 11, 128, (100, 132, 10)), ("cfg2", 3, 40, (130, 36, 40, 10)),                      # tiled, rows aligned
    ("cfg2", 3, 100, (75, 51, 10)), ("cfg2", 2, 300, (37, 41, 33)),                             # rows not aligned, W's end inside a group of four
    ("cfg5", 4, 100, (100, 60, 10)), ("cfg5", 3, 90, (61, 131, 10)), ("cfg5", 3, 64, (100, 128, 128, 10)),
    ("cfg5", 3, 64, (128, 128, 10)),                                                            # matrix-core layers: the separate mix
    ("cfg2", 3, 300, (40, 20)), ("cfg2", 3, 16, (50, 40)),                                      # one layer outside the last-layer kernels
    # from two million floats on every fp32 weight gradient updates its columns, the first layer's the remaining ones too
    ("cfg2", 16, 64, (784, 192, 10)), ("cfg2", 37, 32, (33, 1024, 32, 7)),                      # batches of 32 and 64
    ("cfg2", 21, 100, (784, 132, 40)), ("cfg2", 9, 128, (100, 804, 252, 10)),                   # tiled, rows aligned; 40 classes
    ("cfg2", 70, 40, (784, 40)), ("cfg2", 41, 50, (804, 68, 9, 33, 12)),                        # one layer; layers that do not update
])
@pytest.mark.parametrize("graph", [False, True])
def test_run_is_the_separate_calls(name, M, batch, dims, graph):
    w = workload(name, M=M, batch=batch, n_per_worker=batch + 3, dims=dims)
    inp = inputs_of(w)
    over = dict(momentum=0.9, weight_decay=1e-4)
    calls = make_gpu(w, inp, **over)
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        run = make_gpu(w, inp, **over)
        for net in (calls, run):
            net.x_b.fill_(3.0)                               # every element of the next parameters has to be written
        torch.cuda.synchronize()
        it = 0
        for n in (1, 2, 3):
            run.run(it, n, use_graph=graph)
            side.synchronize()
            for k in range(n):
                calls.step(it + k)
            torch.cuda.synchronize()
            it += n
            assert torch.equal(run.peers, calls.peers)
            for name_ in ("x_a", "x_b", "v", "g"):
                assert torch.equal(getattr(run, name_), getattr(calls, name_)), (name_, it)
            assert torch.equal(run.losses(), calls.losses())
    assert not np.array_equal(run.get("x").cpu().numpy(), inp["X0"])
    calls.close(), run.close()


@pytest.mark.parametrize("name,M,batch,dims", [
    # blocks of 64 columns with the update (one to three of them), data rows of every alignment and of fewer than four features
    ("cfg2", 3, 100, (101, 64, 10)), ("cfg2", 22, 128, (786, 192, 10)), ("cfg2", 5, 40, (3, 36, 10)), ("cfg2", 9, 100, (7, 132, 60, 10)),
    ("cfg2", 40, 90, (787, 148, 60, 10)),
    # 32 x 32 blocks whose rows four waves share, with the update; strips in two and three even parts on batches of 32 and 64
    ("cfg2", 4, 128, (131, 96, 10)), ("cfg2", 3, 256, (45, 68, 10)), ("cfg2", 2, 200, (66, 36)),
    ("cfg2", 3, 32, (70, 320, 10)), ("cfg2", 2, 64, (33, 544, 10)),
])
def test_run_with_narrow_layers(name, M, batch, dims):
    test_run_is_the_separate_calls(name, M, batch, dims, False)


@pytest.mark.parametrize("M,batch,dims,followed,last", RUNS)
@pytest.mark.parametrize("fused", [False, True])
def test_run_of_matrix_core_layers(M, batch, dims, followed, last, fused):
    if not fused:
        return test_run_is_the_separate_calls("cfg5", M, batch, dims, False)
    w = workload("cfg5", M=M, batch=batch, n_per_worker=batch + 3, dims=dims)
    inp = inputs_of(w)
    run, calls = (make_gpu(w, inp, momentum=0.9, weight_decay=1e-4) for _ in range(2))
    nm.netmax_set_fusion(run.ctx, True)
    run.run(0, 3)
    for k in range(3):
        calls.step(k)
    assert torch.equal(run.get("x"), calls.get("x")) and torch.equal(run.v, calls.v) and torch.equal(run.losses(), calls.losses())
    run.close(), calls.close()


@pytest.mark.parametrize("M,batch,dims", [c[:3] for c in RUNS if c[4]])
def test_graph_of_matrix_core_layers(M, batch, dims):
    """Every replay leaves g: the update in weight gradients that also write it."""
    test_run_is_the_separate_calls("cfg5", M, batch, dims, True)


@pytest.mark.parametrize("name,over", [("cfg2", dict(M=5, batch=24, n_per_worker=40, dims=(30, 20, 10))), ("cfg3", dict(M=7, D=5000)),
                                       ("cfg5", dict(M=2, batch=1024, n_per_worker=1100, dims=(20, 8)))])
@pytest.mark.parametrize("n", [1, 15, 16, 17, 35])
def test_draws_ahead_are_the_draws_of_each_iteration(name, over, n):
    """netmax_run draws up to sixteen iterations in one launch: iteration counts around that, and far from zero."""
    w = workload(name, **over)
    inp = inputs_of(w)
    run, calls = make_gpu(w, inp), make_gpu(w, inp)
    first = 2**32 - 3
    run.run(first, n)
    for k in range(n):
        calls.step(first + k)
    assert torch.equal(run.peers, calls.peers)
    assert torch.equal(run.get("x"), calls.get("x")) and torch.equal(run.v, calls.v)
    run.close(), calls.close()
