"""Whole iterations of softmax-regression models in one kernel, at the edges of how its workgroups share the work."""
import numpy as np
import pytest
import torch

import paper_2009_05766_amd as nm
from harness import inputs_of, make_gpu, make_oracle, rel_err_rows
from netmax_inputs import workload
from whole_iteration_cases import GROUPS_OF_UNITS, ONE_WORKGROUP, SLICES, SMALL

pytestmark = pytest.mark.gpu


def _in_one_launch(w, inp, n):
    """Whether netmax_run makes n iterations in one launch whose workgroups wait for each other: with a patience of no polls such a launch, and only
    such a one, reports a fault."""
    net = make_gpu(w, inp)
    nm.netmax_set_barrier_patience(net.ctx, 0)
    net.run(0, n)
    try:
        net.consensus_dist()
        return False
    except nm.NetmaxError as e:
        assert e.code == nm.NETMAX_EDEVICE
        return True
    finally:
        net.close()


def _run_is_calls_and_oracle(over, runs, name="cfg1", kernel=SMALL):
    """kernel: which one makes the longest of the runs in one launch, None: none."""
    w = workload(name, **over)
    inp = inputs_of(w)
    inp["labels"] = np.minimum(inp["labels"], w.dims[-1] - 1).astype(np.int32)
    assert _in_one_launch(w, inp, max(runs)) == (kernel is not None)
    calls, run, o = make_gpu(w, inp), make_gpu(w, inp), make_oracle(w, inp)
    it = 0
    for n in runs:
        run.run(it, n)
        for k in range(n):
            calls.step(it + k)
            assert np.array_equal(calls.peers.cpu().numpy(), o.step(it + k))
        it += n
        assert torch.equal(run.peers, calls.peers)
        for what in ("x", "v", "g"):
            assert torch.equal(run.get(what), calls.get(what)), (what, it)
        assert torch.equal(run.losses(), calls.losses())
    # per iteration a few roundings of every parameter, and the gradient's 1e-5 scaled by the learning rate: 1e-4 over a short run
    assert rel_err_rows(run.get("x").cpu().numpy(), o.X) < 1e-4
    # a row's loss is the logarithm of a sum of 1 or more, which is rounded to 2^-24 of itself: a few of those where the loss is next to zero
    np.testing.assert_allclose(run.losses().cpu().numpy(), o.loss, rtol=1e-4, atol=2.0**-22)
    assert run.consensus_dist() == pytest.approx(o.consensus_dist(), rel=1e-4)      # also reads the barrier's fault flag
    calls.close(), run.close()


@pytest.mark.parametrize("over", [dict(M=3, dims=(7, 3), batch=512, n_per_worker=700), dict(M=3, dims=(7, 3), batch=513, n_per_worker=700),
                                  dict(M=2, dims=(5, 4), batch=1024, n_per_worker=90)])
def test_batches_beyond_the_threads(over):
    """A workgroup has 512 threads; every row of a larger batch has to be drawn and to have its label."""
    _run_is_calls_and_oracle(over, (3, 1, 2, 9))


@pytest.mark.parametrize("dims", [(4, 3), (1, 2), (6, 1), (1, 1)])
def test_divisors_of_one(dims):
    """One piece per data row, one class: positions are divided by 1."""
    _run_is_calls_and_oracle(dict(M=3, dims=dims, batch=24, n_per_worker=50), (2, 1, 9))


@pytest.mark.parametrize("kernel,over", ONE_WORKGROUP)
def test_whole_iterations(kernel, over):
    _run_is_calls_and_oracle(over, (1, 34, 2), kernel=kernel)


def test_runs_on_several_streams():
    """Launches whose workgroups wait for each other run one after the other on a device: two contexts on streams of their own, their runs enqueued
    alternately, and one of them gone before the other runs again."""
    w = workload("cfg1", M=8)
    inp = inputs_of(w)
    calls = make_gpu(w, inp)
    for k in range(60):
        calls.step(k)
    nets = []
    for _ in range(2):
        with torch.cuda.stream(torch.cuda.Stream()):
            nets.append(make_gpu(w, inp))
    torch.cuda.synchronize()
    for k in range(0, 30, 10):
        for net in nets:
            net.run(k, 10)
    nets[0].run(30, 30)
    torch.cuda.synchronize()
    assert torch.equal(nets[0].get("x"), calls.get("x")) and nets[0].consensus_dist() == calls.consensus_dist()
    nets[0].close()
    nets[1].run(30, 30)
    torch.cuda.synchronize()
    assert torch.equal(nets[1].get("x"), calls.get("x")) and nets[1].consensus_dist() == calls.consensus_dist()
    nets[1].close(), calls.close()


@pytest.mark.parametrize("kernel,over", SLICES)
def test_iterations_in_slices(kernel, over):
    _run_is_calls_and_oracle(dict(n_per_worker=over["batch"] + 7, **over), (1, 18, 2), "cfg2", kernel)


@pytest.mark.parametrize("dims", [(784, 10), (104, 96, 10)])
def test_workgroups_that_give_up_are_reported(dims):
    """Patience of zero polls: every wait of the kernel gives up at once, the launch ends, the next consensus distance reports it."""
    w = workload("cfg2", M=4, dims=dims, batch=64, n_per_worker=70)
    inp = inputs_of(w)
    net, calls = make_gpu(w, inp), make_gpu(w, inp)
    nm.netmax_set_barrier_patience(net.ctx, 0)
    net.run(0, 9)
    with pytest.raises(nm.NetmaxError) as e:
        net.consensus_dist()
    assert e.value.code == nm.NETMAX_EDEVICE
    nm.netmax_set_barrier_patience(net.ctx, 1 << 24)
    net.consensus_dist()                                     # the flag is cleared; the parameters stay what they are
    again = make_gpu(w, inp)
    again.run(0, 9)
    for k in range(9):
        calls.step(k)
    assert torch.equal(again.get("x"), calls.get("x"))
    net.close(), calls.close(), again.close()


@pytest.mark.parametrize("kernel,over", GROUPS_OF_UNITS)
def test_iterations_of_resident_perceptrons(kernel, over):
    """One hidden layer: every workgroup keeps 32 units of a worker.  All state, losses and hidden activations are the separate calls' bits;
    the oracle bounds them until a ReLU decision next to zero differs (the tolerance is the one of the other short perceptron runs)."""
    w = workload("cfg2", n_per_worker=over["batch"] + 7, **over)
    inp = inputs_of(w)
    hyper = dict(momentum=0.9, weight_decay=1e-4)
    assert _in_one_launch(w, inp, 18) == (kernel is not None)
    calls, run, o = make_gpu(w, inp, **hyper), make_gpu(w, inp, **hyper), make_oracle(w, inp, **hyper)
    for net in (calls, run):
        net.x_b.fill_(3.0)                                   # every element of the next parameters has to be written
    it = 0
    for n in (1, 18, 2):
        run.run(it, n)
        for k in range(n):
            calls.step(it + k)
            if it + k < 3:
                assert np.array_equal(calls.peers.cpu().numpy(), o.step(it + k))
        if it == 0:
            assert rel_err_rows(run.get("x").cpu().numpy(), o.X) < 1e-5
        it += n
        assert torch.equal(run.peers, calls.peers)
        for what in ("x_a", "x_b", "v", "g"):
            assert torch.equal(getattr(run, what), getattr(calls, what)), (what, it)
        assert torch.equal(run.losses(), calls.losses())
        assert torch.equal(run.hidden(1), calls.hidden(1))
    run.consensus_dist()                                     # reads the barrier's fault flag
    calls.close(), run.close()


@pytest.mark.parametrize("dims,batch", [((784, 10), 64), ((104, 96, 10), 64), ((104, 96, 10), 32)])
@pytest.mark.parametrize("skip", [0, 1, 2, 3])
def test_features_that_start_anywhere(dims, batch, skip):
    """Features inside a larger buffer: netmax_run gives the separate calls' bits, whichever kernels read them."""
    w = workload("cfg2", M=3, dims=dims, batch=batch, n_per_worker=90)
    inp = inputs_of(w)
    flat = torch.zeros(inp["feats"].size + 8, device="cuda")
    inp["feats"] = flat[skip:skip + inp["feats"].size].copy_(torch.from_numpy(inp["feats"]).flatten()).view(inp["feats"].shape)
    inp["labels"] = torch.from_numpy(inp["labels"]).cuda()
    calls, run = make_gpu(w, inp, momentum=0.9), make_gpu(w, inp, momentum=0.9)
    assert run.feats.data_ptr() % 16 == 4 * skip % 16
    run.run(0, 9)
    for k in range(9):
        calls.step(k)
    for what in ("x_a", "x_b", "v", "g"):
        assert torch.equal(getattr(run, what), getattr(calls, what)), what
    assert torch.equal(run.losses(), calls.losses())
    calls.close(), run.close()


@pytest.mark.parametrize("name,over,n", [
    # kernels that take a list of workers: one hidden layer, batches of 32 and 64, self pulls among the draws; softmax regression
    ("cfg2", dict(M=5, dims=(72, 96, 10), batch=32), 40), ("cfg2", dict(M=16, dims=(200, 64, 7), batch=64), 50), ("cfg2", dict(M=40, dims=(40, 32, 16), batch=64), 200),
    ("cfg2", dict(M=6, dims=(1100, 10), batch=40), 30), ("cfg2", dict(M=4, dims=(784, 10), batch=64), 30),
    # more steps than a window of the plan
    ("cfg2", dict(M=3, dims=(16, 32, 3), batch=32), 700),
])
def test_async_steps_in_place(name, over, n):
    """Asynchronous steps on the workers' rows where they lie: draws, x, v, the last gradient of every worker and its loss against the oracle's
    sequential steps; rows of workers that are never drawn keep their bits."""
    w = workload(name, n_per_worker=over["batch"] + 9, **over)
    inp = inputs_of(w)
    gpu, o = make_gpu(w, inp, momentum=0.9), make_oracle(w, inp, momentum=0.9)
    p_act = np.full(w.M, 1.0 / (w.M - 1))
    p_act[1] = 0.0                                           # never active
    x1 = gpu.get("x")[1].clone()
    nm.netmax_set_activity(gpu.ctx, p_act)
    active, peers = (torch.full((n,), -1, dtype=torch.int32, device="cuda") for _ in range(2))
    nm.netmax_async_run(gpu.ctx, 5, n, active, peers)
    o.set_activity(p_act)
    first = 12                                               # a ReLU decision next to zero may differ later on
    want = np.array([o.async_step(5 + k) for k in range(first)])
    assert np.array_equal(active[:first].cpu().numpy(), want[:, 0]) and np.array_equal(peers[:first].cpu().numpy(), want[:, 1])
    again = make_gpu(w, inp, momentum=0.9)
    nm.netmax_set_activity(again.ctx, p_act)
    a2, p2 = (torch.full((n,), -1, dtype=torch.int32, device="cuda") for _ in range(2))
    nm.netmax_async_run(again.ctx, 5, first, a2, p2)
    x = again.get("x")
    assert rel_err_rows(x.cpu().numpy(), o.X) < 1e-4 and rel_err_rows(again.get("v").cpu().numpy(), o.V) < 1e-4
    assert torch.equal(x[1], x1) and torch.equal(gpu.get("x")[1], x1)
    # step by step, every batch of one step: the same bits but for the forms that depend on the number of steps in a batch
    for k in range(first, n):
        nm.netmax_async_run(again.ctx, 5 + k, 1, a2[k:k + 1], p2[k:k + 1])
    assert torch.equal(active, a2) and torch.equal(peers, p2)
    assert rel_err_rows(gpu.get("x").cpu().numpy(), again.get("x").cpu().numpy()) < 1e-3
    gpu.close(), again.close()
