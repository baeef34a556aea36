"""Whole iterations of small softmax-regression models in one kernel, at the edges of how its workgroups share the work."""
import numpy as np
import pytest
import torch

from harness import inputs_of, make_gpu, make_oracle, rel_err_rows
from netmax_inputs import workload

pytestmark = pytest.mark.gpu


def _run_is_calls_and_oracle(over, runs):
    w = workload("cfg1", **over)
    inp = inputs_of(w)
    inp["labels"] = np.minimum(inp["labels"], w.dims[-1] - 1).astype(np.int32)
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
    _run_is_calls_and_oracle(over, (3, 1, 2))


@pytest.mark.parametrize("over", [
    # groups of draws: sixteen iterations, fifteen, five, one
    dict(M=3, dims=(20, 10), batch=64, n_per_worker=90), dict(M=3, dims=(21, 9), batch=65, n_per_worker=90), dict(M=2, dims=(6, 3), batch=200, n_per_worker=230),
    dict(M=2, dims=(3, 2), batch=600, n_per_worker=640),
    # peers counted by more than one wave, by every wave
    dict(M=65, dims=(24, 5), batch=9, n_per_worker=20), dict(M=256, dims=(12, 4), batch=4, n_per_worker=9),
    # matrix-instruction form: one, two and four row tiles; parts of one step, of odd and of even numbers of steps; few vectors and many
    dict(M=3, dims=(128, 10), batch=16, n_per_worker=40), dict(M=5, dims=(384, 16), batch=16, n_per_worker=40), dict(M=3, dims=(128, 7), batch=32, n_per_worker=40),
    dict(M=8, dims=(256, 10), batch=32, n_per_worker=40), dict(M=3, dims=(640, 3), batch=32, n_per_worker=40), dict(M=4, dims=(64, 16), batch=64, n_per_worker=80),
    dict(M=3, dims=(192, 2), batch=64, n_per_worker=80), dict(M=3, dims=(256, 10), batch=64, n_per_worker=80),
])
def test_whole_iterations(over):
    _run_is_calls_and_oracle(over, (1, 34, 2))


def test_runs_on_several_streams():
    """Launches whose workgroups wait for each other take turns on a device: two contexts on streams of their own, their runs enqueued
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
