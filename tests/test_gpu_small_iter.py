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
    np.testing.assert_allclose(run.losses().cpu().numpy(), o.loss, rtol=1e-4)
    assert run.consensus_dist() == pytest.approx(o.consensus_dist(), rel=1e-4)      # also reads the barrier's fault flag
    calls.close(), run.close()


@pytest.mark.parametrize("over", [dict(M=3, dims=(7, 3), batch=512, n_per_worker=700), dict(M=3, dims=(7, 3), batch=513, n_per_worker=700),
                                  dict(M=2, dims=(5, 4), batch=1024, n_per_worker=90)])
def test_batches_beyond_the_threads(over):
    """A workgroup has 512 threads; every row of a larger batch has to be drawn and to have its label."""
    _run_is_calls_and_oracle(over, (3, 1, 2))
