"""The two last-layer kernels at the edges of their tiles: gradients and losses against the oracle."""
import numpy as np
import pytest

from harness import inputs_of, make_gpu, make_oracle, rel_err_rows
from netmax_inputs import workload

pytestmark = pytest.mark.gpu

# as in test_gpu_tile_layers.py: fp32 sums of a few thousand products in another order; bfloat16 against the same operands
TOL = {"f32": 1e-5, "bf16": 1e-3}


@pytest.mark.parametrize("dtype,M,batch,dims", [
    # softmax regression too large for one workgroup, or with bfloat16 operands; one class, 16, 17 and 32 classes
    ("f32", 3, 64, (784, 10)), ("f32", 2, 200, (900, 17)), ("f32", 5, 17, (2500, 32)), ("f32", 2, 256, (801, 16)),
    ("bf16", 3, 64, (784, 10)), ("bf16", 2, 129, (37, 1)), ("bf16", 2, 16, (15, 32)),
    # above a hidden layer: batches around 16 .. 256, hidden widths around the steps of 16 and the eight waves' parts
    ("f32", 2, 15, (20, 17, 10)), ("f32", 2, 1, (20, 1, 2)), ("f32", 3, 100, (30, 129, 31)), ("f32", 2, 255, (30, 16, 16)),
    ("f32", 2, 128, (30, 1030, 10)), ("f32", 2, 256, (20, 131, 32)),
    ("bf16", 2, 100, (30, 300, 10)), ("bf16", 2, 33, (30, 1027, 17)), ("bf16", 2, 250, (20, 47, 32)),
])
def test_last_layer_at_its_edges(ora, dtype, M, batch, dims):
    w = workload("cfg5" if dtype == "bf16" else "cfg2", M=M, batch=batch, n_per_worker=batch + 5, dims=dims)
    inp = inputs_of(w)
    gpu, o = make_gpu(w, inp), make_oracle(w, inp, operands_bf16=dtype == "bf16")
    ora.set_threads(8)
    for it in (0, 3):
        gpu.local_step(it)
        o.local_step(it)
        G = gpu.get("g").cpu().numpy()
        assert np.all(G[:, w.D:] == 0)
        if w.dims[-1] == 1:
            assert np.all(G == 0) and np.all(o.G == 0)
        else:
            assert rel_err_rows(G, o.G) < TOL[dtype]
        np.testing.assert_allclose(gpu.losses().cpu().numpy(), o.loss, rtol=1e-4 if dtype == "bf16" else 1e-5, atol=1e-7)
    ora.set_threads(1)
    gpu.close()
