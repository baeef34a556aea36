"""The tiled layer kernels at the edges of their blocks, steps and load widths: gradients against the oracle."""
import numpy as np
import pytest

from harness import inputs_of, make_gpu, make_oracle, rel_err_rows
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
