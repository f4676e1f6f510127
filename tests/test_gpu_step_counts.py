"""Forward and backward pass at the reduction lengths where the GEMMs' step loop begins, wraps and ends: one to eight steps of
32 over the widths (row GEMMs) and over an expert's rows (weight gradients), with and without a ragged last step, through
the C ABI, against the CPU oracle.  Bar as for the other shapes: max|gpu - oracle| <= 1e-2 * max|oracle| (bf16 storage of
the intermediates: a few 2^-9 each, fp32 accumulation)."""
import numpy as np
import pytest

import oracle
from paper_2603_06626_amd import workloads as wl
from tests.helpers import rel_max_err

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

TOL = 1e-2


@pytest.mark.parametrize("steps", [1, 2, 3, 4, 5, 6, 7, 8])
@pytest.mark.parametrize("ragged", [0, 8])
def test_reduction_lengths_match_the_oracle(steps, ragged):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from tests import gpu_util as gpu

    width = 32 * steps - ragged
    d, f, E, k = width, 32 * (9 - steps) - ragged, 2, 1
    rows = 32 * steps - ragged                  # expert 0; expert 1 gets the step count at the other end
    T = rows + 32 * (9 - steps) - ragged
    _, gates, t = wl.make_custom(T, d, f, E, k, routing="uniform", seed=5, stream=400 + 16 * ragged + steps)
    idx = (np.arange(T) >= rows).astype(np.int32).reshape(T, 1)
    layer = gpu.Layer(T, k, E, d, f)
    layer.build_plan(idx)
    dev = {n: gpu.to_dev(v) for n, v in t.items()}
    gw = gpu.to_dev(gates)
    y = layer.fwd(dev["x"], gw, dev["W1"], dev["W3"], dev["W2"])
    grads = layer.bwd(dev["x"], gw, dev["W1"], dev["W3"], dev["W2"], dev["dY"])
    w = oracle.bf16_bits_to_f32
    ref = oracle.moe_fwd(w(t["x"]), w(gates), idx, w(t["W1"]), w(t["W3"]), w(t["W2"]))
    ref_g = oracle.moe_bwd(w(t["x"]), w(gates), idx, w(t["W1"]), w(t["W3"]), w(t["W2"]), w(t["dY"]))
    assert rel_max_err(gpu.to_f64(y), ref) <= TOL
    for g, r in zip(grads, ref_g):
        assert rel_max_err(gpu.to_f64(g), r) <= TOL
