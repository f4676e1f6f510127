"""Backward pass where its kernels change form, through the C ABI, against the CPU oracle.  Bar as for the other shapes:
max|gpu - oracle| <= 1e-2 * max|oracle| (bf16 storage of the intermediates: a few 2^-9 each, fp32 accumulation)."""
import numpy as np
import pytest

import oracle
from paper_2603_06626_amd import workloads as wl
from tests.helpers import rel_max_err

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

TOL = 1e-2


@pytest.mark.parametrize("T,d,f,E,k,hot", [
    (511, 72, 136, 2, 1, 0),        # mean of 255 rows per expert: dW2 with one register set
    (512, 72, 136, 2, 1, 0),        # 256: with two
    (512, 72, 136, 2, 1, 500),      # the same mean, reductions of 16 and of 1 step
    (768, 264, 264, 3, 1, 768),     # two experts without rows
    (900, 328, 200, 7, 2, 40),      # four tiles of rows, short reductions
])
def test_backward_matches_the_oracle(T, d, f, E, k, hot):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from tests import gpu_util as gpu

    idx, gates, t = wl.make_custom(T, d, f, E, k, routing="uniform", seed=11, stream=700 + T + hot)
    if hot:
        idx = idx.copy()
        idx[:hot] = np.arange(k)
    layer = gpu.Layer(T, k, E, d, f)
    layer.build_plan(idx)
    dev = {n: gpu.to_dev(v) for n, v in t.items()}
    gw = gpu.to_dev(gates)
    layer.fwd(dev["x"], gw, dev["W1"], dev["W3"], dev["W2"])
    grads = layer.bwd(dev["x"], gw, dev["W1"], dev["W3"], dev["W2"], dev["dY"])
    w = oracle.bf16_bits_to_f32
    ref = oracle.moe_bwd(w(t["x"]), w(gates), idx, w(t["W1"]), w(t["W3"]), w(t["W2"]), w(t["dY"]))
    for name, g, r in zip(("dX", "dW1", "dW3", "dW2"), grads, ref):
        assert rel_max_err(gpu.to_f64(g), r) <= TOL, name


@pytest.mark.parametrize("T,d,f,E,k,routing", [
    (64, 72, 136, 1, 1, "uniform"),       # one expert: fewer than four experts in the only group of four
    (3200, 64, 72, 33, 1, "zipf"),        # 4 x 3 steps >= 2 and 8: the heaviest eighth (two groups of four) first in both
    (1055, 64, 520, 33, 1, "zipf"),       # mean of 31 rows: no step, rows first
    (1056, 128, 520, 33, 1, "zipf"),      # 4 x 1 steps against 4 and 36: dW2 and dH heaviest first, dW1/dW3 and dXp rows first
    (1056, 136, 520, 33, 1, "zipf"),      # 6: rows first in both
    (333, 264, 264, 128, 8, "uniform"),   # row tiles whose number is no multiple of 8
])
def test_paired_launches_leave_no_tile_out(T, d, f, E, k, routing):
    """A timed call launches the four products apart; the pairs must give the same bits, whatever their order in the grid."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2603_06626_amd import binding as b
    from tests import gpu_util as gpu

    idx, gates, t = wl.make_custom(T, d, f, E, k, routing=routing, seed=12, stream=900 + T + d)
    layer = gpu.Layer(T, k, E, d, f)
    layer.build_plan(idx)
    dev = {n: gpu.to_dev(v) for n, v in t.items()}
    gw = gpu.to_dev(gates)
    layer.fwd(dev["x"], gw, dev["W1"], dev["W3"], dev["W2"])

    def backward():
        out = [torch.full_like(dev[n], float("nan")) for n in ("x", "W1", "W3", "W2")]
        scratch = torch.full((b.grouter_bwd_scratch_bytes(T, k, d, f),), 255, dtype=torch.uint8, device=gpu.DEV)
        b.grouter_moe_bwd(layer.plan, dev["x"], gw, dev["W1"], dev["W3"], dev["W2"], dev["dY"], layer.ctx, *out, scratch)
        return out

    pairs = backward()
    b.grouter_timing_enable(True)
    try:
        apart = backward()
    finally:
        b.grouter_timing_enable(False)
        b.grouter_timing_read()
    for name, p, a in zip(("dX", "dW1", "dW3", "dW2"), pairs, apart):
        assert bool(torch.isfinite(a.float()).all()), name
        assert torch.equal(p, a), name
