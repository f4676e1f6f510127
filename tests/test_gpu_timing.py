"""Phase timing of the backward pass: every product has a phase of its own, and timing changes no result."""
import pytest

from paper_2603_06626_amd import workloads as wl

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,d,f,E,k", [(256, 128, 256, 8, 2), (37, 520, 264, 5, 3)])
def test_timed_backward_has_four_product_phases_and_the_same_results(T, d, f, E, k):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2603_06626_amd import binding as b
    from tests import gpu_util as gpu

    idx, gates, t = wl.make_custom(T, d, f, E, k, routing="zipf", seed=3, stream=77)
    layer = gpu.Layer(T, k, E, d, f)
    layer.build_plan(idx)
    dev = {n: gpu.to_dev(v) for n, v in t.items()}
    gw = gpu.to_dev(gates)
    layer.fwd(dev["x"], gw, dev["W1"], dev["W3"], dev["W2"])
    plain = layer.bwd(dev["x"], gw, dev["W1"], dev["W3"], dev["W2"], dev["dY"])
    b.grouter_timing_read()
    b.grouter_timing_enable(True)
    try:
        timed = layer.bwd(dev["x"], gw, dev["W1"], dev["W3"], dev["W2"], dev["dY"])
    finally:
        b.grouter_timing_enable(False)
    phases = b.grouter_timing_read()
    for name in ("dW2", "dH", "dW13", "dXp", "dX_reduce"):
        ms, launches = phases[name]
        assert launches == 1 and ms > 0.0, name
    assert sum(n for _, n in phases.values()) == 5
    for a, c in zip(plain, timed):
        assert torch.equal(a, c)
