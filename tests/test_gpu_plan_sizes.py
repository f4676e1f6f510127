"""The routing plan at the sizes where its launch shape changes: chunks of 2048 slots, one launch up to 8192 slots and two
beyond, larger chunks past 256 of them.  All arrays are bit-exact against the stable counting sort of the oracle."""
import numpy as np
import pytest

import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,k,E,dtype", [
    (1, 1, 1, np.int32), (64, 1, 2, np.uint8), (1365, 3, 7, np.int32), (4096, 1, 1024, np.int32), (4097, 1, 5, np.uint8),
    (6143, 1, 64, np.int32), (3072, 2, 256, np.uint8), (2049, 3, 65, np.int32), (524288, 1, 33, np.uint8),
    (524289, 1, 128, np.uint8), (262145, 4, 5, np.int32),
])
def test_plan_at_the_edges_of_its_launch_shapes(T, k, E, dtype):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from tests import gpu_util as gpu

    rng = np.random.default_rng(T + E)
    idx = np.minimum(rng.geometric(min(0.9, 4.0 / E), size=(T, k)) - 1, E - 1).astype(dtype)   # skewed, some experts empty
    layer = gpu.Layer(T, k, E, 8, 8)
    layer.build_plan(torch.from_numpy(idx).to(gpu.DEV))
    for name, got, ref in zip(("counts", "offsets", "row_to_src", "src_to_row"), layer.plan_views(), oracle.plan(idx.astype(np.int32), E)):
        assert np.array_equal(got, ref), name


@pytest.mark.parametrize("T,k,E,dtype", [
    (2048, 1, 3, np.uint8), (2049, 1, 129, np.int32),       # one chunk, one slot in a second
    (1024, 8, 200, np.uint8), (8193, 1, 200, np.int32),     # last plan of one launch, first of two
    (1024, 8, 1024, np.int32), (2731, 3, 513, np.int32),    # one thread per expert compares all loads
    (40, 3, 4, np.int32), (900, 4, 5, np.uint8),            # 256 threads per expert, 128 with ids that do not exist
])
def test_plan_and_load_order_at_the_edges_of_one_launch(T, k, E, dtype):
    """The plan and what depends on the order of experts by load, which the views do not show: a layer whose expert outputs
    differ by expert.  Equal loads occur."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2603_06626_amd import workloads as wl
    from tests import gpu_util as gpu
    from tests.helpers import rel_max_err

    d = f = 8
    idx = np.minimum(np.random.default_rng(T + E).geometric(min(0.9, 6.0 / E), size=(T, k)) - 1, E - 1).astype(dtype)
    _, gates, t = wl.make_custom(T, d, f, E, k, routing="uniform", seed=22, stream=800)
    layer = gpu.Layer(T, k, E, d, f)
    layer.build_plan(torch.from_numpy(idx).to(gpu.DEV))
    for name, got, ref in zip(("counts", "offsets", "row_to_src", "src_to_row"), layer.plan_views(), oracle.plan(idx.astype(np.int32), E)):
        assert np.array_equal(got, ref), name
    dev = {n: gpu.to_dev(v) for n, v in t.items()}
    gw = gpu.to_dev(gates)
    layer.fwd(dev["x"], gw, dev["W1"], dev["W3"], dev["W2"])
    grads = layer.bwd(dev["x"], gw, dev["W1"], dev["W3"], dev["W2"], dev["dY"])
    w = oracle.bf16_bits_to_f32
    ref = oracle.moe_bwd(w(t["x"]), w(gates), idx.astype(np.int32), w(t["W1"]), w(t["W3"]), w(t["W2"]), w(t["dY"]))
    for name, g, r in zip(("dX", "dW1", "dW3", "dW2"), grads, ref):     # bar as for the other shapes
        assert rel_max_err(gpu.to_f64(g), r) <= 1e-2, name


@pytest.mark.parametrize("T,E,dtype", [
    (2048, 1, np.uint8), (2049, 2, np.int32), (4097, 7, np.uint8), (8192, 1, np.int32), (8192, 64, np.uint8), (8192, 1024, np.int32), (8193, 300, np.int32),
])
@pytest.mark.parametrize("where", ["first", "last", "two"])
def test_plan_of_slots_that_pick_one_expert(T, E, dtype, where):
    """All slots on one expert, or all but every 64th, so that the lanes of a wave count the same word."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from tests import gpu_util as gpu

    idx = np.full((T, 1), 0 if where == "first" else E - 1, dtype=dtype)
    if where == "two":
        idx[5::64] = E // 2
    layer = gpu.Layer(T, 1, E, 8, 8)
    layer.build_plan(torch.from_numpy(idx).to(gpu.DEV))
    for name, got, ref in zip(("counts", "offsets", "row_to_src", "src_to_row"), layer.plan_views(), oracle.plan(idx.astype(np.int32), E)):
        assert np.array_equal(got, ref), name


@pytest.mark.parametrize("E,dtype", [(33, np.uint8), (1024, np.int32)])
@pytest.mark.parametrize("where", ["first", "middle", "last"])
def test_a_bad_id_in_any_chunk_is_reported_and_counts_as_expert_0(E, dtype, where):
    """Three chunks of 2048 slots and a ragged fourth, built by two launches."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2603_06626_amd import binding as b
    from tests import gpu_util as gpu

    T, k = 3350, 2
    idx = np.random.default_rng(E).integers(0, E, size=(T, k)).astype(dtype)
    good = idx.copy()
    slot = {"first": 5, "middle": 2048 + 777, "last": T * k - 1}[where]
    idx.reshape(-1)[slot] = 255 if dtype == np.uint8 else -3
    good.reshape(-1)[slot] = 0
    layer = gpu.Layer(T, k, E, 8, 8)
    b.grouter_plan_build(torch.from_numpy(idx).to(gpu.DEV), E, layer.plan)
    with pytest.raises(b.GrouterError) as ei:
        b.grouter_plan_status(layer.plan)
    assert ei.value.code == b.ERR_INDEX_OUT_OF_RANGE
    for name, got, ref in zip(("counts", "offsets", "row_to_src", "src_to_row"), layer.plan_views(), oracle.plan(good.astype(np.int32), E)):
        assert np.array_equal(got, ref), name
    layer.build_plan(good)      # a rebuild in place clears the flag (build_plan asks for the status)


@pytest.mark.parametrize("T,k,E", [(4096, 1, 1024), (4097, 1, 5), (2049, 3, 65), (8200, 1, 1024), (524289, 1, 128)])
def test_layer_on_plans_at_the_edges_of_their_launch_shapes(T, k, E):
    """What the views do not show, the row-to-token map, the load order and the row tiles, by what the layer computes with
    them: y and the gradients against the oracle (bar as for the other shapes)."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2603_06626_amd import workloads as wl
    from tests import gpu_util as gpu
    from tests.helpers import rel_max_err

    d = f = 8
    idx = np.minimum(np.random.default_rng(T).geometric(min(0.9, 4.0 / E), size=(T, k)) - 1, E - 1).astype(np.int32)
    _, gates, t = wl.make_custom(T, d, f, E, k, routing="uniform", seed=21, stream=800 + E)
    layer = gpu.Layer(T, k, E, d, f)
    layer.build_plan(idx)
    dev = {n: gpu.to_dev(v) for n, v in t.items()}
    gw = gpu.to_dev(gates)
    y = layer.fwd(dev["x"], gw, dev["W1"], dev["W3"], dev["W2"])
    grads = layer.bwd(dev["x"], gw, dev["W1"], dev["W3"], dev["W2"], dev["dY"])
    w = oracle.bf16_bits_to_f32
    args = [w(t["x"]), w(gates), idx, w(t["W1"]), w(t["W3"]), w(t["W2"])]
    assert rel_max_err(gpu.to_f64(y), oracle.moe_fwd(*args)) <= 1e-2
    for name, g, r in zip(("dX", "dW1", "dW3", "dW2"), grads, oracle.moe_bwd(*args, w(t["dY"]))):
        assert rel_max_err(gpu.to_f64(g), r) <= 1e-2, name
