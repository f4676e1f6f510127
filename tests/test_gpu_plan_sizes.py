"""The routing plan at the sizes where its launch shape changes: one workgroup up to 4096 slots, chunks of 2048 slots
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
