"""Forward pass at and around the sizes where the kernels for few tokens take over (at most 16 tokens, on few experts at most 64), through the C ABI,
against the CPU oracle.  Bar as for the other shapes: max|gpu - oracle| <= 1e-2 * max|oracle| (bf16 storage of H, O and
y: a few 2^-9 each, fp32 accumulation)."""
import numpy as np
import pytest

import oracle
from paper_2603_06626_amd import workloads as wl
from tests.helpers import rel_max_err

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

TOL = 1e-2


@pytest.mark.parametrize("T,d,f,E,k,repeat", [
    (1, 8, 8, 1, 1, False),         # one K-block and one column block, both mostly masked
    (1, 2048, 1408, 64, 6, False),  # one token at full width
    (2, 72, 136, 5, 3, False),      # K tails of 8, column tails of 8
    (7, 256, 64, 3, 3, False),      # K of exactly one block per wave, one column block
    (15, 264, 520, 9, 2, False),    # one K-block more than the waves share evenly
    (16, 544, 192, 4, 4, False),    # 16 rows in every expert
    (16, 1056, 72, 6, 3, True),     # a token names its expert three times: 48 rows in one expert
    (17, 544, 192, 4, 4, False),    # first size with two row blocks: 17 rows in every expert
    (32, 72, 200, 4, 4, False),     # last size with two, full
    (33, 264, 136, 3, 3, False),    # first with four
    (64, 520, 264, 2, 2, False),    # last with four, full
    (64, 264, 72, 6, 3, True),      # a token names its expert three times: 192 rows in one expert, two tiles
    (65, 264, 136, 3, 3, False),    # first size of the tiled kernels
    (12, 72, 136, 40, 3, False),    # rows that begin inside a line and 32 tiles or more: one XCD per expert
    (16, 200, 264, 64, 4, False),   # the same with five column blocks
    (20, 1032, 1032, 64, 4, False), # more than 16 tokens on many experts: tiled
    (16, 72, 72, 250, 16, False),   # about 163 row tiles on rows that begin inside a line: tiled up to 16 tokens, too
    (13, 72, 72, 250, 16, False),   # about 144: streamed
    (3, 3072, 72, 100, 30, False),  # 66 tiles of gate/up (K = 3072) and 788 of down: both streamed
    (9, 3072, 64, 190, 40, False),  # 168 tiles of gate/up on 3072 rows of weights: tiled; down streamed
    (12, 256, 776, 240, 30, False), # about 192 tiles of down: tiled with K > 768
    (12, 256, 768, 240, 30, False), # the same with K = 768: streamed
    (5, 1024, 256, 70, 20, False),  # more workgroups than CUs, K = 1024: one stage
    (5, 1032, 256, 70, 20, False),  # K = 1032: two
    (8, 704, 512, 8, 2, False),     # 11 column blocks in plain order, 8 in runs
])
def test_few_tokens_match_the_oracle(T, d, f, E, k, repeat):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from tests import gpu_util as gpu

    idx, gates, t = wl.make_custom(T, d, f, E, k, routing="uniform", seed=3, stream=300 + T)
    if repeat:
        idx = np.full_like(idx, 2)
    layer = gpu.Layer(T, k, E, d, f)
    layer.build_plan(idx)
    dev = {n: gpu.to_dev(v) for n, v in t.items()}
    gw = gpu.to_dev(gates)
    y = layer.fwd(dev["x"], gw, dev["W1"], dev["W3"], dev["W2"])
    y_only = layer.fwd_only(dev["x"], gw, dev["W1"], dev["W3"], dev["W2"])
    w = oracle.bf16_bits_to_f32
    ref = oracle.moe_fwd(w(t["x"]), w(gates), idx, w(t["W1"]), w(t["W3"]), w(t["W2"]))
    assert rel_max_err(gpu.to_f64(y), ref) <= TOL
    assert torch.equal(y, y_only)
    # what the forward pass keeps is what the backward pass reads
    grads = layer.bwd(dev["x"], gw, dev["W1"], dev["W3"], dev["W2"], dev["dY"])
    ref_g = oracle.moe_bwd(w(t["x"]), w(gates), idx, w(t["W1"]), w(t["W3"]), w(t["W2"]), w(t["dY"]))
    for g, r in zip(grads, ref_g):
        assert rel_max_err(gpu.to_f64(g), r) <= TOL
