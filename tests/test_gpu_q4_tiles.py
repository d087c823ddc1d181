"""int4 layers of more than 128 tokens (up to eight token tiles per pass)
against the fp64 oracle, packed equal to row-major."""

import numpy as np
import pytest

import oracle
from synth.configs import LayerShape
from tests.gpu_helpers import check_outputs, check_routing, log, make_inputs, run_gpu

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


# The shared expert takes exactly B tokens: 9 tiles (8 + 1), 10 (8 + 2), 13
# (8 + 5), 14 (8 + 6), 15 (8 + 7) and 16, with a ragged or a full last tile.
@pytest.mark.parametrize("B", [129, 144, 145, 197, 224, 226, 241, 256])
def test_int4_eight_tiles(B):
    shape = LayerShape(hidden=384, ffn=256, n_experts=8, top_k=2, cap=4, alpha=0.5, n_shared=1,
                       ffn_shared=128, act="bf16", wdt="q4g32")
    d = make_inputs(shape, B, seed=700 + B, rho=0.7)
    label = f"int4 eight tiles B={B}"
    log(f"[parity] {label}")
    got, _ = run_gpu(shape, d)
    packed, _ = run_gpu(shape, d, packed=True)
    assert np.array_equal(packed["expert_out"], got["expert_out"]), label
    deq = lambda ex: {n: np.stack([oracle.dequant_q4g32(ex[n][e], ex[n + "_s"][e])  # noqa: E731
                                   for e in range(ex[n].shape[0])]).astype(np.float32)
                      for n in ("gate", "up", "down")}
    ref = oracle.forward(d["x"], d["router"], d["conf_w"], deq(d["experts"]), deq(d["shared"]),
                         shape.with_(wdt="f32"))
    check_routing(got, ref, label)
    check_outputs(got, ref, "q4g32", label)
