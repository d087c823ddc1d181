"""fp32 experts at the edges of their token passes (8, 4, 2 or 1 tokens), and the
plain top-k of one token at the edge between its two ranking methods."""

import numpy as np
import pytest

import oracle
from synth.configs import LayerShape
from tests.gpu_helpers import check_outputs, check_routing, log, make_inputs, run_gpu

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


# The shared expert takes exactly B tokens: every remainder of a pass of 8.
@pytest.mark.parametrize("B,hidden", [(1, 64), (2, 320), (3, 256), (4, 64), (5, 192), (6, 64),
                                      (7, 256), (8, 320), (9, 64), (11, 256), (13, 64), (18, 64)])
def test_f32_passes(B, hidden):
    shape = LayerShape(hidden=hidden, ffn=128, n_experts=8, top_k=2, cap=4, alpha=0.5, n_shared=1,
                       ffn_shared=192, act="f32", wdt="f32")
    d = make_inputs(shape, B, seed=900 + B)
    log(f"[f32] B={B} H={hidden}")
    got, _ = run_gpu(shape, d)
    ref = oracle.forward(d["x"], d["router"], d["conf_w"], d["experts"], d["shared"], shape)
    check_routing(got, ref, f"f32 B={B}")
    check_outputs(got, ref, "f32", f"f32 B={B}")


# Logits in eighths (exact, many ties) on a one-hot router; k from 1 to 16 spans
# both rankings, E the slots a lane holds.
@pytest.mark.parametrize("E", [3, 64, 65, 128, 200, 256])
def test_plain_top_k_by_either_ranking(E):
    import paper_2608_15018_amd as s2
    rng = np.random.default_rng(E)
    H = -(-E // 64) * 64
    router = np.zeros((E, H), np.float32)
    router[np.arange(E), np.arange(E)] = 1.0
    for B in (1, 4, 9):
        x = np.zeros((B, H), np.float32)
        x[:, :E] = rng.integers(-16, 17, size=(B, E)) / 8.0
        for k in (1, 2, 11, 12, 16):
            if k >= E:
                continue
            log(f"[select] E={E} B={B} k={k}")
            ref = oracle.route(x, router, k, "f32")
            L = s2.make_layer(hidden=H, ffn=64, n_experts=E, top_k=k, cap=k, alpha=0.0,
                              act="f32", wdt="f32")
            rt = s2.Routing(L, B)
            s2.route(L, torch.from_numpy(x).cuda(), torch.from_numpy(router).cuda(), rt)
            torch.cuda.synchronize()
            got = rt.host()
            np.testing.assert_array_equal(got["plain_idx"], ref["plain_idx"], err_msg=f"k={k}")
            np.testing.assert_array_equal(got["gap"], ref["gap"].astype(np.float32))
