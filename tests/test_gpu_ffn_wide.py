"""The bf16 kernel of large batches (ffn_bf16_wide.hip) against the fp64
oracle, at the edges of its token tiles and of its split of K."""

import numpy as np
import pytest

import oracle
from synth.configs import LayerShape
from tests.gpu_helpers import (assert_same_bits, check_outputs, check_routing, log, make_inputs,
                               run_gpu)

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


# A shared expert takes exactly B tokens: 33 to 256 cover every compiled tile
# count (3 to 16), the last token of a tile and the first of the next, and
# gate-up by K halves (up to 128 tokens) and by token halves.  K spans one run
# of two steps (64), ranges that end on the first or second half's run, and a
# shared width different from the routed one.  2048 columns of 8 experts are
# the least that this kernel takes up to 64 tokens (packed: 127).
@pytest.mark.parametrize("B,hidden,ffn,ffn_shared", [
    (33, 64, 2048, 64), (48, 128, 2112, 64), (49, 192, 2048, 320), (65, 320, 2176, 192),
    (96, 128, 2048, 128), (97, 64, 2112, 64), (112, 192, 2048, 64), (128, 256, 192, 448),
    (129, 64, 128, 64), (160, 320, 64, 192), (193, 128, 192, 320), (208, 64, 64, 128),
    (209, 192, 128, 64), (256, 256, 320, 192)])
def test_wide_tiles_and_k_edges(B, hidden, ffn, ffn_shared):
    check(B, hidden, ffn, ffn_shared)


# Where the register-only kernel stays, in both layouts or (65 to 127 tokens) in
# the packed one: narrow experts (down K by one wave below 256 columns, shared
# ones counted) and few units; from 128 tokens on, narrow experts of more than
# 1024 down units.
@pytest.mark.parametrize("B,hidden,ffn,ffn_shared,E", [
    (33, 128, 192, 64, 8), (64, 192, 64, 320, 8), (64, 64, 1920, 64, 8), (65, 64, 1920, 64, 8),
    (96, 320, 256, 192, 8), (127, 128, 256, 64, 8), (100, 320, 64, 64, 255),
    (128, 320, 64, 64, 255), (200, 384, 64, 320, 200)])
def test_large_batches_on_few_or_narrow_units(B, hidden, ffn, ffn_shared, E):
    check(B, hidden, ffn, ffn_shared, E)


def check(B, hidden, ffn, ffn_shared, E=8):
    shape = LayerShape(hidden=hidden, ffn=ffn, n_experts=E, top_k=2, cap=4, alpha=0.5,
                       n_shared=1, ffn_shared=ffn_shared)
    d = make_inputs(shape, B, seed=500 + B, rho=0.7)
    label = f"wide B={B} H={hidden} F={ffn} Fs={ffn_shared} E={E}"
    log(f"[wide] {label}")
    rows, _ = run_gpu(shape, d)
    packed, dw = run_gpu(shape, d, packed=True)
    one, _ = run_gpu(shape, d, dw, packed=True, fused=True)
    assert_same_bits(one, packed, label + " one call")
    assert np.array_equal(rows["expert_out"], packed["expert_out"]), label
    ref = oracle.forward(d["x"], d["router"], d["conf_w"], d["experts"], d["shared"], shape)
    check_routing(rows, ref, label)
    check_outputs(rows, ref, shape.wdt, label)
    check_outputs(packed, ref, shape.wdt, label + " packed")
