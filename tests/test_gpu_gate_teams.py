"""The gating kernel's per-token ranking by teams of lanes (a wave, or a row of
16 lanes) and by the threshold search, against the fp64 oracle on dyadic
logits with many exact ties, and the one-call layer's ranking inside the gating
launch against the four calls."""

import numpy as np
import pytest

import oracle
from synth.configs import LayerShape
from tests.gpu_helpers import assert_same_bits, check_routing, log, make_inputs, run_gpu

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


# Expert counts at the edges of a team's slots (1, 4, 8, 16 a row lane; 1, 2, 4
# a wave lane) and not multiples of 4; token counts at the edges of a wave per
# token (16), of a row group (4) and of a workgroup pass (64).  k at the edges
# of taking maxima: by 8, 16, 32 and more tokens up to 3 / 5 / 12 / 16 of 17 to
# 64 experts, 6 / 7 / 8 / 13 of 65 to 128, 7 / 8 / 6 / 13 of more, 8 / 16 / 16 /
# 16 of at most 16; in the routing's ranking up to 5, 8 and 11.
@pytest.mark.parametrize("E,k,cap", [(2, 1, 1), (3, 2, 2), (16, 8, 12), (16, 9, 12), (16, 15, 16),
                                     (17, 16, 17), (63, 5, 9), (63, 6, 9), (64, 3, 12),
                                     (64, 4, 12), (64, 12, 16), (64, 13, 16), (66, 3, 40),
                                     (127, 16, 20), (128, 7, 14), (128, 8, 14), (128, 9, 14),
                                     (129, 5, 7), (200, 6, 9), (200, 7, 9), (255, 16, 30),
                                     (256, 11, 100), (256, 13, 100), (256, 14, 100)])
def test_ties_over_team_edges(E, k, cap):
    import paper_2608_15018_amd as s2
    rng = np.random.default_rng(E * 31 + k)
    H = -(-E // 64) * 64
    router = np.zeros((E, H), np.float32)
    router[np.arange(E), np.arange(E)] = 1.0
    for B in (1, 3, 5, 8, 9, 16, 17, 32, 33, 63, 65, 256):
        # eighths in [-2, 2]: with alpha 0.5 every g, bias and biased logit is exact
        x = np.zeros((B, H), np.float32)
        x[:, :E] = rng.integers(-16, 17, size=(B, E)) / 8.0
        w = (rng.random(B) < 0.7).astype(np.float32)
        w[0] = 1.0
        log(f"[gate] E={E} k={k} cap={cap} B={B}")
        r = oracle.route(x, router, k, "f32")
        for flags in (0, 1, 2 | 4):
            ref = oracle.reuse_gate(r["logits"], r["gap"], r["plain_idx"], w, k, cap, 0.5, flags)
            L = s2.make_layer(hidden=H, ffn=64, n_experts=E, top_k=k, cap=cap, alpha=0.5,
                              flags=flags, act="f32", wdt="f32")
            rt = s2.Routing(L, B)
            s2.route(L, torch.from_numpy(x).cuda(), torch.from_numpy(router).cuda(), rt)
            s2.reuse_gate(L, torch.from_numpy(w).cuda(), rt)
            torch.cuda.synchronize()
            got, label = rt.host(), f"E={E} B={B} flags={flags}"
            for n in ("pref", "idx", "count", "offset", "slot", "uniq"):
                np.testing.assert_array_equal(got[n], ref[n], err_msg=f"{n} {label}")
            # k terms of at most 1, each within 1e-6, and their sum's rounding
            assert np.abs(got["gate_w"] - ref["gate_w"]).max() <= 5e-6, label


# hidden 256: logits in one slice of H, as the rows launch adds them.  1024
# (512 in fp32): the routing slices H for 32 experts and fewer, where the gate
# must not rank what the rows launch would compute, but not for 36.  k beyond
# taking maxima: ranked by the search, up to 16 tokens inside the launch.
@pytest.mark.parametrize("E,k,B,hidden,act", [
    (40, 4, 9, 256, "bf16"), (64, 6, 33, 256, "bf16"), (64, 6, 64, 256, "bf16"),
    (64, 6, 65, 256, "bf16"), (36, 3, 24, 256, "bf16"), (100, 8, 17, 256, "bf16"),
    (128, 8, 32, 256, "bf16"), (128, 8, 33, 256, "bf16"), (32, 4, 24, 256, "bf16"),
    (32, 4, 24, 1024, "bf16"), (8, 2, 40, 1024, "bf16"), (36, 4, 24, 1024, "bf16"),
    (32, 4, 24, 512, "f32"), (32, 4, 24, 256, "f32"), (36, 4, 40, 512, "f32"),
    (64, 10, 12, 256, "bf16"), (64, 10, 40, 256, "bf16"), (16, 9, 40, 256, "bf16"),
    (200, 12, 16, 256, "bf16"), (200, 12, 17, 256, "bf16"), (64, 13, 32, 256, "bf16")])
def test_ranking_inside_the_gating_launch(E, k, B, hidden, act):
    shape = LayerShape(hidden=hidden, ffn=64, n_experts=E, top_k=k, cap=min(E, 2 * k), alpha=0.5,
                       act=act, wdt=act)
    d = make_inputs(shape, B, seed=E + B, rho=0.5)
    label = f"E={E} k={k} B={B} H={hidden} {act}"
    log(f"[gate] one call {label}")
    four, dw = run_gpu(shape, d)
    one, _ = run_gpu(shape, d, dw, fused=True)
    assert_same_bits(one, four, label)
    ref = oracle.forward(d["x"], d["router"], d["conf_w"], d["experts"], d["shared"], shape)
    check_routing(one, ref, label)


# A token whose logits are all the NaN of all bits set (in fp32 or in bf16, so
# with a key of 0 or 0xFFFF but for the clamp): it still gets k experts, and the
# other tokens' plain ranking is theirs (g, and so a biased selection, is NaN
# for the whole batch).  By maxima and by search, in the small-batch gate, one
# token a wave, and rows.
@pytest.mark.parametrize("bits", [-1, -0x10000])
@pytest.mark.parametrize("E,k,B,alpha", [(64, 3, 2, 0.0), (64, 12, 2, 0.0), (40, 3, 6, 0.5),
                                         (40, 9, 6, 0.5), (200, 4, 20, 0.5), (200, 12, 40, 0.5)])
def test_nan_logits_still_select_k_experts(E, k, B, alpha, bits):
    import paper_2608_15018_amd as s2
    H = -(-E // 64) * 64
    rng = np.random.default_rng(E + k)
    x = np.zeros((B, H), np.float32)
    x[:, :E] = rng.permuted(np.tile(np.arange(E), (B, 1)), axis=1) / 8.0
    r = oracle.route(x, np.eye(E, H, dtype=np.float32), k, "f32")
    x[1] = np.array([bits], np.int32).view(np.float32)[0]
    log(f"[gate] NaN row E={E} k={k} B={B}")
    L = s2.make_layer(hidden=H, ffn=64, n_experts=E, top_k=k, cap=k, alpha=alpha, act="f32",
                      wdt="f32")
    rt = s2.Routing(L, B)
    s2.route(L, torch.from_numpy(x).cuda(), torch.eye(E, H).cuda(), rt)
    s2.reuse_gate(L, torch.ones(B).cuda(), rt)
    torch.cuda.synchronize()
    got = rt.host()
    for n in ("plain_idx", "idx"):
        assert (np.diff(got[n], axis=1) > 0).all() and got[n].min() >= 0 and got[n].max() < E, n
    others = np.arange(B) != 1
    np.testing.assert_array_equal(got["plain_idx"][others], r["plain_idx"][others])
    assert got["count"].sum() == B * k
    np.testing.assert_array_equal(np.sort(got["slot"]), np.arange(B * k))
