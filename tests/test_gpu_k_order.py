"""Order in which the bf16 expert FFN adds along K, on sums that the order
decides: 2^30 and -2^30 cancel, and a 1 after them survives only where all
three are added by one wave.  Contiguous ranges of K per wave (at most 16
tokens; row-major rows a multiple of 4 KB) keep them together, runs of two or
four steps dealt to the waves (17 tokens and more otherwise) do not."""

import numpy as np
import pytest

from tests.gpu_helpers import log

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

F = 2048


def experts(H):
    """Two experts whose gate and down rows hold 2^30, -2^30, 1 in the steps
    (of 32) 0, 2, 3 and 0, 4, 5; up rows pick x[0]."""
    w = {"gate": torch.zeros(2, F, H), "up": torch.zeros(2, F, H), "down": torch.zeros(2, H, F)}
    w["gate"][:, :, 0], w["gate"][:, :, 64], w["gate"][:, :, 96] = 2.0 ** 30, -(2.0 ** 30), 1.0
    w["up"][:, :, 0] = 1.0
    w["down"][:, :, 0], w["down"][:, :, 128], w["down"][:, :, 160] = 2.0 ** 30, -(2.0 ** 30), 1.0
    return {n: t.to(torch.bfloat16).cuda() for n, t in w.items()}


@pytest.mark.parametrize("H,B,packed,together", [
    (2048, 1, True, True), (2048, 4, False, True), (2048, 5, True, True), (2048, 16, True, True),
    (2048, 16, False, True), (2112, 8, False, True), (2048, 24, False, True),
    (2048, 24, True, False), (2112, 24, False, False), (2048, 33, True, False),
    (2048, 33, False, False)])
def test_k_ranges(H, B, packed, together):
    import paper_2608_15018_amd as s2
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    log(f"[k order] H={H} B={B} packed={packed}")
    dev = (experts(H), {})
    if packed:
        dev, w = s2.pack_expert_weights(dev, "bf16")
    else:
        w = s2.make_weights(*dev)
    layer = s2.make_layer(hidden=H, ffn=F, n_experts=2, top_k=1, cap=1, alpha=0.0,
                          flags=s2.PACKED_WEIGHTS if packed else 0)
    x = torch.ones(B, H, dtype=torch.bfloat16, device="cuda")
    router = torch.zeros(2, H, dtype=torch.bfloat16, device="cuda")
    router[0, 0] = 1.0
    h = float((torch.sigmoid(torch.tensor(1.0))).to(torch.bfloat16))  # silu(1) x[0]
    for fused in (True, False):
        p = s2.VerifyPass(layer, B, fused=fused)
        y = p(x, router, torch.ones(B, device="cuda"), w)
        torch.cuda.synchronize()
        assert np.array_equal(y.cpu().numpy(), np.full((B, H), h if together else 0.0, np.float32))
