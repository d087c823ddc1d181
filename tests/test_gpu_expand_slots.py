"""s2moe_expand where a tree's viable nodes outnumber the bitsets kept in LDS
(more trees than compute units), against the expansion oracle, exactly."""

import numpy as np
import pytest

from tests.test_gpu_expand import KEYS, X, compare, log, random_batch, run_gpu

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


# Bitsets of 40 KB: about 160 of 200 slots at L = 6, E = 256; 16 (the minimum)
# at 8 KB a node; ids in 16-byte chunks or not (L k a multiple of 4 or not),
# two and four nodes a thread.  T_AR 64 makes most nodes viable.
@pytest.mark.parametrize("N,L,E,k", [(200, 6, 256, 5), (120, 48, 128, 8), (90, 17, 512, 3),
                                     (300, 12, 200, 4), (600, 4, 250, 3), (18, 64, 1024, 2)])
def test_more_viable_nodes_than_bitsets(N, L, E, k):
    rng = np.random.default_rng(N + L)
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    T = cus + 40
    few = random_batch(rng, 8, N, L, E, k)
    a = [np.ascontiguousarray(np.concatenate([v] * (T // 8 + 1))[:T]) for v in few]
    for t_ar, t_exp in ((64.0, 0.5 / (L * k)), (1.5, 0.05 / (L * k))):
        log(f"[expand] slots T={T} N={N} L={L} E={E} k={k} T_AR={t_ar}")
        got = run_gpu(*a, E, t_ar, t_exp)
        ref = X.expand(few[0], few[1], few[2], few[3], E, t_ar, t_exp, few[4], few[5])
        for first in (0, 8, T - T % 8 - 8):
            compare({n: got[n][first:first + 8] for n in KEYS}, ref, f"slots from {first}")
