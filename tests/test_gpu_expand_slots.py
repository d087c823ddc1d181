"""s2moe_expand where a launch keeps fewer bitsets than a tree has viable
nodes and leaves the tree to the next launch, and where the bitsets take all
of a workgroup's LDS, against the expansion oracle, exactly."""

import numpy as np
import pytest

from tests.test_gpu_expand import KEYS, X, compare, log, random_batch, run_gpu

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


# More trees than compute units (256 on MI355X): one launch or, by `per_cu`
# trees a unit, bitsets of half a unit's LDS and then of all of it (1), or a
# quarter first (2).  Bitsets of quarter / half / all:
#   (200, 6, 256)    192 / 200       (120, 48, 128)  46 / 100 / 120
#   (90, 17, 512)     32 /  69 / 90  (300, 12, 200)  89 / 196 / 300
#   (600, 4, 250)    240 / 560 / 600 (38, 64, 512)    - /  18 /  38, one union
#   (18, 64, 1024)     - /   - / 18  (104, 48, 256)  21 /  48 / 104, one union
# Ids in 16-byte chunks or not (L k a multiple of 4 or not), one to three
# nodes a thread.  T_AR 64 makes most nodes viable, 4 some.
@pytest.mark.parametrize("per_cu", [1, 2])
@pytest.mark.parametrize("N,L,E,k", [(200, 6, 256, 5), (120, 48, 128, 8), (90, 17, 512, 3),
                                     (300, 12, 200, 4), (600, 4, 250, 3), (38, 64, 512, 5),
                                     (18, 64, 1024, 2), (104, 48, 256, 3)])
def test_more_viable_nodes_than_bitsets(N, L, E, k, per_cu):
    rng = np.random.default_rng(N + L)
    T = per_cu * torch.cuda.get_device_properties(0).multi_processor_count + 40
    few = random_batch(rng, 8, N, L, E, k)
    tiled = lambda v: np.ascontiguousarray(np.concatenate([v] * (T // 8 + 1))[:T])  # noqa: E731
    a = [tiled(v) for v in few]
    for t_ar, t_exp in ((64.0, 0.5 / (L * k)), (4.0, 0.1 / (L * k)), (1.5, 0.05 / (L * k))):
        log(f"[expand] slots T={T} N={N} L={L} E={E} k={k} T_AR={t_ar}")
        got = run_gpu(*a, E, t_ar, t_exp)
        ref = X.expand(few[0], few[1], few[2], few[3], E, t_ar, t_exp, few[4], few[5])
        compare(got, {n: tiled(ref[n]) for n in KEYS}, f"slots T_AR={t_ar}")


# The largest trees that are accepted at (L, E): one union for all waves
# (4 to 16 KB a node), or one per wave (140 bytes a node).
@pytest.mark.parametrize("L,E,k", [(128, 1024, 3), (128, 513, 2), (48, 256, 8), (61, 200, 3),
                                   (35, 32, 4), (127, 64, 1)])
def test_trees_that_fill_the_lds(L, E, k):
    import paper_2608_15018_amd as s2
    N = s2.expand_max_nodes(L, E, k)
    few = random_batch(np.random.default_rng(L + E), 8, N, L, E, k, ragged=False)
    for t_ar, t_exp in ((64.0, 0.5 / (L * k)), (1.5, 0.05 / (L * k))):
        log(f"[expand] full T=8 N={N} L={L} E={E} k={k} T_AR={t_ar}")
        got = run_gpu(*few, E, t_ar, t_exp)
        compare(got, X.expand(few[0], few[1], few[2], few[3], E, t_ar, t_exp, few[4], few[5]),
                f"full T_AR={t_ar}")
