"""The union of row bitmaps in front of the contraction, by the number of rows: full rounds of twelve, and two, four, eight or twelve for those
that are left; bitmaps of fewer words than a workgroup has threads, of one word and of two for each thread with the last ones shared, of more
than two.  Lists and selections against the oracle; the plan whose union is a kernel of its own gives the same lists."""
import numpy as np
import pytest

from gpu_harness import GpuCase, assert_close_logprobs, assert_topb_matches

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("V,d", [(3000, 24), (32768, 8), (40000, 8), (50001, 8), (70000, 8)])
@pytest.mark.parametrize("B", [1, 2, 3, 5, 9, 12, 13, 14, 15, 16, 17, 20, 21, 24, 25, 26, 29, 32])
def test_rows_of_every_remainder(V, d, B):
    rng = np.random.default_rng(V + B)
    W, K, T, t = 6, 4, 70, 4
    E = rng.standard_normal((V, d)).astype(np.float32)
    perms = np.stack([rng.permutation(d)[:K] for _ in range(3 * W)]).astype(np.int32)
    gc = GpuCase(E, perms, rng.permutation(V)[:T].astype(np.int32), W)
    H = rng.standard_normal((B, d)).astype(np.float32) / np.sqrt(d)
    H[B // 2] = E[V - 1]                                                       # (a row whose word is in the last bit)
    bs = -np.sort(rng.random(B)).astype(np.float32)
    ref = gc.oracle_sentence(H, bs, B, threshold=t)
    assert ref.cand[-1] == V - 1
    for opts in (dict(fused=1), dict(fused=0)):
        gc.tables.reset_options()
        gc.tables.set_options(**opts)
        gb, gw, gs, sp, ws = gc.step(H, bs, 1, B, threshold=t)
        assert np.array_equal(gc.tables.debug_candidates(ws, sp, 0), ref.cand)
        assert_close_logprobs(gc.tables.debug_logprobs(ws, sp, 0, cap=len(ref.cand)), ref)
        assert_topb_matches(gb[0], gw[0], gs[0], ref, bs)
    gc.tables.reset_options()
