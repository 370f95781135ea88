"""The union of bitmaps in front of the contraction: rows of one word, of fewer and more words than a chunk of four, of more chunks than
threads; fewer and more bitmaps than are asked for at a time; hidden rows that come to LDS meanwhile, whose number of floats is a
multiple of four or not, and hidden rows that have no room there; with hit thresholds and with many beams hashed in parts.  The plan with
the union in a kernel of its own and the selection in the same kernel as the contraction give the same bits."""
import numpy as np
import pytest

from gpu_harness import GpuCase, assert_close_logprobs, assert_topb_matches

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("V,S,B,T,t,d,bf16", [
    (20, 1, 3, 5, 2, 24, False), (100, 2, 5, 10, 2, 33, False), (130, 1, 17, 10, 3, 70, True), (4000, 1, 12, 300, 4, 1001, False),
    (4000, 3, 9, 300, 4, 263, False), (4000, 1, 32, 300, 5, 1536, False), (4000, 1, 30, 300, 1, 1024, True), (5000, 2, 31, 300, 1, 999, False),
    (140000, 1, 2, 300, 5, 24, False), (140000, 2, 5, 300, 6, 40, True)])
def test_union_and_contraction(V, S, B, T, t, d, bf16):
    rng = np.random.default_rng(V + d)
    W, K = 8, 4
    E = rng.standard_normal((V, d)).astype(np.float32)
    if bf16:
        E = (E.view(np.uint32) >> 16).astype(np.uint16)
    perms = np.stack([rng.permutation(d)[:K] for _ in range((4 if t == 1 else 2) * W)]).astype(np.int32)
    topfreq = rng.permutation(V)[:T].astype(np.int32)
    gc = GpuCase(E, perms, topfreq, W)
    H = rng.standard_normal((S * B, d)).astype(np.float32) / np.sqrt(d)
    bs = -np.sort(rng.random(S * B)).astype(np.float32)
    got = {}
    for plan, opts in (("two", dict(fused=1)), ("one", dict(fused=1, one_launch=1)), ("three", dict(fused=0))):
        gc.tables.reset_options()
        gc.tables.set_options(**opts)
        gb, gw, gs, sp, ws = gc.step(H, bs, S, B, threshold=t)
        cands = [gc.tables.debug_candidates(ws, sp, s) for s in range(S)]
        lps = [gc.tables.debug_logprobs(ws, sp, s, cap=len(cands[s])) for s in range(S)]
        got[plan] = (gb, gw, gs, *cands, *lps)
    gc.tables.reset_options()
    assert all(np.array_equal(x, y) for x, y in zip(got["two"], got["one"]))
    assert all(np.array_equal(got["two"][3 + s], got["three"][3 + s]) for s in range(S))
    for s in range(S):
        rows = slice(s * B, (s + 1) * B)
        ref = gc.oracle_sentence(H[rows], bs[rows], B, threshold=t)
        assert np.array_equal(got["two"][3 + s], ref.cand)
        assert_close_logprobs(got["two"][3 + S + s], ref)
        assert_topb_matches(got["two"][0][s], got["two"][1][s], got["two"][2][s], ref, bs[rows])
