"""Lists of nothing but the first tiles: every word has the same codes and no hidden row shares one, so that a list is the top-frequent
words, as many as fill those tiles.  The workgroup that ends such a step in the contraction's kernel reads ids that it has stored
itself.  Hit thresholds, and many beams hashed in parts; one and two row groups, rows that end in a partial chunk, as many tiles as are made at
most.  (words_expected: what the plan goes by, words that collide by chance alone.)"""
import math

import numpy as np
import pytest

from gpu_harness import GpuCase, assert_close_logprobs, assert_topb_matches

pytestmark = pytest.mark.gpu

SHAPES = [(4, 2, 704, 2, 4000, 100, False), (4, 2, 704, 2, 4000, 101, True), (1, 12, 2048, 2, 8000, 1001, False), (1, 17, 2048, 2, 6000, 130, False),
          (1, 30, 2048, 1, 6000, 1536, False), (1, 30, 2048, 1, 6000, 1531, True)]


def words_expected(S, B, T, t, V, W, K, u):
    m = W * K ** -u
    below = sum(math.exp(-m) * m ** i / math.factorial(i) for i in range(t))
    return V - (V - T) * below ** B


@pytest.mark.parametrize("S,B,T,t,V,d,bf16", SHAPES)
def test_lists_of_the_first_tiles_alone(S, B, T, t, V, d, bf16):
    rng = np.random.default_rng(V + d)
    W, K, u = 8, 4, 4 if t == 1 else 2
    assert words_expected(S, B, T, t, V, W, K, u) > 16 * (256 // S) and T % 16 == 0     # a tile and more for each workgroup, by chance alone
    e = rng.standard_normal(d).astype(np.float32)
    E = rng.uniform(0.5, 1.5, (V, 1)).astype(np.float32) * e
    if bf16:
        E = (E.view(np.uint32) >> 16).astype(np.uint16)
    perms = np.stack([rng.permutation(d)[:K] for _ in range(u * W)]).astype(np.int32)
    gc = GpuCase(E, perms, np.arange(T, dtype=np.int32), W)
    H = (-rng.uniform(0.5, 1.5, (S * B, 1)).astype(np.float32) * e / np.sqrt(d)).astype(np.float32)
    bs = -np.sort(rng.random(S * B)).astype(np.float32)
    got = {}
    for plan, opts in (("two", {}), ("one", dict(one_launch=1))):
        gc.tables.reset_options()
        gc.tables.set_options(**opts)
        for _ in range(3):
            gb, gw, gs, sp, ws = gc.step(H, bs, S, B, threshold=t)
            lps = [gc.tables.debug_logprobs(ws, sp, s, cap=T) for s in range(S)]
            assert all(np.array_equal(gc.tables.debug_candidates(ws, sp, s), np.arange(T)) for s in range(S))
            got.setdefault(plan, (gb, gw, gs, *lps))
            assert all(np.array_equal(x, y) for x, y in zip(got[plan], (gb, gw, gs, *lps)))
    gc.tables.reset_options()
    assert all(np.array_equal(x, y) for x, y in zip(got["two"], got["one"]))
    for s in range(S):
        rows = slice(s * B, (s + 1) * B)
        ref = gc.oracle_sentence(H[rows], bs[rows], B, threshold=t)
        assert np.array_equal(ref.cand, np.arange(T))
        assert_close_logprobs(got["two"][3 + s], ref)
        assert_topb_matches(got["two"][0][s], got["two"][1][s], got["two"][2][s], ref, bs[rows])
