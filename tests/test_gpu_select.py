"""The selection where its number of records per lane and of lanes per hidden row changes: lists of 64, 128, 256, 512 and 1024
tiles and one word more, and of several times what fits in registers, 1 to 65 beams; scores apart, close together, tied by the hundred
(more tiles than are opened at once, more keys than are ranked by ballot) and all the same (the exact select).  The list is all of V: every word is a top-frequent one.  Of equal scores
the lower beam comes first, then the lower word."""
import numpy as np
import pytest

from gpu_harness import GpuCase, assert_close_logprobs, assert_order_of_ties, assert_topb_matches

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("V", [16, 1024, 1025, 2048, 2049, 4096, 4097, 8193, 16384, 16385, 24577, 40003])
@pytest.mark.parametrize("B", [1, 16, 17, 32, 33, 40, 64, 65])
def test_records_per_lane(V, B):
    rng = np.random.default_rng(V + B)
    d, S = 16, 2
    perms = np.stack([rng.permutation(d)[:4] for _ in range(4)]).astype(np.int32)
    for distinct in (V, 40, 1):
        E = rng.standard_normal((min(V, distinct), d)).astype(np.float32)[np.arange(V) % min(V, distinct)]
        gc = GpuCase(E, perms, np.arange(V, dtype=np.int32), 2)
        gc.tables.set_options(fused=0)
        H = rng.standard_normal((S * B, d)).astype(np.float32)
        bs = -np.sort(rng.random(S * B)).astype(np.float32)
        gb, gw, gs, sp, ws = gc.step(H, bs, S, B)
        for s in range(S):
            rows = slice(s * B, (s + 1) * B)
            ref = gc.oracle_sentence(H[rows], bs[rows], B)
            assert len(ref.cand) == V
            assert_close_logprobs(gc.tables.debug_logprobs(ws, sp, s, cap=V), ref)
            assert_topb_matches(gb[s], gw[s], gs[s], ref, bs[rows])
            assert_order_of_ties(gb[s], gw[s], gs[s], distinct)


# 2000 words: no more tiles than are opened at once for any threshold; then some hundred to several thousand (more than are listed)
# reach a row's or the lanes' threshold, and the listed ones' own is found.  The first beam far ahead: all results are of one row.
@pytest.mark.parametrize("full", [False, True])
@pytest.mark.parametrize("V", [2000, 8193, 16384, 40003])
@pytest.mark.parametrize("B", [2, 16, 17, 32, 33, 50, 64])
def test_close_scores(V, B, full):
    rng = np.random.default_rng(V + B)
    d, S = 16, 2
    perms = np.stack([rng.permutation(d)[:4] for _ in range(4)]).astype(np.int32)
    gc = GpuCase(rng.standard_normal((V, d)).astype(np.float32), perms, np.arange(V, dtype=np.int32), 2)
    gc.tables.set_options(fused=0)
    H = (0.05 * rng.standard_normal((S * B, d))).astype(np.float32)
    for bs in (-np.sort(rng.random(S * B)).astype(np.float32) * 0.05, np.where(np.arange(S * B) % B == 0, 0, -9).astype(np.float32)):
        gb, gw, gs, sp, ws = gc.step(H, bs, S, B, full_vocab=full)
        for s in range(S):
            rows = slice(s * B, (s + 1) * B)
            ref = gc.oracle_sentence(H[rows], bs[rows], B, full_vocab=full)
            assert_close_logprobs(gc.tables.debug_logprobs(ws, sp, s, cap=V), ref)
            assert_topb_matches(gb[s], gw[s], gs[s], ref, bs[rows])


# tiles that reach the threshold, and keys: 200 of each; 257 to some thousand; as many as the lists hold; more than they hold
@pytest.mark.parametrize("fused", [0, 1])
@pytest.mark.parametrize("V,distinct,B", [(8000, 40, 1), (8000, 40, 16), (8000, 40, 17), (8000, 40, 64), (8000, 20, 10), (8000, 20, 32),
                                          (4096, 1, 16), (8192, 2, 32), (16000, 4, 2), (16384, 16, 4)])
def test_tied_rows(V, distinct, B, fused):
    """Hidden rows and beam scores the same too: beam 0 has all results, the lowest copies of the best word, in order."""
    rng = np.random.default_rng(V + B + distinct)
    d = 16
    perms = np.stack([rng.permutation(d)[:4] for _ in range(4)]).astype(np.int32)
    E = rng.standard_normal((distinct, d)).astype(np.float32)[np.arange(V) % distinct]
    gc = GpuCase(E, perms, np.arange(V, dtype=np.int32), 2)
    gc.tables.set_options(fused=fused)
    h = rng.standard_normal(d).astype(np.float32)
    best = int(np.argmax(E[:distinct].astype(np.float64) @ h))
    gb, gw, gs, _, _ = gc.step(np.tile(h, (B, 1)), np.full(B, -1.5, np.float32), 1, B)
    assert np.all(gb == 0) and np.array_equal(gw[0], best + distinct * np.arange(B)) and np.all(gs == gs[0, 0])
