"""All words, a few hidden rows: every split of the words over waves and rounds (one wave of 16 words to several rounds of twelve), rows
of less than a step, of a ring of steps and one more element, rows that end inside a chunk, one to three groups of hidden rows,
pitched rows of E."""
import numpy as np
import pytest

import workloads
from gpu_harness import GpuCase, assert_close_logprobs, assert_order_of_ties, assert_topb_matches, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ty", ["fp32", "bf16"])
@pytest.mark.parametrize("V,d,S,B", [(8209, 8, 1, 1), (8210, 19, 1, 16), (8225, 255, 2, 8), (16385, 256, 1, 5), (12289, 257, 1, 17),
                                     (9001, 513, 3, 16), (36881, 64, 1, 16), (49153, 100, 1, 3), (100003, 33, 4, 4), (20011, 1000, 1, 12),
                                     (70001, 48, 1, 48), (40001, 641, 3, 13)])
def test_all_words_few_rows(V, d, S, B, ty):
    rng = np.random.default_rng(V + d + B)
    E = (rng.standard_normal((V, d)) / np.sqrt(d)).astype(np.float32)
    if ty == "bf16":
        E = workloads.f32_to_bf16_bits(E)
    perms = np.stack([rng.permutation(d)[:4] for _ in range(2)]).astype(np.int32)
    pitched = np.zeros((V, d + 3), E.dtype)
    pitched[:, :d] = E
    gc = GpuCase(E, perms, np.arange(4, dtype=np.int32), 2, E_dev=to_dev(pitched)[:, :d])
    H = (4.0 * rng.standard_normal((S * B, d))).astype(np.float32)
    bs = -np.sort(rng.random(S * B)).astype(np.float32)
    for _ in range(2):
        gb, gw, gs, sp, ws = gc.step(H, bs, S, B, full_vocab=True)
    for s in range(S):
        rows = slice(s * B, (s + 1) * B)
        ref = gc.oracle_sentence(H[rows], bs[rows], B, full_vocab=True)
        assert_close_logprobs(gc.tables.debug_logprobs(ws, sp, s, cap=V), ref)
        assert_topb_matches(gb[s], gw[s], gs[s], ref, bs[rows])


# Records of 256 and 384 words (k_logits_pass) and of 64 (k_logits_few; 64 rows: k_logits_rows): a few tiles opened, more than two
# sweeps (the threshold is found again), more keys than the list holds and more tiles than its list (the general path).
@pytest.mark.parametrize("V,d,ty", [(50003, 64, "fp32"), (90001, 64, "bf16"), (20011, 16, "fp32")])
@pytest.mark.parametrize("distinct", [1, 40, 400, 2000])
@pytest.mark.parametrize("B", [1, 12, 16, 17, 40, 64])
def test_all_words_tied(V, d, ty, distinct, B):
    """Word w has the embedding of word w % distinct: logits equal bit for bit, so that the order (beam, then word) says what comes
    out.  With the same hidden row and beam score for all beams everything is beam 0's; with scores far apart too; a beam apart by less
    than its words leaves those to the oracle, each set of equal words by its lowest."""
    rng = np.random.default_rng(V + B + distinct)
    E = (rng.standard_normal((distinct, d)) / np.sqrt(d)).astype(np.float32)
    if ty == "bf16":
        E = workloads.f32_to_bf16_bits(E)
    perms = np.stack([rng.permutation(d)[:4] for _ in range(2)]).astype(np.int32)
    gc = GpuCase(E[np.arange(V) % distinct], perms, np.arange(4, dtype=np.int32), 2)
    h = (4.0 * rng.standard_normal(d)).astype(np.float32)
    H = np.tile(h, (B, 1))
    for bs in (np.full(B, -1.5, np.float32), -20.0 * np.arange(1, B + 1, dtype=np.float32)):
        gb, gw, gs, sp, ws = gc.step(H, bs, 1, B, full_vocab=True)
        ref = gc.oracle_sentence(H[:1], bs[:1], B, full_vocab=True)
        best = int(np.argmax(ref.lp[0][:distinct]))
        if V // distinct >= B:
            assert np.all(gb == 0) and np.array_equal(gw[0], best + distinct * np.arange(B)) and np.all(gs == gs[0, 0])
        assert_close_logprobs(gc.tables.debug_logprobs(ws, sp, 0, cap=V)[:1], ref)
    H = (4.0 * rng.standard_normal((B, d))).astype(np.float32)
    bs = -np.sort(rng.random(B)).astype(np.float32)
    gb, gw, gs, sp, ws = gc.step(H, bs, 1, B, full_vocab=True)
    assert_topb_matches(gb[0], gw[0], gs[0], gc.oracle_sentence(H, bs, B, full_vocab=True), bs)
    assert_order_of_ties(gb[0], gw[0], gs[0], distinct)
