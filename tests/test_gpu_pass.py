"""All words, a few hidden rows (k_logits_pass): splits of the words over four to twelve waves and one to five rounds, rows of less than a
step of 64 bytes, of one, of a ring of 16 steps, one element less and one more, rows that end inside a chunk, one to three groups of
hidden rows, pitched rows of E.  That the calls are this kernel's is checked with the other plans (test_host_plans.py)."""
import numpy as np
import pytest

import workloads
from gpu_harness import GpuCase, assert_close_logprobs, assert_order_of_ties, assert_topb_matches, to_dev

pytestmark = pytest.mark.gpu

# type, V, d, pitch, S, B, waves of a workgroup, times 16 words for each
SHAPES = [
    ("fp32", 57345, 8, 11, 1, 1, 8, 2), ("fp32", 66001, 16, 19, 1, 16, 9, 2), ("fp32", 34000, 19, 22, 1, 16, 9, 1),
    ("fp32", 8225, 150, 153, 2, 8, 4, 1), ("fp32", 12289, 257, 260, 1, 17, 4, 1), ("fp32", 17001, 255, 258, 1, 5, 5, 1),
    ("fp32", 22003, 32, 64, 3, 5, 6, 1), ("fp32", 26001, 300, 303, 1, 48, 7, 1), ("fp32", 31000, 601, 604, 1, 12, 8, 1),
    ("fp32", 33001, 1000, 1000, 1, 12, 9, 1), ("fp32", 38000, 48, 51, 2, 20, 10, 1), ("fp32", 44003, 100, 103, 1, 3, 11, 1),
    ("fp32", 48001, 641, 644, 3, 11, 12, 1), ("fp32", 75001, 33, 36, 4, 4, 10, 2), ("fp32", 86003, 20, 23, 1, 31, 11, 2),
    ("fp32", 93001, 64, 64, 1, 48, 12, 2), ("fp32", 100003, 256, 259, 2, 2, 9, 3), ("fp32", 137003, 17, 20, 1, 7, 12, 3),
    ("fp32", 125003, 9, 12, 1, 20, 8, 4), ("fp32", 200003, 16, 16, 1, 2, 10, 5),
    ("bf16", 140001, 24, 27, 1, 1, 12, 3), ("bf16", 150001, 32, 32, 2, 8, 10, 4), ("bf16", 200003, 33, 36, 1, 16, 10, 5),
    ("bf16", 100003, 513, 516, 3, 5, 9, 3), ("bf16", 80001, 512, 512, 1, 12, 10, 2), ("bf16", 90003, 511, 514, 2, 3, 11, 2),
    ("bf16", 70001, 601, 604, 1, 3, 9, 2), ("bf16", 90003, 40, 43, 1, 12, 11, 2), ("bf16", 17003, 1001, 1004, 1, 7, 5, 1),
    ("bf16", 125003, 150, 150, 4, 4, 8, 4),
]


@pytest.mark.parametrize("ty,V,d,pitch,S,B,waves,rounds", SHAPES)
def test_all_words_few_rows(ty, V, d, pitch, S, B, waves, rounds):
    rng = np.random.default_rng(V + d + B)
    E = (rng.standard_normal((V, d)) / np.sqrt(d)).astype(np.float32)
    if ty == "bf16":
        E = workloads.f32_to_bf16_bits(E)
    perms = np.stack([rng.permutation(d)[:4] for _ in range(2)]).astype(np.int32)
    pitched = np.zeros((V, pitch), E.dtype)
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


# Records of 256 and 352 words (k_logits_pass; of bf16 words 9 to 16 beams) and of 64 (k_logits_few; 64 rows: k_logits_rows): a few tiles
# opened, more than two sweeps (the threshold is found again), more keys than the list holds and more tiles than its list (the general path).
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
