"""All words, a few hidden rows: every split of the words over waves and rounds (one wave of 16 words to several rounds of twelve), rows
of less than a step, of a ring of steps and one more element, rows that end inside a chunk, one to three groups of hidden rows,
pitched rows of E."""
import numpy as np
import pytest

import workloads
from gpu_harness import GpuCase, assert_close_logprobs, assert_topb_matches, to_dev

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
