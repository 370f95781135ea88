"""Candidate lists where their making changes: spans from a few ids to a thousand (walked one by one, or all of a chunk's in groups
of four, two, four or eight groups in flight per thread), bitmaps written by one workgroup and by four, top-frequent words in
one piece and scattered."""
import numpy as np
import pytest

from gpu_harness import GpuCase

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("V", [257, 3001, 20011, 65536, 65537, 65600, 131071, 200003])
@pytest.mark.parametrize("K,B", [(2, 9), (4, 3), (16, 11)])
def test_lists_against_the_oracle(V, K, B):
    rng = np.random.default_rng(V + K)
    d, W, S = 40, 13, 3
    perms = np.stack([rng.permutation(d)[:K] for _ in range(3 * W)]).astype(np.int32)
    E = rng.standard_normal((V, d)).astype(np.float32)
    topfreq = rng.permutation(V)[:min(V, 1500)] if K == 4 else np.arange(min(V, 1100))
    gc = GpuCase(E, perms, topfreq.astype(np.int32), W)
    gc.tables.set_options(fused=0)
    H = rng.standard_normal((S * B, d)).astype(np.float32)
    _, _, _, sp, ws = gc.step(H, np.zeros(S * B, np.float32), S, B)
    for s in range(S):
        want = gc.index.candidates(H[s * B:(s + 1) * B], gc.topfreq)
        assert np.array_equal(gc.tables.debug_candidates(ws, sp, s), want)


@pytest.mark.parametrize("S", [64, 65])
def test_as_many_sentences_as_are_split(S):
    rng = np.random.default_rng(S)
    V, d, W, B = 65573, 24, 5, 2
    perms = np.stack([rng.permutation(d)[:8] for _ in range(3 * W)]).astype(np.int32)
    gc = GpuCase(rng.standard_normal((V, d)).astype(np.float32), perms, np.arange(V - 700, V, dtype=np.int32), W)
    H = rng.standard_normal((S * B, d)).astype(np.float32)
    _, _, _, sp, ws = gc.step(H, np.zeros(S * B, np.float32), S, B)
    for s in range(S):
        want = gc.index.candidates(H[s * B:(s + 1) * B], gc.topfreq)
        assert np.array_equal(gc.tables.debug_candidates(ws, sp, s), want), s
