"""The selection where its number of records per lane and of lanes per hidden row changes: lists of 64, 128, 256, 512 and 1024
tiles and one word more, 1 to 65 beams; scores apart, tied by the hundred (more tiles than are opened at once, more keys than
are ranked by ballot) and all the same (the exact select).  The list is all of V: every word is a top-frequent one."""
import numpy as np
import pytest

from gpu_harness import GpuCase, assert_close_logprobs, assert_topb_matches

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("V", [16, 1024, 1025, 2048, 2049, 4096, 4097, 8193, 16384, 16385])
@pytest.mark.parametrize("B", [1, 16, 17, 40, 64, 65])
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
