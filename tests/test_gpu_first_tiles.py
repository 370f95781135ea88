"""Hit thresholds: the first tiles of the lists, made beside the hashing where the top-frequent list is expected to fill them.  Lists that
begin with the ids 0, 1, 2, ... and lists that do not (the top-frequent list begins at 3, or leaves one id out, which a sentence may
hit or not); a last top-frequent word in the middle of a tile; lists of nothing but those tiles; shuffled and repeated ids; one to
four sentences, one and two row groups; with the selection in a kernel of its own and in the same one.  The plan with the union in a
kernel of its own, which makes every tile of every list, gives the same bits."""
import numpy as np
import pytest

from gpu_harness import GpuCase, assert_close_logprobs, assert_topb_matches

pytestmark = pytest.mark.gpu

LISTS = {
    "from 0": lambda T, rng: np.arange(T),
    "shuffled": lambda T, rng: rng.permutation(T),
    "repeated": lambda T, rng: np.concatenate([rng.permutation(T - 40), np.arange(40)]),
    "from 3": lambda T, rng: np.arange(3, T + 3),
    "but 17": lambda T, rng: np.delete(np.arange(T + 1), 17),
}


@pytest.mark.parametrize("name", LISTS)
@pytest.mark.parametrize("S,B,T,t,d,bf16", [(4, 2, 704, 2, 100, False), (4, 2, 711, 9, 100, True), (1, 12, 2600, 2, 1001, False), (2, 17, 1300, 5, 130, False),
                                            (3, 5, 900, 3, 24, True)])
def test_lists_and_their_first_tiles(name, S, B, T, t, d, bf16):
    rng = np.random.default_rng(T + d)
    V, W, K = 4000, 8, 4
    E = rng.standard_normal((V, d)).astype(np.float32)
    if bf16:
        E = (E.view(np.uint32) >> 16).astype(np.uint16)
    perms = np.stack([rng.permutation(d)[:K] for _ in range(2 * W)]).astype(np.int32)
    topfreq = LISTS[name](T, rng).astype(np.int32)
    gc = GpuCase(E, perms, topfreq, W)
    H = rng.standard_normal((S * B, d)).astype(np.float32) / np.sqrt(d)
    bs = -np.sort(rng.random(S * B)).astype(np.float32)
    got = {}
    for plan, opts in (("two", {}), ("one", dict(one_launch=1)), ("three", dict(fused=0))):
        gc.tables.reset_options()
        gc.tables.set_options(**opts)
        gb, gw, gs, sp, ws = gc.step(H, bs, S, B, threshold=t)
        cands = [gc.tables.debug_candidates(ws, sp, s) for s in range(S)]
        lps = [gc.tables.debug_logprobs(ws, sp, s, cap=len(cands[s])) for s in range(S)]
        got[plan] = (gb, gw, gs, *cands, *lps)
    gc.tables.reset_options()
    for plan in ("one", "three"):
        assert all(np.array_equal(x, y) for x, y in zip(got["two"], got[plan])), plan
    for s in range(S):
        rows = slice(s * B, (s + 1) * B)
        ref = gc.oracle_sentence(H[rows], bs[rows], B, threshold=t)
        assert np.array_equal(got["two"][3 + s], ref.cand)
        assert_close_logprobs(got["two"][3 + S + s], ref)
        assert_topb_matches(got["two"][0][s], got["two"][1][s], got["two"][2][s], ref, bs[rows])
