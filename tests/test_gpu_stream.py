"""The contraction of many tiles at the edges of its units, and the selection of winners that share a tile:
rows of one step, of a unit, of every number of parts and a bit more, odd lengths, both element types, one and
two row groups and several of them; few and many sentences (workgroups of their own, dealt to them, and an even cut),
lists of less than a tile up to several blocks of tiles."""
import numpy as np
import pytest

import workloads
from gpu_harness import GpuCase, assert_close_logprobs, assert_topb_matches
from test_gpu_parity import run_and_check

pytestmark = pytest.mark.gpu

_SHAPES = [
    # V, d, T, (S, B) ...
    (700, 8, 300, [(9, 3), (12, 17)]),
    (300, 63, 7, [(20, 1), (9, 16)]),
    (900, 129, 513, [(10, 5), (3, 40)]),
    (2500, 255, 1100, [(9, 20), (70, 2)]),
    (600, 516, 250, [(11, 16), (9, 33)]),
    (500, 780, 100, [(9, 4), (10, 17)]),
    (9000, 1000, 5000, [(9, 2), (9, 18)]),
    (400, 1025, 90, [(10, 12), (9, 20)]),
    (300, 1281, 130, [(9, 16)]),
    (350, 1666, 60, [(17, 3)]),
    (260, 2047, 40, [(9, 17)]),
]


def _case(V, d, T, bf16, run=1):
    """run: words in a row that are near copies of each other."""
    rng = np.random.default_rng(V + 3 * d)
    E = rng.standard_normal((V, d)).astype(np.float32)
    E = (E[np.arange(V) // run * run] + 0.05 * rng.standard_normal((V, d)).astype(np.float32)) / np.sqrt(d)
    K = min(4, d)
    perms = np.stack([rng.permutation(d)[:K] for _ in range(9)]).astype(np.int32)
    E = E.astype(np.float32)
    return rng, GpuCase(workloads.f32_to_bf16_bits(E) if bf16 else E, perms, np.arange(T, dtype=np.int32), 3)


@pytest.mark.parametrize("bf16", [False, True], ids=["fp32", "bf16"])
@pytest.mark.parametrize("shape", _SHAPES, ids=lambda s: "V%d-d%d" % s[:2])
def test_many_tiles(shape, bf16):
    V, d, T, calls = shape
    rng, gc = _case(V, d, T, bf16)
    for S, B in calls:
        H = (3.0 * rng.standard_normal((S * B, d))).astype(np.float32)
        run_and_check(None, gc, H, rng.standard_normal(S * B).astype(np.float32), S, B)


@pytest.mark.parametrize("bf16", [False, True], ids=["fp32", "bf16"])
@pytest.mark.parametrize("d", [132, 192, 196, 256, 260, 320, 384, 448, 508, 512, 520, 580, 700, 768])
def test_last_parts_of_every_length(d, bf16):
    """Rows of two and three parts whose last has one, some or all of its steps, with and without a partial chunk (bf16: of
    one and two), in one and two row groups."""
    rng, gc = _case(500, d + (2 if d % 3 == 0 else 0), 150, bf16)
    for S, B in [(9, 5), (9, 18)]:
        H = (3.0 * rng.standard_normal((S * B, gc.d))).astype(np.float32)
        run_and_check(None, gc, H, rng.standard_normal(S * B).astype(np.float32), S, B)


@pytest.mark.parametrize("V,T", [(1500, 40), (20000, 700)], ids=["few", "many"])
@pytest.mark.parametrize("B", [17, 32, 33, 50])
@pytest.mark.parametrize("d", [300, 430, 512])
def test_row_groups_of_two_parts(d, B, V, T):
    """Two, three and four times 16 rows, on either side of the tiles from which groups of 32 are taken."""
    rng, gc = _case(V, d, T, False)
    H = (3.0 * rng.standard_normal((4 * B, d))).astype(np.float32)
    run_and_check(None, gc, H, rng.standard_normal(4 * B).astype(np.float32), 4, B)


@pytest.mark.parametrize("run", [2, 3, 5, 16])
@pytest.mark.parametrize("B", [1, 2, 7, 16])
def test_winners_that_share_a_tile(B, run):
    rng, gc = _case(1500, 40, 400, False, run)
    words = gc.E[rng.integers(0, 1500, 2 * B)]
    H = (6.0 * words * np.sqrt(40.0) / np.sqrt((words * words).sum(1, keepdims=True)) / 2).astype(np.float32)
    run_and_check(None, gc, H, np.linspace(0, -1, 2 * B).astype(np.float32), 2, B)


@pytest.mark.parametrize("bf16", [False, True], ids=["fp32", "bf16"])
@pytest.mark.parametrize("d", [2050, 2052, 2056])
def test_longer_rows_end_in_a_split_round(d, bf16):
    """Rows too long for k_logits_stream, that end in a partial chunk of 16 bytes (or not): few tiles, all of them in
    the last round, which splits k."""
    rng, gc = _case(300, d, 60, bf16)
    for S, B in [(9, 3), (9, 17)]:
        H = (3.0 * rng.standard_normal((S * B, d))).astype(np.float32)
        run_and_check(None, gc, H, rng.standard_normal(S * B).astype(np.float32), S, B)


@pytest.mark.parametrize("bf16", [False, True], ids=["fp32", "bf16"])
@pytest.mark.parametrize("S,d", [(40, 600), (100, 300), (40, 40)])
def test_sentences_dealt_to_workgroups(S, d, bf16):
    """Numbers of sentences that would leave many workgroups without work if every sentence had as many on every XCD."""
    rng, gc = _case(3000, d, 1500, bf16)
    H = (3.0 * rng.standard_normal((S * 3, d))).astype(np.float32)
    run_and_check(None, gc, H, rng.standard_normal(S * 3).astype(np.float32), S, 3)


@pytest.mark.parametrize("bf16", [False, True], ids=["fp32", "bf16"])
@pytest.mark.parametrize("S,B", [(8, 12), (33, 3), (70, 3)])
@pytest.mark.parametrize("d", [100, 700])
def test_lists_of_different_lengths(d, S, B, bf16):
    """A few lists many times as long as the others: their sentences get more workgroups."""
    V = 24000
    rng = np.random.default_rng(S + d)
    E = rng.standard_normal((V, d)).astype(np.float32) / np.sqrt(d)
    E[:V // 2] = E[0] + 0.01 * E[:V // 2]                # (half of all words share their codes)
    E = E.astype(np.float32)
    perms = np.stack([rng.permutation(d)[:8] for _ in range(12)]).astype(np.int32)
    gc = GpuCase(workloads.f32_to_bf16_bits(E) if bf16 else E, perms, np.arange(600, dtype=np.int32), 3)
    H = (3.0 * rng.standard_normal((S, B, d))).astype(np.float32)
    H[1] = 3.0 * np.sqrt(d) * E[0]
    H[S - 2, 0] = H[1, 0]
    H = H.reshape(S * B, d)
    counts = [len(gc.index.candidates(H[s * B:(s + 1) * B], gc.topfreq)) for s in range(S)]
    assert counts[1] > 4 * np.median(counts)
    run_and_check(None, gc, H, rng.standard_normal(S * B).astype(np.float32), S, B)


@pytest.mark.parametrize("bf16", [False, True], ids=["fp32", "bf16"])
@pytest.mark.parametrize("B", [3, 18])
@pytest.mark.parametrize("d", [40, 100, 200, 300, 600, 1000, 1500, 2047])
def test_tiles_cut_evenly(d, B, bf16):
    """More sentences than workgroups (eight here, of one or two row groups): all tiles in a row, a workgroup goes from one
    sentence to the next, and through several blocks of candidates; rows of one and two steps and of several numbers of parts."""
    S = 20
    rng, gc = _case(1200, d, 700, bf16)
    gc.tables.set_options(logits_grid=8)
    H = (3.0 * rng.standard_normal((S * B, d))).astype(np.float32)
    run_and_check(None, gc, H, rng.standard_normal(S * B).astype(np.float32), S, B)


def test_more_sentences_than_workgroups():
    """Several times 64 sentences on eight workgroups, short lists."""
    S, B, d = 150, 2, 24
    rng, gc = _case(900, d, 0, False)
    gc.tables.set_options(logits_grid=8)
    H = (3.0 * rng.standard_normal((S * B, d))).astype(np.float32)
    H[2 * B:70 * B] = H[:1]                              # (one list for all of these)
    run_and_check(None, gc, H, rng.standard_normal(S * B).astype(np.float32), S, B)


@pytest.mark.parametrize("bf16", [False, True], ids=["fp32", "bf16"])
@pytest.mark.parametrize("B,d", [(3, 130), (3, 300), (18, 300)])
def test_lists_of_several_blocks(B, d, bf16):
    """Lists so long that a workgroup takes its candidates in several blocks, with masked words (logits that are made
    again) in the first, a middle and the last block."""
    S, V = 60, 12000
    rng, gc = _case(V, d, V, bf16)
    E = gc.E.copy()
    masked = [5, 16 * 8 * 34, V - 3]
    E[masked, 7] = 0xFF80 if bf16 else -np.inf
    gc = GpuCase(E, gc.perms, np.arange(V, dtype=np.int32), 3)
    H = (3.0 * rng.standard_normal((S * B, d))).astype(np.float32)
    H[:, 7] = 1.0
    bs = rng.standard_normal(S * B).astype(np.float32)
    gb, gw, gs, sp, ws = gc.step(H, bs, S, B)
    for s in (0, 17, S - 1):
        rows = slice(s * B, (s + 1) * B)
        with np.errstate(invalid="ignore"):
            ref = gc.oracle_sentence(H[rows], bs[rows], B)
        lp = gc.tables.debug_logprobs(ws, sp, s, cap=len(ref.cand))
        assert np.all(np.isneginf(lp[:, masked]))
        ref.lp[:, masked] = ref.logits[:, masked] = -1e30
        lp[:, masked] = -1e30
        assert_close_logprobs(lp, ref)
        assert_topb_matches(gb[s], gw[s], gs[s], ref, bs[rows])


@pytest.mark.parametrize("V,T", [(3000, 100), (12000, 3000)], ids=["few", "many"])
@pytest.mark.parametrize("B,d", [(33, 516), (40, 1000), (64, 1024)])
def test_one_sentence_of_many_beams(V, T, B, d):
    """One sentence of 33 to 64 beams on either side of the number of candidates from which all its rows are taken at
    once, and both kernels where the other one is the rule."""
    rng, gc = _case(V, d, T, False)
    H = (3.0 * rng.standard_normal((B, d))).astype(np.float32)
    bs = rng.standard_normal(B).astype(np.float32)
    for estage, t in ((-1, 1), (-1, 2), (0, 1), (1, 1)):
        gc.tables.set_options(logits_estage=estage)
        run_and_check(None, gc, H, bs, 1, B, threshold=t)
