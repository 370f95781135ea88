"""Embeddings that mask a word (the type's lowest value, -inf) and hidden values at the end of the fp32 range,
through every contraction driver: the masked words get a hugely negative or -inf log-probability, every other
result stays what the oracle says.  The hidden values that meet a masked element are 1 and 0.5, whose lower
bf16 planes are zero; the elements lie at both ends of the row and in its middle."""
import numpy as np
import pytest

import workloads
from gpu_harness import GpuCase, assert_close_logprobs, assert_topb_matches

pytestmark = pytest.mark.gpu

# driver: S, B, V, full vocabulary, options, hidden sizes, element types
_HIDDEN = (200, 203)                     # whole 16-byte chunks that fill no step or unit; a partial chunk
_BOTH = ("fp32", "bf16")
_DRIVERS = {
    "rows": (4, 20, 9000, True, {}, _HIDDEN, _BOTH),
    "few": (1, 12, 9000, True, {}, _HIDDEN, _BOTH),
    "few, two row groups": (2, 12, 9000, True, {}, _HIDDEN, _BOTH),
    "few, three row groups": (4, 12, 9000, True, {}, _HIDDEN, ("fp32",)),
    "pass": (1, 12, 78000, True, {}, _HIDDEN, _BOTH),
    "pass, two row groups": (2, 12, 33000, True, {}, _HIDDEN, ("fp32",)),
    "pass, three row groups": (4, 11, 33000, True, {}, _HIDDEN, ("fp32",)),
    "stream": (9, 5, 1200, False, {}, (24, 200, 203), _BOTH),
    "stream, two row groups": (9, 20, 1200, False, {}, (200, 203), _BOTH),
    "stream, four parts": (9, 3, 1200, False, {}, (1540,), ("bf16",)),
    "stream, all words": (2, 5, 700, True, {}, (203,), _BOTH),
    "fused": (1, 5, 1200, False, {}, (200, 201, 203), _BOTH),
    "fused, t = 1 and parts": (1, 20, 1200, False, {"part_rows": 7}, (203,), _BOTH),
    "hidden rows in memory": (9, 20, 1200, False, {"logits_hlds": 0}, (200, 203), _BOTH),
    "k over 16 waves": (2, 5, 1200, False, {"fused": 0}, (203,), _BOTH),
    "k over 4 waves": (1, 70, 1200, False, {"logits_waves": 4}, (203,), _BOTH),
    "candidate rows in LDS": (2, 40, 1200, False, {}, (516, 1000), ("fp32",)),
    "hidden rows in LDS": (9, 5, 1200, False, {"logits_hlds": 1}, (200, 203), _BOTH),
    "hidden rows in LDS, two row groups": (9, 20, 1200, False, {"logits_hlds": 1}, (200, 203), _BOTH),
}
_CASES = [(n, d, ty) for n, (_, _, _, _, _, ds, tys) in _DRIVERS.items() for d in ds for ty in tys]


def _inputs(name, d, ty):
    S, B, V, full, options, _, _ = _DRIVERS[name]
    rng = np.random.default_rng(d + len(name))
    E = (rng.standard_normal((V, d)) / np.sqrt(d)).astype(np.float32)
    H = (4.0 * rng.standard_normal((S * B, d))).astype(np.float32)
    return rng, S, B, V, full, options, E, H


def _check(rng, S, B, V, full, options, E, H, ty):
    """Log-probabilities and winners of every sentence; returns how many words had none."""
    perms = np.stack([rng.permutation(E.shape[1])[:4] for _ in range(9)]).astype(np.int32)
    gc = GpuCase(workloads.f32_to_bf16_bits(E) if ty == "bf16" else E, perms, np.arange(min(V, 600), dtype=np.int32), 3)
    gc.tables.set_options(**options)
    bs = rng.standard_normal(S * B).astype(np.float32)
    gb, gw, gs, sp, ws = gc.step(H, bs, S, B, full_vocab=full)
    masked = 0
    for s in range(S):
        rows = slice(s * B, (s + 1) * B)
        with np.errstate(invalid="ignore"):
            ref = gc.oracle_sentence(H[rows], bs[rows], B, full_vocab=full)
        lp = gc.tables.debug_logprobs(ws, sp, s, cap=len(ref.cand))
        out = ref.lp < -1e30             # a masked word: as unlikely as the oracle says, if fp32 can say it
        assert np.all(lp[out] < -1e30) and np.all(np.isneginf(lp[np.isneginf(ref.lp)]))
        masked += int(out.sum())
        ref = ref._replace(lp=np.where(out, -1e30, ref.lp), logits=np.where(out, -1e30, ref.logits))
        assert_close_logprobs(np.where(out, np.float32(-1e30), lp), ref)
        assert_topb_matches(gb[s], gw[s], gs[s], ref, bs[rows])
    return masked


@pytest.mark.parametrize("value", ["lowest", "-inf"])
@pytest.mark.parametrize("case", _CASES, ids=lambda c: "%s-%d-%s" % c)
def test_masked_words(case, value):
    rng, S, B, V, full, options, E, H = _inputs(*case)
    d, ty = case[1:]
    low = -np.inf if value == "-inf" else np.float32(-3.3895314e38) if ty == "bf16" else np.finfo(np.float32).min
    for word, k in ((3, 0), (17, d // 2), (40, d - 2), (599, d - 1)):
        H[:, k] = 1.0
        H[::3, k] = 0.5
        E[word, k] = low
    assert _check(rng, S, B, V, full, options, E, H, ty) == 4 * S * B


@pytest.mark.parametrize("case", _CASES, ids=lambda c: "%s-%d-%s" % c)
def test_largest_hidden_values(case):
    rng, S, B, V, full, options, E, H = _inputs(*case)
    E[:, 5] = 0.0                        # the values meet nothing but zeros
    E[17, 5] = 2.0 ** -120
    H[0, 5], H[S * B - 1, 5] = np.finfo(np.float32).max, np.finfo(np.float32).min
    assert _check(rng, S, B, V, full, options, E, H, case[2]) == 0


@pytest.mark.parametrize("case", _CASES, ids=lambda c: "%s-%d-%s" % c)
def test_tiles_and_records_without_a_word(case):
    """A hundred words in a row masked: whole tiles of 16 and whole records of 64 with nothing but -inf."""
    rng, S, B, V, full, options, E, H = _inputs(*case)
    H[:, 5] = 1.0
    E[60:160, 5] = -np.inf
    assert _check(rng, S, B, V, full, options, E, H, case[2]) == 100 * S * B


@pytest.mark.parametrize("case", [c for c in _CASES if c[1] in (203, 1000)], ids=lambda c: "%s-%d-%s" % c)
def test_a_hidden_row_of_nan_is_alone(case):
    """A beam whose hidden row holds a NaN has no results; the others of its sentence have theirs."""
    rng, S, B, V, full, options, E, H = _inputs(*case)
    perms = np.stack([rng.permutation(E.shape[1])[:4] for _ in range(9)]).astype(np.int32)
    gc = GpuCase(workloads.f32_to_bf16_bits(E) if case[2] == "bf16" else E, perms, np.arange(min(V, 600), dtype=np.int32), 3)
    gc.tables.set_options(**options)
    H[1, 20] = np.nan
    bs = rng.standard_normal(S * B).astype(np.float32)
    gb, gw, gs, sp, ws = gc.step(H, bs, S, B, full_vocab=full)
    for s in range(S):
        rows = slice(s * B, (s + 1) * B)
        ref = gc.oracle_sentence(H[rows], bs[rows], B, full_vocab=full)
        lp = gc.tables.debug_logprobs(ws, sp, s, cap=len(ref.cand))
        bad = np.isnan(ref.lp)
        assert bad.sum() == (len(ref.cand) if s == 0 else 0) and np.array_equal(bad, np.isnan(lp))
        ref = ref._replace(lp=np.where(bad, -1e30, ref.lp), logits=np.where(bad, -1e30, ref.logits))
        assert_close_logprobs(np.where(bad, np.float32(-1e30), lp), ref)
        assert_topb_matches(gb[s], gw[s], gs[s], ref, bs[rows])
