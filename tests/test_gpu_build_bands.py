"""Tables whose slots come out of the sort's scan, with a band's chunks on one XCD: seven, eight, nine, sixteen and seventeen bands (all, and a
last round of some), vocabularies of one and several chunks and pieces of a wave, words that share one code; every band's words and
the step's lists against the oracle; and permutations out of range, which this build's first kernel reports."""
import numpy as np
import pytest

from gpu_harness import GpuCase, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("W", [7, 8, 9, 16, 17])
@pytest.mark.parametrize("V", [1, 70, 2049, 33001])
def test_every_band(V, W):
    rng = np.random.default_rng(V + W)
    d, K, u = 24, 8, 4
    E = rng.standard_normal((V, d)).astype(np.float32)
    E[: V // 3] = E[0]
    perms = np.stack([rng.permutation(d)[:K] for _ in range(u * W)]).astype(np.int32)
    gc = GpuCase(E, perms, np.arange(min(V, 30), dtype=np.int32), W)
    for w in range(W):
        keys, offs, words = gc.tables.debug_csr(w)
        okeys = np.sort(gc.index.bucket_keys(w))
        buckets = [gc.index.bucket(w, int(k)) for k in okeys]
        assert np.array_equal(keys, okeys) and np.array_equal(words, np.concatenate(buckets))
        assert np.array_equal(np.diff(offs), [len(b) for b in buckets])
    H = rng.standard_normal((3, d)).astype(np.float32)
    _, _, _, sp, ws = gc.step(H, np.zeros(3, np.float32), 1, 3)
    assert np.array_equal(gc.tables.debug_candidates(ws, sp, 0), gc.oracle_sentence(H, np.zeros(3), 3).cand)


@pytest.mark.parametrize("bad", [-1, 24, 2**31 - 1])
@pytest.mark.parametrize("P,at", [(32, 0), (32, 31), (64, 40)])
def test_positions_outside_a_row(P, at, bad):
    import paper_1806_00588_amd as lsh
    rng = np.random.default_rng(P)
    perms = np.stack([rng.permutation(24)[:8] for _ in range(P)]).astype(np.int32)
    perms[at, at % 8] = bad
    E = to_dev(rng.standard_normal((3000, 24)).astype(np.float32))
    with pytest.raises(lsh.LshBeamError):
        lsh.build_tables(E, to_dev(perms), 8, P // 4)
