"""The table build at the edges of its kernels: vocabularies around one and several chunks of the sort,
codes of one, two and three passes, bands whose words share one code, rows of every alignment, windows
longer than the registers hold, many permutations per row -- bucket for bucket against the oracle; and
permutations out of range."""
import numpy as np
import pytest

import oracle
import workloads
from gpu_harness import GpuCase, to_dev

pytestmark = pytest.mark.gpu

_SHAPES = [
    # V, d, K, u, W, bf16, equal rows
    (1, 2, 2, 1, 1, False, False),
    (63, 9, 3, 2, 3, True, False),
    (4096, 33, 8, 4, 2, False, False),
    (4097, 16, 2, 12, 2, True, False),
    (5000, 77, 16, 4, 5, True, False),
    (9001, 40, 8, 8, 2, False, False),
    (3000, 64, 4, 15, 3, False, False),
    (20000, 130, 24, 4, 3, False, True),
    (2500, 515, 8, 3, 100, True, False),
]


@pytest.mark.parametrize("shape", _SHAPES, ids=lambda s: "V%d-d%d-K%d-u%d-W%d" % s[:5])
def test_build_matches_the_oracle(shape):
    V, d, K, u, W, bf16, equal = shape
    rng = np.random.default_rng(V + d)
    E = rng.standard_normal((V, d)).astype(np.float32)
    if equal:                                       # long spans: most words are one of two vectors
        E[: V - V // 8] = E[rng.integers(0, 2, V - V // 8)]
    E = workloads.f32_to_bf16_bits(E) if bf16 else E
    perms = np.stack([rng.permutation(d)[:K] for _ in range(u * W)]).astype(np.int32)
    gc = GpuCase(E, perms, np.zeros(0, np.int32), W)
    assert np.array_equal(gc.tables.debug_embedding_codes(), oracle.band_codes(oracle.wta_codes(E, perms), W, K))
    assert gc.tables.debug_build_info()[0]
    for w in range(W) if W < 10 else (0, 1, W - 1):
        keys, offs, words = gc.tables.debug_csr(w)
        okeys = np.sort(gc.index.bucket_keys(w))
        buckets = [gc.index.bucket(w, int(k)) for k in okeys]
        assert np.array_equal(keys, okeys) and np.array_equal(words, np.concatenate(buckets))
        assert np.array_equal(np.diff(offs), [len(b) for b in buckets])
        for k in okeys[:: max(1, len(okeys) // 50)]:
            assert np.array_equal(gc.tables.debug_bucket(w, int(k)), gc.index.bucket(w, int(k)))


@pytest.mark.parametrize("V,d,K,u,W,direct", [(20000, 40, 4, 7, 3, True), (5000, 40, 4, 7, 3, False), (9000, 30, 2, 13, 4, True),
                                              (70000, 200, 16, 4, 8, True), (30000, 24, 16, 4, 12, False)])
def test_direct_tables_of_codes_of_several_passes(V, d, K, u, W, direct):
    """Codes of 13 to 16 bits, sorted in two passes: direct tables where cuckoo tables for the keys would be no smaller (their
    number known to be large, or counted), cuckoo tables otherwise; bucket for bucket, absent codes too, and the lists of a
    hit threshold, which read where the vocabulary slices begin in a span."""
    rng = np.random.default_rng(V)
    E = rng.standard_normal((V, d)).astype(np.float32)
    if V == 30000:                                  # (few codes come up)
        E = E[rng.integers(0, 500, V)]
    perms = np.stack([rng.permutation(d)[:K] for _ in range(u * W)]).astype(np.int32)
    gc = GpuCase(E, perms, np.arange(40, dtype=np.int32), W)
    bits = u * (K - 1).bit_length()
    assert (gc.tables.debug_cuckoo_shape(0)[0] == 2 << bits) == direct
    for w in (0, W - 1):
        keys, offs, words = gc.tables.debug_csr(w)
        okeys = np.sort(gc.index.bucket_keys(w))
        assert np.array_equal(keys, okeys) and np.array_equal(words, np.concatenate([gc.index.bucket(w, int(k)) for k in okeys]))
        for k in okeys[:: len(okeys) // 40]:
            assert np.array_equal(gc.tables.debug_bucket(w, int(k)), gc.index.bucket(w, int(k)))
        for k in np.setdiff1d(np.arange(0, 1 << bits, (1 << bits) // 50), okeys)[:10]:
            assert gc.tables.debug_bucket(w, int(k)) is None
    H = E[[7, V // 2, V - 1]] + 0.05 * rng.standard_normal((3, d)).astype(np.float32)
    for t in (1, 2):
        _, _, _, sp, ws = gc.step(H, np.zeros(3, np.float32), 1, 3, threshold=t)
        assert np.array_equal(gc.tables.debug_candidates(ws, sp, 0), gc.oracle_sentence(H, np.zeros(3), 3, threshold=t).cand)


@pytest.mark.parametrize("V", [1, 127, 129, 513, 2048 * 4 + 1, 40001])
def test_slices_of_direct_tables(V):
    """Codes few enough for direct tables: the slots and the places where the vocabulary slices begin in every span
    come out of the sort's counters.  The hit-count kernel reads both: its lists at V around the edges of slices and of
    the sort's chunks, and those of the cuckoo tables a short chain asks for, against the oracle's."""
    import os
    d, K, u, W, B, t = 24, 4, 2, 9, 3, 3
    rng = np.random.default_rng(V)
    E = rng.standard_normal((V, d)).astype(np.float32)
    perms = np.stack([rng.permutation(d)[:K] for _ in range(u * W)]).astype(np.int32)
    H = rng.standard_normal((B, d)).astype(np.float32)
    bs = np.zeros(B, np.float32)
    for chain in (None, "64"):
        if chain:
            os.environ["LSHBEAM_CUCKOO_CHAIN"] = chain
        try:
            gc = GpuCase(E, perms, np.arange(min(V, 3), dtype=np.int32), W)
        finally:
            os.environ.pop("LSHBEAM_CUCKOO_CHAIN", None)
        _, _, _, sp, ws = gc.step(H, bs, 1, B, threshold=t)
        assert np.array_equal(gc.tables.debug_candidates(ws, sp, 0), gc.oracle_sentence(H, bs, B, threshold=t).cand)


def test_permutations_out_of_range_are_refused():
    import paper_1806_00588_amd as lsh
    E = to_dev(np.random.default_rng(0).standard_normal((500, 12)).astype(np.float32))
    perms = np.tile(np.arange(4, dtype=np.int32), (300, 1))
    for bad in (-1, 12, 1 << 30):
        p = perms.copy()
        p[299, 3] = bad
        with pytest.raises(lsh.binding.LshBeamError):
            lsh.build_tables(E, to_dev(p), 4, 100)
    lsh.build_tables(E, to_dev(perms), 4, 100).close()


def test_a_handle_holds_its_tables_and_no_more():
    """Codes, ids and slots for the keys there are -- not for all 65536 a band could have, and not what the build
    worked in; a freed handle's memory is given back by release_kept, and freeing nothing does nothing."""
    import torch
    import paper_1806_00588_amd as lsh
    from paper_1806_00588_amd import binding
    V, d, K, u, W = 30000, 20, 16, 4, 12
    rng = np.random.default_rng(11)
    E = to_dev(rng.standard_normal((500, d)).astype(np.float32)[rng.integers(0, 500, V)])
    perms = to_dev(np.stack([rng.permutation(d)[:K] for _ in range(u * W)]).astype(np.int32))
    lsh.build_tables(E, perms, K, W).close()          # (whatever a first build brings with it)
    binding.release_kept()
    free = torch.cuda.mem_get_info()[0]
    t = lsh.build_tables(E, perms, K, W)
    slots = sum(t.debug_cuckoo_shape(w)[0] for w in range(W))
    assert slots <= W * 2048                          # at most 500 keys a band
    binding.release_kept()
    held = free - torch.cuda.mem_get_info()[0]
    assert held <= 2 * 4 * V * W + 32 * slots + (6 << 20), held      # (blocks of 2 MiB)
    t.close()
    kept = free - torch.cuda.mem_get_info()[0]
    assert kept <= 192 << 20
    binding.load_library().lsh_free_tables(None)
    assert free - torch.cuda.mem_get_info()[0] == kept
    binding.release_kept()
    assert torch.cuda.mem_get_info()[0] == free


def test_released_memory_shows_at_once():
    """After release_kept the free memory holds all of what was kept, blocks of whole and of partial 2 MiB pages, each time."""
    import time
    import torch
    import paper_1806_00588_amd as lsh
    from paper_1806_00588_amd import binding
    V, d, K, u, W = 30000, 20, 16, 4, 12
    rng = np.random.default_rng(11)
    E = to_dev(rng.standard_normal((500, d)).astype(np.float32)[rng.integers(0, 500, V)])
    perms = to_dev(np.stack([rng.permutation(d)[:K] for _ in range(u * W)]).astype(np.int32))
    lsh.build_tables(E, perms, K, W).close()
    binding.release_kept()
    time.sleep(0.05)
    free = torch.cuda.mem_get_info()[0]
    for _ in range(30):
        lsh.build_tables(E, perms, K, W).close()
        assert torch.cuda.mem_get_info()[0] < free
        binding.release_kept()
        assert torch.cuda.mem_get_info()[0] == free
