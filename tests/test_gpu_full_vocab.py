"""The contraction of the full-vocabulary step at the edges of its tiles: rows of one and several row
tiles and groups, vocabularies around the 16- and 64-word tiles, hidden sizes around the blocks of 32 and
128 k and the 16-byte chunks, both element types."""
import numpy as np
import pytest

from test_gpu_parity import run_and_check
from gpu_harness import GpuCase
import workloads

pytestmark = pytest.mark.gpu

_SHAPES = [
    # V, d, (S, B) ...
    (1, 8, [(1, 1), (3, 7)]),
    (63, 9, [(1, 16), (1, 17)]),
    (65, 31, [(2, 16), (3, 11), (7, 7)]),
    (257, 33, [(1, 48), (7, 7), (1, 64), (5, 13)]),
    (300, 129, [(1, 2), (4, 16), (6, 16), (9, 9)]),
    (1025, 260, [(1, 33), (10, 10), (20, 16), (25, 20)]),
    (4100, 1000, [(2, 12), (32, 10)]),
]


@pytest.mark.parametrize("bf16", [False, True], ids=["fp32", "bf16"])
@pytest.mark.parametrize("shape", _SHAPES, ids=lambda s: "V%d-d%d" % s[:2])
def test_full_vocabulary_tiles(shape, bf16):
    V, d, calls = shape
    rng = np.random.default_rng(V * 7 + d)
    E = (rng.standard_normal((V, d)) / np.sqrt(d)).astype(np.float32)
    K = min(8, d)
    perms = np.stack([rng.permutation(d)[:K] for _ in range(4)]).astype(np.int32)
    gc = GpuCase(workloads.f32_to_bf16_bits(E) if bf16 else E, perms, np.zeros(0, np.int32), 2)
    for S, B in calls:
        H = (4.0 * rng.standard_normal((S * B, d))).astype(np.float32)
        bs = rng.standard_normal(S * B).astype(np.float32)
        run_and_check(None, gc, H, bs, S, B, full_vocab=True)
