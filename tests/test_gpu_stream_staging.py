"""The streamed tiles' hidden rows on both sides of the line from which they come through LDS, by the parts of a row that LDS holds: all of them, two of three
or four, one of the two or four that two row groups have.  Lists alike, and a few many times as long as the others, where some workgroups are
dealt to another sentence than the one known in front and some keep theirs."""
import numpy as np
import pytest

import workloads
from gpu_harness import GpuCase
from test_gpu_parity import run_and_check

pytestmark = pytest.mark.gpu

CALLS = [(d, B) for ds, bs in (((40, 128), (12, 16, 17, 32)), ((129, 300, 512), (1, 7, 8, 16, 17, 30)), ((513, 1000, 1025, 1536, 1537, 2045), (1, 2, 3, 16)))
         for d in ds for B in bs]


@pytest.mark.parametrize("differ", [False, True], ids=["alike", "differ"])
@pytest.mark.parametrize("d,B", CALLS)
def test_hidden_rows_through_lds(d, B, differ):
    S, V = 16, 8000
    rng = np.random.default_rng(S + d)
    E = rng.standard_normal((V, d)).astype(np.float32) / np.sqrt(d)
    if differ:
        E[:V // 2] = E[0] + 0.01 * E[:V // 2]            # (half of all words share their codes)
    E = E.astype(np.float32)
    perms = np.stack([rng.permutation(d)[:8] for _ in range(12)]).astype(np.int32)
    gc = GpuCase(workloads.f32_to_bf16_bits(E), perms, np.arange(V - 500, V, dtype=np.int32), 3)
    H = (3.0 * rng.standard_normal((S, B, d))).astype(np.float32)
    if differ:
        H[1] = 3.0 * np.sqrt(d) * E[0]
        H[S - 2, 0] = H[1, 0]
    H = H.reshape(S * B, d)
    counts = [len(gc.index.candidates(H[s * B:(s + 1) * B], gc.topfreq)) for s in range(S)]
    assert (counts[1] > 2 * np.median(counts)) == differ
    run_and_check(None, gc, H, rng.standard_normal(S * B).astype(np.float32), S, B)
