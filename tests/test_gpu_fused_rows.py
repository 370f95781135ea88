"""The fused kernel's candidate rows on both sides of the line from which lanes load them for each other: rows of one step for each wave and a bit more, whole
and partial last chunks, pitches that put rows at any multiple of an element's bytes; one and two row groups, a tile and several tiles for
each workgroup. """
import numpy as np
import pytest

import workloads
from gpu_harness import GpuCase, assert_close_logprobs, assert_topb_matches

pytestmark = pytest.mark.gpu

ROWS = [(ty, d, ld) for ty, ds in (("fp32", (256, 257, 260, 262, 1000, 1003)), ("bf16", (512, 513, 520, 524, 1000, 1001)))
        for d in ds for ld in (d, d + 1, (d + 15) // 16 * 16)]


@pytest.mark.parametrize("S,B,V,T", [(1, 12, 3000, 300), (2, 5, 12000, 7000), (1, 21, 3000, 1000)])
@pytest.mark.parametrize("ty,d,ld", ROWS)
def test_rows_of_the_fused_kernel(ty, d, ld, S, B, V, T):
    import torch
    rng = np.random.default_rng(d + ld)
    E = (rng.standard_normal((V, d)) / np.sqrt(d)).astype(np.float32)
    perms = np.stack([rng.permutation(d)[:4] for _ in range(9)]).astype(np.int32)
    if ty == "bf16":
        E = workloads.f32_to_bf16_bits(E)
    wide = torch.full((V, ld), -1 if ty == "bf16" else float("nan"), dtype=torch.int16 if ty == "bf16" else torch.float32, device="cuda")
    wide[:, :d] = torch.from_numpy(E.view(np.int16) if ty == "bf16" else E).cuda()
    gc = GpuCase(E, perms, np.arange(T, dtype=np.int32), 3, E_dev=wide[:, :d])
    H = (3.0 * rng.standard_normal((S * B, d))).astype(np.float32)
    bs = -np.sort(rng.random(S * B)).astype(np.float32)
    for one in (0, 1):
        gc.tables.reset_options()
        gc.tables.set_options(fused=1, one_launch=one)
        gb, gw, gs, sp, ws = gc.step(H, bs, S, B)
        for s in range(S):
            rows = slice(s * B, (s + 1) * B)
            ref = gc.oracle_sentence(H[rows], bs[rows], B)
            assert np.array_equal(gc.tables.debug_candidates(ws, sp, s), ref.cand)
            assert_close_logprobs(gc.tables.debug_logprobs(ws, sp, s, cap=len(ref.cand)), ref)
            assert_topb_matches(gb[s], gw[s], gs[s], ref, bs[rows])
    gc.tables.reset_options()
