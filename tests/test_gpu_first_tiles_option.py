"""First tiles as many as the option first_tiles asks for, with the same bits as none: hit thresholds, and many beams hashed in parts; one and two
row groups; rows that end in a partial chunk; a top-frequent list that fills the most tiles that are made and more; fewer tiles than it fills.
Top-frequent lists that do not begin 0, 1, 2, ... up to the last word of those tiles: nothing is made beside the hashing, which shows in a
workspace that holds nothing but a mark behind the end of the lists.  Several steps in the same workspace, and a replayed graph."""
import numpy as np
import pytest

from gpu_harness import GpuCase, assert_close_logprobs, assert_topb_matches, to_dev

pytestmark = pytest.mark.gpu

MOST = 128
#         S, B,  T,    t, V,    d,    bf16
SHAPES = [(4, 2, 704, 2, 4000, 100, False), (4, 3, 711, 3, 4000, 101, True), (1, 12, 2600, 3, 4000, 1001, False), (2, 17, 1300, 4, 4000, 131, False),
          (1, 17, 2300, 3, 4000, 1003, True), (3, 5, 900, 3, 4000, 8, True), (1, 30, 2100, 1, 5000, 1536, False), (2, 31, 1000, 1, 4000, 1401, True)]


def lists(T, n):
    a = np.arange(T)
    last, third = a.copy(), a.copy()
    last[[n - 1, T - 1]] = last[[T - 1, n - 1]] if T > n else [T + 1, T + 1]
    third[2] = T + 5
    return {"from 0": a, "last of them elsewhere": last, "third missing": third, "from 3": a + 3, "backwards": a[::-1].copy()}


def _blocks(S, B, t, d, W):
    return S * B * 4 if t > 1 else S * -(-B // min(max(1, 12288 // d), 1024 // W, B))


@pytest.mark.parametrize("S,B,T,t,V,d,bf16", SHAPES)
def test_forced_first_tiles(S, B, T, t, V, d, bf16):
    rng = np.random.default_rng(T + d)
    W, K, u = 8, 4, 4 if t == 1 else 2
    E = rng.standard_normal((V, d)).astype(np.float32)
    if bf16:
        E = (E.view(np.uint32) >> 16).astype(np.uint16)
    perms = np.stack([rng.permutation(d)[:K] for _ in range(u * W)]).astype(np.int32)
    gc = GpuCase(E, perms, np.arange(T, dtype=np.int32), W)
    H = rng.standard_normal((S * B, d)).astype(np.float32) / np.sqrt(d)
    bs = -np.sort(rng.random(S * B)).astype(np.float32)
    n = min(T // 16, MOST, (256 - _blocks(S, B, t, d, W)) // S)
    assert n > 1

    def step(**opts):
        gc.tables.reset_options()
        gc.tables.set_options(fused=1, **opts)
        gb, gw, gs, sp, ws = gc.step(H, bs, S, B, threshold=t)
        cands = [gc.tables.debug_candidates(ws, sp, s) for s in range(S)]
        lps = [gc.tables.debug_logprobs(ws, sp, s, cap=len(cands[s])) for s in range(S)]
        return (gb, gw, gs, *cands, *lps)

    for name, ids in lists(T, 16 * n).items():
        gc.topfreq = ids.astype(np.int32)
        gc.topfreq_dev = to_dev(gc.topfreq)
        want = step(first_tiles=0)
        for opts in (dict(first_tiles=MOST), dict(first_tiles=n - 1), dict(first_tiles=1), dict(first_tiles=MOST, one_launch=1), dict(first_tiles=0)):
            assert all(np.array_equal(x, y) for x, y in zip(want, step(**opts))), (name, opts)
        for s in range(S):
            rows = slice(s * B, (s + 1) * B)
            ref = gc.oracle_sentence(H[rows], bs[rows], B, threshold=t)
            assert np.array_equal(want[3 + s], ref.cand), name
            assert_close_logprobs(want[3 + S + s], ref)
            assert_topb_matches(want[0][s], want[1][s], want[2][s], ref, bs[rows])
    gc.tables.reset_options()


@pytest.mark.parametrize("shuffled", [False, True])
@pytest.mark.parametrize("t,B", [(9, 3), (1, 30)])
def test_nothing_is_made_for_other_lists(t, B, shuffled):
    """A top-frequent list of 400 words, 25 tiles: if it begins otherwise (200 words, each twice), nothing is written behind the end of the
    candidate list, where those tiles would be."""
    import torch
    rng = np.random.default_rng(t)
    V, T, W, K, u = 4000, 400, 8, 4, 4 if t == 1 else 2
    d = 1536 if t == 1 else 64
    e = rng.standard_normal(d).astype(np.float32)
    E = rng.uniform(0.5, 1.5, (V, 1)).astype(np.float32) * e                   # (every word in one bucket, no hidden row there)
    perms = np.stack([rng.permutation(d)[:K] for _ in range(u * W)]).astype(np.int32)
    ids = np.arange(T) if not shuffled else np.arange(T)[::-1] // 2            # (shuffled: 200 words, each twice)
    gc = GpuCase(E, perms, ids.astype(np.int32), W)
    H = (-rng.uniform(0.5, 1.5, (B, 1)).astype(np.float32) * e).astype(np.float32)
    bs = -np.sort(rng.random(B)).astype(np.float32)
    gc.tables.set_options(fused=1, first_tiles=MOST)
    gc.step(H, bs, 1, B, threshold=t)
    (ws,) = gc._ws.values()
    ws.fill_(0xA5)
    torch.cuda.synchronize()
    _, _, _, sp, ws = gc.step(H, bs, 1, B, threshold=t)
    C = len(gc.tables.debug_candidates(ws, sp, 0))
    assert C == len(set(ids))
    up = lambda x: (x + 255) // 256 * 256
    at, pitch = up(V * 4) + up(4), (V + 63) // 64 * 64
    raw = ws.cpu().numpy()[at:at + B * pitch * 4].view(np.uint32).reshape(B, pitch)
    assert np.all(raw[:, C:] == 0xA5A5A5A5) and not np.any(raw[:, :C] == 0xA5A5A5A5)
    gc.tables.reset_options()


def test_first_tiles_in_a_replayed_graph():
    import torch
    from paper_1806_00588_amd import binding
    rng = np.random.default_rng(3)
    V, d, S, B, T, t, W, K = 4000, 200, 2, 5, 900, 3, 8, 4
    E = rng.standard_normal((V, d)).astype(np.float32)
    perms = np.stack([rng.permutation(d)[:K] for _ in range(2 * W)]).astype(np.int32)
    gc = GpuCase(E, perms, np.arange(T, dtype=np.int32), W)
    gc.tables.set_options(fused=1, first_tiles=MOST)
    sp = binding.step_params(S, B, T, t, False)
    ws = torch.empty(binding.step_workspace_bytes(gc.tables, sp), dtype=torch.uint8, device="cuda")
    H, bs = torch.zeros(S * B, d, device="cuda"), -torch.rand(S * B, device="cuda").sort().values
    out = [torch.empty(S, B, dtype=x, device="cuda") for x in (torch.int32, torch.int32, torch.float32)]
    tf = gc.topfreq_dev.clone()
    go = lambda: binding.decode_step(gc.tables, H, bs, tf, sp, ws, *out)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        go()
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        go()
    for i in range(6):                                                         # (the top-frequent list changes between replays too)
        H.copy_(torch.from_numpy(rng.standard_normal((S * B, d)).astype(np.float32) / np.sqrt(d)))
        tf.copy_(gc.topfreq_dev.flip(0) if i % 3 == 1 else gc.topfreq_dev + (i % 3 == 2) * 7)
        graph.replay()
        torch.cuda.synchronize()
        got = [x.clone() for x in out]
        gc.tables.set_options(fused=1, first_tiles=0)
        go()
        torch.cuda.synchronize()
        assert all(torch.equal(x, y) for x, y in zip(got, out)), i
        gc.tables.set_options(fused=1, first_tiles=MOST)
    gc.tables.reset_options()
