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


def _logits(gc, H, S, B):
    """The step's logits, from its workspace (behind the candidate counts; rows are pitched to 64 words)."""
    import torch
    ws = gc.step(H, np.zeros(S * B, np.float32), S, B, full_vocab=True)[4]
    at, pitch = (4 * S + 255) // 256 * 256, (gc.V + 63) // 64 * 64
    return ws[at:at + 4 * S * B * pitch].view(torch.float32).view(S * B, pitch)[:, :gc.V].double()


@pytest.mark.parametrize("n", [1, 2, 4, 16, 0], ids=lambda n: "%d" % n if n else "all")
@pytest.mark.parametrize("case", [("rows", 9000, 5, 16, False), ("rows", 9000, 5, 16, True), ("few", 9000, 2, 12, False),
                                  ("few", 9000, 2, 12, True), ("pass", 33000, 1, 12, False), ("pass", 78000, 1, 12, True)],
                         ids=lambda c: "%s-%s" % (c[0], "bf16" if c[4] else "fp32"))
def test_logits_are_as_near_as_fp32_sums(case, n):
    """Logits with n products that are not zero (0: all) against fp64, beside a chain of fused multiply-adds in fp32.
    The error, over the sum of the products' sizes, is no larger in the mean square; and of a single product no
    larger than rounding it once: half a unit, 2^-24, and what the smaller planes' own sum loses, 2^-8 of that."""
    import torch
    _, V, S, B, bf16 = case
    d = 600
    rng = np.random.default_rng(V + B + n)
    E = (rng.standard_normal((V, d)) / np.sqrt(d)).astype(np.float32)
    if n:
        keep = np.zeros((V, d), np.float32)
        np.put_along_axis(keep, np.argpartition(rng.random((V, d)), n, axis=1)[:, :n], 1.0, axis=1)
        E *= keep
    H = (4.0 * rng.standard_normal((S * B, d))).astype(np.float32)
    bits = workloads.f32_to_bf16_bits(E)
    if bf16:
        E = (bits.astype(np.uint32) << 16).view(np.float32)
    perms = np.stack([rng.permutation(d)[:4] for _ in range(4)]).astype(np.int32)
    gc = GpuCase(bits if bf16 else E, perms, np.zeros(0, np.int32), 2)
    e, h = torch.from_numpy(E).cuda().double(), torch.from_numpy(H).cuda().double()
    exact, size = h @ e.T, h.abs() @ e.abs().T
    chain = torch.zeros(S * B, V, device="cuda")
    for k in range(d):                   # (a product of two fp32 values is exact in fp64)
        chain = (chain.double() + torch.outer(h[:, k], e[:, k])).float()

    def error(x):
        r = (x.double() - exact) / size
        return r.square().mean().sqrt().item(), r.abs().max().item()
    got, ref = error(_logits(gc, H, S, B)), error(chain)
    assert got[0] <= 1.02 * ref[0], (got, ref)
    if n == 1:
        assert got[1] <= 2.0 ** -24 * (1 + 2.0 ** -7), got


@pytest.mark.parametrize("d", [1028, 1100, 1300, 1536, 1800, 2048])
def test_long_rows_of_few_tiles(d):
    """Vocabularies so small that the streamed tiles take them: logits no further from fp64 than those of the kernel for
    large ones, whose error (root mean square, over the products' sizes) is 0.33 of a chain of fp32 sums'."""
    import torch
    V, S, B = 1000, 8, 12
    rng = np.random.default_rng(d)
    E = (rng.standard_normal((V, d)) / np.sqrt(d)).astype(np.float32)
    H = (4.0 * rng.standard_normal((S * B, d))).astype(np.float32)
    gc = GpuCase(E, np.stack([rng.permutation(d)[:4] for _ in range(4)]).astype(np.int32), np.zeros(0, np.int32), 2)
    e, h = torch.from_numpy(E).cuda().double(), torch.from_numpy(H).cuda().double()
    exact, size = h @ e.T, h.abs() @ e.abs().T
    chain = torch.zeros(S * B, V, device="cuda")
    for k in range(d):
        chain = (chain.double() + torch.outer(h[:, k], e[:, k])).float()
    got, ref = (((x.double() - exact) / size).square().mean().sqrt().item() for x in (_logits(gc, H, S, B), chain))
    assert got <= 0.34 * ref, (got, ref)


@pytest.mark.parametrize("S, B", [(2, 12), (5, 16)])
@pytest.mark.parametrize("bf16", [False, True], ids=["fp32", "bf16"])
def test_without_planes(S, B, bf16):
    """logits_planes = 0: the fp32 instructions, as k_logits_hlds has them, and not the planes' result."""
    import torch
    rng = np.random.default_rng(S)
    E = (rng.standard_normal((9000, 300)) / 17).astype(np.float32)
    H = (4.0 * rng.standard_normal((S * B, 300))).astype(np.float32)
    perms = np.stack([rng.permutation(300)[:4] for _ in range(4)]).astype(np.int32)
    gc = GpuCase(workloads.f32_to_bf16_bits(E) if bf16 else E, perms, np.zeros(0, np.int32), 2)
    planes = _logits(gc, H, S, B)
    gc.tables.set_option("logits_planes", 0)
    without = _logits(gc, H, S, B)
    gc.tables.set_option("logits_hlds", 1)
    assert torch.equal(without, _logits(gc, H, S, B))
    assert not torch.equal(without, planes)
    assert (without - planes).abs().max() < 1e-4
