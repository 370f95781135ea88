"""How many first tiles are made beside the hashing, on the CPU: the GPU tests' shapes reach what they are for; calls whose lists are too short for
them take none, many beams hashed in parts among them; never more than there are words, idle CUs and ids that a workgroup looks at."""
import math
import os
import random
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def tiles(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("rule") / "host_first_tiles")
    subprocess.check_call([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), "--offload-arch=gfx950", "-std=c++17", "-O1", "-w", "-o", exe,
                           os.path.join(ROOT, "tests", "host_first_tiles.hip")])

    def run(calls):
        """calls: (S, B, T, V, blocks, words, wanted)"""
        out = subprocess.run([exe], input="".join("%d %d %d %d %d %.17g %d\n" % c for c in calls), capture_output=True, text=True, check=True)
        return [int(x) for x in out.stdout.split()]
    return run


def _call(S, B, T, t, V, W, K, u, blocks=None, wanted=-1):
    m = W * K ** -u
    below = sum(math.exp(-m) * m ** i / math.factorial(i) for i in range(t))
    return S, B, T, V, S * B * 4 if blocks is None else blocks, V - (V - min(T, V)) * below ** B, wanted


def test_shapes_of_the_gpu_tests(tiles):
    import test_gpu_first_tiles_only as only
    calls = [_call(S, B, T, t, V, 8, 4, 4 if t == 1 else 2, None if t > 1 else S * 4) for S, B, T, t, V, _, _ in only.SHAPES]
    assert tiles(calls) == [s[2] // 16 for s in only.SHAPES]


def test_calls_that_take_them_and_calls_that_do_not(tiles):
    calls = {"500 bands": (_call(1, 12, 1000, 5, 40000, 500, 8, 3), 62),
             "few words, long lists": (_call(4, 2, 1132, 4, 3637, 174, 8, 3), 56),
             "lists of a third of a tile": (_call(4, 7, 211, 5, 9750, 259, 8, 3), 0),
             "few of a long list's tiles": (_call(1, 12, 500, 3, 60000, 500, 8, 3), 0),
             # 0.9 of a tile for each workgroup: 5 us lost with them
             "30 beams hashed in parts": (_call(1, 30, 1000, 1, 40000, 8, 8, 4, 4), 0),
             "30 beams, longer lists": (_call(1, 30, 1000, 1, 60000, 8, 8, 4, 4), 62),
             "16 bands, 12 beams in parts": (_call(1, 12, 1000, 1, 40000, 16, 8, 3, 2), 62)}
    assert dict(zip(calls, tiles([c for c, _ in calls.values()]))) == {k: n for k, (_, n) in calls.items()}


def test_limits(tiles):
    rng = random.Random(5)
    calls = [(S, rng.randint(1, 32), rng.randint(0, 4000), rng.randint(1, 5000), rng.randint(1, 400), rng.uniform(0, 1e5), rng.choice([-1, 0, 1, 30, 1000]))
             for S in (1, 2, 3, 4, 5, 7, 8, 64) for _ in range(400)]
    for c, n in zip(calls, tiles(calls)):
        S, B, T, V, blocks, words, wanted = c
        most = min(T // 16, V // 16, 128, max(0, 256 - blocks) // S)
        assert 0 <= n <= most and (wanted < 0 or n == min(wanted, most)), c
