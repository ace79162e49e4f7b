"""The grouped GEMM's tile schedule, walked on the host: every tile once, the load even."""
import itertools
import os
import random
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def walk(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("schedule") / "tile_schedule")
    subprocess.check_call(["g++", "-std=c++17", "-O2", "-Wall", "-I", os.path.join(ROOT, "paper_2404_05019_amd", "csrc"),
                           os.path.join(ROOT, "tests", "tile_schedule_main.cpp"), "-o", exe])

    def run(calls):
        text = "\n".join(" ".join(map(str, c[:8] + [len(c[8]) - 1] + c[8])) for c in calls)
        out = subprocess.run([exe], input=text, stdout=subprocess.PIPE, text=True, check=True, timeout=300).stdout.splitlines()
        assert len(out) == len(calls)
        return out
    return run


def _offsets(rng, E, most):
    off = [0]
    for _ in range(E):
        off.append(off[-1] + rng.choice([0, 1, 127, 128, 129, 255, 256, 257, rng.randrange(most + 1)]))
    return off


@pytest.mark.parametrize("cat", [0, 1])
def test_every_tile_once(walk, cat):
    rng = random.Random(5)
    calls = []
    for bm, nt, split, slots in itertools.product([128, 256] if cat else [64, 128, 256], [1, 2, 3, 8], [0, 1], [1, 5, 32, 64]):
        for _ in range(6):
            off = _offsets(rng, rng.choice([1, 2, 8, 17, 64]) + cat, rng.choice([40, 600, 3000]))
            if off[-1] == 0:
                off[-1] = 1
            xrows = 0 if cat else rng.choice([0, 1, 700, 4096])
            calls.append([cat, bm, nt, 2 * rng.randrange(8, 70), split, {64: 2, 128: 4, 256: 8}[bm], slots, xrows, off])
        if not cat:                                  # the extra segment alone: the launch that has the gate on the side
            calls.append([0, bm, nt, 2 * rng.randrange(2, 70), 0, bm // 32, slots, rng.choice([1, bm, bm + 1, 3001]), [0]])
    for call, line in zip(calls, walk(calls)):
        assert line.replace(" ", "").isdigit(), (call, line)
        # the XCDs' shares differ by a tile of each of the two ranges at most, and the last round is one tile long
        longest, total = map(int, line.split())
        nk, slots = call[3], call[6]
        assert longest <= total / (8 * slots) + nk * (1 + 2 / slots), (call, line)


def test_short_tiles_fill_the_round_of_the_full_ones(walk):
    """44 row tiles of experts and 28 of tokens without a routed row, four column tiles, 32 workgroups on
    an XCD: 22 full and 14 short tiles each, so nobody does more than one full tile or two short ones."""
    off = [1024 * e for e in range(12)] + [72 * 256]
    longest, total = map(int, walk([[1, 256, 4, 128, 1, 8, 32, 0, off]])[0].split())
    assert (longest, total) == (128, (44 * 128 + 28 * 64) * 4)
