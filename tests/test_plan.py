"""The plan of a fused step launch (tile height, z chunk, store hint), built with the
address and undefined-behaviour sanitizers and driven on the CPU: every chunk length of
the cost model tried by hand gives the same plan, and the longest lattices that the
library accepts are planned without overflow."""
import os
import random
import shutil
import subprocess
import time

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def planner(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("g++ is needed")
    exe = str(tmp_path_factory.mktemp("plan") / "plan")
    r = subprocess.run(["g++", "-O1", "-g", "-std=c++17", "-fsanitize=address,undefined", "-fno-sanitize-recover=all",
                        "-I" + os.path.join(ROOT, "paper_2403_15773_amd", "csrc"),
                        os.path.join(ROOT, "tests", "plan_main.cpp"), "-o", exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]

    def run(cases):
        text = "\n".join(" ".join(str(int(v)) for v in c) for c in cases)
        r = subprocess.run([exe], input=text, capture_output=True, text=True, timeout=100)
        assert r.returncode == 0, r.stderr[-3000:]
        lines = [ln.split() for ln in r.stdout.splitlines()]
        const = [float(v) for v in lines[0]]
        return const, [tuple(int(v) for v in ln) for ln in lines[1:]]

    return run


def _by_hand(c, const):
    """(rows, chunk, work items) of the cheapest plan: every number of chunks tried."""
    nx, ny, nz, phase, wide, half, cus, chunk, rows, _ = c
    cap, wide_cost, half_cost, fill2, fill1 = const

    def best(r):
        tiles = -(-nx // 32) * -(-ny // r)
        f = 1.0 if r == 16 else (half_cost if half else wide_cost)
        found = None
        for k in range(1, nz + 1):
            lz = min(chunk, nz) if chunk else -(-nz // k)
            if not chunk and lz > cap:
                continue
            w = tiles * -(-nz // lz)
            cost = float(-(-w // cus)) * (0.5 * (2 * lz + (fill2 if phase else fill1))) * f
            if found is None or cost <= found[0]:
                found = (cost, lz, w)
            if chunk:
                break
        return found

    b16 = best(16)
    if not wide or rows == 16:
        return 16, b16[1], b16[2]
    b20 = best(20)
    return (20, b20[1], b20[2]) if rows == 20 or b20[0] < b16[0] else (16, b16[1], b16[2])


def test_plan_is_the_cheapest_of_all_chunk_lengths(planner):
    rng = random.Random(7)
    cases = []
    for _ in range(400):
        phase = rng.random() < 0.7
        wide = phase and rng.random() < 0.8
        cases.append((rng.randint(1, 520), rng.randint(1, 520), int(2 ** rng.uniform(0, 11)), phase, wide, rng.random() < 0.4,
                      rng.choice([256, 256, 64, 304, 1]), rng.choice([0, 0, 0, 1, 7, 128, 5000]),
                      rng.choice([0, 0, 16, 20]) if wide else 0, 1 << 30))
    const, got = planner(cases)
    for c, g in zip(cases, got):
        assert g[:3] == _by_hand(c, const), c


@pytest.mark.parametrize("nx,ny,nz", [(1, 1, 1100000000), (1, 1, 2**31 - 1), (4, 1, 2**31 - 1), (33, 1, 260000000),
                                      (1, 2**30 - 1, 7), (2**29, 1, 15)])
def test_longest_lattices_are_planned_without_overflow(planner, nx, ny, nz):
    cases = [(nx, ny, nz, phase, phase, half, 256, chunk, 0, 44 * nx * ny * nz)
             for phase in (0, 1) for half in (0, 1) for chunk in (0, 1, 2**31 - 1)]
    t = time.perf_counter()
    _, got = planner(cases)
    assert time.perf_counter() - t < 10.0
    for c, (rows, lz, items, _, launches) in zip(cases, got):
        assert 1 <= lz <= nz and items == -(-nx // 32) * -(-ny // rows) * -(-nz // lz)
        assert launches == -(-items // 4194303)  # each within 2^32 - 1 threads
        if c[7]:
            assert lz == min(c[7], nz)
        elif nz > 1000000:  # workgroups are plenty: the longest chunks cost least
            assert lz == 128


def test_store_hint(planner):
    mb = 1 << 20
    cases = [(c[0], 64, 64, 1, 1, c[1], 256, 0, 0, c[2]) for c in
             [(61, 0, 13 * mb), (61, 0, 14 * mb), (64, 0, 100 * mb), (64, 0, 128 * mb), (64, 0, 129 * mb), (96, 0, 900 * mb),
              (96, 1, 900 * mb), (128, 1, 900 * mb), (128, 1, 100 * mb), (250, 0, 900 * mb)]]
    _, got = planner(cases)
    assert [g[3] for g in got] == [1, 0, 0, 0, 1, 1, 0, 1, 0, 0]


@pytest.mark.parametrize("half,shape,rows", [
    # two components on 256 compute units: the height that is at least 3.5 % faster in each of the
    # 16-bit types (us a step on 16 and 20 rows, FP16 and FP16Q)
    (1, (103, 97, 514), 20),   # 171 162, 175 164
    (1, (119, 161, 196), 20),  # 116 111, 118 111
    (1, (66, 38, 415), 20),    # 52.1 50.0, 52.6 50.4
    (1, (128, 128, 512), 16),  # 192 214, 198 218
    (1, (237, 41, 113), 16),   # 44.2 56.2, 44.9 56.2
    (1, (398, 396, 510), 16),  # 1859 1987, 1986 2097
    (1, (171, 102, 105), 16),  # 59.6 66.3, 60.3 66.2
    # binary32
    (0, (119, 161, 196), 20),  # 116 111
    (0, (128, 128, 512), 16),  # 185 202
    (0, (398, 396, 510), 16),  # 2134 2250
    (0, (52, 203, 69), 16),    # 30.7 35.7
])
def test_faster_tile_height_is_taken(planner, half, shape, rows):
    _, got = planner([shape + (1, 1, half, 256, 0, 0, 1 << 30)])
    assert got[0][0] == rows
