"""The split of the attention kernel's work, compiled for the host: every tile of
every (sequence, head group) pair falls to exactly one workgroup, the parts of a
pair are numbered in order and stored in slots of their own below the
allocation, and no more workgroups have work than the grid holds.  Over random
ragged batches with empty lists on both sides of 64 sequences, every number of
KV heads together, and the batches of the GPU tests, whose form (aligned parts
or straddled ranges) and heads together are pinned here."""
import ctypes
import os
import random
import subprocess

import numpy as np
import pytest

from paper_2512_11221_amd import build

HERE = os.path.dirname(os.path.abspath(__file__))
GRID = 256                              # workgroups resident on the device, one per CU


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("split") / "split_check.so")
    subprocess.run([build.hipcc(), "-x", "hip", "--offload-host-only", "-O1", "-std=c++17", "-fPIC", "-shared",
                    os.path.join(HERE, "split", "split_check.cpp"), "-o", out], check=True,
                   stdout=subprocess.PIPE, stderr=subprocess.STDOUT)
    return ctypes.CDLL(out)


def _ints(x):
    return (ctypes.c_int32 * max(1, len(x)))(*x)


def _heads(lib, plen, hkv, row_bytes, t=1):
    launch = ctypes.c_int()
    hw = lib.split_layout(_ints(plen), len(plen), t, hkv, row_bytes, GRID, ctypes.byref(launch))
    assert 1 <= launch.value <= GRID
    return hw, launch.value


def _pieces(lib, n_active, hkv, hw, tile, grid=GRID):
    groups = hkv // hw
    cap = len(n_active) * groups + 2 * grid + 8
    out, info = (ctypes.c_int32 * (9 * cap))(), (ctypes.c_int32 * 4)()
    k = lib.split_pieces(_ints(n_active), len(n_active), hkv, hw, grid, tile, out, cap, info)
    assert k <= cap
    return np.array(out[:9 * k], dtype=np.int64).reshape(k, 9), list(info)


def _check(lib, n_active, hkv, hw, tile, grid=GRID):
    p, (live, aligned, groups, _) = _pieces(lib, n_active, hkv, hw, tile, grid)
    assert 0 <= live <= grid
    seen = {}
    for w, b, n, g, t0, t1, parts, part, slot in p.tolist():
        assert 0 <= w < live and n == n_active[b] and 0 <= g < groups and 0 <= t0 < t1 <= -(-n // tile)
        seen.setdefault((b, g), []).append((t0, t1, parts, part, slot, w))
    assert set(seen) == {(b, g) for b, n in enumerate(n_active) if n for g in range(groups)}
    for (b, g), rows in seen.items():
        rows.sort()
        assert rows[0][0] == 0 and rows[-1][1] == -(-n_active[b] // tile)
        for (x, y) in zip(rows, rows[1:]):
            assert x[1] == y[0]                                    # no gap, no overlap
        for i, (_, _, parts, part, slot, _) in enumerate(rows):
            assert parts == len(rows) and part == i
            assert slot - part == rows[0][4]                       # consecutive slots: first + part
    slots = p[:, 8][p[:, 6] > 1]                                   # of the pairs with partials
    assert len(np.unique(slots)) == len(slots)
    # a slot holds the heads of a group; the allocation, in groups: workgroups + pairs
    assert len(slots) == 0 or (slots.min() >= 0 and slots.max() < grid + len(n_active) * groups)
    return aligned, live, p


def test_random_batches(lib):
    rng = random.Random(5)
    forms = set()
    for _ in range(1500):
        batch = rng.choice([1, 2, 3, 5, 8, 17, 63, 64, 65, 66, 130, 257, 1024])
        hkv = rng.choice([1, 2, 4, 8, 16, 32])
        hw = rng.choice([h for h in (1, 2, 4, 8) if h <= hkv])
        top = int(2 ** rng.uniform(0, 15 if batch < 64 else 11))
        n = [0 if rng.random() < 0.2 else rng.randint(1, top) for _ in range(batch)]
        aligned, live, _ = _check(lib, n, hkv, hw, rng.choice([16, 32, 64]), rng.choice([256, 256, 304, 7]))
        forms.add((bool(aligned), live > 0))
    assert forms >= {(True, True), (False, True)}


@pytest.mark.parametrize("batch", [1, 64, 65])
def test_nothing_to_do(lib, batch):
    _, live, p = _check(lib, [0] * batch, 8, 1, 32)
    assert live == 0 and len(p) == 0


def test_launch_covers_the_workgroups_with_work(lib):
    """Lists up to plen + t long, shorter ones after freezing: the launched
    workgroups are at least those with work (further ranges would be walked in
    turn by the same workgroups)."""
    rng = random.Random(9)
    for _ in range(600):
        batch = rng.choice([1, 2, 8, 33, 64, 100])
        hkv, row = rng.choice([(1, 128), (2, 256), (8, 256), (8, 512), (32, 256), (32, 128)])
        t = rng.randint(1, 40)
        plen = [rng.randint(0, int(2 ** rng.uniform(0, 13))) for _ in range(batch)]
        hw, launch = _heads(lib, plen, hkv, row, t)
        full = [p + t for p in plen]
        for n in (full, [max(1, int(x * rng.uniform(0.2, 1))) for x in full]):
            _, live, _ = _check(lib, n, hkv, hw, lib.split_tile(row))
            assert live <= launch


# the batches of the GPU tests: (list lengths at the first step, KV heads, row bytes) ->
# heads together and whether the parts are aligned
B128 = [901 if b == 3 else (1 if b % 7 == 2 else 6 + 13 * b % 90) for b in range(130)]
SHARED = lambda batch: [2 + (97 * b * b + 31 * b) % 700 for b in range(batch)]
GPU_CASES = {
    "plan-ragged": ([1, 2901, 3101, 41, 4201], 8, 256, 1, False),
    "plan-hh": ([3001, 2601, 3401], 8, 256, 1, True),
    "plan-g8": ([2901, 3301, 2501], 4, 256, 1, True),
    "plan-rows-512": ([3101, 2801, 3301], 8, 512, 1, True),
    "plan-rows-128": ([3101, 2801, 3301], 8, 128, 1, True),
    "tiles-b64": (B128[:64], 8, 128, 2, False),
    "tiles-b65": (B128[:65], 8, 128, 4, False),
    "tiles-b130": (B128, 8, 128, 8, False),
    "tiles-room": ([66201], 8, 128, 1, True),
    "room-b66": ([8701] * 66, 8, 128, 8, False),
    "room-b8": ([72001] * 8, 8, 128, 8, True),
    "poisoned": ([577], 8, 256, 1, True),
    "poisoned-b66": ([65] * 66, 8, 256, 4, True),
    "shared-64-b16": (SHARED(16), 32, 128, 2, True),
    "shared-64-b32": (SHARED(32), 32, 128, 4, False),
    "shared-64-b70": (SHARED(70), 32, 128, 8, False),
    "shared-128-b40": (SHARED(40), 8, 256, 2, False),
    "shared-128-b300": (SHARED(300), 8, 256, 8, False),
}


@pytest.mark.parametrize("name", sorted(GPU_CASES))
def test_forms_of_the_gpu_cases(lib, name):
    n, hkv, row, want_hw, want_aligned = GPU_CASES[name]
    hw, _ = _heads(lib, [x - 1 for x in n], hkv, row)
    aligned, _, _ = _check(lib, n, hkv, hw, lib.split_tile(row))
    assert (hw, bool(aligned)) == (want_hw, want_aligned)


def test_the_benchmarks_copy_of_the_rule(lib):
    """bench.py states the relevance and list bytes from its own copy of the rule."""
    import bench
    rng = random.Random(11)
    for _ in range(500):
        hkv, row = rng.choice([(1, 128), (2, 256), (8, 256), (8, 512), (32, 256), (32, 128)])
        plen = [rng.randint(0, int(2 ** rng.uniform(0, 16))) for _ in range(rng.choice([1, 2, 8, 33, 64, 100, 500]))]
        assert bench.heads_together(plen, hkv, row, GRID) == _heads(lib, plen, hkv, row)[0]
