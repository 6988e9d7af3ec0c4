"""What a call launches, seen without a GPU: the library runs on a runtime that only prints its launches (fake_hip.c), in a process
of its own."""
from __future__ import annotations

import json
import os
import re
import subprocess
import sys

import pytest

from paper_2412_21124_amd import binding as B

HERE = os.path.dirname(os.path.abspath(__file__))
STATS, ADAMW, GBAR, COORD = B.NT_DO_STATS, B.NT_DO_ADAMW, B.NT_WRITE_GBAR, B.NT_COORD_TEST
FULL = STATS | ADAMW

# calls from stdin, one JSON list per line; fabricated pointers, as nothing is ever dereferenced
CLIENT = """
import ctypes, json, struct, sys
fake = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
lib = ctypes.CDLL(sys.argv[2])
vp, i64 = ctypes.c_void_p, ctypes.c_int64
for line in sys.stdin:
    c = json.loads(line)
    fake.fake_set(c["device"], c["capture"])
    hyper = struct.pack("6d4qiI", 1e-3, 0.9, 0.95, 1e-8, 0.1, 0.1, 1, 64, 0, 1, 1, c["flags"])
    shard = struct.pack("2i2q", 0, 1, 0, c["whole"]) if c["whole"] else None
    J, d, g = c["J"], c["d"], c["gdtype"]
    tail = (vp(0x2000), vp(0x3000), vp(0x4000), vp(0x5000), hyper, shard, vp(0x6000), ctypes.c_size_t(1 << 40), vp(0x7000),
            vp(c["stream"]))
    if c["table"]:
        rc = lib.normtest_step_rows(vp(0x1000), g, i64(J), i64(d), *tail)
    else:
        rc = lib.normtest_step(vp(0x1000), g, i64(J), i64(d), i64(d), *tail)
    print("rc", rc, flush=True)
"""


def _call(J, gdtype, d, flags, whole=0, table=False, device=0, stream=0, capture=0):
    return dict(J=J, gdtype=gdtype, d=d, flags=flags, whole=whole, table=table, device=device, stream=stream, capture=capture)


@pytest.fixture(scope="module")
def launches(tmp_path_factory):
    """Function from a list of calls to the launches of each: (kernel, template arguments, blocks, threads, dynamic LDS);
    `counters` then holds for each call where the blocks of its k_step_end count themselves, None without one."""
    fake = str(tmp_path_factory.mktemp("fake") / "libfakehip.so")
    subprocess.run(["gcc", "-std=gnu99", "-Wall", "-Wextra", "-Werror", "-shared", "-fPIC", os.path.join(HERE, "fake_hip.c"), "-o", fake],
                   check=True)

    def run(calls):
        out = subprocess.run([sys.executable, "-c", CLIENT, fake, B.lib()._name], check=True, capture_output=True, text=True,
                             input="".join(json.dumps(c) + "\n" for c in calls)).stdout
        got, now, run.counters, counter = [], [], [], []
        for line in out.splitlines():
            if line.startswith("rc "):
                assert line == "rc 0"
                got.append(now)
                run.counters.append(int(counter[0], 16) if counter else None)
                now = []
            else:
                name, grid, block, lds, *counter = line.split()
                now.append((re.search(r"\d(k_[a-z_0-9]*[a-z])", name).group(1), re.findall(r"L[ib](\d+)E", name), int(grid), int(block),
                            int(lds)))
        assert len(got) == len(calls) and not now
        return got

    return run


def _names(step):
    return [k[0] for k in step]


# A step of a few tiles counts its blocks in memory of the library, which is a device's own.  On a stream of another device than
# the current one, and in a graph, it takes the reduction kernel instead.
def test_counters_are_those_of_the_streams_device(launches):
    call = dict(J=4, gdtype=B.NT_F32, d=100_000, flags=FULL)
    got = launches([_call(**call), _call(**call, stream=1), _call(**call, stream=3 << 16, device=3), _call(**call, stream=1 << 16),
                    _call(**call, stream=2 << 16, device=1), _call(**call, capture=1)])
    assert [_names(s) for s in got] == [["k_step_end"]] * 3 + [["k_step", "k_finalize"]] * 3


# One tile, up to 16 rows in the classes of short vectors and beyond 16 rows wherever short tiles are walked, also as a part of a longer vector
@pytest.mark.parametrize("gdtype", [B.NT_BF16, B.NT_F32])
@pytest.mark.parametrize("flags", [FULL, STATS, STATS | GBAR, FULL | COORD])
def test_one_tile_is_one_launch(launches, gdtype, flags):
    calls = [_call(J, gdtype, d, flags, whole) for J in (2, 8, 16) for d in (1, 4096) for whole in (0, 1 << 20)]
    calls += [_call(J, gdtype, d, flags, whole) for J in (17, 24, 33, 512) for d in (1, 2048) for whole in (0, 1 << 20, 1 << 22)]
    if flags == STATS:   # short tiles at any length
        calls += [_call(J, gdtype, 2048, flags, 1 << 30) for J in (17, 33, 512)]
    assert [_names(s) for s in launches(calls)] == [["k_step_end"]] * len(calls)


# Beyond 16 rows steps that write per coordinate run in generations of blocks of 8192 coordinates, or in short tiles where too much of
# the last generation would be empty: the last length on either side of every edge, in 32nds of a generation.
G = 1 << 23
EDGES = [(J, g, f, 64, 0) for J in (17, 20) for g in (B.NT_BF16, B.NT_F32) for f in (FULL, STATS | GBAR, ADAMW)]
EDGES += [(J, B.NT_F32, f, 64, 0) for J in (21, 32) for f in (FULL, STATS | GBAR, ADAMW)]
EDGES += [(J, B.NT_BF16, f, 64, 8) for J in (21, 32) for f in (FULL, STATS | GBAR, ADAMW)]
EDGES += [(33, B.NT_BF16, FULL, 26, 12, 4), (47, B.NT_BF16, FULL, 26, 12, 4), (48, B.NT_BF16, FULL, 24, 12, 4), (33, B.NT_F32, FULL, 24, 4, 0),
          (33, B.NT_BF16, STATS | GBAR, 26, 12, 4), (100, B.NT_BF16, STATS | GBAR, 26, 12, 4), (33, B.NT_F32, STATS | GBAR, 26, 8, 0),
          (33, B.NT_BF16, ADAMW, 26, 12, 4), (63, B.NT_BF16, ADAMW, 26, 12, 4), (64, B.NT_BF16, ADAMW, 26, 10, 2), (33, B.NT_F32, ADAMW, 24, 2, 0)]


@pytest.mark.parametrize("J,gdtype,flags,first,after", [(*e[:4], e[4:]) for e in EDGES])
def test_generations_of_blocks(launches, J, gdtype, flags, first, after):
    start = first * G // 32
    full = -(-start // G)
    lengths, want = [start - 1, start, full * G], [False, True, True]
    for k, left in enumerate(after):
        lengths += [(full + k) * G + 1, (full + k) * G + left * G // 32, (full + k) * G + left * G // 32 + 1, (full + k + 1) * G]
        want += [left == 0, True if left == 0 else False, True, True]
    lengths += [3 * G + 1, 4 * G + 1]
    want += [True, True]
    got = launches([_call(J, gdtype, d, flags) for d in lengths])
    for d, long_class, step in zip(lengths, want, got):
        shape = ("256", "8") if J <= 20 else ("128", "16")
        assert all(tuple(k[1][2:4]) == (shape if long_class else ("256", "2")) for k in step if k[0].startswith("k_step")), d
        if long_class:   # launches of whole generations: 256 CUs x 4 blocks
            assert [k[2] for k in step if k[0].startswith("k_step")].count(1024) == d // G


# Beyond 16 rows the shortest vectors run in tiles of 1024 coordinates: bf16 rows shared by two or four waves, fp32 rows in blocks of 256
# threads; both sides of the length, which is the whole vector's.
@pytest.mark.parametrize("flags", [FULL, STATS, STATS | GBAR, ADAMW])
def test_tiles_of_the_shortest_vectors(launches, flags):
    edge = 1 << 18
    cases = [(17, B.NT_BF16, (1002, 512)), (32, B.NT_BF16, (1002, 512)), (33, B.NT_BF16, (1004, 1024)), (600, B.NT_BF16, (1004, 1024)),
             (17, B.NT_F32, (0, 256)), (600, B.NT_F32, (0, 256))]
    for J, g, (j_t, block) in cases:
        short, ends, past, part = launches([_call(J, g, 2049, flags), _call(J, g, edge, flags), _call(J, g, edge + 1, flags),
                                            _call(J, g, 1025, flags, edge + 1)])
        for step, grid in ((short, 3), (ends, 256)):
            assert [(k[0], int(k[1][0]), int(k[1][2]), k[2], k[3]) for k in step] == [("k_step_end", j_t, block, grid, block)]
        assert [(k[0], k[1][2:4], k[2]) for k in part] == [("k_step_end", ["512", "1"], 1)]
        assert _names(past) == (["k_step_end"] if flags == ADAMW else ["k_step", "k_finalize"])
        assert (past[0][1][2:4], past[0][2]) == (["512", "1"], 129)


# ... but few rows of a vector that fits one tile of 2048 coordinates, where there are sums: both sides of each count of rows and length
@pytest.mark.parametrize("flags", [FULL, STATS, STATS | GBAR, ADAMW])
def test_one_tile_of_the_shortest_vectors(launches, flags):
    calls = [_call(J, g, d, flags) for g, few, half in ((B.NT_BF16, 56, 24), (B.NT_F32, 40, 16)) for J in (17, half, half + 1, few, few + 1)
             if J > 16 for d in (1, 1024, 1025, 2048, 2049)]
    calls.append(_call(17, B.NT_BF16, 2000, flags, 2049))
    for c, step in zip(calls, launches(calls)):
        few, half = (56, 24) if c["gdtype"] == B.NT_BF16 else (40, 0)
        one = flags != ADAMW and c["d"] <= 2048 and not c["whole"] and c["J"] <= (few if c["d"] > 1024 else half)
        (name, args, grid, _, _), = step
        assert name == "k_step_end" and grid == (1 if one else -(-c["d"] // 1024)), c
        assert (args[0] == "0" and args[2:4] == ["512", "1"]) == one, c


# The blocks of a step that ends in one launch count themselves in words that no other stream has, as a launch may wait on its stream
# for as long as it likes.  A stream that finds no place among them takes the reduction kernel.
def test_counters_are_a_streams_own(launches):
    base, places = 0x10000000, 4096   # see fake_hip.c; streams that have words
    few = [(s << 16, s) for s in (0, 3, 0, 3)] + [(s, 0) for s in (1, 2, 5, 0, 6, 5, 2, 1, 6)]   # (stream, device)
    many = [(s, 0) for s in range(17, 6017)]
    asked = few + many + many[:50]
    steps = launches([_call(4, B.NT_F32, 100_000, FULL, stream=s, device=dev) for s, dev in asked])
    words = dict(zip(asked, launches.counters))
    for who, word, step in zip(asked, launches.counters, steps):
        assert word == words[who] and _names(step) == (["k_step_end"] if word else ["k_step", "k_finalize"])
        assert word or who in many
    own = [w for w in words.values() if w]
    assert len(own) == len(set(own)) > places // 2
    assert all(base <= w < base + 4 * places and w % 4 == 0 for w in own)


# Dynamic LDS that keeps one block of 1024 threads on a CU (160 KB), or two or three of 512 of the statistics that store the mean.
def test_blocks_held_per_cu(launches):
    cases = [((8, B.NT_BF16, 1 << 25, FULL), 0), ((8, B.NT_BF16, (1 << 25) + 1, FULL), 1), ((4, B.NT_BF16, 1 << 28, FULL), 0),
             ((3, B.NT_F32, 1 << 24, FULL), 0), ((3, B.NT_F32, (1 << 24) + 1, FULL), 1), ((8, B.NT_BF16, 1 << 23, ADAMW), 0),
             ((8, B.NT_BF16, (1 << 23) + 1, ADAMW), 1), ((8, B.NT_BF16, 1 << 28, ADAMW), 0), ((7, B.NT_BF16, 1 << 24, ADAMW), 0)]
    cases += [((J, g, d, STATS | GBAR), held if d > 1 << 25 else 0) for d in (1 << 25, (1 << 25) + 1)
              for J, g, held in ((4, B.NT_BF16, 0), (5, B.NT_BF16, 3), (6, B.NT_BF16, 2), (9, B.NT_BF16, 2), (2, B.NT_F32, 0), (3, B.NT_F32, 2))]
    cases += [((9, B.NT_BF16, 1 << 26, STATS), 0), ((20, B.NT_BF16, 1 << 26, STATS | GBAR), 0)]
    for (call, held), step in zip(cases, launches([_call(*c) for c, _ in cases])):
        for k in step:
            if k[0].startswith("k_step"):
                assert (163840 // k[4] if k[4] else 0) == held, (call, k)


# The record, the partials of all tiles and those of all groups fit in the bytes that a step of these rows asks for, at both sides of
# every number of tiles where the groups change; and the built-in scratch holds as much as it did when groups had one size.
def test_partials_fit_in_the_workspace(launches):
    calls = [_call(J, g, n * tile + more, flags) for J, tile, flags in ((8, 4096, FULL), (4, 4096, STATS | GBAR), (2, 8192, STATS),
                                                                       (24, 2048, FULL), (40, 2048, STATS), (40, 8192, STATS | GBAR))
             for g in (B.NT_BF16, B.NT_F32) for n in (2560, 4096, 1 << 16, (1 << 17) - 1, 1 << 17, 1 << 18) for more in (0, 1)]
    groups = set()
    for c, step in zip(calls, launches(calls)):
        tiles = sum(k[2] for k in step if k[0].startswith("k_step"))
        n = sum(k[2] for k in step if k[0] == "k_reduce_end")
        assert 256 + 40 * tiles + 80 * n <= B.normtest_workspace_bytes(c["J"], c["d"]), c
        groups.add(n)
    assert {0, 6, 32, 33, 64, 65, 128} <= groups
    for J in (2, 16, 17, 512):
        assert B.normtest_static_max_coords(J) == (1_716_281_344 if J <= 16 else 858_140_672)
        d = [k * (1 << 26) // 3 for k in range(1, 100)]
        sizes = [B.normtest_workspace_bytes(J, x) for x in sorted(d + [(1 << 16) * 2048, (1 << 16) * 2048 + 1, (1 << 16) * 4096, (1 << 16) * 4096 + 1])]
        assert sizes == sorted(sizes)
