"""The order in which query tiles of the packed prefill are launched, and the rows that they have (host only: the schedule builder, compiled with g++)."""
import os
import shutil
import subprocess

import numpy as np
import pytest

from paper_2602_06072_amd import workloads as wl

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2602_06072_amd", "csrc")


@pytest.fixture(scope="module")
def tiles_of(tmp_path_factory):
    """(q_lens, contexts, (Hq, Hkv, d)) -> (row shift, [(request, tile of the request, rows, key tiles)] in launch order), of a device with 256 units"""
    if shutil.which("g++") is None:
        pytest.skip("needs g++")
    exe = str(tmp_path_factory.mktemp("launch_order") / "driver")
    srcs = [os.path.join(CSRC, f) for f in ("planner.cpp", "schedule.cpp", "trie.cpp", "api.cpp")]
    srcs.append(os.path.join(ROOT, "tests", "native", "launch_order_driver.cpp"))
    build = subprocess.run(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", *srcs, "-L/opt/rocm/lib", "-lamdhip64",
                            "-Wl,-rpath,/opt/rocm/lib", "-o", exe], capture_output=True, text=True)
    assert build.returncode == 0, build.stderr[-3000:]

    def run(ql, ctx, heads):
        ql = np.asarray(ql, dtype=np.int64)
        line = " ".join(str(x) for x in (*heads, len(ql), *ql, *(ql + np.asarray(ctx))))
        out = subprocess.run([exe], input=line + "\n", capture_output=True, text=True, timeout=60)
        assert out.returncode == 0, out
        head, tiles = out.stdout.split("|")
        starts = np.concatenate([[0], np.cumsum(ql)])
        found = []
        for x in tiles.split():
            row, rows, n_kv = (int(v) for v in x.split(","))
            req = int(np.searchsorted(starts, row, side="right")) - 1
            found.append((req, row - int(starts[req]), rows, n_kv))
        return int(head.split()[0]), found
    return run


def classes(tiles):
    longest = max(t[3] for t in tiles)
    return [int(np.floor(np.log2(longest // t[3]))) for t in tiles]


def is_by_request(tiles):
    """A request's tiles are together (a tile of several requests counts as its first one's)."""
    seen = [t[0] for t in tiles]
    return all(seen[i] == seen[i - 1] or seen[i] not in seen[:i] for i in range(1, len(seen)))


RAGGED = np.random.default_rng(4).integers(140, 480, size=28)


# one query head per KV head, lists of a few key tiles, several rounds of workgroups
@pytest.mark.parametrize("ql, heads", [([512] * 32, (32, 32, 128)), ([200] * 64, (16, 16, 128)), ([380] * 73, (32, 32, 128)), ([205] * 143, (32, 32, 128)),
                                       (RAGGED, (32, 32, 128)), (wl.config2_lengths(0), (32, 32, 128))])
def test_short_lists_of_one_head_stay_by_request(tiles_of, ql, heads):
    shift, tiles = tiles_of(ql, 0, heads)
    assert shift == 2 and is_by_request(tiles)


@pytest.mark.parametrize("ql, heads", [([512] * 16, (16, 16, 128)), ([1000] * 24, (16, 16, 128)), ([2048] * 8, (8, 8, 64)), ([1000] * 3, (16, 16, 128)), ([200] * 64, (16, 16, 64)),
                                       ([512] * 16, (24, 8, 128)), ([512] * 16, (32, 8, 128)), ([200] * 64, (32, 8, 128))])
def test_launches_end_with_short_lists(tiles_of, ql, heads):
    _, tiles = tiles_of(ql, 0, heads)
    h = classes(tiles)
    assert h == sorted(h) and len(set(h)) > 1 and not is_by_request(tiles)


# with a compute unit for every tile of 128 rows and head: tiles of 128 rows where the one with the longest list has a wave without rows, several heads to a workgroup where it is full
@pytest.mark.parametrize("ql, ctx, heads, shift", [([382, 407], 0, (8, 2, 128), 2), ([315, 400, 554, 490], 0, (8, 2, 128), 2), ([440] * 2, 0, (16, 8, 64), 2), ([211] * 6, 1161, (8, 1, 128), 2),
                                                   ([608], 0, (16, 2, 128), 2), ([609], 0, (16, 2, 128), 0), ([1000], 0, (16, 2, 128), 0), ([128] * 2, 4000, (32, 8, 128), 0),
                                                   ([505] * 3, 0, (8, 4, 128), 1), ([461, 852, 403], 0, (16, 2, 128), 2), ([57] * 7, 2500, (32, 8, 128), 2), ([128] + [20] * 12, [1000] + [0] * 12, (16, 8, 128), 2)])
def test_rows_of_a_tile_in_launches_that_leave_units_idle(tiles_of, ql, ctx, heads, shift):
    found, tiles = tiles_of(ql, ctx, heads)
    assert found == shift and (shift < 2 or is_by_request(tiles))            # (all workgroups start at once: nothing to end earlier)
    if np.size(ctx) == 1 and shift == 2:
        assert tiles_of(list(ql) * 24, ctx, heads)[0] == {1: 2, 2: 1}.get(heads[0] // heads[1], 0)          # (more of the same fill the chip)


@pytest.mark.parametrize("heads", [(8, 1, 128), (16, 2, 64), (16, 4, 128), (32, 8, 128), (8, 4, 64), (16, 8, 128), (6, 1, 128)])
def test_tiles_of_several_heads_cover_every_row_once(tiles_of, heads):
    """Every row of every request in one tile of 32 or 64 rows, which sees the keys up to its last row's; sets of four tiles dealt over the XCDs leave none out."""
    rng = np.random.default_rng(heads[0])
    for _ in range(12):
        n = int(rng.integers(1, 60))
        ql, ctx = rng.integers(1, int(rng.choice([40, 300, 2500])), size=n), rng.integers(0, int(rng.choice([1, 100, 5000])), size=n)
        shift, tiles = tiles_of(ql, ctx, heads)
        if shift == 2:
            continue                               # (a launch that leaves units idle)
        want = {(i, t, min(32 << shift, int(ql[i]) - t)) for i in range(n) for t in range(0, int(ql[i]), 32 << shift)}
        assert sorted(t[:3] for t in tiles) == sorted(want)
        assert all(n_kv == (int(ctx[i]) + t + rows + 63) // 64 for i, t, rows, n_kv in tiles)
