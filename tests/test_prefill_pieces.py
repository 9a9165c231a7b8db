"""Key-tile lists that the packed prefill cuts into pieces (host only: the schedule builder, compiled with g++): every list whole or in pieces that
follow one another, with what a workgroup has to know of its piece; and which launches get pieces."""
import os
import shutil
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2602_06072_amd", "csrc")


@pytest.fixture(scope="module")
def tables_of(tmp_path_factory):
    """(q_lens, contexts, (Hq, Hkv, d)) -> (row shift, row shift of the pieces, bytes of partial results, tiles, pieces, merges, list of the pieces)"""
    if shutil.which("g++") is None:
        pytest.skip("needs g++")
    exe = str(tmp_path_factory.mktemp("prefill_pieces") / "driver")
    srcs = [os.path.join(CSRC, f) for f in ("planner.cpp", "schedule.cpp", "trie.cpp", "api.cpp")]
    srcs.append(os.path.join(ROOT, "tests", "native", "prefill_pieces_driver.cpp"))
    build = subprocess.run(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", *srcs, "-L/opt/rocm/lib", "-lamdhip64",
                            "-Wl,-rpath,/opt/rocm/lib", "-o", exe], capture_output=True, text=True)
    assert build.returncode == 0, build.stderr[-3000:]

    def run(ql, ctx, heads):
        ql = np.asarray(ql, dtype=np.int64)
        line = " ".join(str(x) for x in (*heads, len(ql), *ql, *(ql + np.asarray(ctx))))
        out = subprocess.run([exe], input=line + "\n", capture_output=True, text=True, timeout=60)
        assert out.returncode == 0, out
        head, *tables = out.stdout.split("|")
        words = [np.asarray(x.split(), dtype=np.int64) for x in tables]
        return (*(int(x) for x in head.split()), words[0].reshape(-1, 16), words[1].reshape(-1, 16), words[2].reshape(-1, 4), words[3].reshape(-1, 2))
    return run


def byte(word, w):
    return int(word) >> (8 * w) & 0xFF


HEADS = [(8, 8, 128), (4, 1, 128), (32, 8, 64), (12, 2, 128), (5, 1, 64), (6, 2, 128), (16, 2, 128)]


@pytest.mark.parametrize("heads", HEADS)
def test_pieces_follow_one_another(tables_of, heads):
    """Against the definition: rows t .. of a request see the keys up to their own; 64 keys to a key tile, 32 rows to a wave."""
    Hq, Hkv, d = heads
    rng = np.random.default_rng(Hq)
    cut = 0
    for _ in range(25):
        n = int(rng.integers(1, 12))
        ql = rng.integers(1, int(rng.choice([10, 140, 700])), size=n)
        ctx = rng.integers(0, int(rng.choice([500, 3000, 20000])), size=n)
        shift, piece_shift, part_bytes, tiles, pieces, merges, entries = tables_of(ql, ctx, heads)
        if len(merges) == 0:
            assert len(pieces) == 0 and part_bytes == 0
            continue
        cut += 1
        rows, mates = 32 << piece_shift, 4 >> piece_shift
        assert piece_shift == {1: 2, 2: 1, 3: 2, 4: 0, 5: 2, 6: 1, 8: 0}[Hq // Hkv]
        q0, k0 = np.concatenate([[0], np.cumsum(ql)]), np.concatenate([[0], np.cumsum(ql + ctx)])
        want = {int(q0[i]) + t: (i, t) for i in range(n) for t in range(0, int(ql[i]), rows)}
        slots = []
        for row, (i, t) in want.items():
            mine = [p for p in pieces if p[5] == row]
            n_rows = min(rows, int(ql[i]) - t)
            sees = int(ctx[i]) + t + n_rows
            n_kv = (sees + 63) // 64
            mine.sort(key=lambda p: p[8])
            end = 0
            for p in mine:
                assert p[4] == n_rows | 1 << 16 and p[6] == k0[i] and p[7] == k0[i] + ctx[i] + t + 1 and p[1] > 0
                for e in range(p[1]):
                    at = end + e
                    first, info = entries[p[0] + e]
                    keys = min(info & 0xFF, p[14] - first)           # (a shared list goes on to the request's last key)
                    assert first == k0[i] + 64 * at and keys == min(64, sees - 64 * at)
                    if e < 3:
                        assert (p[8 + e], p[11 + e]) == (first, info)
                for e in range(p[1], 3):
                    assert (p[8 + e], p[11 + e]) == tuple(entries[p[0] + p[1] - 1])
                for w in range(4 if piece_shift == 2 else rows // 32):
                    last = min(n_rows, 32 * (w + 1))
                    own = (int(ctx[i]) + t + last + 63) // 64 if 32 * w < n_rows else 0
                    begin, stop = min(byte(p[2], w), p[1]), p[1] - byte(p[3], w)
                    assert stop >= max(0, min(p[1], own - end))      # all that a wave sees; what it does not see may be left to its mask
                    if own > 0:
                        assert begin == 0 and (stop == max(0, min(p[1], own - end)) or n_kv - own >= 255)
                end += p[1]
            assert end == n_kv
            mine_slots = [int(p[15]) - 1 for p in mine]
            if len(mine) == 1:
                assert mine_slots == [-1]
                continue
            assert mine_slots == list(range(mine_slots[0], mine_slots[0] + len(mine)))
            assert [list(m) for m in merges if m[2] == row] == [[mine_slots[0], len(mine), row, n_rows]]
            slots += mine_slots
        assert len(pieces) == sum(1 for p in pieces if int(p[5]) in want)
        assert sorted(slots) == list(range(len(slots))) and len(merges) == len({m[2] for m in merges})
        # a record of 32 rows of a head: the accumulators and 16 bytes a lane
        assert part_bytes == len(slots) * Hkv * (Hq // Hkv // mates) * 4 * 64 * (2 * d + 16)
    assert cut >= 5


# a handful of rows or a chunk behind a long context, few heads; and launches that fill the chip or have no list worth a second launch
@pytest.mark.parametrize("ql, ctx, heads, cut", [
    ([64], 8000, (8, 8, 128), True), ([16], 2000, (32, 8, 128), True), ([128], 8192, (32, 8, 128), True), ([4096], 0, (4, 1, 128), True), ([64], 8000, (8, 8, 64), True),
    ([30] * 20 + [5], [0] * 20 + [9000], (32, 8, 128), True),
    ([1024], 8192, (32, 8, 128), False), ([512] * 8, 0, (8, 8, 64), False), ([400], 400, (8, 8, 128), False), ([1000], 0, (32, 8, 128), False), ([200] * 64, 0, (32, 8, 128), False),
    ([1] * 4, 8000, (8, 8, 128), False)])          # (a decode plan)
def test_which_launches_get_pieces(tables_of, ql, ctx, heads, cut):
    assert (len(tables_of(ql, ctx, heads)[5]) > 0) == cut
