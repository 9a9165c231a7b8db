"""Which of the two prefill bodies a batch takes (host only: the tables of a plan say it).  Measured on batches of both kinds;
results do not depend on it.  And what building the tables costs."""
import time

import numpy as np
import pytest

from paper_2602_06072_amd import binding as pk
from paper_2602_06072_amd import workloads as wl


def bound(ql, ctx, Hq, Hkv, d):
    ql = np.asarray(ql, dtype=np.int32)
    plan = pk.pack_plan(ql + np.asarray(ctx, dtype=np.int32), ql, token_budget=16384)
    assert plan.workspace_bytes(Hq, Hkv, d, pk.PK_BF16) > 0
    return plan


# n requests of L rows behind ctx tokens: short key lists on a full chip, launches of little work, few workgroups
@pytest.mark.parametrize("Hq, Hkv, d, n, L, ctx", [
    (64, 8, 128, 8, 128, 0), (32, 8, 128, 64, 200, 0), (64, 8, 128, 256, 130, 0), (32, 8, 128, 32, 512, 0), (32, 8, 128, 16, 1024, 0),
    (64, 8, 64, 64, 200, 0), (64, 8, 64, 512, 300, 0), (32, 8, 64, 21, 768, 0), (32, 8, 64, 14, 128, 2000), (8, 8, 64, 8, 512, 0),
    (32, 8, 128, 1, 512, 8192), (8, 8, 64, 1, 64, 8000)])
def test_launches_of_little_work(Hq, Hkv, d, n, L, ctx):
    assert bound([L] * n, [ctx] * n, Hq, Hkv, d).stat(8) == 1


@pytest.mark.parametrize("Hq, Hkv, d, n, L, ctx", [
    (64, 8, 128, 32, 1024, 8192), (32, 8, 128, 1, 1024, 8192), (32, 8, 128, 16, 2048, 0), (32, 8, 128, 16, 128, 2000),
    (32, 8, 64, 8, 4096, 0), (32, 8, 64, 1, 4096, 8192), (64, 8, 64, 16, 2048, 0)])
def test_launches_of_much_work(Hq, Hkv, d, n, L, ctx):
    assert bound([L] * n, [ctx] * n, Hq, Hkv, d).stat(8) == 0


@pytest.mark.parametrize("d", [64, 128])
def test_idle_tiles_of_the_padded_schedule_do_not_count(d):
    """One long prompt among short ones: the padded grid has a tile for every 128 rows of the longest one in every request."""
    plan = bound([8192] + [100] * 30, [0] * 31, 32, 8, d)
    assert plan.stat(7) == 31 * 64 and plan.stat(8) == 0 and plan.stat(9) == 0


# many short prompts: a query tile per request where the waves of a workgroup take several heads, tiles of 128 rows and one head otherwise
@pytest.mark.parametrize("ql", [[16] * 512, [256] * 64, wl.config2_lengths(0)], ids=["512 x 16", "64 x 256", "64 ragged"])
def test_tables_of_tiles_of_several_heads_are_no_slower_to_build(ql):
    """The best of 40 runs each in turn: a fifth beyond the tables of one head per KV head, which do not have such tiles."""
    ql = np.asarray(ql, dtype=np.int32)
    best = {}
    for _ in range(40):
        for heads in ((32, 8), (8, 1), (16, 16)):
            plan = pk.pack_plan(ql, ql, token_budget=16384)
            begin = time.perf_counter()
            plan.workspace_bytes(*heads, 128, pk.PK_BF16)
            best[heads] = min(best.get(heads, 1.0), time.perf_counter() - begin)
    assert max(best[32, 8], best[8, 1]) <= 1.2 * best[16, 16], best


# waves of a workgroup, query rows of a tile: chunks of a 70B-shaped layer, lists too short for eight waves, two, four, six and eight heads per KV head, odd numbers
@pytest.mark.parametrize("ql, ctx, Hq, Hkv, d, waves, rows", [
    (*wl.config5_structure(0)[:2], 64, 8, 128, 8, 32), (*wl.config5_structure(0)[:2], 64, 8, 64, 4, 32), (wl.config2_lengths(0), [0] * 64, 32, 8, 128, 4, 32),
    ([128] * 16, [12000] * 16, 32, 8, 128, 8, 64), ([128] * 16, [12000] * 16, 32, 16, 128, 8, 128), ([128] * 20, [12000] * 20, 48, 8, 128, 8, 128),
    ([128] * 16, [6000] * 16, 32, 8, 128, 4, 32), ([200] * 64, [0] * 64, 16, 8, 128, 4, 64), ([200] * 64, [0] * 64, 24, 8, 128, 4, 128), ([200] * 64, [0] * 64, 8, 8, 128, 4, 128)])
def test_waves_and_rows_of_a_workgroup(ql, ctx, Hq, Hkv, d, waves, rows):
    plan = bound(ql, ctx, Hq, Hkv, d)
    assert (plan.stat(11), plan.stat(12)) == (waves, rows)
    plan.workspace_bytes(Hq, Hkv, d, pk.PK_F32)
    assert (plan.stat(11), plan.stat(12)) == (0, 0)
