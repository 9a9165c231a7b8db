"""Which short decode batches are served by workgroups, and that PK_TUNE_DECODE_SPLIT changes the split of the work items and not the
kernel (host only: the tables say both)."""
import numpy as np
import pytest

from paper_2602_06072_amd import binding as pk


@pytest.mark.parametrize("kv, shared, waves", [
    ([300, 900, 2000, 3000], False, 4), ([1500] * 24, False, 4), ([8, 20, 32] * 20, False, 1), ([700] * 16, True, 1)])
def test_split_knob_keeps_the_kernel(kv, shared, waves):
    kv = np.asarray(kv, dtype=np.int32)
    pid, plen = (np.zeros_like(kv), np.full_like(kv, 200)) if shared else (None, None)
    plan = pk.pack_plan(kv, np.ones_like(kv), pid, plen, 1 << 20)
    plan.workspace_bytes(32, 8, 128, pk.PK_BF16)
    own = plan.stat(5)
    assert plan.stat(10) == waves
    for split in (32, 250, 512, 4096, 0):
        plan.tune(pk.TUNE_DECODE_SPLIT, split)
        plan.workspace_bytes(32, 8, 128, pk.PK_BF16)
        assert plan.stat(10) == waves and plan.stat(5) == ((split + 31) // 32 * 32 or own)
        assert shared or plan.stat(3) >= sum(-(-int(x) // plan.stat(5)) for x in kv)


# lengths, heads, waves per item: one workgroup merges the partial results of all query heads of a KV head
@pytest.mark.parametrize("kv, Hq, Hkv, waves", [
    ([4000], 64, 4, 1), ([4000], 32, 2, 1), ([4000, 800], 64, 8, 1), ([3000, 2500], 64, 4, 1), ([4000], 32, 8, 4), ([4000], 8, 2, 4),
    ([3000] * 8, 64, 4, 4), ([1500], 64, 4, 4), ([2500], 64, 8, 4), ([40000, 9000, 33000, 5, 20000, 768], 64, 4, 4)])
def test_short_batches_with_many_merged_rows(kv, Hq, Hkv, waves):
    plan = pk.pack_plan(np.asarray(kv, dtype=np.int32), np.ones(len(kv), dtype=np.int32), None, None, 32768)
    plan.workspace_bytes(Hq, Hkv, 128, pk.PK_BF16)
    assert plan.stat(10) == waves
