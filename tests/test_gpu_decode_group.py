"""Decode batches whose work items are served by workgroups: items shorter than the workgroup has waves, requests of one item
and of as many partial results as one batch of the merge holds, one more, and two batches."""
import numpy as np
import pytest
import torch

from paper_2602_06072_amd import binding as pk
from paper_2602_06072_amd import workloads as wl
from tests import helpers as H

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.mark.parametrize("out_f32", [True, False])
@pytest.mark.parametrize("heads", [(1, 1, 64), (16, 1, 128), (8, 2, 64), (3, 3, 128)])
@pytest.mark.parametrize("case", ["tiles", "parts", "parts_reversed", "private_prefix"])
def test_decode_by_workgroups(case, heads, out_f32):
    Hq, Hkv, d = heads
    unit = 384 * 128 // d                          # the shortest split, of which these batches are cut
    kv = np.asarray([1, 31, 32, 33, 95, 96, 97, 127, 128, 129, 160, 161, 190, 255, 257], dtype=np.int32)
    pid = plen = None
    if case != "tiles":
        kv = np.asarray([2 * unit, 5, 8 * unit, unit + 1, 9 * unit - 31, 16 * unit, unit], dtype=np.int32)
        if case == "parts_reversed":
            kv = np.ascontiguousarray(kv[::-1])
        if case == "private_prefix":                # shared segments of one request each
            pid, plen = np.arange(len(kv), dtype=np.int32), (kv // 3).astype(np.int32)
    w = wl.make_paged(f"group_{case}", kv, Hq, Hkv, d, 32768, 16, 90 + len(case), prefix_ids=pid, prefix_lens=plen, device=DEV,
                      keep_f32=False)
    plan = pk.pack_plan(kv, np.ones_like(kv), pid, plen, 32768)
    ws = pk.new_workspace(plan, Hq, Hkv, d, pk.PK_BF16)
    buf = pk.new_kv_buf(plan, Hkv, d, pk.PK_BF16, fill=0x7F)
    pk.kv_reorganize(plan, w.k_pages, w.v_pages, torch.from_numpy(w.block_table).to(DEV), buf, ws)
    if torch.cuda.get_device_properties(0).multi_processor_count == 256:
        assert plan.stat(5) >= unit and (plan.stat(4) >= 37) == (case != "tiles")   # (a wave each would have 128)
    want = H.oracle_paged_decode(w, False)
    got = []
    for _ in range(3):                              # the counts of finished items are back at zero for the next launch
        out = torch.full(w.q.shape, float("nan"), dtype=torch.float32 if out_f32 else torch.bfloat16, device=DEV)
        pk.packed_decode_attn(plan, w.q, buf, out, w.scale, Hkv, ws)
        torch.cuda.synchronize()
        got.append(out)
        H.assert_close(out.float().cpu().numpy(), want, 0, f"decode by workgroups, {case}, {heads}")
    assert torch.equal(got[0], got[1]) and torch.equal(got[0], got[2])      # partial results in the order of their slots
    # the same plan with a wave per item: another split of the same sums, each side within its own rounding of the
    # oracle: P in bf16 (relative 2^-9 of values below 4), and the output's own rounding if it is bf16
    plan.tune(pk.TUNE_DECODE_SPLIT, 128)
    ws = pk.new_workspace(plan, Hq, Hkv, d, pk.PK_BF16)
    out = torch.full_like(got[0], float("nan"))
    pk.packed_decode_attn(plan, w.q, buf, out, w.scale, Hkv, ws)
    torch.cuda.synchronize()
    assert plan.stat(5) == 128
    assert float((out.float() - got[0].float()).abs().max()) <= 2 * 4 * 2.0 ** -9 * (1 if out_f32 else 2)
