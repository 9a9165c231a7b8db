"""Decode batches whose work items are served by workgroups: items shorter than the workgroup has waves, requests of one item
and of as many partial results as one batch of the merge holds, one more, and two batches; the merge through the fixed scratch, in
replays of a captured graph, and with two plans in turns on one workspace."""
import ctypes

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
        # (short batches with more than 64 merged rows per KV head stay with waves: at most four of sixteen here, more in the test below)
        most = 16 if Hq // Hkv < 16 else 4
        kv = np.asarray([2 * unit, 5, most // 2 * unit, unit + 1, (most // 2 + 1) * unit - 31, most * unit, unit], dtype=np.int32)
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
        assert plan.stat(5) >= unit and (plan.stat(4) >= (37 if Hq // Hkv < 16 else 13)) == (case != "tiles")   # (a wave each would have 128)
    waves = plan.stat(10)
    assert waves == 4
    want = H.oracle_paged_decode(w, False)
    got = []
    for _ in range(3):                              # the counts of finished items are back at zero for the next launch
        out = torch.full(w.q.shape, float("nan"), dtype=torch.float32 if out_f32 else torch.bfloat16, device=DEV)
        pk.packed_decode_attn(plan, w.q, buf, out, w.scale, Hkv, ws)
        torch.cuda.synchronize()
        got.append(out)
        H.assert_close(out.float().cpu().numpy(), want, 0, f"decode by workgroups, {case}, {heads}")
    assert torch.equal(got[0], got[1]) and torch.equal(got[0], got[2])      # partial results in the order of their slots
    # the same plan with the split that a wave per item would have: the kernel is the same (another split of the same sums, each
    # side within its own rounding of the oracle: P in bf16 (relative 2^-9 of values below 4), and the output's own rounding if it is bf16)
    plan.tune(pk.TUNE_DECODE_SPLIT, 128)
    ws = pk.new_workspace(plan, Hq, Hkv, d, pk.PK_BF16)
    out = torch.full_like(got[0], float("nan"))
    pk.packed_decode_attn(plan, w.q, buf, out, w.scale, Hkv, ws)
    torch.cuda.synchronize()
    assert plan.stat(5) == 128 and plan.stat(10) == waves
    assert float((out.float() - got[0].float()).abs().max()) <= 2 * 4 * 2.0 ** -9 * (1 if out_f32 else 2)


def batch(kv, seed):
    """A decode batch, its plan, buffer and the result of the workspace call."""
    kv = np.asarray(kv, dtype=np.int32)
    w = wl.make_paged(f"merge_{seed}", kv, 8, 2, 128, 32768, 16, seed, device=DEV, keep_f32=False)
    plan = pk.pack_plan(kv, np.ones_like(kv), None, None, 32768)
    ws = pk.new_workspace(plan, 8, 2, 128, pk.PK_BF16)
    buf = pk.new_kv_buf(plan, 2, 128, pk.PK_BF16)
    pk.kv_reorganize(plan, w.k_pages, w.v_pages, torch.from_numpy(w.block_table).to(DEV), buf, ws)
    ref = torch.full(w.q.shape, float("nan"), dtype=torch.float32, device=DEV)
    pk.packed_decode_attn(plan, w.q, buf, ref, w.scale, 2, ws)
    torch.cuda.synchronize()
    assert plan.stat(10) == 4 and plan.stat(4) > 0
    H.assert_close(ref.cpu().numpy(), H.oracle_paged_decode(w, False), 0, f"batch {seed}")
    return w, plan, ws, buf, ref


def test_many_partial_results_of_sixteen_rows():
    """Sixteen query heads of a KV head and as many as 17 partial results: three batches of the merge, two passes of the workgroup."""
    kv = np.asarray([40000, 9000, 33000, 5, 20000, 768], dtype=np.int32)
    w = wl.make_paged("sixteen", kv, 64, 4, 128, 32768, 16, 65, device=DEV, keep_f32=False)
    plan = pk.pack_plan(kv, np.ones_like(kv), None, None, 32768)
    ws = pk.new_workspace(plan, 64, 4, 128, pk.PK_BF16)
    buf = pk.new_kv_buf(plan, 4, 128, pk.PK_BF16)
    pk.kv_reorganize(plan, w.k_pages, w.v_pages, torch.from_numpy(w.block_table).to(DEV), buf, ws)
    if torch.cuda.get_device_properties(0).multi_processor_count == 256:
        assert plan.stat(10) == 4 and -(-40000 // plan.stat(5)) > 16
    got = []
    for _ in range(2):
        out = torch.full(w.q.shape, float("nan"), dtype=torch.float32, device=DEV)
        pk.packed_decode_attn(plan, w.q, buf, out, w.scale, 4, ws)
        torch.cuda.synchronize()
        got.append(out)
    H.assert_close(got[0].cpu().numpy(), H.oracle_paged_decode(w, False), 0, "many partial results of sixteen rows")
    assert torch.equal(got[0], got[1])


def test_merge_through_the_fixed_scratch_and_in_replays():
    w, plan, ws, buf, ref = batch([2000, 100, 6000, 900, 800, 5000], 61)
    other = batch([3000, 60, 2000, 2500], 62)
    L = pk.lib()
    plan_s = pk.pack_plan(w.kv_lens, np.ones(w.n, dtype=np.int32), None, None, 32768)

    def call(plan, w, buf, out, stream):
        rc = L.pk_packed_decode_attn_static(plan.handle, w.q.data_ptr(), buf.data_ptr(), out.data_ptr(), ctypes.c_float(w.scale),
                                            8, 2, 128, pk.PK_BF16, pk.PK_F32, ctypes.c_void_p(stream.cuda_stream))
        assert rc == 0, L.pk_last_error().decode()

    def eager(plan, w, buf, ref):
        out = torch.full_like(ref, float("nan"))
        call(plan, w, buf, out, torch.cuda.current_stream())
        torch.cuda.synchronize()
        assert torch.equal(out, ref)

    plan_o = pk.pack_plan(other[0].kv_lens, np.ones(other[0].n, dtype=np.int32), None, None, 32768)
    for _ in range(2):                              # the second call uploads nothing, another plan's call in between everything
        eager(plan_s, w, buf, ref)
        eager(plan_s, w, buf, ref)
        eager(plan_o, other[0], other[3], other[4])
    eager(plan_s, w, buf, ref)
    out = torch.full_like(ref, float("nan"))
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        call(plan_s, w, buf, out, torch.cuda.current_stream())
        call(plan_s, w, buf, out, torch.cuda.current_stream())
    torch.cuda.synchronize()
    for rep in range(4):
        out.fill_(float("nan"))
        again = torch.full_like(ref, float("nan"))
        pk.packed_decode_attn(plan, w.q, buf, again, w.scale, 2, ws)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, ref) and torch.equal(again, ref), f"replay {rep}"


def test_two_plans_in_turns_on_one_workspace():
    a, b = batch([2000, 100, 6000, 900, 800, 5000], 63), batch([5000, 60, 4000, 2500], 64)
    ws = max((a[2], b[2]), key=lambda t: t.numel())
    for turn in range(3):
        for w, plan, _, buf, ref in (a, b):
            for _ in range(2):
                out = torch.full_like(ref, float("nan"))
                pk.packed_decode_attn(plan, w.q, buf, out, w.scale, 2, ws)
                torch.cuda.synchronize()
                assert torch.equal(out, ref), f"turn {turn} {w.name}"
