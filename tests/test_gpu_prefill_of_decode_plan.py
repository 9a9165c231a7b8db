"""The packed prefill call on a plan of one query row per request, whose prefill tables are built and uploaded at the first such call: against the oracle and the decode
call, on workspaces that the plan is bound to in turns, and captured."""
import numpy as np
import pytest
import torch

from paper_2602_06072_amd import binding as pk
from paper_2602_06072_amd import workloads as wl
from tests import helpers as H

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.mark.parametrize("n", [1, 7, 40, 300])             # (a tile for each of them, and tiles that many share)
@pytest.mark.parametrize("Hq, Hkv, d", [(8, 2, 128), (16, 16, 64), (12, 2, 128)])
def test_prefill_and_decode_of_one_plan(n, Hq, Hkv, d):
    kv = np.random.default_rng(n).integers(1, 700, size=n).astype(np.int32)
    ones = np.ones_like(kv)
    w = wl.make_ragged("one row each", kv, ones, Hq, Hkv, d, 2048, 23, device=DEV, keep_f32=False)
    plan = pk.pack_plan(kv, ones, token_budget=2048)
    workspaces = [pk.new_workspace(plan, Hq, Hkv, d, pk.PK_BF16) for _ in range(2)]
    want = H.oracle_ragged(w, False)
    buf = pk.new_kv_buf(plan, Hkv, d, pk.PK_BF16)
    # the rows as pages of one token
    starts = np.concatenate([[0], np.cumsum(kv)])
    table = np.zeros((n, int(kv.max())), dtype=np.int32)
    for i in range(n):
        table[i, : kv[i]] = np.arange(starts[i], starts[i + 1])
    pages = [x.view(-1, 1, Hkv, d) for x in (w.k, w.v)]
    outs = []
    for ws in workspaces + workspaces[:1]:
        pk.kv_reorganize(plan, *pages, torch.from_numpy(table).to(DEV), buf, ws)
        decoded, filled, again = (torch.full(w.q.shape, float("nan"), dtype=torch.float32, device=DEV) for _ in range(3))
        pk.packed_decode_attn(plan, w.q, buf, decoded, w.scale, Hkv, ws)
        pk.packed_prefill_attn(plan, w.q, w.k, w.v, filled, w.scale, ws)
        pk.packed_decode_attn(plan, w.q, buf, again, w.scale, Hkv, ws)
        torch.cuda.synchronize()
        H.assert_close(filled.cpu().numpy(), want, 0, f"prefill of a decode plan {n} {Hq}/{Hkv} {d}")
        H.assert_close(decoded.cpu().numpy(), want, 0, f"decode {n} {Hq}/{Hkv} {d}")
        assert torch.equal(decoded, again)
        outs.append(filled)
    assert torch.equal(outs[0], outs[1]) and torch.equal(outs[0], outs[2])
    assert plan.stat(6) > 0 and plan.stat(1) >= plan.stat(0) == int(kv.sum())


def test_first_prefill_call_captured():
    kv = np.random.default_rng(2).integers(1, 400, size=60).astype(np.int32)
    w = wl.make_ragged("captured", kv, np.ones_like(kv), 8, 2, 128, 2048, 24, device=DEV, keep_f32=False)
    other = pk.pack_plan(kv, kv, token_budget=2048)            # (a staging buffer and the kernels are there from here on)
    pk.plan_bind(other, 8, 2, 128, pk.PK_BF16, pk.new_workspace(other, 8, 2, 128, pk.PK_BF16))
    ref = torch.empty(w.q.shape, dtype=torch.float32, device=DEV)
    plans = [pk.pack_plan(kv, np.ones_like(kv), token_budget=2048) for _ in range(2)]
    ws = [pk.new_workspace(p, 8, 2, 128, pk.PK_BF16) for p in plans]
    pk.packed_prefill_attn(plans[0], w.q, w.k, w.v, ref, w.scale, ws[0])
    out = torch.empty_like(ref)
    pk.plan_bind(plans[1], 8, 2, 128, pk.PK_BF16, ws[1])
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        pk.packed_prefill_attn(plans[1], w.q, w.k, w.v, out, w.scale, ws[1])
    for rep in range(3):
        out.fill_(float("nan"))
        pk.packed_prefill_attn(plans[0], w.q, w.k, w.v, ref, w.scale, ws[0])
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, ref), f"replay {rep}"


@pytest.mark.parametrize("inside", ["prefill", "bind and prefill"])
def test_calls_behind_a_capture_that_has_not_run(inside):
    """An eager call, and one of another capture, find their tables whether or not the first graph ever runs.  (Zeros as tables would leave the output as it is.)"""
    kv = np.random.default_rng(3).integers(1, 400, size=60).astype(np.int32)
    w = wl.make_ragged("captured", kv, np.ones_like(kv), 8, 2, 128, 2048, 25, device=DEV, keep_f32=False)
    plans = [pk.pack_plan(kv, np.ones_like(kv), token_budget=2048) for _ in range(3)]
    ws = [torch.zeros(p.workspace_bytes(8, 2, 128, pk.PK_BF16), dtype=torch.uint8, device=DEV) for p in plans]
    outs = [torch.full(w.q.shape, float("nan"), dtype=torch.float32, device=DEV) for _ in range(5)]
    pk.packed_prefill_attn(plans[0], w.q, w.k, w.v, outs[0], w.scale, ws[0])      # (eager all the way, and kernels that are loaded)
    if inside == "prefill":
        for p, x in zip(plans[1:], ws[1:]):
            pk.plan_bind(p, 8, 2, 128, pk.PK_BF16, x)
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())

    def capture(p, x, out):
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=side):
            if inside != "prefill":
                pk.plan_bind(p, 8, 2, 128, pk.PK_BF16, x)
            pk.packed_prefill_attn(p, w.q, w.k, w.v, out, w.scale, x)
        return graph
    graphs = [capture(p, x, outs[1]) for p, x in zip(plans[1:], ws[1:])]
    pk.packed_prefill_attn(plans[1], w.q, w.k, w.v, outs[2], w.scale, ws[1])      # eager, behind a capture
    graphs.append(capture(plans[2], ws[2], outs[3]))                               # captured, behind another capture
    torch.cuda.synchronize()
    graphs[2].replay()
    pk.packed_prefill_attn(plans[2], w.q, w.k, w.v, outs[4], w.scale, ws[2])
    torch.cuda.synchronize()
    for x in (2, 3, 4):
        assert torch.equal(outs[x], outs[0]), x
    for rep in range(3):
        for graph in graphs[:2]:
            outs[1].fill_(float("nan"))
            pk.packed_prefill_attn(plans[0], w.q, w.k, w.v, outs[0], w.scale, ws[0])
            torch.cuda.synchronize()
            graph.replay()
            torch.cuda.synchronize()
            assert torch.equal(outs[1], outs[0]), rep
