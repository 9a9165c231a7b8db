"""The output of the prefill launches of little work on both sides of 2 MiB, from where it is written through the L2 (fp32 rows by way of LDS): fp32 rounded to
bf16 is the bf16 output bit for bit, whichever way either took, also in the mixed step; and the oracle."""
import numpy as np
import pytest
import torch

from paper_2602_06072_amd import binding as pk
from paper_2602_06072_amd import workloads as wl
from tests import helpers as H

pytestmark = pytest.mark.gpu
DEV = "cuda"


# bytes in bf16, in fp32: both below, one on each side, both above
@pytest.mark.parametrize("values, sides", [(300_000, (0, 0)), (800_000, (0, 1)), (1_600_000, (1, 1))])
@pytest.mark.parametrize("Hq, Hkv, d", [(16, 4, 128), (32, 8, 64), (16, 16, 128), (18, 3, 128), (30, 6, 64)])
def test_both_outputs(values, sides, Hq, Hkv, d):
    ql, left = [], values // (Hq * d)
    while left > 0:
        ql.append(min(left, (33, 130, 1, 64, 95, 31, 7, 200)[len(ql) % 8]))
        left -= ql[-1]
    ql = np.asarray(ql, dtype=np.int32)
    ctx = np.arange(len(ql), dtype=np.int32) * 61 % 150
    elements = int(ql.sum()) * Hq * d
    assert (elements * 2 >= 2 << 20, elements * 4 >= 2 << 20) == sides
    w = wl.make_ragged("output", ql + ctx, ql, Hq, Hkv, d, 2048, 17, device=DEV, keep_f32=False)
    dec = wl.small_paged(seed=18, n=3, lo=1, hi=200, Hq=Hq, Hkv=Hkv, d=d, token_budget=500, device=DEV, keep_f32=False)
    dplan = pk.pack_plan(dec.kv_lens, np.ones_like(dec.kv_lens), None, None, 500)
    dws = pk.new_workspace(dplan, Hq, Hkv, d, pk.PK_BF16)
    buf = pk.new_kv_buf(dplan, Hkv, d, pk.PK_BF16)
    pk.kv_reorganize(dplan, dec.k_pages, dec.v_pages, torch.from_numpy(dec.block_table).to(DEV), buf, dws)
    plan = pk.pack_plan(w.kv_lens, w.q_lens, token_budget=w.token_budget)
    ws = pk.new_workspace(plan, Hq, Hkv, d, pk.PK_BF16)
    outs = {}
    for dtype in (torch.float32, torch.bfloat16):
        guard = torch.full((elements + 256,), float("nan"), dtype=dtype, device=DEV)     # (nothing behind the output is written)
        out, fused = guard[:elements].view(w.q.shape), torch.full(w.q.shape, float("nan"), dtype=dtype, device=DEV)
        pk.packed_prefill_attn(plan, w.q, w.k, w.v, out, w.scale, ws)
        pk.packed_mixed_step(plan, w.q, w.k, w.v, fused, ws, dplan, dec.q, buf, torch.empty_like(dec.q, dtype=dtype), dws, w.scale)
        torch.cuda.synchronize()
        assert plan.stat(8) == 1 and torch.isnan(guard[elements:]).all()
        assert torch.isfinite(out).all() and torch.equal(out, fused)
        outs[dtype] = out
    assert torch.equal(outs[torch.float32].to(torch.bfloat16), outs[torch.bfloat16])
    H.assert_close(outs[torch.float32].cpu().numpy(), H.oracle_ragged(w, False), 0, f"{values} {Hq}/{Hkv} {d}")
