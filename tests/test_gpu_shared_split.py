"""Decode batches whose shared segments are cut otherwise than the suffixes, shorter and longer: against the oracle, with both outputs, twice on one workspace."""
import numpy as np
import pytest
import torch

from paper_2602_06072_amd import binding as pk
from paper_2602_06072_amd import workloads as wl
from tests import helpers as H

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.mark.parametrize("out_f32", [True, False])
@pytest.mark.parametrize("n, own, families, prefix, heads, shorter", [
    (180, 33, 11, 2000, (16, 16, 128), True), (280, 63, 34, 900, (32, 8, 128), True), (124, 30, 30, 1600, (32, 8, 64), True),
    (40, 350, 20, 2743, (16, 2, 128), False), (64, 56, 16, 2459, (28, 4, 128), False)])
def test_shared_segments_with_their_own_split(n, own, families, prefix, heads, shorter, out_f32):
    Hq, Hkv, d = heads
    rng = np.random.default_rng(n)
    fam = (np.arange(n) * families // n).astype(np.int32)
    plen = rng.integers(prefix * 3 // 4, prefix + 1, families).astype(np.int32)[fam]
    kv = (plen + rng.integers(1, 2 * own, n)).astype(np.int32)
    w = wl.make_paged("split", kv, Hq, Hkv, d, 32768, 16, n, prefix_ids=fam, prefix_lens=plen, device=DEV, keep_f32=False)
    plan = pk.pack_plan(kv, np.ones_like(kv), fam, plen, 32768)
    ws = pk.new_workspace(plan, Hq, Hkv, d, pk.PK_BF16)
    buf = pk.new_kv_buf(plan, Hkv, d, pk.PK_BF16, fill=0x7F)
    pk.kv_reorganize(plan, w.k_pages, w.v_pages, torch.from_numpy(w.block_table).to(DEV), buf, ws)
    items = plan.stat(3)
    rows = list(range(0, n, max(1, n // 24)))
    want = H.oracle_paged_decode(w, False, rows)
    got = []
    for _ in range(2):
        out = torch.full(w.q.shape, float("nan"), dtype=torch.float32 if out_f32 else torch.bfloat16, device=DEV)
        pk.packed_decode_attn(plan, w.q, buf, out, w.scale, Hkv, ws)
        torch.cuda.synchronize()
        got.append(out)
        H.assert_close(out[rows].float().cpu().numpy(), want, 0, f"shared split {n} {heads}")
    assert torch.equal(got[0], got[1]) and torch.isfinite(got[0].float()).all()
    if torch.cuda.get_device_properties(0).multi_processor_count == 256:
        plan.tune(pk.TUNE_DECODE_SPLIT, plan.stat(5))
        plan.workspace_bytes(Hq, Hkv, d, pk.PK_BF16)
        assert (items > plan.stat(3)) == shorter and items != plan.stat(3)
