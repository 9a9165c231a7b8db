"""The fused mixed step (prefill tiles and decode work items of one continuous-batching step in one
launch) against the two separate calls and against the oracle."""
import numpy as np
import pytest
import torch

from paper_2602_06072_amd import binding as pk
from paper_2602_06072_amd import workloads as wl
from tests import helpers as H

pytestmark = pytest.mark.gpu
DEV = "cuda"


def run_both(p, d, budget_p, budget_d, out_dtype=torch.float32):
    plan_p = pk.pack_plan(p.kv_lens, p.q_lens, token_budget=budget_p)
    ones = np.ones(d.n, dtype=np.int32)
    plan_d = pk.pack_plan(d.kv_lens, ones, d.prefix_ids, d.prefix_lens, budget_d)
    ws_p = pk.new_workspace(plan_p, p.Hq, p.Hkv, p.d, pk.PK_BF16)
    ws_d = pk.new_workspace(plan_d, d.Hq, d.Hkv, d.d, pk.PK_BF16)
    buf = pk.new_kv_buf(plan_d, d.Hkv, d.d, pk.PK_BF16)
    pk.kv_reorganize(plan_d, d.k_pages, d.v_pages, torch.from_numpy(d.block_table).to(DEV), buf, ws_d)
    sep_p = torch.full(p.q.shape, float("nan"), dtype=out_dtype, device=DEV)
    sep_d = torch.full(d.q.shape, float("nan"), dtype=out_dtype, device=DEV)
    pk.packed_prefill_attn(plan_p, p.q, p.k, p.v, sep_p, p.scale, ws_p)
    pk.packed_decode_attn(plan_d, d.q, buf, sep_d, d.scale, d.Hkv, ws_d)
    torch.cuda.synchronize()
    fus_p = torch.full(p.q.shape, float("nan"), dtype=out_dtype, device=DEV)
    fus_d = torch.full(d.q.shape, float("nan"), dtype=out_dtype, device=DEV)
    pk.packed_mixed_step(plan_p, p.q, p.k, p.v, fus_p, ws_p, plan_d, d.q, buf, fus_d, ws_d, p.scale)
    torch.cuda.synchronize()
    assert torch.equal(fus_p, sep_p) and torch.equal(fus_d, sep_d)      # same arithmetic per tile and per work item
    return fus_p, fus_d


@pytest.mark.parametrize("case", ["more_prefill", "more_decode", "families", "d64", "d64_families"])
def test_mixed_step_small(case):
    kwp = dict(seed=80, n=7, lo=5, hi=300, Hq=8, Hkv=2, d=128, token_budget=400, ctx_hi=200, device=DEV, keep_f32=False)
    kwd = dict(seed=81, n=9, lo=1, hi=500, Hq=8, Hkv=2, d=128, token_budget=900, device=DEV, keep_f32=False)
    if case == "more_decode":
        kwp.update(n=1, lo=20, hi=40, ctx_hi=0)
        kwd.update(n=60, hi=900)
    elif case == "families":
        kwd.update(n=30, families=3, prefix_lo=40, prefix_hi=300)
    elif case == "d64":
        kwp.update(d=64)
        kwd.update(d=64)
    elif case == "d64_families":
        kwp.update(d=64, n=12, hi=700)
        kwd.update(d=64, n=40, families=4, prefix_lo=40, prefix_hi=300)
    p, d = wl.small_ragged(**kwp), wl.small_paged(**kwd)
    fus_p, fus_d = run_both(p, d, p.token_budget, d.token_budget)
    H.assert_close(fus_p.cpu().numpy(), H.oracle_ragged(p, False), 0, f"mixed step {case}: prefill half")
    H.assert_close(fus_d.cpu().numpy(), H.oracle_paged_decode(d, False), 0, f"mixed step {case}: decode half")


@pytest.mark.parametrize("waves", [4, 1])
@pytest.mark.parametrize("light", [1, 0])
@pytest.mark.parametrize("d", [64, 128])
def test_mixed_step_kernels(d, light, waves):
    """Each prefill body beside each kind of decode workgroup; requests of one and of several partial results."""
    kv, ql = [700, 300, 129, 64, 1000], [90, 300, 1, 64, 40]
    if not light:
        kv, ql = H.with_long_requests(kv, ql)
    p = wl.make_ragged("kernels", np.asarray(kv, np.int32), np.asarray(ql, np.int32), 4 if light else 32, 2 if light else 8, d, 4096, 98, device=DEV,
                       keep_f32=False)
    dkv = np.asarray([9000, 40, 3000, 700, 500, 33] * 4, dtype=np.int32)
    pid = plen = None
    if waves == 1:                                        # a shared prefix: items of several requests
        pid, plen = np.zeros_like(dkv), np.full_like(dkv, 32)
    dec = wl.make_paged("kernels", dkv, p.Hq, p.Hkv, d, 1 << 18, 16, 99, prefix_ids=pid, prefix_lens=plen, device=DEV, keep_f32=False)
    plan_p = pk.pack_plan(p.kv_lens, p.q_lens, token_budget=4096)
    plan_d = pk.pack_plan(dec.kv_lens, np.ones_like(dkv), pid, plen, 1 << 18)
    for plan in (plan_p, plan_d):
        plan.workspace_bytes(p.Hq, p.Hkv, d, pk.PK_BF16)
    assert plan_p.stat(8) == light and plan_d.stat(10) == waves and plan_d.stat(4) > 0
    for out_dtype in (torch.float32, torch.bfloat16):
        fus_p, fus_d = run_both(p, dec, 4096, 1 << 18, out_dtype)
        H.assert_close(fus_p.float().cpu().numpy(), H.oracle_ragged(p, False), 0, f"mixed step: prefill half, d {d}")
        H.assert_close(fus_d.float().cpu().numpy(), H.oracle_paged_decode(dec, False), 0, f"mixed step: decode half, d {d}")


@pytest.mark.parametrize("prefill, rows", [(40, 12), (33, 260), (16, 300), (9, 64)])
def test_mixed_step_order_of_workgroups(prefill, rows):
    """Runs of 256 workgroups: 5 prefill to 1 decode, 5 to 3 (two left over), 2 to 3 (one decode run left over),
    2 to 1 with a remainder in both kinds."""
    p = wl.small_ragged(seed=90, n=prefill, lo=100, hi=128, Hq=32, Hkv=8, d=64, token_budget=2048, ctx_hi=70,
                        device=DEV, keep_f32=False)
    d = wl.small_paged(seed=91, n=rows, lo=1, hi=120, Hq=32, Hkv=8, d=64, token_budget=2048, device=DEV, keep_f32=False)
    run_both(p, d, p.token_budget, d.token_budget, torch.bfloat16)


@pytest.mark.parametrize("out_dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("heads, n, lo, hi", [((64, 2), 4, 200, 256), ((64, 4), 24, 20, 90), ((8, 4), 20, 130, 256),
                                              ((32, 16), 9, 128, 257), ((12, 2), 30, 1, 256)])
def test_eight_waves_to_a_workgroup(heads, n, lo, hi, out_dtype):
    """Long key lists, full rounds: the prefill call has eight waves to a workgroup, the fused step four on the same query tiles, with
    the same arithmetic per query row.  2, 6, 16 and 32 heads per KV head, tiles of one request and of several."""
    rng = np.random.default_rng(95)
    ql = rng.integers(lo, hi + 1, size=n).astype(np.int32)
    kv = ql + rng.integers(2200, 2700, size=n).astype(np.int32)
    kv, ql = H.with_eight_waves(kv, ql, *heads, 1 << 17, rows=128)
    p = wl.make_ragged("pair", kv, ql, heads[0], heads[1], 128, 1 << 17, 96, device=DEV, keep_f32=False)
    d = wl.small_paged(seed=97, n=5, lo=1, hi=100, Hq=heads[0], Hkv=heads[1], d=128, token_budget=500, device=DEV, keep_f32=False)
    plan = pk.pack_plan(kv, ql, token_budget=1 << 17)
    plan.workspace_bytes(heads[0], heads[1], 128, pk.PK_BF16)
    assert plan.stat(11) == 8 and plan.stat(12) == (32 if heads[0] // heads[1] >= 16 else 128)
    assert heads != (12, 2) or plan.stat(6) < sum((x + 127) // 128 for x in ql)       # some tiles are shared
    fus_p, _ = run_both(p, d, 1 << 17, 500, out_dtype)
    req = rng.integers(0, len(ql), size=300)
    rows = np.stack([req, rng.integers(0, heads[0], size=300), rng.integers(0, ql[req])], axis=1).astype(np.int32)
    start = np.concatenate([[0], np.cumsum(ql)])
    got = fus_p.float().cpu().numpy()[start[rows[:, 0]] + rows[:, 2], rows[:, 1]]
    H.assert_close(got, H.oracle_ragged(p, False, rows=rows), 0, f"eight waves, {heads}")


def test_mixed_step_with_an_empty_half_and_bad_arguments():
    p = wl.small_ragged(seed=82, n=3, lo=5, hi=100, Hq=4, Hkv=2, d=128, token_budget=200, device=DEV, keep_f32=False)
    d = wl.small_paged(seed=83, n=4, lo=1, hi=100, Hq=4, Hkv=2, d=128, token_budget=200, device=DEV, keep_f32=False)
    plan_p = pk.pack_plan(p.kv_lens, p.q_lens, token_budget=200)
    plan_d = pk.pack_plan(d.kv_lens, np.ones(d.n, dtype=np.int32), None, None, 200)
    empty = pk.pack_plan([], token_budget=16)
    ws_p = pk.new_workspace(plan_p, 4, 2, 128, pk.PK_BF16)
    ws_d = pk.new_workspace(plan_d, 4, 2, 128, pk.PK_BF16)
    buf = pk.new_kv_buf(plan_d, 2, 128, pk.PK_BF16)
    pk.kv_reorganize(plan_d, d.k_pages, d.v_pages, torch.from_numpy(d.block_table).to(DEV), buf, ws_d)
    out_p = torch.full(p.q.shape, float("nan"), dtype=torch.float32, device=DEV)
    out_d = torch.full(d.q.shape, float("nan"), dtype=torch.float32, device=DEV)
    pk.packed_mixed_step(plan_p, p.q, p.k, p.v, out_p, ws_p, empty, d.q, buf, out_d, ws_d, p.scale)
    pk.packed_mixed_step(empty, p.q, p.k, p.v, out_p, ws_p, plan_d, d.q, buf, out_d, ws_d, p.scale)
    torch.cuda.synchronize()
    H.assert_close(out_p.cpu().numpy(), H.oracle_ragged(p, False), 0, "prefill half alone")
    H.assert_close(out_d.cpu().numpy(), H.oracle_paged_decode(d, False), 0, "decode half alone")
    with pytest.raises(pk.PackInferError):            # one workspace for both plans
        pk.packed_mixed_step(plan_p, p.q, p.k, p.v, out_p, ws_p, plan_d, d.q, buf, out_d, ws_p, p.scale)
    with pytest.raises(pk.PackInferError):            # the decode plan must be a decode plan
        pk.packed_mixed_step(plan_p, p.q, p.k, p.v, out_p, ws_p, plan_p, d.q, buf, out_d, ws_d, p.scale)


def test_mixed_step_config5_full_size():
    """Configuration 5 at the size bench.py runs through the fused entry point: bit-equal to the two
    separate calls (whose outputs the full-size parity tests compare with the oracle), and the decode
    half against the oracle on every long request plus 60 others."""
    w = wl.config5(0, device=DEV)
    fus_p, fus_d = run_both(w.prefill, w.decode, w.prefill.token_budget, w.decode.token_budget, out_dtype=torch.bfloat16)
    d = w.decode
    rng = np.random.default_rng(8)
    long_ = [int(i) for i in np.where(d.kv_lens > 16000)[0][::6]]
    reqs = sorted(set(long_) | set(int(i) for i in rng.choice(d.n, size=60, replace=False)))
    got = fus_d.float()[torch.as_tensor(reqs, device=DEV)].cpu().numpy()
    H.assert_close(got, H.oracle_paged_decode(d, False, reqs), 0, "cfg5 fused step: decode half")
