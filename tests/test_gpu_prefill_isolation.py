"""Query rows that share a wave, a tile or a launch must not see each other's values: a NaN or an infinity in one
row of Q or K reaches the rows that attend to it and no other.  Rows next to it may take another path through the
online softmax (the wave as a whole re-does a half tile), so they are compared within the usual tolerance of two bf16
kernels; rows of other waves are compared bit for bit."""
import numpy as np
import pytest
import torch

from paper_2602_06072_amd import binding as pk
from paper_2602_06072_amd import workloads as wl
from tests import helpers as H

pytestmark = pytest.mark.gpu
DEV = "cuda"


def prefill(w, padded=False, out_dtype=torch.float32):
    plan = pk.pack_plan(w.kv_lens, w.q_lens, token_budget=w.token_budget)
    ws = pk.new_workspace(plan, w.Hq, w.Hkv, w.d, pk.PK_BF16)
    out = torch.full(w.q.shape, 7.0, dtype=out_dtype, device=DEV)
    (pk.padded_prefill_attn if padded else pk.packed_prefill_attn)(plan, w.q, w.k, w.v, out, w.scale, ws)
    torch.cuda.synchronize()
    return out, plan


@pytest.mark.parametrize("light", [1, 0])
@pytest.mark.parametrize("d", [128, 64])
def test_lanes_without_a_query_hold_nobody_elses_row(d, light):
    """Partly filled waves with unmasked key tiles; the first query row of the batch holds a NaN.  Tiles are not
    shared here, so every row behind the first wave of request 0 is in another wave than that row."""
    ql = np.asarray([200, 17, 45, 100, 9], dtype=np.int32)
    kv = ql + np.asarray([0, 500, 300, 130, 700], dtype=np.int32)
    if not light:
        kv, ql = H.with_long_requests(kv, ql)
    w = wl.make_ragged("padding", kv, ql, 4 if light else 32, 2, d, 1024, 21, DEV, keep_f32=False)
    clean = {p: prefill(w, p)[0] for p in (False, True)}
    w.q[0] = float("nan")
    for padded in (False, True):
        got, plan = prefill(w, padded)
        assert plan.stat(6) == len(ql) + 1                 # one tile a request, two for the first: nothing shared
        assert plan.stat(8) == light and (not padded or plan.stat(9) == light)
        assert torch.equal(got[32:], clean[padded][32:])
        assert torch.isnan(got[0]).all()


BAD = {"q_first": ("q", 0, float("nan")), "q_middle": ("q", 77, float("nan")), "q_inf": ("q", 41, float("inf")),
       "k_nan": ("k", 25, float("nan")), "k_inf": ("k", 60, float("inf")), "k_first": ("k", 0, float("nan"))}


@pytest.mark.parametrize("case", list(BAD))
@pytest.mark.parametrize("heads", [(4, 2, 128), (4, 2, 64), (16, 2, 128), (12, 2, 128), (12, 4, 128), (16, 2, 64)])
@pytest.mark.parametrize("launch", ["packed", "padded", "mixed"])
def test_nonfinite_values_reach_only_the_rows_that_see_them(launch, heads, case):
    """Both bodies and head dimensions, several heads of a request to a workgroup and (three heads per KV head, and six with eight waves) tiles
    of several requests; eight waves with 16/2 and 12/2 heads.  A NaN makes exactly the rows that see it NaN; what a row that sees an infinity gives is not asked."""
    Hq, Hkv, d = heads
    waves = 8 if heads in ((16, 2, 128), (12, 2, 128)) else 4
    n, budget = (150, 8192) if waves == 4 else (40, 8192) if Hq == 16 else (30, 1 << 18)
    rng = np.random.default_rng(51)
    ql = rng.integers(5, 61, size=n).astype(np.int32)
    ctx = rng.integers(600, 901, size=n) if Hq > 4 else rng.integers(0, 300, size=n)
    kv = (ql + ctx).astype(np.int32)
    if waves == 8:
        kv, ql = H.with_eight_waves(kv, ql, Hq, Hkv, budget, rows=1 if Hq == 16 else 128)
    w = wl.make_ragged("isolation", kv, ql, Hq, Hkv, d, budget, 52, DEV, keep_f32=False)
    dec = wl.small_paged(seed=53, n=4, lo=1, hi=90, Hq=Hq, Hkv=Hkv, d=d, token_budget=500, device=DEV, keep_f32=False)
    dplan = pk.pack_plan(dec.kv_lens, np.ones_like(dec.kv_lens), None, None, 500)
    dws = pk.new_workspace(dplan, Hq, Hkv, d, pk.PK_BF16)
    buf = pk.new_kv_buf(dplan, Hkv, d, pk.PK_BF16)
    pk.kv_reorganize(dplan, dec.k_pages, dec.v_pages, torch.from_numpy(dec.block_table).to(DEV), buf, dws)

    def run(out_dtype):
        if launch != "mixed":
            return prefill(w, launch == "padded", out_dtype)[0]
        plan = pk.pack_plan(w.kv_lens, w.q_lens, token_budget=w.token_budget)
        ws = pk.new_workspace(plan, Hq, Hkv, d, pk.PK_BF16)
        out = torch.full(w.q.shape, 7.0, dtype=out_dtype, device=DEV)
        pk.packed_mixed_step(plan, w.q, w.k, w.v, out, ws, dplan, dec.q, buf, torch.empty_like(dec.q, dtype=out_dtype), dws, w.scale)
        torch.cuda.synchronize()
        return out

    plan = prefill(w)[1]
    assert plan.stat(11) == waves and (plan.stat(12) < 128 or plan.stat(6) < len(ql))     # tiles of 128 rows: shared by requests
    assert plan.stat(12) == {1: 32, 2: 64, 3: 128, 6: 128, 8: 32}[Hq // Hkv]
    # (of the padded schedule, whose lists are not shared, both kinds are light with one head per workgroup)
    assert plan.stat(8) == int(Hq == 4)
    clean = {t: run(t).float() for t in (torch.float32, torch.bfloat16)}
    which, req, value = BAD[case]
    req %= n
    q0 = int(w.q_lens[:req].sum())
    sees = torch.zeros(w.q.shape[:2], dtype=torch.bool, device=DEV)
    if which == "q":
        row = q0 + int(ql[req]) // 2 if req else 0
        heads_hit = slice(None) if req == 0 else slice(1, 2)
        w.q[row, heads_hit, 5] = value
        sees[row, heads_hit] = True
    else:                                                  # a key half way through the request's own queries
        t = int(ql[req]) // 2
        w.k[int(w.kv_start[req]) + int(ctx[req]) + t, Hkv - 1, 3] = value
        sees[q0 + t: q0 + int(ql[req]), (Hkv - 1) * (Hq // Hkv):] = True
    for out_dtype, want in clean.items():
        got = run(out_dtype).float()
        H.assert_close(got[~sees].cpu().numpy(), want[~sees].cpu().numpy(), 0, f"{case} {launch} {heads}")
        if np.isnan(value):
            assert torch.isnan(got[sees]).all()
