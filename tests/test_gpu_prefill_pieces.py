"""Prefill launches of few workgroups whose key-tile lists are cut into pieces, and the launch that puts the pieces together, against the oracle: all kinds of query
tiles, lists that end inside a piece for some waves, whole lists beside cut ones, a workspace full of NaNs, captured and in the mixed step."""
import numpy as np
import pytest
import torch

from paper_2602_06072_amd import binding as pk
from paper_2602_06072_amd import workloads as wl
from tests import helpers as H

pytestmark = pytest.mark.gpu
DEV = "cuda"
SHAPES = {
    "few rows": ([64], [8000]),
    "edges": ([1, 31, 33, 65, 128], [2000, 900, 63, 64 * 40 - 1, 5000]),
    "causal": ([1400, 97], [0, 0]),
    "straggler": ([20] * 12 + [5], [3] * 12 + [9000]),
    "counters": ([200], [16500]),                  # more than 255 key tiles: what a wave skips does not fit its counter
}


def ready(w, fill=None):
    plan = pk.pack_plan(w.kv_lens, w.q_lens, token_budget=w.token_budget)
    ws = pk.new_workspace(plan, w.Hq, w.Hkv, w.d, pk.PK_BF16)
    if fill is not None:
        ws.fill_(fill)
    pk.plan_bind(plan, w.Hq, w.Hkv, w.d, pk.PK_BF16, ws)
    return plan, ws


def batch(shape, heads, seed):
    ql, ctx = (np.asarray(x, dtype=np.int32) for x in SHAPES[shape])
    return wl.make_ragged(shape, ql + ctx, ql, *heads, 16384, seed, device=DEV, keep_f32=False)


@pytest.mark.parametrize("shape", list(SHAPES))
@pytest.mark.parametrize("heads", [(8, 8, 128), (4, 1, 128), (8, 2, 64), (12, 2, 128), (5, 1, 64), (6, 2, 128), (4, 2, 64)])
def test_pieces_against_the_oracle(heads, shape):
    w = batch(shape, heads, 91)
    plan, ws = ready(w, 255)                       # (whatever was in the workspace)
    assert plan.stat(13) > plan.stat(6) and plan.stat(8) == 1
    rng = np.random.default_rng(92)
    req = rng.integers(0, w.n, size=150)
    rows = np.stack([req, rng.integers(0, w.Hq, size=150), rng.integers(0, w.q_lens[req])], axis=1).astype(np.int32)
    at = (np.concatenate([[0], np.cumsum(w.q_lens)])[rows[:, 0]] + rows[:, 2], rows[:, 1])
    want = H.oracle_ragged(w, False, rows=rows)
    outs = {}
    for dtype in (torch.float32, torch.bfloat16):
        outs[dtype] = torch.full(w.q.shape, float("nan"), dtype=dtype, device=DEV)
        pk.packed_prefill_attn(plan, w.q, w.k, w.v, outs[dtype], w.scale, ws)
        torch.cuda.synchronize()
        assert torch.isfinite(outs[dtype]).all()
        H.assert_close(outs[dtype].float().cpu().numpy()[at], want, 0, f"{shape} {heads} {dtype}")
    assert torch.equal(outs[torch.float32].to(torch.bfloat16), outs[torch.bfloat16])


@pytest.mark.parametrize("heads", [(8, 8, 128), (8, 2, 64), (12, 2, 128)])
def test_nonfinite_values_reach_only_the_rows_that_see_them(heads):
    w = batch("edges", heads, 93)
    plan, ws = ready(w)

    def run():
        out = torch.full(w.q.shape, 7.0, dtype=torch.float32, device=DEV)
        pk.packed_prefill_attn(plan, w.q, w.k, w.v, out, w.scale, ws)
        torch.cuda.synchronize()
        return out
    clean = run()
    q0, k0 = np.concatenate([[0], np.cumsum(w.q_lens)]), np.concatenate([[0], np.cumsum(w.kv_lens)])
    sees = torch.zeros(w.q.shape[:2], dtype=torch.bool, device=DEV)
    w.q[int(q0[1]) + 7, 0, 5] = float("nan")
    sees[int(q0[1]) + 7, 0] = True
    w.k[int(k0[3]) + 64 * 40 - 1 + 40, 0, 3] = float("nan")            # in the last piece, seen by the rows from 40 on
    sees[int(q0[3]) + 40: int(q0[4]), : w.Hq // w.Hkv] = True
    got = run()
    assert torch.isnan(got[sees]).all() and torch.isfinite(got[~sees]).all()
    H.assert_close(got[~sees].cpu().numpy(), clean[~sees].cpu().numpy(), 0, f"beside a NaN {heads}")
    assert torch.equal(got[: int(q0[1])], clean[: int(q0[1])]) and torch.equal(got[int(q0[4]):], clean[int(q0[4]):])


@pytest.mark.parametrize("heads", [(8, 8, 128), (8, 2, 64), (12, 2, 128)])
@pytest.mark.parametrize("ctx", [1500, 2000, 3000, 8000])
def test_infinite_values_stay_infinite(heads, ctx):
    """An infinite value among those that every row sees, in the last piece or in the first: every row of its KV head and column is infinite, as in whole lists."""
    ql = np.asarray([64], dtype=np.int32)
    w = wl.make_ragged("infinite", ql + ctx, ql, *heads, 16384, 97, device=DEV, keep_f32=False)
    w.v[ctx - 10, 0, 3] = float("inf")
    w.v[20, w.Hkv - 1, 40] = float("-inf")
    plan, ws = ready(w)
    assert plan.stat(13) > 1
    r = w.Hq // w.Hkv
    for pipeline in (0, 1):                        # (1: whole lists)
        plan.tune(pk.TUNE_PREFILL_PIPELINE, pipeline)
        out = torch.full(w.q.shape, float("nan"), dtype=torch.float32, device=DEV)
        pk.packed_prefill_attn(plan, w.q, w.k, w.v, out, w.scale, ws)
        torch.cuda.synchronize()
        assert (out[:, :r, 3] == float("inf")).all() and (out[:, -r:, 40] == float("-inf")).all(), (pipeline, plan.stat(13))
        out[:, :r, 3] = out[:, -r:, 40] = 0
        assert torch.isfinite(out).all()


@pytest.mark.parametrize("heads", [(8, 2, 128), (8, 2, 64)])
def test_pieces_in_the_mixed_step_and_in_a_graph(heads):
    """The same bits in every launch; two plans take turns on the tables and partial results of a workspace each."""
    w = batch("straggler", heads, 94)
    dec = wl.small_paged(seed=95, n=5, lo=1, hi=3000, Hq=w.Hq, Hkv=w.Hkv, d=w.d, token_budget=500, device=DEV, keep_f32=False)
    dplan = pk.pack_plan(dec.kv_lens, np.ones_like(dec.kv_lens), None, None, 500)
    dws = pk.new_workspace(dplan, w.Hq, w.Hkv, w.d, pk.PK_BF16)
    buf = pk.new_kv_buf(dplan, w.Hkv, w.d, pk.PK_BF16)
    pk.kv_reorganize(dplan, dec.k_pages, dec.v_pages, torch.from_numpy(dec.block_table).to(DEV), buf, dws)
    plan, ws = ready(w)
    assert plan.stat(13) > 0
    alone, fused, captured = (torch.full_like(w.q, float("nan")) for _ in range(3))
    d_alone, d_fused = torch.empty_like(dec.q), torch.empty_like(dec.q)
    pk.packed_prefill_attn(plan, w.q, w.k, w.v, alone, w.scale, ws)
    pk.packed_decode_attn(dplan, dec.q, buf, d_alone, dec.scale, w.Hkv, dws)
    pk.packed_mixed_step(plan, w.q, w.k, w.v, fused, ws, dplan, dec.q, buf, d_fused, dws, w.scale)
    torch.cuda.synchronize()
    assert torch.isfinite(alone.float()).all() and torch.equal(alone, fused) and torch.equal(d_alone, d_fused)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        pk.packed_prefill_attn(plan, w.q, w.k, w.v, captured, w.scale, ws)
    for rep in range(3):
        captured.fill_(float("nan"))
        pk.packed_mixed_step(plan, w.q, w.k, w.v, fused, ws, dplan, dec.q, buf, d_fused, dws, w.scale)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(captured, alone), f"replay {rep}"


def test_tuned_pipeline_takes_whole_lists():
    w = batch("edges", (8, 2, 128), 96)
    plan, ws = ready(w)
    outs = []
    for pipeline in (0, 1, 0):
        plan.tune(pk.TUNE_PREFILL_PIPELINE, pipeline)
        outs.append(torch.full_like(w.q, float("nan")))
        pk.packed_prefill_attn(plan, w.q, w.k, w.v, outs[-1], w.scale, ws)
    torch.cuda.synchronize()
    assert torch.equal(outs[0], outs[2])
    assert (outs[0].float() - outs[1].float()).abs().max() <= 4e-2     # (each within 2e-2 of the reference)


@pytest.mark.parametrize("heads", [(8, 8, 128), (8, 2, 64), (12, 2, 128)])
def test_references_near_and_far_from_zero_meet(heads):
    """Pieces whose scores are some octaves beside pieces whose scores are so large that their reference is a score, with either the greater, and pieces that all lie far below
    zero.  The best key of a row is alone or has equals, bit for bit, and leads the others by far more than any rounding."""
    w = batch("edges", heads, 98)
    assert ready(w)[0].stat(13) > 0
    q0, k0 = np.concatenate([[0], np.cumsum(w.q_lens)]), np.concatenate([[0], np.cumsum(w.kv_lens)])
    for i in range(w.n):
        q, k, ctx = w.q[int(q0[i]): int(q0[i + 1])], w.k[int(k0[i]): int(k0[i + 1])], int(w.kv_lens[i] - w.q_lens[i])
        if i == 4:                                 # 32 factors, repeated, all below zero
            q.fill_(1e16)
            k.copy_((-1e15 * (2.0 - (torch.arange(k.shape[0], device=DEV) * 7 % 32).float() / 32)).view(-1, 1, 1).expand(k.shape))
            continue
        q.copy_(q.abs() * 1e3)
        k.zero_()                                  # a score of zero, but for a few keys spread over the context: above (one after the other the best) or below
        for j, pos in enumerate(np.linspace(0, ctx - 1, 9).astype(int)):
            k[int(pos)] = (1e6 if i % 2 else -1e6) * 2.0 ** (j if i == 1 else 9 - j)
    plan, ws = ready(w, 255)
    out = torch.full(w.q.shape, float("nan"), dtype=torch.float32, device=DEV)
    pk.packed_prefill_attn(plan, w.q, w.k, w.v, out, w.scale, ws)
    torch.cuda.synchronize()
    H.assert_close(out.cpu().numpy(), H.oracle_ragged(w, False), 0, f"near and far {heads}")


@pytest.mark.parametrize("heads", [(8, 8, 128), (8, 8, 64)])
def test_whole_lists_beside_a_decode_half_that_outlasts_them(heads):
    """The mixed step's prefill half is that of whole lists (which the padded call has) beside long decode work, and in pieces beside short; the decode half is the decode call's."""
    Hq, Hkv, d = heads
    ql, ctx = np.asarray([64], dtype=np.int32), np.asarray([2000], dtype=np.int32)
    w = wl.make_ragged("chunk", ql + ctx, ql, *heads, 16384, 99, device=DEV, keep_f32=False)
    plan, ws = ready(w)
    assert plan.stat(13) > 1
    pieces, whole = (torch.full(w.q.shape, float("nan"), dtype=torch.float32, device=DEV) for _ in range(2))
    pk.packed_prefill_attn(plan, w.q, w.k, w.v, pieces, w.scale, ws)
    pk.padded_prefill_attn(plan, w.q, w.k, w.v, whole, w.scale, ws)
    want = H.oracle_ragged(w, False)
    torch.cuda.synchronize()
    assert not torch.equal(pieces, whole)
    for n, lo, hi, expected in ((3, 50, 400, pieces), (40, 3500 * 128 // d, 4500 * 128 // d, whole)):
        dec = wl.small_paged(seed=100, n=n, lo=lo, hi=hi, Hq=Hq, Hkv=Hkv, d=d, token_budget=8192, device=DEV, keep_f32=False)
        dplan = pk.pack_plan(dec.kv_lens, np.ones_like(dec.kv_lens), None, None, 8192)
        dws = pk.new_workspace(dplan, Hq, Hkv, d, pk.PK_BF16)
        buf = pk.new_kv_buf(dplan, Hkv, d, pk.PK_BF16)
        pk.kv_reorganize(dplan, dec.k_pages, dec.v_pages, torch.from_numpy(dec.block_table).to(DEV), buf, dws)
        out = torch.full(w.q.shape, float("nan"), dtype=torch.float32, device=DEV)
        d_alone, d_fused = (torch.full(dec.q.shape, float("nan"), dtype=torch.float32, device=DEV) for _ in range(2))
        pk.packed_decode_attn(dplan, dec.q, buf, d_alone, dec.scale, Hkv, dws)
        pk.packed_mixed_step(plan, w.q, w.k, w.v, out, ws, dplan, dec.q, buf, d_fused, dws, w.scale)
        torch.cuda.synchronize()
        assert torch.equal(out, expected) and torch.equal(d_fused, d_alone), n
        H.assert_close(out.cpu().numpy(), want, 0, f"beside {n} decode rows {heads}")
