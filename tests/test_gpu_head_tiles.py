"""Query tiles of 32 or 64 rows whose workgroups take several heads of a KV head (even numbers of heads per KV head), and tiles of 128
rows and one head, of one request or of several (odd numbers), against the padded schedule, which has 128 rows, one head and one request to a tile
whatever the heads: a row's arithmetic does not depend on its tile, so the results are the same bits.  Rows and contexts around the edges of
tiles, lists around 64 and 128 entries (they are read 64 at a time), both bodies, four and eight waves, both outputs."""
import numpy as np
import pytest
import torch

from paper_2602_06072_amd import binding as pk
from paper_2602_06072_amd import workloads as wl
from tests import helpers as H

pytestmark = pytest.mark.gpu
DEV = "cuda"
EDGES = [1, 2, 31, 32, 33, 63, 64, 65, 96, 127, 128, 129, 160, 257]


def compare(ql, ctx, Hq, Hkv, d, what, light, out=torch.bfloat16, budget=1 << 14):
    ql = np.asarray(ql, dtype=np.int32)
    kv = ql + np.asarray(ctx, dtype=np.int32)
    w = wl.make_ragged(what, kv, ql, Hq, Hkv, d, budget, 77, device=DEV, keep_f32=False)
    plan = pk.pack_plan(w.kv_lens, w.q_lens, token_budget=budget)
    ws = pk.new_workspace(plan, Hq, Hkv, d, pk.PK_BF16)
    got = torch.full(w.q.shape, float("nan"), dtype=out, device=DEV)
    want = torch.full(w.q.shape, float("nan"), dtype=out, device=DEV)
    pk.packed_prefill_attn(plan, w.q, w.k, w.v, got, w.scale, ws)
    pk.padded_prefill_attn(plan, w.q, w.k, w.v, want, w.scale, ws)
    torch.cuda.synchronize()
    assert light is None or plan.stat(8) == light, what
    assert torch.isfinite(want).all() and torch.equal(got, want), what
    return plan


# heads per KV head: 1, 2, 3, 4, 5, 6, 8, 12, 16
@pytest.mark.parametrize("Hq, Hkv", [(2, 2), (4, 2), (3, 1), (8, 2), (5, 1), (6, 1), (16, 2), (12, 1), (16, 1)])
@pytest.mark.parametrize("d", [64, 128])
def test_edges_in_launches_of_little_work(d, Hq, Hkv):
    rng = np.random.default_rng(Hq)
    ctx = rng.permutation([0, 0, 1, 31, 32, 33, 63, 64, 65, 100, 127, 128, 129, 500])
    compare(EDGES, ctx, Hq, Hkv, d, f"edges {Hq}/{Hkv} d {d}", 1)
    # many requests of few rows: the tiles of 128 rows hold several
    ql = rng.integers(1, 70, 200)
    plan = compare(ql, rng.integers(0, 200, 200), Hq, Hkv, d, f"short ones {Hq}/{Hkv} d {d}", 1, torch.float32)
    assert Hq < 5 or plan.stat(6) < 200


# the same rows, more or fewer of them than a tile of 128 rows and head for every compute unit: with several heads to a workgroup, and without
@pytest.mark.parametrize("Hq, Hkv", [(4, 2), (4, 1), (8, 2), (6, 1), (16, 2)])
@pytest.mark.parametrize("reps", [1, 4])
@pytest.mark.parametrize("d", [64, 128])
def test_edges_on_both_sides_of_a_full_chip(d, reps, Hq, Hkv):
    ctx = np.arange(len(EDGES) * reps) * 37 % 200
    compare(EDGES * reps, ctx, Hq, Hkv, d, f"edges x {reps} {Hq}/{Hkv} d {d}", 1, torch.float32 if Hq == 6 else torch.bfloat16)


@pytest.mark.parametrize("Hq, Hkv", [(16, 16), (16, 8), (24, 8), (32, 8), (30, 5), (64, 8), (48, 4), (64, 4)])
@pytest.mark.parametrize("d", [64, 128])
def test_edges_in_launches_of_much_work(d, Hq, Hkv):
    ctx = [0, 63, 64, 65, 4000, 4031, 4032, 4033, 4095, 8063, 8064, 8130, 8191, 8256]
    reps = 2 if Hq >= 32 else 3
    compare(EDGES * reps, ctx * reps, Hq, Hkv, d, f"long lists {Hq}/{Hkv} d {d}", 0, torch.float32 if Hq == 32 else torch.bfloat16)


# Eight waves, for 2 x 128, 4 x 64 or 8 x 32 heads and rows (tiles of 64 rows of which the second half is empty among them): short lists in a batch that
# is long on average.
@pytest.mark.parametrize("Hq, Hkv, rows", [(8, 4, 128), (8, 2, 64), (12, 2, 128), (16, 2, 32)])
def test_edges_with_eight_waves(Hq, Hkv, rows):
    kv, ql = H.with_eight_waves([x + 63 * n for n, x in enumerate(EDGES)], EDGES, Hq, Hkv, 1 << 14, rows=128)
    plan = compare(ql, kv - ql, Hq, Hkv, 128, f"eight waves {Hq}/{Hkv}", 0)
    assert plan.stat(11) == 8 and plan.stat(12) == rows


@pytest.mark.parametrize("out", [torch.bfloat16, torch.float32])
def test_tiles_of_several_requests_with_eight_waves(out):
    """Two heads of 128 rows with six heads per KV head: the rows of a wave may be of two requests."""
    ql = np.random.default_rng(81).integers(1, 70, 30)
    kv, ql = H.with_eight_waves(ql + np.arange(30) * 37, ql, 12, 2, 1 << 18, rows=128)
    plan = compare(ql, kv - ql, 12, 2, 128, "eight waves, shared tiles", 0, out, 1 << 18)
    assert plan.stat(11) == 8 and plan.stat(12) == 128 and plan.stat(6) < len(ql) - 10


# Rounds of eight-wave workgroups that are full, and lists of some 190 key tiles: 256 (2 x 240 with six heads per KV head) such
# workgroups, 512 of four waves, of which two share a compute unit.  The mixed step works on the same tables with four waves.
@pytest.mark.parametrize("Hq, Hkv, n", [(64, 8, 8), (32, 8, 16), (32, 16, 16), (48, 8, 20)])
def test_long_lists_with_eight_waves(Hq, Hkv, n):
    ql = ([128, 127, 97, 113, 128, 98, 126, 100] * 3)[:n]
    ctx = [12000 + 64 * (x % 5) + x % 3 for x in range(n)]
    plan = compare(ql, ctx, Hq, Hkv, 128, f"eight waves, long lists {Hq}/{Hkv}", 0, torch.float32 if n == 8 else torch.bfloat16)
    assert plan.stat(11) == 8
    w = wl.make_ragged("long lists", np.asarray(ql, np.int32) + np.asarray(ctx, np.int32), np.asarray(ql, np.int32), Hq, Hkv, 128, 1 << 14, 78, device=DEV,
                       keep_f32=False)
    d = wl.small_paged(seed=79, n=3, lo=1, hi=100, Hq=Hq, Hkv=Hkv, d=128, token_budget=500, device=DEV, keep_f32=False)
    plan, plan_d = pk.pack_plan(w.kv_lens, w.q_lens, token_budget=1 << 14), pk.pack_plan(d.kv_lens, np.ones_like(d.kv_lens), None, None, 500)
    ws, ws_d = pk.new_workspace(plan, Hq, Hkv, 128, pk.PK_BF16), pk.new_workspace(plan_d, Hq, Hkv, 128, pk.PK_BF16)
    buf = pk.new_kv_buf(plan_d, Hkv, 128, pk.PK_BF16)
    pk.kv_reorganize(plan_d, d.k_pages, d.v_pages, torch.from_numpy(d.block_table).to(DEV), buf, ws_d)
    alone, fused = torch.full_like(w.q, float("nan")), torch.full_like(w.q, float("nan"))
    pk.packed_prefill_attn(plan, w.q, w.k, w.v, alone, w.scale, ws)
    pk.packed_mixed_step(plan, w.q, w.k, w.v, fused, ws, plan_d, d.q, buf, torch.empty_like(d.q), ws_d, w.scale)
    torch.cuda.synchronize()
    assert torch.isfinite(alone.float()).all() and torch.equal(alone, fused)
    rng = np.random.default_rng(80)
    req = rng.integers(0, n, size=100)
    rows = np.stack([req, rng.integers(0, Hq, size=100), rng.integers(0, w.q_lens[req])], axis=1).astype(np.int32)
    at = (np.concatenate([[0], np.cumsum(ql)])[rows[:, 0]] + rows[:, 2], rows[:, 1])
    H.assert_close(alone.float().cpu().numpy()[at], H.oracle_ragged(w, False, rows=rows), 0, f"eight waves, long lists {Hq}/{Hkv}")


@pytest.mark.parametrize("Hq, Hkv, d", [(8, 2, 128), (8, 2, 64), (4, 2, 128), (3, 1, 64)])
def test_tuned_pipeline_and_back(Hq, Hkv, d):
    """The register-staged kernel works on the same tables: the pipeline may change between two calls on a bound plan."""
    ql, kv = np.asarray([40, 300, 7, 64], np.int32), np.asarray([400, 300, 9, 129], np.int32)
    w = wl.make_ragged("tuned", kv, ql, Hq, Hkv, d, 1 << 14, 3, device=DEV, keep_f32=False)
    plan = pk.pack_plan(kv, ql, token_budget=1 << 14)
    ws = pk.new_workspace(plan, Hq, Hkv, d, pk.PK_BF16)
    outs = []
    for pipeline in (0, 1, 0):
        plan.tune(pk.TUNE_PREFILL_PIPELINE, pipeline)
        outs.append(torch.full_like(w.q, float("nan")))
        pk.packed_prefill_attn(plan, w.q, w.k, w.v, outs[-1], w.scale, ws)
    torch.cuda.synchronize()
    assert torch.equal(outs[0], outs[2])
    assert (outs[0].float() - outs[1].float()).abs().max() <= 4e-2      # (each within 2e-2 of the reference)
