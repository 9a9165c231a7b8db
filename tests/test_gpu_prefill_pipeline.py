"""The prefill pipeline where its parts begin and end: key lists of one to three tiles (prologue and last turn alone) and around
64 and 128 entries (the list is read 64 entries at a time), last tiles of which a wave sees one half only, tiles that rows of
other requests skip at the start and the end of the list; four and eight waves, both head
dimensions, and the same for launches of little work, which have a body of their own (`light`: what plan.stat(8) says)."""
import numpy as np
import pytest
import torch

from paper_2602_06072_amd import binding as pk
from paper_2602_06072_amd import workloads as wl
from tests import helpers as H

pytestmark = pytest.mark.gpu
DEV = "cuda"
TAILS = {"half": 1, "half_full": 32, "second_half": 33, "full": 64}     # keys of the last tile


def check(kv, ql, Hq, Hkv, d, what, light, rows=None, budget=1 << 16):
    w = wl.make_ragged(f"pipe_{what}", np.asarray(kv, np.int32), np.asarray(ql, np.int32), Hq, Hkv, d, budget, 31, device=DEV,
                       keep_f32=False)
    plan = pk.pack_plan(w.kv_lens, w.q_lens, token_budget=budget)
    ws = pk.new_workspace(plan, Hq, Hkv, d, pk.PK_BF16)
    out = torch.full(w.q.shape, float("nan"), dtype=torch.float32, device=DEV)
    pk.packed_prefill_attn(plan, w.q, w.k, w.v, out, w.scale, ws)
    torch.cuda.synchronize()
    assert plan.stat(8) == light, what
    got = out.cpu().numpy()
    if rows is None:
        H.assert_close(got, H.oracle_ragged(w, False), 0, what)
    else:                                           # as many rows as that, any request
        rng = np.random.default_rng(32)
        start = np.concatenate([[0], np.cumsum(w.q_lens)])
        assert np.all(np.isfinite(got))
        req = rng.integers(0, w.n, size=rows)
        r = np.stack([req, rng.integers(0, Hq, size=rows), rng.integers(0, np.asarray(w.q_lens)[req])], axis=1).astype(np.int32)
        H.assert_close(got[start[r[:, 0]] + r[:, 2], r[:, 1]], H.oracle_ragged(w, False, rows=r), 0, what)
    return plan


@pytest.mark.parametrize("tail", TAILS)
@pytest.mark.parametrize("tiles", [1, 2, 3, 4, 63, 64, 65, 66, 127, 128, 129])
@pytest.mark.parametrize("d", [64, 128])
def test_key_lists(d, tiles, tail):
    kv = 64 * (tiles - 1) + TAILS[tail]
    ql = [min(kv, 3 * n + 1) for n in range(7)]
    check([kv], [min(kv, 37)], 2, 1, d, f"{tiles} tiles, {tail}, d {d}", 1)
    plan = check([kv] * 7, ql, 64, 8, d, f"{tiles} tiles, {tail}, d {d}, a full chip", int(tiles <= 4))
    assert plan.stat(6) == 7                        # a tile for every request
    if tiles <= 4:                                  # lists as short in a launch of much work
        plan = check(*H.with_long_requests([kv] * 7, ql), 32, 8, d, f"{tiles} tiles, {tail}, d {d}, with long ones", 0)
        assert plan.stat(6) == 7 + H.LONG


@pytest.mark.parametrize("d", [64, 128])
def test_tiles_of_several_requests(d):
    """Enough tiles that requests share them: a wave skips the key tiles of the requests that it holds no rows of."""
    six = [700, 64, 65, 1300, 33, 31], [30, 2, 33, 31, 31, 1]
    check(six[0] * 6, six[1] * 6, 16, 8, d, f"shared tiles of six, d {d}", 1)
    plan = check(six[0] * 20, six[1] * 20, 64, 8, d, f"shared tiles of six, d {d}, much work", 0, rows=2000)
    assert plan.stat(6) < 60
    n = 90
    ql = np.random.default_rng(5).integers(1, 60, n)
    check(ql + np.arange(n) * 7, ql, 16, 8, d, f"shared tiles, d {d}", 1)
    n = 130
    ql = np.random.default_rng(5).integers(1, 60, n)
    plan = check(ql + np.arange(n) * 7, ql, 48, 16, d, f"shared tiles, d {d}, much work", 0, rows=2000)
    assert plan.stat(6) < 60


@pytest.mark.parametrize("tail", TAILS)
def test_eight_waves(tail):
    """Lists of one to four tiles and around 64 and 128 entries, in a batch that is long on average."""
    kv = np.asarray([64 * t + TAILS[tail] for t in (0, 1, 2, 3, 30, 62, 63, 64, 65, 126, 127, 128)], dtype=np.int32)
    ql = np.minimum(kv, [1, 31, 32, 33, 64, 96, 127, 128, 17, 65, 97, 40])
    kv, ql = H.with_eight_waves(kv, ql, 16, 2, 1 << 14)
    plan = check(kv, ql, 16, 2, 128, f"eight waves, {tail}", 0, budget=1 << 14)
    assert plan.stat(11) == 8
