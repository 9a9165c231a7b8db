"""GPU parity where the online softmax is stressed rather than the schedule: score maxima that keep
growing along the keys, a dominant key late or first in a request, scores far below zero, scores of
large magnitude.  The prefill kernels take their exponentials against a reference that moves only
when it must and re-do a half tile when it does; these inputs make it move at every tile, by a lot,
or never.  Same oracle, same tolerances as everywhere else."""
import numpy as np
import pytest
import torch

from paper_2602_06072_amd import binding as pk
from paper_2602_06072_amd import workloads as wl
from tests import helpers as H

pytestmark = pytest.mark.gpu
DEV = "cuda"


def shape_scores(q, k, kv_start, kv_lens, case, rng):
    """Rewrites q and k (bf16 tensors on the device, token-major) in place."""
    if case == "ramp":                 # key norms grow along every request: the row maximum rises tile after tile
        for s, L in zip(kv_start, kv_lens):
            f = torch.linspace(0.2, 6.0, int(L), device=k.device).view(-1, 1, 1)
            k[s:s + L] = (k[s:s + L].float() * f).to(k.dtype)
    elif case == "falling":            # ... or falls: the first tile sets a reference that is never raised again
        for s, L in zip(kv_start, kv_lens):
            f = torch.linspace(6.0, 0.05, int(L), device=k.device).view(-1, 1, 1)
            k[s:s + L] = (k[s:s + L].float() * f).to(k.dtype)
    elif case in ("late_outlier", "first_outlier"):
        q.copy_(q.abs())               # every score against an all-positive key is large and positive
        for s, L in zip(kv_start, kv_lens):
            pos = s + (int(L) - 1 - int(rng.integers(0, min(int(L), 40))) if case == "late_outlier" else 0)
            k[pos] = 2.0
    elif case == "far_below_zero":     # all scores around -100 nats: the reference starts far from zero
        q.copy_(q.abs())
        k.copy_(-(k.abs()) * 1.5)
    elif case == "jumps":              # a few keys per request, spread out, each larger than everything before it
        q.copy_(q.abs())
        for s, L in zip(kv_start, kv_lens):
            n_j = max(1, int(L) // 90)
            for j, pos in enumerate(sorted(rng.choice(int(L), size=n_j, replace=False))):
                k[s + int(pos)] = 0.25 * (j + 1)
    else:
        raise ValueError(case)


CASES = ["ramp", "falling", "late_outlier", "first_outlier", "far_below_zero", "jumps"]


@pytest.fixture
def sized(request):
    """(kv, ql) -> a batch for one of the prefill bodies (the pipeline with four waves to a workgroup or, with D = 128, eight) with its
    heads; `.light` and `.waves`: what plan.stat(8) and plan.stat(11) say of it."""
    def batch(kv, ql):
        if batch.light:
            return np.asarray(kv, dtype=np.int32), np.asarray(ql, dtype=np.int32), 4, 2
        return (*H.with_long_requests(kv, ql), 33, 3) if batch.waves == 4 else (*H.with_eight_waves(kv, ql, 16, 2, 1024), 16, 2)
    batch.light = int(request.param == "light")
    batch.waves = 8 if request.param == "eight_waves" else 4
    return batch


BODIES = pytest.mark.parametrize("d, sized", [(128, "light"), (128, "four_waves"), (128, "eight_waves"), (64, "light"), (64, "four_waves")],
                                 indirect=["sized"])


@BODIES
@pytest.mark.parametrize("case", CASES)
def test_prefill_softmax_extremes(case, d, sized):
    rng = np.random.default_rng(100 * CASES.index(case) + d)
    kv, ql, Hq, Hkv = sized([700 + 333, 300, 129, 64, 1500], [700, 300, 129, 64, 1500])
    w = wl.make_ragged(f"extreme_{case}", kv, ql, Hq, Hkv, d, 1024, 5, DEV, keep_f32=False)
    shape_scores(w.q, w.k, w.kv_start, w.kv_lens, case, rng)
    want = H.oracle_ragged(w, False)
    for padded, pipeline in ((False, 0), (True, 0), (False, 1)):
        plan = pk.pack_plan(w.kv_lens, w.q_lens, token_budget=w.token_budget)
        plan.tune(pk.TUNE_PREFILL_PIPELINE, pipeline)
        ws = pk.new_workspace(plan, w.Hq, w.Hkv, w.d, pk.PK_BF16)
        out = torch.full(w.q.shape, float("nan"), dtype=torch.float32, device=DEV)
        (pk.padded_prefill_attn if padded else pk.packed_prefill_attn)(plan, w.q, w.k, w.v, out, w.scale, ws)
        torch.cuda.synchronize()
        assert plan.stat(9 if padded else 8) == sized.light and plan.stat(11) == sized.waves
        H.assert_close(out.cpu().numpy(), want, 0, f"prefill {case} d={d} padded={padded} pipeline={pipeline}")


@pytest.mark.parametrize("case", CASES)
def test_decode_softmax_extremes(case):
    rng = np.random.default_rng(100 * CASES.index(case) + 7)
    plen = np.asarray([608] * 6 + [0] * 4, dtype=np.int32)     # whole pages: the family shares all of them physically
    pid = np.asarray([0] * 6 + [-1] * 4, dtype=np.int32)
    kv = (plen + np.asarray([5, 40, 260, 1, 33, 700, 3000, 64, 31, 129])).astype(np.int32)
    w = wl.make_paged(f"extreme_dec_{case}", kv, 8, 2, 128, 2048, 16, 3, prefix_ids=pid, prefix_lens=plen,
                      device=DEV, keep_f32=False)
    # the pages are rewritten in place through the block table; a family's prefix pages are the same
    # physical pages for every member, so whatever is written there is seen by all of them
    tok_k = []
    for i in range(w.n):
        L = int(kv[i])
        blocks = torch.from_numpy(w.block_table[i, :(L + 15) // 16].astype(np.int64)).to(DEV)
        tok_k.append((blocks, L))
    q = w.q
    flat_k = w.k_pages.view(-1, w.Hkv, w.d)                # [pages * 16, Hkv, d]
    if case in ("ramp", "falling"):
        f_all = torch.linspace(0.3, 5.0, flat_k.shape[0], device=DEV).view(-1, 1, 1)
        if case == "falling":
            f_all = f_all.flip(0)
        flat_k.copy_((flat_k.float() * f_all).to(flat_k.dtype))
    elif case == "far_below_zero":
        q.copy_(q.abs()); flat_k.copy_(-(flat_k.abs()) * 1.5)
    else:
        q.copy_(q.abs())
        for i, (blocks, L) in enumerate(tok_k):
            own = L - int(plen[i])                         # tokens of the request's own suffix
            if case == "first_outlier":
                t = 0
            elif case == "late_outlier":
                t = L - 1 - int(rng.integers(0, min(own, 20)))
            else:
                t = int(plen[i]) + int(rng.integers(0, own))
            flat_k[int(blocks[t // 16]) * 16 + t % 16] = 2.0 if case != "jumps" else 0.5
    ones = np.ones(w.n, dtype=np.int32)
    plan = pk.pack_plan(w.kv_lens, ones, w.prefix_ids, w.prefix_lens, w.token_budget, 0)
    ws = pk.new_workspace(plan, w.Hq, w.Hkv, w.d, pk.PK_BF16)
    buf = pk.new_kv_buf(plan, w.Hkv, w.d, pk.PK_BF16)
    bt = torch.from_numpy(w.block_table).to(DEV)
    pk.kv_reorganize(plan, w.k_pages, w.v_pages, bt, buf, ws)
    out = torch.full(w.q.shape, float("nan"), dtype=torch.float32, device=DEV)
    pk.packed_decode_attn(plan, w.q, buf, out, w.scale, w.Hkv, ws)
    torch.cuda.synchronize()
    want = H.oracle_paged_decode(w, False)
    H.assert_close(out.cpu().numpy(), want, 0, f"decode {case}")
    out2 = torch.full(w.q.shape, float("nan"), dtype=torch.float32, device=DEV)
    pk.padded_decode_attn(plan, w.q, w.k_pages, w.v_pages, bt, out2, w.scale, ws)
    torch.cuda.synchronize()
    H.assert_close(out2.cpu().numpy(), want, 0, f"padded decode {case}")


@BODIES
def test_prefill_scores_beyond_the_exponent_range(d, sized):
    """Row maxima that jump by more than 127 octaves inside a request (a probability against the old
    reference overflows to infinity in bf16 and fp32) and rows all of whose scores lie thousands of
    nats below zero.  Rows are one-hot or nearly: an error of a score of magnitude S is at most
    S * d * 2^-24 (fp32 sums of exact products), 2e-2 for the largest here, and only keys of equal
    score share a row, so the usual tolerance holds."""
    kv, ql, Hq, Hkv = sized([513, 200, 97, 1000], [513, 200, 97, 1000])
    w = wl.make_ragged("exponent_range", kv, ql, Hq, Hkv, d, 1024, 9, DEV, keep_f32=False)
    w.q.copy_(w.q.abs())
    s0 = w.kv_start
    for pos, value in ((0, -4.0), (40, 12.0), (64, 30.0), (130, 60.0), (131, -60.0), (300, 100.0)):
        w.k[int(s0[0]) + pos] = value
        w.k[int(s0[3]) + pos + 500] = value
    w.k[int(s0[1]):int(s0[2])] = -(w.k[int(s0[1]):int(s0[2])].abs() + 20.0)
    want = H.oracle_ragged(w, False)
    plan = pk.pack_plan(w.kv_lens, w.q_lens, token_budget=w.token_budget)
    ws = pk.new_workspace(plan, w.Hq, w.Hkv, w.d, pk.PK_BF16)
    out = torch.full(w.q.shape, float("nan"), dtype=torch.float32, device=DEV)
    pk.packed_prefill_attn(plan, w.q, w.k, w.v, out, w.scale, ws)
    torch.cuda.synchronize()
    assert plan.stat(8) == sized.light and plan.stat(11) == sized.waves
    got = out.cpu().numpy()
    lo, hi = int(s0[1]), int(s0[2])                        # scores around -2000 nats there: checked loosely below
    keep = np.r_[0:lo, hi:got.shape[0]]
    H.assert_close(got[keep], want[keep], 0, f"exponent range d={d}")
    # bf16 keys of magnitude 20..23 step by 2^-3: many keys share a row; the score error above (|score| up to
    # 3000 nats: 3000 * 128 * 2^-24 = 2.3e-2) moves a probability by that fraction and an output of |v| <= 5 by 5 times it
    assert np.abs(got[lo:hi] - want[lo:hi]).max() <= 2e-2 + 5 * 2.3e-2


def check_prefill_launches(w, want, keep, what, light):
    """Packed and padded prefill and the prefill half of the fused step against `want`, on the rows `keep`."""
    dec = wl.small_paged(seed=3, n=3, lo=1, hi=90, Hq=w.Hq, Hkv=w.Hkv, d=w.d, token_budget=500, device=DEV, keep_f32=False)
    dplan = pk.pack_plan(dec.kv_lens, np.ones_like(dec.kv_lens), None, None, 500)
    dws = pk.new_workspace(dplan, w.Hq, w.Hkv, w.d, pk.PK_BF16)
    buf = pk.new_kv_buf(dplan, w.Hkv, w.d, pk.PK_BF16)
    pk.kv_reorganize(dplan, dec.k_pages, dec.v_pages, torch.from_numpy(dec.block_table).to(DEV), buf, dws)
    plan = pk.pack_plan(w.kv_lens, w.q_lens, token_budget=w.token_budget)
    ws = pk.new_workspace(plan, w.Hq, w.Hkv, w.d, pk.PK_BF16)
    for launch in ("packed", "padded", "mixed"):
        out = torch.full(w.q.shape, float("nan"), dtype=torch.float32, device=DEV)
        if launch == "mixed":
            dout = torch.full(dec.q.shape, float("nan"), dtype=torch.float32, device=DEV)
            pk.packed_mixed_step(plan, w.q, w.k, w.v, out, ws, dplan, dec.q, buf, dout, dws, w.scale)
        else:
            (pk.padded_prefill_attn if launch == "padded" else pk.packed_prefill_attn)(plan, w.q, w.k, w.v, out, w.scale, ws)
        torch.cuda.synchronize()
        H.assert_close(out.cpu().numpy()[keep], want[keep], 0, f"{what} {launch}")
    assert plan.stat(8) == light and plan.stat(9) == light
    return plan


@BODIES
def test_prefill_rows_with_every_score_far_below_zero(d, sized):
    """Scaled scores around -1e31 .. -1e33.  A row's keys repeat 32 factors a 32nd apart: the nearest to zero that it
    sees stand alone against the rest by far more than any rounding, and equal keys have equal scores."""
    kv, ql, Hq, Hkv = sized([200, 100, 33, 400], [200, 60, 33, 150])
    w = wl.make_ragged("far_below", kv, ql, Hq, Hkv, d, 1024, 31, DEV, keep_f32=False)
    w.q.fill_(1e16)
    f = 2.0 - (torch.arange(w.k.shape[0], device=DEV) * 7 % 32).float() / 32
    w.k.copy_((-1e15 * f.view(-1, 1, 1)).expand(w.k.shape))
    plan = check_prefill_launches(w, H.oracle_ragged(w, False), slice(None), f"scores far below zero d={d}", sized.light)
    assert plan.stat(11) == sized.waves


def rows_that_rounding_cannot_turn(w, rows):
    """Of the rows (request, head, t): those whose best key leads every key that is not a copy of it by more than 40
    nats and twice what fp32 sums can be off by, d * 2^-24 of the sum of |q c k c| each."""
    k64 = w.k.double().cpu()
    q0 = np.concatenate([[0], np.cumsum(w.q_lens)])
    keep = np.zeros(len(rows), dtype=bool)
    for x, (i, h, t) in enumerate(rows):
        seen = int(w.kv_lens[i] - w.q_lens[i] + t + 1)
        kk = k64[int(w.kv_start[i]):int(w.kv_start[i]) + seen, h // (w.Hq // w.Hkv)]
        qq = w.q[int(q0[i]) + int(t), h].double().cpu()
        s = kk @ qq
        best = int(s.argmax())
        other = ~(kk == kk[best]).all(dim=1)
        off = 2 * w.d * 2.0 ** -24 * float((kk.abs() @ qq.abs()).max())
        keep[x] = not bool(other.any()) or float(s[best] - s[other].max()) > off + 40 / w.scale
    return keep


@pytest.mark.parametrize("heads", [(4, 2, 128), (4, 2, 64), (16, 2, 128), (30, 10, 128), (30, 10, 64)])
@pytest.mark.parametrize("size", [3e3, 1e5, 1e6, 1e9])
def test_prefill_with_large_finite_scores(size, heads):
    """Scaled scores of 1e7 to 1e19: a reference rounded to fp32 is off by up to many octaves there, more than the
    exponentials can take.  Copies of a key, in other key tiles too, have the same score and share the row.  Rows where
    the rounding of the sums decides between two keys are left out (under 1 in 50)."""
    Hq, Hkv, d = heads
    kv = np.asarray([513, 200, 97, 640], dtype=np.int32)
    ql = np.asarray([513, 60, 97, 300], dtype=np.int32)
    if Hq == 30:                                          # the pipeline with one head per workgroup
        kv, ql = H.with_long_requests(kv, ql)
    elif Hq == 16:                                        # and with eight waves
        kv, ql = H.with_eight_waves(kv, ql, Hq, Hkv, 4096)
    w = wl.make_ragged("large_scores", kv, ql, Hq, Hkv, d, 4096, 33, DEV, keep_f32=False)
    w.q.mul_(size)
    w.k.mul_(size)
    rng = np.random.default_rng(34)
    for s, L in zip(w.kv_start, w.kv_lens):
        a, b = rng.integers(0, int(L), size=(2, int(L) // 3))
        w.k[int(s) + torch.from_numpy(b).to(DEV)] = w.k[int(s) + torch.from_numpy(a).to(DEV)]
    req = np.where(rng.random(600) < 0.1, rng.integers(0, len(ql), size=600), rng.integers(0, 4, size=600))
    rows = np.stack([req, rng.integers(0, Hq, size=600), rng.integers(0, ql[req])], axis=1).astype(np.int32)
    keep = rows_that_rounding_cannot_turn(w, rows)
    assert keep.mean() > 0.98
    rows = rows[keep]
    at = (np.concatenate([[0], np.cumsum(ql)])[rows[:, 0]] + rows[:, 2], rows[:, 1])
    want = np.zeros(tuple(w.q.shape), dtype=np.float32)
    want[at] = H.oracle_ragged(w, False, rows=rows)
    plan = check_prefill_launches(w, want, at, f"scores of {size * size:g} {heads}", int(Hq == 4))
    assert plan.stat(11) == (8 if Hq == 16 else 4)
