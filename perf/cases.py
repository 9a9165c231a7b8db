"""Cases for timing the public entry points of paper_2602_06072_amd on one GPU.

listed() and draw() give cases, prepare() makes what a serving program has in hand before the call
(tensors on the GPU and, where it keeps one, the bound plan), run() makes one pass through
paper_2602_06072_amd.binding, work() states what a pass cannot do without and tolerance() how far two
correct implementations may be apart.

The lengths of a case come from its own "structure" number, so that work() knows them; the tensor
values come from the seed and are N(0,1) rounded to bf16, as everywhere in this repository.  The fp32
entry points (a plain-FMA debugging aid) and the padded ones (the comparison that the packed calls
are held against) are not work that a user has done, and no case times them.

path      one pass is
prefill   packed_prefill_attn of one layer (plan "kept": the plan and its workspace are there, as in
          every layer but the first; plan "new": pack_plan, workspace, plan_bind and the call, as for
          the first layer of a new batch)
decode    packed_decode_attn on a group buffer that is there
loop      one step of a decode loop on one plan: kv_append of the new rows, packed_decode_attn_grown
relayout  kv_reorganize with a plan that is there
regroup   the first decode step after a (re)grouping: pack_plan, workspace, plan_bind, kv_reorganize,
          packed_decode_attn
mixed     packed_mixed_step: the prefill chunks and the decode rows of one step, one layer
"""
import math

import numpy as np
import torch

from paper_2602_06072_amd import binding as pk
from paper_2602_06072_amd import workloads as wl

DEV = "cuda"


def _prefill(name, n, q_lo, q_hi, q_mid, sigma, ctx_hi, heads, budget, plan="kept", out="bf16", structure=0):
    """n requests; query lengths uniform in [q_lo, q_hi] (sigma 0) or lognormal around q_mid, clipped;
    context before them uniform in [0, ctx_hi]."""
    Hq, Hkv, d = heads
    return dict(name=name, path="prefill", n=n, q_lo=q_lo, q_hi=q_hi, q_mid=q_mid, sigma=sigma, ctx_hi=ctx_hi,
                Hq=Hq, Hkv=Hkv, d=d, budget=budget, plan=plan, out=out, structure=structure)


def _decode(name, path, n, lo, hi, mid, sigma, heads, budget, families=0, prefix_lo=0, prefix_hi=0, tree=False,
            headroom=0, page=16, out="bf16", structure=0):
    """n requests; private lengths uniform in [lo, hi] (sigma 0) or lognormal around mid, clipped; with
    families > 0 the requests are dealt evenly to that many families whose shared prefix is uniform in
    [prefix_lo, prefix_hi]; with tree the families lie below one common root of prefix_lo tokens."""
    Hq, Hkv, d = heads
    return dict(name=name, path=path, n=n, lo=lo, hi=hi, mid=mid, sigma=sigma, Hq=Hq, Hkv=Hkv, d=d, budget=budget,
                families=families, prefix_lo=prefix_lo, prefix_hi=prefix_hi, tree=tree, headroom=headroom, page=page,
                out=out, structure=structure)


def listed():
    return [
        # the smallest batch: a handful of short prompts, few heads; a new batch every pass (8 x 16..512, the
        # tiny configuration): planning, table upload and launch latency count
        _prefill("prefill_tiny_new_plan", 8, 16, 512, 0, 0.0, 0, (8, 8, 64), 1024, plan="new"),
        # one layer of an 8B-shaped model on 64 prompts of very different lengths
        _prefill("prefill_8b_ragged", 64, 8, 8192, 256, 1.2, 0, (32, 8, 128), 16384),
        # chunked prefill of a 70B-shaped layer: chunks of 512..2048 tokens behind up to 16384 tokens of context
        _prefill("prefill_70b_chunks", 32, 512, 2048, 0, 0.0, 16384, (64, 8, 128), 16384),
        # long prompts of equal order with head dimension 64, fp32 output for a caller that goes on in fp32
        _prefill("prefill_d64_long", 8, 3500, 4600, 0, 0.0, 0, (32, 8, 64), 16384, out="f32"),
        # interactive decode: four users, a layer of an 8B-shaped model; latency bound
        _decode("decode_small", "decode", 4, 300, 3000, 0, 0.0, (32, 8, 128), 8192, structure=3),
        # heterogeneous decode batch: 256 rows, lengths over three orders of magnitude
        _decode("decode_8b_hetero", "decode", 256, 32, 32768, 512, 1.5, (32, 8, 128), 16384),
        # shared-prefix decode: 16 families of 8 (one document, several questions)
        _decode("decode_8b_families", "decode", 128, 16, 512, 0, 0.0, (32, 8, 128), 16384, families=16,
                prefix_lo=1024, prefix_hi=4096),
        # nested prefixes: one system prompt, 16 documents below it, 128 requests
        _decode("decode_8b_tree", "decode", 128, 16, 512, 0, 0.0, (32, 8, 128), 8192, families=16,
                prefix_lo=1024, prefix_hi=3072, tree=True),
        # one step of a decode loop in the headroom of a plan, head dimension 64
        _decode("loop_d64", "loop", 200, 32, 8192, 700, 1.0, (32, 8, 64), 8192, headroom=32),
        # consolidation of a heterogeneous batch's pages into the group buffers
        _decode("relayout_8b", "relayout", 256, 32, 32768, 512, 1.5, (32, 8, 128), 16384),
        # a decode batch that is regrouped: new plan, consolidation, first step; some shared prefixes
        _decode("regroup_8b", "regroup", 48, 100, 1500, 0, 0.0, (32, 8, 128), 8192, families=6, prefix_lo=200,
                prefix_hi=1200, headroom=16, structure=5),
        # the largest: a whole continuous-batching step of a 70B-shaped layer, chunks as above + 480 decode rows,
        # four fifths of them short and one fifth of 16384..65536 tokens
        dict(name="mixed_70b", path="mixed", n=32, q_lo=512, q_hi=2048, q_mid=0, sigma=0.0, ctx_hi=16384, Hq=64, Hkv=8,
             d=128, budget=16384, out="bf16", structure=0, rows=480, row_lo=128, row_hi=2048, row_long=0.2,
             long_lo=16384, long_hi=65536),
    ]


# ---------------------------------------------------------------------------------------------
# drawn cases
# ---------------------------------------------------------------------------------------------

HEADS = [(8, 8, 64), (32, 8, 64), (32, 8, 128), (32, 8, 128), (64, 8, 128), (64, 8, 128), (8, 2, 128), (16, 2, 128),
         (4, 1, 128), (16, 16, 128)]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_once(rng):
    heads = rng.choice(HEADS)
    path = rng.choice(["prefill", "prefill", "prefill", "decode", "decode", "decode", "loop", "relayout", "regroup", "mixed"])
    s = rng.randrange(1 << 20)
    budget = rng.choice([2048, 8192, 16384])
    out = rng.choice(["bf16", "bf16", "bf16", "f32"])
    if path == "prefill":
        n = _log(rng, 1, 64)
        mid = max(8, _log(rng, 200, 60000) // n)
        sigma = rng.choice([0.0, 0.3, 1.2])
        return _prefill("", n, max(1, mid // (2 if sigma == 0 else 16)), min(16384, mid * (2 if sigma == 0 else 8)), mid, sigma,
                        rng.choice([0, 0, _log(rng, 16, 16384)]), heads, budget, rng.choice(["kept", "kept", "new"]), out, s)
    if path == "mixed":
        n, mid = _log(rng, 1, 24), _log(rng, 64, 2048)
        row_hi = _log(rng, 64, 4096)
        return dict(path="mixed", n=n, q_lo=max(1, mid // 4), q_hi=mid, q_mid=0, sigma=0.0, ctx_hi=_log(rng, 16, 16384),
                    Hq=heads[0], Hkv=heads[1], d=heads[2], budget=budget, out=out, structure=s, rows=_log(rng, 1, 400),
                    row_lo=max(1, row_hi // 16), row_hi=row_hi, row_long=rng.choice([0.0, 0.1, 0.2]),
                    long_lo=row_hi, long_hi=8 * row_hi)
    n = _log(rng, 1, 480)
    mid = min(32768, max(16, _log(rng, 500, 900000) // n))
    sigma = rng.choice([0.0, 0.7, 1.5])
    families = rng.choice([0, 0, max(1, n // rng.choice([2, 5, 8]))]) if n > 1 else 0
    hi_p = _log(rng, 32, 4096)
    c = _decode("", path, n, max(1, mid // (2 if sigma == 0 else 16)), min(65536, mid * (2 if sigma == 0 else 16)), mid, sigma, heads,
                budget, families, max(1, hi_p // 4) if families else 0, hi_p if families else 0,
                bool(families) and path == "decode" and rng.random() < 0.5,
                rng.choice([1, 8, 32]) if path == "loop" else rng.choice([0, 0, 16]), rng.choice([16, 16, 16, 128, 256, 7]), out, s)
    return c


def _cost(case):
    w = work(case)
    return w["bytes"] / 5e12 + w["flops"] / (1e15 if case["path"] in ("prefill", "mixed") else 1e18)


def draw(rng):
    while True:
        c = _draw_once(rng)
        c.pop("name", None)
        if _cost(c) <= 6e-3:           # under half of the largest listed case
            return c


# ---------------------------------------------------------------------------------------------
# structure of a case (lengths, families): the same for every seed
# ---------------------------------------------------------------------------------------------

def _lengths(rng, n, lo, hi, mid, sigma):
    if sigma == 0.0:
        return rng.integers(lo, hi + 1, size=n).astype(np.int32)
    x = np.exp(rng.normal(math.log(mid), sigma, size=n))
    return np.clip(np.rint(x), lo, hi).astype(np.int32)


def _prefill_lengths(case):
    rng = np.random.default_rng(case["structure"])
    q = _lengths(rng, case["n"], case["q_lo"], case["q_hi"], case["q_mid"], case["sigma"])
    ctx = rng.integers(0, case["ctx_hi"] + 1, size=case["n"]).astype(np.int32)
    return q, q + ctx


def _decode_structure(case):
    """(private lengths, family of every request or None, prefix length of every family, length of the root)."""
    rng = np.random.default_rng(case["structure"] + 1)
    if case["path"] == "mixed":
        is_long = rng.random(case["rows"]) < case["row_long"]
        short = rng.integers(case["row_lo"], case["row_hi"] + 1, size=case["rows"])
        return np.where(is_long, rng.integers(case["long_lo"], case["long_hi"] + 1, size=case["rows"]), short).astype(np.int32), None, None, 0
    own = _lengths(rng, case["n"], case["lo"], case["hi"], case["mid"], case["sigma"])
    if not case["families"]:
        return own, None, None, 0
    family = (np.arange(case["n"]) * case["families"] // case["n"]).astype(np.int32)
    plen = rng.integers(case["prefix_lo"], case["prefix_hi"] + 1, size=case["families"]).astype(np.int32)
    return own, family, plen, case["prefix_lo"] if case["tree"] else 0


def work(case):
    """Each input read once, each output written once; shared prefixes once."""
    Hq, Hkv, d = case["Hq"], case["Hkv"], case["d"]
    osize = 4 if case["out"] == "f32" else 2
    nbytes = flops = 0
    if case["path"] in ("prefill", "mixed"):
        q, kv = (x.astype(np.int64) for x in _prefill_lengths(case))
        pairs = int((q * (kv - q) + q * (q + 1) // 2).sum())
        flops += 4 * d * Hq * pairs
        nbytes += int(q.sum()) * Hq * d * (2 + osize) + int(kv.sum()) * Hkv * d * 4
    if case["path"] != "prefill":
        own, family, plen, root = _decode_structure(case)
        n = len(own)
        unique, total = int(own.sum()), int(own.sum())
        if family is not None:
            unique += int(plen[np.unique(family)].sum()) + root
            total += int(plen[family].sum()) + root * n
        grown = _loop_step(case) + 1 if case["path"] == "loop" else 0
        if case["path"] in ("relayout", "regroup"):
            nbytes += 2 * unique * Hkv * d * 4
        if case["path"] != "relayout":
            nbytes += (unique + n * grown) * Hkv * d * 4 + n * Hq * d * (2 + osize)
            flops += 4 * d * Hq * (total + n * grown)
        if case["path"] == "loop":
            nbytes += 2 * n * Hkv * d * 4
    return {"bytes": nbytes, "flops": flops}


def _loop_step(case):
    return case["headroom"] // 2


def tolerance(case):
    if case["path"] == "relayout":
        return "exact"
    # Against the path in 64 bits: rel 1.9e-3 .. 2.3e-3 (bf16 out), 1.1e-3 .. 1.6e-3 (fp32 out: what is left is P
    # rounded to bf16), max 0.005 .. 0.043; about four times that.
    return {"rel": 8e-3 if case["out"] == "bf16" else 6e-3, "max": 0.15}


# ---------------------------------------------------------------------------------------------
# what a program has in hand, and one pass
# ---------------------------------------------------------------------------------------------

def _out(case, shape):
    return torch.empty(shape, dtype=torch.float32 if case["out"] == "f32" else torch.bfloat16, device=DEV)


def _bound(plan, case):
    ws = pk.new_workspace(plan, case["Hq"], case["Hkv"], case["d"], pk.PK_BF16)
    pk.plan_bind(plan, case["Hq"], case["Hkv"], case["d"], pk.PK_BF16, ws)
    return ws


def _prepare_prefill(case, seed):
    ql, kl = _prefill_lengths(case)
    w = wl.make_ragged("prefill", kl, ql, case["Hq"], case["Hkv"], case["d"], case["budget"], seed, device=DEV)
    s = dict(kv_lens=kl, q_lens=ql, q=w.q, k=w.k, v=w.v, out=_out(case, w.q.shape), scale=w.scale)
    if case.get("plan") != "new":
        s["plan"] = pk.pack_plan(kl, ql, token_budget=case["budget"])
        s["ws"] = _bound(s["plan"], case)
    return s


def _decode_plan(case, s):
    if s["tree"] is not None:
        return pk.pack_plan_tree(s["kv_lens"], s["ones"], *s["tree"], token_budget=case["budget"], headroom=case["headroom"])
    return pk.pack_plan(s["kv_lens"], s["ones"], s["prefix_ids"], s["prefix_lens"], case["budget"], case.get("headroom", 0))


def _prepare_decode(case, seed):
    own, family, plen, root = _decode_structure(case)
    Hq, Hkv, d = case["Hq"], case["Hkv"], case["d"]
    page = case.get("page", 16)
    pid = pl = tree = None
    if family is None:
        w = wl.make_paged("decode", own, Hq, Hkv, d, case["budget"], page, seed, device=DEV)
    elif root:
        fams = len(plen)
        tree = (np.asarray([-1] + [0] * fams, np.int32), np.concatenate([[root], plen]).astype(np.int32), family + 1)
        w = wl.make_paged_tree("decode", own, *tree, Hq, Hkv, d, case["budget"], page, seed, device=DEV)
    else:
        pid, pl = family, plen[family]
        w = wl.make_paged("decode", own + pl, Hq, Hkv, d, case["budget"], page, seed, prefix_ids=pid, prefix_lens=pl, device=DEV)
    s = dict(kv_lens=w.kv_lens, ones=np.ones_like(w.kv_lens), prefix_ids=pid, prefix_lens=pl, tree=tree, q=w.q,
             k_pages=w.k_pages, v_pages=w.v_pages, block_table=torch.from_numpy(w.block_table).to(DEV), scale=w.scale,
             out=_out(case, w.q.shape))
    plan = _decode_plan(case, s)
    s["kv_buf"] = pk.new_kv_buf(plan, Hkv, d, pk.PK_BF16)
    if case["path"] == "regroup":
        return s                        # (the buffer is kept for the life of the server; the plan is made in the pass)
    s["plan"], s["ws"] = plan, _bound(plan, case)
    if case["path"] == "relayout":
        return s
    pk.kv_reorganize(plan, s["k_pages"], s["v_pages"], s["block_table"], s["kv_buf"], s["ws"])
    if case["path"] == "loop":          # the steps before the one that is timed, and that one's new rows
        for t in range(_loop_step(case) + 1):
            g = torch.Generator(device=DEV).manual_seed(seed * 1009 + t)
            shape = (2, w.n, Hkv, d)
            rows = torch.randn(shape, generator=g, device=DEV, dtype=torch.float32).to(torch.bfloat16)
            s["k_new"], s["v_new"] = rows[0], rows[1]
            if t < _loop_step(case):
                pk.kv_append(plan, s["k_new"], s["v_new"], s["kv_buf"], t, s["ws"])
    torch.cuda.synchronize()
    del s["k_pages"], s["v_pages"], s["block_table"]
    return s


def prepare(case, seed):
    s = {"case": dict(case)}
    if case["path"] in ("prefill", "mixed"):
        s["prefill"] = _prepare_prefill(case, seed)
    if case["path"] != "prefill":
        s["decode"] = _prepare_decode(case, seed)
    return s


def run(state):
    case = state["case"]
    p, s = state.get("prefill"), state.get("decode")
    Hkv = case["Hkv"]
    if case["path"] == "prefill":
        if case["plan"] == "new":
            plan = pk.pack_plan(p["kv_lens"], p["q_lens"], token_budget=case["budget"])
            return pk.packed_prefill_attn(plan, p["q"], p["k"], p["v"], p["out"], p["scale"], _bound(plan, case))
        return pk.packed_prefill_attn(p["plan"], p["q"], p["k"], p["v"], p["out"], p["scale"], p["ws"])
    if case["path"] == "decode":
        return pk.packed_decode_attn(s["plan"], s["q"], s["kv_buf"], s["out"], s["scale"], Hkv, s["ws"])
    if case["path"] == "loop":
        t = _loop_step(case)
        pk.kv_append(s["plan"], s["k_new"], s["v_new"], s["kv_buf"], t, s["ws"])
        pk.packed_decode_attn_grown(s["plan"], s["q"], s["kv_buf"], s["out"], s["scale"], t + 1, Hkv, s["ws"])
        return s["out"], s["kv_buf"].view(torch.int16)
    if case["path"] == "relayout":
        pk.kv_reorganize(s["plan"], s["k_pages"], s["v_pages"], s["block_table"], s["kv_buf"], s["ws"])
        return s["kv_buf"].view(torch.int16)
    if case["path"] == "regroup":
        plan = _decode_plan(case, s)
        ws = _bound(plan, case)
        pk.kv_reorganize(plan, s["k_pages"], s["v_pages"], s["block_table"], s["kv_buf"], ws)
        pk.packed_decode_attn(plan, s["q"], s["kv_buf"], s["out"], s["scale"], Hkv, ws)
        return s["out"], s["kv_buf"].view(torch.int16)
    return pk.packed_mixed_step(p["plan"], p["q"], p["k"], p["v"], p["out"], p["ws"],
                                s["plan"], s["q"], s["kv_buf"], s["out"], s["ws"], p["scale"])
