"""Tables of many plans bound one after the other while the stream is busy: the host runs out of staging buffers, waits for one or copies from pageable memory, and
every plan's call finds its own tables.  (When it waits and when it does not: test_table_uploads.py.)"""
import numpy as np
import pytest
import torch

from paper_2602_06072_amd import binding as pk
from paper_2602_06072_amd import workloads as wl

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.mark.parametrize("busy_first", [False, True])
def test_many_binds_ahead_of_the_gpu(busy_first):
    Hq, Hkv, d = 8, 2, 64
    rng = np.random.default_rng(3)
    calls = []
    for i in range(100):                            # (more than the 64 buffers of the pool)
        lens = rng.integers(1, 120, 6).astype(np.int32)
        w = wl.make_ragged("ahead", lens, lens, Hq, Hkv, d, 1024, 100 + i, device=DEV, keep_f32=False)
        calls.append((lens, w, torch.full(w.q.shape, float("nan"), dtype=torch.float32, device=DEV)))

    def run(lens, w, out):
        plan = pk.pack_plan(lens, lens, token_budget=1024)
        ws = pk.new_workspace(plan, Hq, Hkv, d, pk.PK_BF16)
        pk.plan_bind(plan, Hq, Hkv, d, pk.PK_BF16, ws)
        pk.packed_prefill_attn(plan, w.q, w.k, w.v, out, w.scale, ws)
        return plan, ws

    want = []
    for lens, w, out in calls:                      # one at a time
        keep = run(lens, w, out)
        torch.cuda.synchronize()
        want.append(out.clone())
        out.fill_(float("nan"))
        del keep
    a = torch.randn(8192, 8192, device=DEV, dtype=torch.bfloat16)
    torch.cuda.synchronize()
    for _ in range(12 if busy_first else 0):        # some 10 ms: longer than the host takes to fill the pool, and than it waits for a buffer
        torch.mm(a, a)
    keep = [run(*c) for c in calls]
    torch.cuda.synchronize()
    assert len(keep) == len(calls)
    for (_, _, out), x in zip(calls, want):
        assert torch.equal(out, x)
