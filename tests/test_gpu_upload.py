"""The table upload of a bind: a kernel up to 160 KiB, a copy command above; staging buffers that are reused
while the stream is still behind."""
import numpy as np
import pytest
import torch

from paper_2602_06072_amd import binding as pk
from paper_2602_06072_amd import workloads as wl
from tests import helpers as H

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.mark.parametrize("n", [1, 150, 700, 1300, 1500, 6000])
def test_decode_parity_over_the_sizes_of_the_tables(n):
    """3 KB of tables; part of one pass of the upload kernel's lanes; more than one (82 KB); below the limit (154 KB); the
    copy command (177 and 700 KB)."""
    w = wl.small_paged(seed=300 + n, n=n, lo=1, hi=40, Hq=4, Hkv=1, d=64, token_budget=512, device=DEV, keep_f32=False)
    plan = pk.pack_plan(w.kv_lens, np.ones_like(w.kv_lens), None, None, w.token_budget)
    ws = pk.new_workspace(plan, w.Hq, w.Hkv, w.d, pk.PK_BF16)
    ws.fill_(0x7F)
    kv_buf = pk.new_kv_buf(plan, w.Hkv, w.d, pk.PK_BF16)
    out = torch.full(w.q.shape, float("nan"), dtype=torch.float32, device=DEV)
    pk.plan_bind(plan, w.Hq, w.Hkv, w.d, pk.PK_BF16, ws)
    pk.kv_reorganize(plan, w.k_pages, w.v_pages, torch.from_numpy(w.block_table).to(DEV), kv_buf, ws)
    pk.packed_decode_attn(plan, w.q, kv_buf, out, w.scale, w.Hkv, ws)
    torch.cuda.synchronize()
    H.assert_close(out.cpu().numpy(), H.oracle_paged_decode(w, False), 0, f"decode, {n} requests")


def test_many_new_batches_without_a_synchronisation():
    """More binds in flight than there are staging buffers (64), all on one workspace a stream; every batch must get its
    own tables, on either of two streams.  Matrix products ahead of them keep the streams busy until every buffer is
    out; the bind after that waits for its stream to drain, and those that follow reuse buffers."""
    rng = np.random.default_rng(310)
    w = wl.small_ragged(seed=311, n=40, lo=1, hi=300, Hq=8, Hkv=2, d=64, token_budget=512, device=DEV, keep_f32=False)
    total = int(w.q_lens.sum())
    batches = []
    for _ in range(90):                             # the same rows cut into other requests each time
        cuts = np.sort(rng.choice(np.arange(1, total), size=int(rng.integers(5, 200)), replace=False))
        batches.append(np.diff(np.concatenate([[0], cuts, [total]])).astype(np.int32))

    def run(lens, ws, out):
        plan = pk.pack_plan(lens, lens, token_budget=512)
        pk.plan_bind(plan, 8, 2, 64, pk.PK_BF16, ws)
        pk.packed_prefill_attn(plan, w.q, w.k, w.v, out, w.scale, ws)
        return plan

    biggest = np.full(total // 2, 2, dtype=np.int32)
    nbytes = max(pk.pack_plan(x, x, token_budget=512).workspace_bytes(8, 2, 64, pk.PK_BF16) for x in batches + [biggest])
    spaces = [torch.empty(nbytes, dtype=torch.uint8, device=DEV) for _ in range(2)]
    streams = [torch.cuda.Stream() for _ in range(2)]
    want = []
    for lens in batches:
        out = torch.empty_like(w.q)
        run(lens, spaces[0], out)
        torch.cuda.synchronize()
        want.append(out)
    got = [torch.full_like(w.q, float("nan")) for _ in batches]
    torch.cuda.synchronize()
    x = torch.randn(8192, 8192, dtype=torch.bfloat16, device=DEV)
    y = [torch.mm(x, x) for _ in streams]
    torch.cuda.synchronize()
    for st, z in zip(streams, y):
        with torch.cuda.stream(st):
            for _ in range(60):
                torch.mm(x, x, out=z)
    ahead = [st.record_event() for st in streams]
    plans = []
    for i, lens in enumerate(batches):
        if i == 64:
            assert not any(e.query() for e in ahead)       # nothing has been uploaded yet
        with torch.cuda.stream(streams[i % 2]):
            plans.append(run(lens, spaces[i % 2], got[i]))
    torch.cuda.synchronize()
    for i in range(len(batches)):
        assert torch.equal(got[i], want[i]), f"batch {i}"
