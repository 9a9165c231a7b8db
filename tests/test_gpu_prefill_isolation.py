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


@pytest.mark.parametrize("d", [128, 64])
def test_lanes_without_a_query_hold_nobody_elses_row(d):
    """Partly filled waves with unmasked key tiles; the first query row of the batch holds a NaN.  Tiles are not
    shared here, so every row behind the first wave of request 0 is in another wave than that row."""
    ql = np.asarray([200, 17, 45, 100, 9], dtype=np.int32)
    kv = ql + np.asarray([0, 500, 300, 130, 700], dtype=np.int32)
    w = wl.make_ragged("padding", kv, ql, 4, 2, d, 1024, 21, DEV, keep_f32=False)
    clean = {p: prefill(w, p)[0] for p in (False, True)}
    w.q[0] = float("nan")
    for padded in (False, True):
        got, plan = prefill(w, padded)
        assert plan.stat(6) == 6                           # one tile a request, two for the first: nothing shared
        assert torch.equal(got[32:], clean[padded][32:])
        assert torch.isnan(got[0]).all()
