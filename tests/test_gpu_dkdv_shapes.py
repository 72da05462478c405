"""The two workgroup shapes of the dkdv pass: eight waves for packings with few (key tile, kv head) workgroups, four waves
beyond.  Groups end inside, at and just past a 32-key block, a 128-key tile and a 32-row step; prompts and responses
cross them."""
import pytest
import torch

from paper_2511_18871_amd import binding as B
from paper_2511_18871_amd import workloads as W
from parity import gate, oracle_bwd, to64

pytestmark = pytest.mark.gpu

EDGES = [W.Group(1, []), W.Group(32, []), W.Group(31, [1, 1]), W.Group(33, [95]), W.Group(0, [128, 1]), W.Group(127, [2]),
         W.Group(128, [128]), W.Group(130, [30, 64, 33]), W.Group(65, [0, 200, 7]), W.Group(64, [64, 64])]


@pytest.mark.parametrize("resp_rows", [False, True])
@pytest.mark.parametrize("heads", [(16, 8), (8, 8), (12, 4)])
@pytest.mark.parametrize("repeats", [1, 6])                # (12, 4), once: eight waves and per-head partial sums
def test_dkdv_at_tile_edges(heads, repeats, resp_rows):
    w = W.Workload("edges", EDGES * repeats, heads[0], heads[1], 128, torch.bfloat16, 810 + heads[0])
    t = W.make_tensors(w)
    pl, Gs, rl, sc = w.prompt_lens(), w.Gs(), w.resp_lens_flat(), w.softmax_scale
    if resp_rows:                                          # by definition: no upstream gradient on the prompt rows
        at = 0
        for g in w.groups:
            t.d_o[at:at + g.prompt_len] = 0
            at += g.total
    q, k, v, d_o = t.q.cuda(), t.k.cuda(), t.v.cuda(), t.d_o.cuda()
    o, lse = B.sp_attn_fwd_batched(q, k, v, pl, Gs, rl, sc)
    dk0 = torch.zeros_like(k)
    dv0 = torch.zeros_like(v)
    flags = B.SP_FLAG_RESPONSE_ROWS | B.SP_FLAG_ACCUMULATE_DKDV if resp_rows else 0
    _, dk, dv = B.sp_attn_bwd_batched_ex(q, k, v, o, lse, d_o, pl, Gs, rl, sc, flags, dq=torch.zeros_like(q), dk=dk0, dv=dv0)
    torch.cuda.synchronize()
    _, rdk, rdv, _, _ = oracle_bwd(w, t)
    gate("dK", to64(dk), rdk, w.dtype)
    gate("dV", to64(dv), rdv, w.dtype)
