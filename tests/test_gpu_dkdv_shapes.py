"""The workgroup shapes of the dkdv pass: eight waves with per-head partial sums and without, four waves.  Groups end inside,
at and just past a 32-key block, a 128-key tile and a 32-row step; prompts and responses cross them.  In response-rows mode the
results are added to what the buffers hold, or replace it whatever it is."""
import pytest
import torch

from paper_2511_18871_amd import binding as B
from paper_2511_18871_amd import workloads as W
from parity import gate, oracle_bwd, to64

pytestmark = pytest.mark.gpu

EDGES = [W.Group(1, []), W.Group(32, []), W.Group(31, [1, 1]), W.Group(33, [95]), W.Group(0, [128, 1]), W.Group(127, [2]),
         W.Group(128, [128]), W.Group(130, [30, 64, 33]), W.Group(65, [0, 200, 7]), W.Group(64, [64, 64])]


# (16, 8) and (12, 4), once: partial sums; (8, 8), once, and (12, 4), three times: eight waves, one and three q heads; beyond: four
@pytest.mark.parametrize("mode", ["all_rows", "accumulate", "overwrite"])
@pytest.mark.parametrize("heads", [(16, 8), (8, 8), (12, 4)])
@pytest.mark.parametrize("repeats", [1, 3, 6])
def test_dkdv_at_tile_edges(heads, repeats, mode):
    w = W.Workload("edges", EDGES * repeats, heads[0], heads[1], 128, torch.bfloat16, 810 + heads[0])
    t = W.make_tensors(w)
    pl, Gs, rl, sc = w.prompt_lens(), w.Gs(), w.resp_lens_flat(), w.softmax_scale
    flags = {"all_rows": 0, "accumulate": B.SP_FLAG_RESPONSE_ROWS | B.SP_FLAG_ACCUMULATE_DKDV, "overwrite": B.SP_FLAG_RESPONSE_ROWS}[mode]
    assert B.sp_attn_dkdv_waves(pl, Gs, rl, *heads, flags) == (8 if repeats == 1 or (heads, repeats) == ((12, 4), 3) else 4)
    q, k, v, d_o = t.q.cuda(), t.k.cuda(), t.v.cuda(), t.d_o.cuda()
    if mode != "all_rows":                                 # by definition: no upstream gradient on the prompt rows
        at = 0
        for g in w.groups:
            t.d_o[at:at + g.prompt_len] = 0
            at += g.total
    o, lse = B.sp_attn_fwd_batched(q, k, v, pl, Gs, rl, sc)
    gen = torch.Generator().manual_seed(5)
    start = [torch.randn(t.k.shape, generator=gen).to(torch.bfloat16) if mode == "accumulate" else torch.full_like(t.k, float("nan"))
             for _ in range(2)]
    _, dk, dv = B.sp_attn_bwd_batched_ex(q, k, v, o, lse, d_o, pl, Gs, rl, sc, flags, dq=torch.zeros_like(q),
                                         dk=start[0].cuda(), dv=start[1].cuda())
    torch.cuda.synchronize()
    _, rdk, rdv, _, _ = oracle_bwd(w, t)
    for name, got, ref, old in zip(("dK", "dV"), (dk, dv), (rdk, rdv), start):
        gate(name, to64(got), ref + to64(old) if mode == "accumulate" else ref, w.dtype)
