"""Workgroups of the forward and of the dq pass hold (32 rows, q head) items of one kv head, row block first: every
ratio of q to kv heads cuts a row tile differently, and a group's end can fall inside any item of any workgroup."""
import pytest
import torch

from paper_2511_18871_amd import binding as B
from paper_2511_18871_amd import workloads as W
from parity import gate, gate_lse, oracle_bwd, to64

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("steps", [0, 1 << 20])            # force either workgroup shape (eight and four waves)
@pytest.mark.parametrize("heads", [(1, 1), (2, 1), (6, 2), (4, 1), (10, 2), (7, 1), (16, 2), (9, 1)])
def test_every_head_ratio_with_groups_ending_in_any_item(heads, steps):
    groups = [W.Group(1, []), W.Group(31, [1]), W.Group(33, [31, 32, 33]), W.Group(0, [160]), W.Group(255, [2, 65])]
    w = W.Workload(f"items{heads}", groups, heads[0], heads[1], 128, torch.bfloat16, 700 + heads[0])
    t = W.make_tensors(w)
    pl, Gs, rl, sc = w.prompt_lens(), w.Gs(), w.resp_lens_flat(), w.softmax_scale
    q, k, v, d_o = t.q.cuda(), t.k.cuda(), t.v.cuda(), t.d_o.cuda()
    try:
        B.set_small_shape_steps(steps)
        o, lse = B.sp_attn_fwd_batched(q, k, v, pl, Gs, rl, sc)
        dq, dk, dv = B.sp_attn_bwd_batched(q, k, v, o, lse, d_o, pl, Gs, rl, sc)
        torch.cuda.synchronize()
    finally:
        B.set_small_shape_steps(-1)
    rdq, rdk, rdv, ro, rlse = oracle_bwd(w, t)
    gate("O", to64(o), ro, w.dtype)
    gate_lse(to64(lse), rlse, w.dtype)
    gate("dQ", to64(dq), rdq, w.dtype)
    gate("dK", to64(dk), rdk, w.dtype)
    gate("dV", to64(dv), rdv, w.dtype)
