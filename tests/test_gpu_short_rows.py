"""Rows that see at most 64 keys are computed beside the dq pass's row tiles, two or three (segment, q head) pairs to a
workgroup: prompts and responses around 64 keys, empty responses (also a group's last), odd counts of pairs, and a
backward whose stages run apart."""
import pytest
import torch

from paper_2511_18871_amd import binding as B
from paper_2511_18871_amd import workloads as W
from parity import gate, oracle_bwd, to64

pytestmark = pytest.mark.gpu

GROUPS = [W.Group(1, [0]), W.Group(63, [1, 2, 0]), W.Group(64, [5, 70]), W.Group(30, [33, 34, 35]), W.Group(0, [64, 65, 0]),
          W.Group(200, []), W.Group(10, [100, 0])]


@pytest.mark.parametrize("steps", [0, 1 << 20])            # either workgroup shape of the dq pass
@pytest.mark.parametrize("heads,groups", [((1, 1), GROUPS), ((7, 1), GROUPS[1:]), ((6, 3), GROUPS[:3])])
def test_short_rows_in_one_call_and_in_stages(heads, groups, steps):
    w = W.Workload("short", groups, heads[0], heads[1], 128, torch.bfloat16, 900 + heads[0])
    t = W.make_tensors(w)
    pl, Gs, rl, sc = w.prompt_lens(), w.Gs(), w.resp_lens_flat(), w.softmax_scale
    q, k, v, d_o = t.q.cuda(), t.k.cuda(), t.v.cuda(), t.d_o.cuda()
    try:
        B.set_small_shape_steps(steps)
        o, lse = B.sp_attn_fwd_batched(q, k, v, pl, Gs, rl, sc)
        one = B.sp_attn_bwd_batched(q, k, v, o, lse, d_o, pl, Gs, rl, sc)
        o2, lse2 = B.sp_attn_fwd_batched(q, k, v, pl, Gs, rl, sc)
        apart = [torch.empty_like(q), torch.empty_like(k), torch.empty_like(v)]
        for stage in (B.SP_BWD_STAGE_ROWSUM, B.SP_BWD_STAGE_DQ, B.SP_BWD_STAGE_DKDV):
            B.sp_attn_bwd_batched_stages(q, k, v, o2, lse2, d_o, pl, Gs, rl, sc, stage, o2._sp_workspace, *apart)
        torch.cuda.synchronize()
    finally:
        B.set_small_shape_steps(-1)
    for name, got, also, ref in zip(("dQ", "dK", "dV"), one, apart, oracle_bwd(w, t)):
        gate(name, to64(got), ref, w.dtype)
        assert torch.equal(got, also), name


@pytest.mark.parametrize("heads", [1, 8])
@pytest.mark.parametrize("responses", [300, 4000])
def test_prompt_gradients_under_many_short_responses(responses, heads):
    """A prompt of 10 tokens under responses of 35, whose every row sees fewer than 64 keys, against batched per-sample attention."""
    Lp, n, d = 10, 35, 128
    gen = torch.Generator(device="cuda").manual_seed(responses)
    T = Lp + responses * n
    q, k, v, d_o = (torch.randn(T, heads, d, generator=gen, device="cuda").to(torch.bfloat16) for _ in range(4))
    pack, sc = ([Lp], [responses], [n] * responses), d ** -0.5
    o, lse = B.sp_attn_fwd_batched(q, k, v, *pack, sc)
    dq, dk, dv = B.sp_attn_bwd_batched(q, k, v, o, lse, d_o, *pack, sc)
    torch.cuda.synchronize()
    idx = torch.cat([torch.arange(Lp).expand(responses, Lp), Lp + torch.arange(responses * n).view(responses, n)], 1).cuda()
    mask = torch.ones(Lp + n, Lp + n, device="cuda").tril().bool()
    for h in {0, heads - 1}:
        Q, K, V = (x[:, h].float()[idx].contiguous().requires_grad_() for x in (q, k, v))
        G = d_o[:, h].float()[idx].contiguous()
        G[1:, :Lp] = 0                                    # the prompt's own rows count once
        S = (Q * sc) @ K.transpose(1, 2).contiguous()
        (torch.softmax(S.masked_fill(~mask, float("-inf")), -1) @ V).backward(G)
        for name, got, x in (("dQ", dq, Q), ("dK", dk, K), ("dV", dv, V)):
            ref = torch.zeros(T, d, dtype=torch.float64, device="cuda").index_add_(0, idx.reshape(-1), x.grad.double().view(-1, d))
            gate(f"{name} head {h}", to64(got[:, h]), to64(ref), torch.bfloat16)
