"""Response rows only, in one call: the rowsum is part of the dq pass, which also writes the zeros that the dkdv pass reads for the
prompt rows of its first row tile.  Prompts that end at every place of a 64-row tile that matters, outputs and gradients of the
prompt rows as NaN, both shapes; bitwise equal to the stages."""
import pytest
import torch

from paper_2511_18871_amd import binding as B
from paper_2511_18871_amd import workloads as W
from parity import gate, oracle_bwd, to64

pytestmark = pytest.mark.gpu

ENDS = [0, 1, 31, 32, 33, 63, 64, 65, 95, 96, 97, 160]


@pytest.mark.parametrize("heads,shape", [((4, 2), 0), ((4, 2), 1 << 20), ((8, 8), 1 << 20)])
def test_prompt_rows_take_no_part(heads, shape):
    w = W.Workload("ends", [W.Group(e, [40, 70, 3]) for e in ENDS] * 2, *heads, 128, torch.bfloat16, 640)
    t = W.make_tensors(w)
    pack, sc = (w.prompt_lens(), w.Gs(), w.resp_lens_flat()), w.softmax_scale
    prompt, at = torch.zeros(w.total_tokens, dtype=torch.bool), 0
    for g in w.groups:
        prompt[at:at + g.prompt_len] = True
        at += g.total
    t.d_o[prompt] = 0
    q, k, v, d_o = t.q.cuda(), t.k.cuda(), t.v.cuda(), t.d_o.cuda()
    B.set_small_shape_steps(shape)
    try:
        o, lse = B.sp_attn_fwd_batched(q, k, v, *pack, sc)
        o[prompt.cuda()] = float("nan")
        lse[:, prompt.cuda()] = float("nan")
        ws = torch.full((B.workspace_bytes(True, q.shape[0], len(pack[0]), len(pack[2]), *heads, 128, B.SP_BF16),), 255, dtype=torch.uint8,
                        device="cuda")                    # NaN wherever a call writes nothing
        nan = lambda: [torch.full_like(x, float("nan")) for x in (q, k, v)]
        one = B.sp_attn_bwd_batched_ex(q, k, v, o, lse, d_o, *pack, sc, B.SP_FLAG_RESPONSE_ROWS, *nan(), workspace=ws)
        staged = nan()
        for stage in (1, 4, 2):
            B.sp_attn_bwd_batched_ex(q, k, v, o, lse, d_o, *pack, sc, B.SP_FLAG_RESPONSE_ROWS, *staged, workspace=ws, stages=stage)
        torch.cuda.synchronize()
    finally:
        B.set_small_shape_steps(-1)
    rdq, rdk, rdv, _, _ = oracle_bwd(w, t)
    assert one[0][prompt.cuda()].isnan().all()
    gate("dQ", to64(one[0][~prompt.cuda()]), rdq[~prompt.numpy()], w.dtype)
    gate("dK", to64(one[1]), rdk, w.dtype)
    gate("dV", to64(one[2]), rdv, w.dtype)
    for name, a, b in zip(("dQ", "dK", "dV"), one, staged):
        assert torch.equal(a.nan_to_num(7.0), b.nan_to_num(7.0)), name
