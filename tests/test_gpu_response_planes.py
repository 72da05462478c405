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


EMPTY = [W.Group(1, []), W.Group(33, []), W.Group(257, []), W.Group(70, [0, 0]), W.Group(95, [0])]
BESIDE = EMPTY + [W.Group(e, [40, 70, 3]) for e in (0, 33, 64, 95)]


# groups without response tokens: no row of them takes part, so nothing writes their planes.  Split over the q heads (one group
# alone, several, with two row parts), eight waves, four waves
@pytest.mark.parametrize("accumulate", [False, True])
@pytest.mark.parametrize("groups,heads,waves", [*(([g], (4, 2), 8) for g in EMPTY), (BESIDE, (4, 2), 8), (BESIDE + [W.Group(600, [200])], (4, 2), 8),
                                                (BESIDE, (8, 8), 8), (BESIDE * 8, (8, 8), 4)])
def test_groups_without_responses_add_nothing(groups, heads, waves, accumulate):
    w = W.Workload("empty", groups, *heads, 128, torch.bfloat16, 641)
    t = W.make_tensors(w)
    pack, sc = (w.prompt_lens(), w.Gs(), w.resp_lens_flat()), w.softmax_scale
    flags = B.SP_FLAG_RESPONSE_ROWS | (B.SP_FLAG_ACCUMULATE_DKDV if accumulate else 0)
    assert B.sp_attn_dkdv_waves(*pack, *heads, flags) == waves
    empty, at = torch.zeros(w.total_tokens, dtype=torch.bool), 0
    for g in w.groups:
        t.d_o[at:at + g.prompt_len] = 0
        empty[at:at + g.total] = g.total == g.prompt_len
        at += g.total
    q, k, v, d_o = t.q.cuda(), t.k.cuda(), t.v.cuda(), t.d_o.cuda()
    o, lse = B.sp_attn_fwd_batched(q, k, v, *pack, sc)
    start = 1.0 if accumulate else float("nan")
    args = (q.shape[0], len(pack[0]), len(pack[2]), *heads, 128, B.SP_BF16)
    results = []
    for stages in ((7,), (1, 4, 2)):
        ws = torch.full((B.workspace_bytes(True, *args),), 255, dtype=torch.uint8, device="cuda")      # NaN wherever a call writes nothing
        out = [torch.zeros_like(q), torch.full_like(k, start), torch.full_like(v, start)]
        for stage in stages:
            B.sp_attn_bwd_batched_ex(q, k, v, o, lse, d_o, *pack, sc, flags, *out, workspace=ws, stages=stage)
        results.append(out)
    torch.cuda.synchronize()
    _, rdk, rdv, _, _ = oracle_bwd(w, t)
    for i, ref in ((1, rdk), (2, rdv)):
        got = results[0][i]
        assert torch.all(got[empty.cuda()] == (start if accumulate else 0.0))
        assert torch.equal(got, results[1][i])
        gate("dK" if i == 1 else "dV", to64(got), ref + (1.0 if accumulate else 0.0), w.dtype)
