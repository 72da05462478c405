"""Key tiles of the head-split dkdv pass in one and in two row parts, and both within a packing: longest tiles of seven, eight
and nine steps, several groups, short prompts whose rows are swept twice, in response-rows mode added to what the buffers hold;
one call and stages bit for bit."""
import pytest
import torch

from paper_2511_18871_amd import binding as B
from paper_2511_18871_amd import workloads as W
from parity import gate, oracle_bwd, to64

pytestmark = pytest.mark.gpu

PACKS = {
    "seven_steps": [W.Group(100, [348])],
    "eight_steps": [W.Group(100, [349])],
    "nine_steps_mid_tile": [W.Group(129, [200, 0, 90, 95])],
    "short_prompt": [W.Group(5, [600, 30])],
    "one_long_one_short": [W.Group(700, [60, 1, 120]), W.Group(30, [40, 9])],
    "no_prompt": [W.Group(0, [700, 300])],
    "long_prompt_responses": [W.Group(64, [64] * 20)],
}


@pytest.mark.parametrize("mode", ["all_rows", "accumulate"])
@pytest.mark.parametrize("name", list(PACKS))
def test_row_parts(name, mode):
    w = W.Workload(name, PACKS[name], 4, 2, 128, torch.bfloat16, 770)
    t = W.make_tensors(w)
    pack, sc = (w.prompt_lens(), w.Gs(), w.resp_lens_flat()), w.softmax_scale
    flags = B.SP_FLAG_RESPONSE_ROWS | B.SP_FLAG_ACCUMULATE_DKDV if mode == "accumulate" else 0
    if flags:
        at = 0
        for g in w.groups:
            t.d_o[at:at + g.prompt_len] = 0
            at += g.total
    q, k, v, d_o = t.q.cuda(), t.k.cuda(), t.v.cuda(), t.d_o.cuda()
    o, lse = B.sp_attn_fwd_batched(q, k, v, *pack, sc)
    start = lambda: [torch.zeros_like(q), *(torch.ones_like(k) if flags else torch.full_like(k, float("nan")) for _ in range(2))]
    one, staged = start(), start()
    B.sp_attn_bwd_batched_ex(q, k, v, o, lse, d_o, *pack, sc, flags, *one)
    for stage in (1, 4, 2):
        B.sp_attn_bwd_batched_ex(q, k, v, o, lse, d_o, *pack, sc, flags, *staged, stages=stage)
    torch.cuda.synchronize()
    _, rdk, rdv, _, _ = oracle_bwd(w, t)
    for what, got, other, ref in (("dK", one[1], staged[1], rdk), ("dV", one[2], staged[2], rdv)):
        assert torch.equal(got, other), what
        gate(what, to64(got), ref + 1.0 if flags else ref, w.dtype)
