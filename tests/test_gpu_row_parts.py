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
    # (room for partial sums of pieces, which take this pass's place where they are used, is left out)
    ws = torch.empty(B.kept_workspace_bytes(w.total_tokens, len(w.groups), len(pack[2]), 4, 2, 128, B.SP_BF16), dtype=torch.uint8, device="cuda")
    o, lse = B.sp_attn_fwd_batched(q, k, v, *pack, sc, workspace=ws)
    start = lambda: [torch.zeros_like(q), *(torch.ones_like(k) if flags else torch.full_like(k, float("nan")) for _ in range(2))]
    one, staged = start(), start()
    B.sp_attn_bwd_batched_ex(q, k, v, o, lse, d_o, *pack, sc, flags, *one, workspace=ws)
    for stage in (1, 4, 2):
        B.sp_attn_bwd_batched_ex(q, k, v, o, lse, d_o, *pack, sc, flags, *staged, stages=stage, workspace=ws)
    torch.cuda.synchronize()
    _, rdk, rdv, _, _ = oracle_bwd(w, t)
    for what, got, other, ref in (("dK", one[1], staged[1], rdk), ("dV", one[2], staged[2], rdv)):
        assert torch.equal(got, other), what
        gate(what, to64(got), ref + 1.0 if flags else ref, w.dtype)


# longest tiles of eight steps: up to 72 workgroups two row parts, beyond one
BY_WORKGROUPS = {"56_workgroups": [W.Group(60, [440])] * 3, "76_workgroups": [W.Group(60, [440])] * 4}


@pytest.mark.parametrize("mode", ["all_rows", "response_rows"])
@pytest.mark.parametrize("name", [*PACKS, *BY_WORKGROUPS])
def test_which_key_tiles_have_two_row_parts(name, mode):
    """The second set of partial sums, at the workspace's end, is written for tiles of eight and more steps, and for no others."""
    w = W.Workload(name, {**PACKS, **BY_WORKGROUPS}[name], 4, 2, 128, torch.bfloat16, 771)
    t, T = W.make_tensors(w), w.total_tokens
    pack, sc = (w.prompt_lens(), w.Gs(), w.resp_lens_flat()), w.softmax_scale
    q, k, v, d_o = t.q.cuda(), t.k.cuda(), t.v.cuda(), t.d_o.cuda()
    want, at = torch.zeros(T, dtype=torch.bool), 0
    for g in w.groups:
        ends = [g.prompt_len + sum(g.resp_lens[:i + 1]) for i in range(len(g.resp_lens))]
        for s0 in range(0, g.total, 128):
            s1 = min(s0 + 128, g.total)
            row_end = g.total if s0 < g.prompt_len else min(e for e in ends if e >= s1)
            row_lo = max(s0, g.prompt_len) if mode == "response_rows" else s0
            want[at + s0:at + s1] = -(-row_end // 64) - row_lo // 64 >= 8
        at += g.total
    none = {"seven_steps"} if mode == "all_rows" else {"seven_steps", "eight_steps", "nine_steps_mid_tile", "one_long_one_short"}
    assert want.any() == (name not in none)
    if name == "76_workgroups":
        want[:] = False
    o_lo = torch.empty_like(q)
    o, lse = B.sp_attn_fwd_batched_ex(q, k, v, *pack, sc, 0, o_lo=o_lo)
    behind = B.workspace_bytes(True, T, len(w.groups), len(pack[2]), 4, 2, 128, B.SP_BF16) + B.reserve_bytes(T, 4, 128, B.SP_BF16)
    ws = torch.full((behind + B.row_parts_bytes(T, len(w.groups), 4, 2, B.SP_BF16),), 255, dtype=torch.uint8, device="cuda")
    B.sp_attn_bwd_batched_ex(q, k, v, o, lse, d_o, *pack, sc, B.SP_FLAG_RESPONSE_ROWS if mode == "response_rows" else 0, o_lo=o_lo, workspace=ws)
    torch.cuda.synchronize()
    written = (ws[behind:].view(torch.int32) != -1).view(2, 2, T, 2 * 128)
    assert torch.equal(written.all(3).all(1).all(0).cpu(), want) and torch.equal(written.any(3).any(1).any(0).cpu(), want)
