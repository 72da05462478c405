"""The dkdv pass in pieces of key tiles: few groups, whose prompt tiles every row sees, with short prompts (swept twice), none, and
several tiles of prompt; all ways in which kv heads fall onto the chip; response rows only, added to what the buffers hold; and the same
bits from one call, from stages, and again."""
import pytest
import torch

from paper_2511_18871_amd import binding as B
from paper_2511_18871_amd import workloads as W
from parity import gate, oracle_bwd, to64

pytestmark = pytest.mark.gpu

PACKS = {
    "short_prompts": [W.Group(60, [70] * 12), W.Group(17, [90, 31, 0, 200, 64])],
    "one_tile_prompt": [W.Group(128, [129, 300, 1, 250, 64, 65])],
    "three_tile_prompt": [W.Group(300, [256] * 4), W.Group(5, [3])],
    "long_response": [W.Group(70, [900]), W.Group(0, [130, 40])],
    "prompt_alone": [W.Group(1500, []), W.Group(65, [40])],
}


@pytest.mark.parametrize("heads", [(4, 2), (28, 4), (16, 8), (6, 3), (8, 1), (16, 16)])
@pytest.mark.parametrize("name", list(PACKS))
def test_pieces(name, heads):
    w = W.Workload(name, PACKS[name], *heads, 128, torch.bfloat16, 780)
    t = W.make_tensors(w)
    pack, sc = (w.prompt_lens(), w.Gs(), w.resp_lens_flat()), w.softmax_scale
    assert B.sp_attn_pieces(*pack, *heads)[0]
    q, k, v, d_o = t.q.cuda(), t.k.cuda(), t.v.cuda(), t.d_o.cuda()
    o, lse = B.sp_attn_fwd_batched(q, k, v, *pack, sc)
    nan = lambda: [torch.full_like(x, float("nan")) for x in (q, k, v)]
    one, again, staged = nan(), nan(), nan()
    B.sp_attn_bwd_batched_ex(q, k, v, o, lse, d_o, *pack, sc, 0, *one)
    B.sp_attn_bwd_batched_ex(q, k, v, o, lse, d_o, *pack, sc, 0, *again)
    for stage in (1, 4, 2):
        B.sp_attn_bwd_batched_ex(q, k, v, o, lse, d_o, *pack, sc, 0, *staged, stages=stage)
    torch.cuda.synchronize()
    for x, y, z in zip(one, again, staged):
        assert torch.equal(x, y) and torch.equal(x, z)
    for what, got, ref in zip(("dQ", "dK", "dV"), one, oracle_bwd(w, t)):
        gate(what, to64(got), ref, w.dtype)


@pytest.mark.parametrize("groups,prompt,responses,length,words,pieces", [
    (27, 28, 19, 41, 760, 216), (27, 58, 17, 14, 706, 108),      # the list takes the arguments' place of the table
    (19, 23, 24, 7, 631, 114),                                   # beside the table
    (24, 23, 21, 7, 724, 0)])                                    # pieces do not pay for the launch that a table in memory takes
def test_parts_do_not_depend_on_the_table(groups, prompt, responses, length, words, pieces):
    """Tables of 631 to 760 words, beside most of which a kernel's arguments (768) have no room for the list of pieces."""
    w = W.Workload("tables", [W.Group(prompt, [length] * responses)] * groups, 4, 2, 128, torch.bfloat16, 783)
    pack = (w.prompt_lens(), w.Gs(), w.resp_lens_flat())
    assert (len(B.sp_attn_segment_table(*pack)), len(B.sp_attn_pieces(*pack, 4, 2)[0])) == (words, pieces)
    t = W.make_tensors(w)
    pack, sc = (w.prompt_lens(), w.Gs(), w.resp_lens_flat()), w.softmax_scale
    q, k, v, d_o = t.q.cuda(), t.k.cuda(), t.v.cuda(), t.d_o.cuda()
    o, lse = B.sp_attn_fwd_batched(q, k, v, *pack, sc)
    one = B.sp_attn_bwd_batched(q, k, v, o, lse, d_o, *pack, sc)
    staged = [torch.full_like(x, float("nan")) for x in (q, k, v)]
    for stage in (1, 4, 2):
        B.sp_attn_bwd_batched_ex(q, k, v, o, lse, d_o, *pack, sc, 0, *staged, stages=stage)
    torch.cuda.synchronize()
    for what, x, y, ref in zip(("dQ", "dK", "dV"), one, staged, oracle_bwd(w, t)):
        assert torch.equal(x, y)
        gate(what, to64(x), ref, w.dtype)


@pytest.mark.parametrize("name", list(PACKS))
def test_pieces_of_response_rows_accumulate(name):
    w = W.Workload(name, PACKS[name], 8, 2, 128, torch.bfloat16, 781)
    t = W.make_tensors(w)
    at = 0
    for g in w.groups:
        t.d_o[at:at + g.prompt_len] = 0
        at += g.total
    pack, sc = (w.prompt_lens(), w.Gs(), w.resp_lens_flat()), w.softmax_scale
    assert bool(B.sp_attn_pieces(*pack, 8, 2, B.SP_FLAG_RESPONSE_ROWS)[0]) == (name != "prompt_alone")
    q, k, v, d_o = t.q.cuda(), t.k.cuda(), t.v.cuda(), t.d_o.cuda()
    o, lse = B.sp_attn_fwd_batched(q, k, v, *pack, sc)
    _, dk, dv = B.sp_attn_bwd_batched_ex(q, k, v, o, lse, d_o, *pack, sc, B.SP_FLAG_RESPONSE_ROWS | B.SP_FLAG_ACCUMULATE_DKDV,
                                         dq=torch.zeros_like(q), dk=torch.ones_like(k), dv=torch.ones_like(v))
    torch.cuda.synchronize()
    _, rdk, rdv, _, _ = oracle_bwd(w, t)
    gate("dK", to64(dk), rdk + 1.0, w.dtype)
    gate("dV", to64(dv), rdv + 1.0, w.dtype)


@pytest.mark.parametrize("heads", [(4, 2), (28, 4)])
def test_sums_stay_in_their_room(heads):
    """Pieces are used (their sums are written), nothing lies behind the workspace, and without the room whole tiles give the same gradients."""
    w = W.Workload("room", PACKS["short_prompts"], *heads, 128, torch.bfloat16, 782)
    t, T = W.make_tensors(w), w.total_tokens
    pack, sc = (w.prompt_lens(), w.Gs(), w.resp_lens_flat()), w.softmax_scale
    q, k, v, d_o = t.q.cuda(), t.k.cuda(), t.v.cuda(), t.d_o.cuda()
    n, r = len(w.groups), len(pack[2])
    behind = (B.workspace_bytes(True, T, n, r, *heads, 128, B.SP_BF16) + B.reserve_bytes(T, heads[0], 128, B.SP_BF16)
              + B.row_parts_bytes(T, n, *heads, B.SP_BF16))
    full = B.full_workspace_bytes(T, n, r, *heads, 128, B.SP_BF16)
    ws = torch.full((full + 4096,), 255, dtype=torch.uint8, device="cuda")
    o, lse = B.sp_attn_fwd_batched(q, k, v, *pack, sc, workspace=ws[:full])
    got = B.sp_attn_bwd_batched(q, k, v, o, lse, d_o, *pack, sc, workspace=ws[:full])
    torch.cuda.synchronize()
    assert (ws[behind:full] != 255).any() and (ws[full:] == 255).all()
    ws[:] = 255
    o, lse = B.sp_attn_fwd_batched(q, k, v, *pack, sc, workspace=ws[:full - 1])
    whole = B.sp_attn_bwd_batched(q, k, v, o, lse, d_o, *pack, sc, workspace=ws[:full - 1])
    torch.cuda.synchronize()
    assert (ws[behind:] == 255).all()
    for x, y in zip(got, whole):
        # one bf16 rounding of sums in another order
        assert float((x.float() - y.float()).norm() / y.float().norm()) < 1e-3
