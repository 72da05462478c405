"""The forward of response rows and the dq pass with key loops in parts: few rows under long prompts, response rows only and all rows, ragged ends of
keys, rows that see no key of a part, all ways in which kv heads fall onto the chip; the gradients of stages and of a second call bit for
bit, and what a workspace without the room gives."""
import pytest
import torch

from paper_2511_18871_amd import binding as B
from paper_2511_18871_amd import workloads as W
from parity import gate, gate_lse, oracle_bwd, to64

pytestmark = pytest.mark.gpu

PACKS = {
    "two_prompts": [W.Group(1400, [20, 5, 0, 33]), W.Group(1089, [1, 70])],
    "prompt_alone": [W.Group(1601, [])],
    "long_response": [W.Group(3, [1500]), W.Group(40, [30])],
    "no_prompt": [W.Group(0, [64, 1300, 40])],
}


def _setup(name, heads, seed, resp_only=False):
    w = W.Workload(name, PACKS[name], *heads, 128, torch.bfloat16, seed)
    t = W.make_tensors(w)
    resp, at = torch.ones(w.total_tokens, dtype=torch.bool), 0
    for g in w.groups:
        resp[at:at + g.prompt_len] = False
        at += g.total
    if resp_only:
        t.d_o[~resp] = 0
    return w, t, resp, (w.prompt_lens(), w.Gs(), w.resp_lens_flat(), w.softmax_scale)


# all rows of these fill the chip, or nearly: whole key loops
WHOLE = {(n, (28, 4)) for n in PACKS} | {("two_prompts", (8, 8)), ("two_prompts", (8, 1))}


@pytest.mark.parametrize("heads", [(4, 2), (28, 4), (8, 8), (6, 3), (8, 1)])
@pytest.mark.parametrize("name", list(PACKS))
def test_all_rows(name, heads):
    w, t, _, pk = _setup(name, heads, 790)
    assert bool(B.sp_attn_pieces(*pk[:3], *heads, 0, True)[0]) == ((name, heads) not in WHOLE)
    q, k, v, d_o = t.q.cuda(), t.k.cuda(), t.v.cuda(), t.d_o.cuda()
    o, lse = B.sp_attn_fwd_batched(q, k, v, *pk)
    nan = lambda: [torch.full_like(x, float("nan")) for x in (q, k, v)]
    one, again, staged = nan(), nan(), nan()
    B.sp_attn_bwd_batched_ex(q, k, v, o, lse, d_o, *pk, 0, *one)
    B.sp_attn_bwd_batched_ex(q, k, v, o, lse, d_o, *pk, 0, *again)
    for stage in (1, 4, 2):
        B.sp_attn_bwd_batched_ex(q, k, v, o, lse, d_o, *pk, 0, *staged, stages=stage)
    torch.cuda.synchronize()
    for x, y, z in zip(one, again, staged):
        assert torch.equal(x, y) and torch.equal(x, z)
    *grads, ro, rlse = oracle_bwd(w, t)
    gate("O", to64(o), ro, w.dtype)
    gate_lse(to64(lse), rlse, w.dtype)
    for what, got, ref in zip(("dQ", "dK", "dV"), one, grads):
        gate(what, to64(got), ref, w.dtype)


@pytest.mark.parametrize("heads", [(4, 2), (8, 8), (28, 4)])
@pytest.mark.parametrize("name", ["two_prompts", "long_response"])
def test_response_rows_only(name, heads):
    w, t, resp, pk = _setup(name, heads, 791, True)
    assert bool(B.sp_attn_pieces(*pk[:3], *heads, B.SP_FLAG_RESPONSE_ROWS, True)[0]) == ((name, heads) != ("long_response", (28, 4)))
    q, k, v, d_o = t.q.cuda(), t.k.cuda(), t.v.cuda(), t.d_o.cuda()
    fl = B.SP_FLAG_RESPONSE_ROWS
    o, lse = B.sp_attn_fwd_batched_ex(q, k, v, *pk, fl, o=torch.full_like(q, 7.0), lse=torch.full((heads[0], w.total_tokens), 7.0, device="cuda"))
    dq, dk, dv = B.sp_attn_bwd_batched_ex(q, k, v, o, lse, d_o, *pk, fl, dq=torch.full_like(q, 7.0))
    torch.cuda.synchronize()
    rdq, rdk, rdv, ro, rlse = oracle_bwd(w, t)
    idle = ~resp.cuda()
    assert (o[idle] == 7).all() and (lse[:, idle] == 7).all() and (dq[idle] == 7).all()
    gate("O", to64(o)[resp], ro[resp], w.dtype)
    gate_lse(to64(lse)[:, resp], rlse[:, resp], w.dtype)
    gate("dQ", to64(dq)[resp], rdq[resp], w.dtype)
    gate("dK", to64(dk), rdk, w.dtype)
    gate("dV", to64(dv), rdv, w.dtype)


def test_the_last_round_in_parts():
    """More workgroups than places: those of full rounds stay whole, the last round's are cut; a table in memory.  Against float64, one kv
    head and its q heads."""
    Lp, lens, heads, kvh, rep, d, fl = 8192, W.ragged_lengths(5100, 16, 64, 256), (40, 8), 3, 5, 128, B.SP_FLAG_RESPONSE_ROWS
    T, pk = Lp + sum(lens), ([Lp], [16], lens)
    words, sums, first_slot, n_slots = B.sp_attn_pieces(*pk, *heads, fl, True)
    assert first_slot == 64 and n_slots > 0 and -(-T // 128) * heads[0] > 2048       # (a small call has its table in the arguments)
    gen = torch.Generator(device="cuda").manual_seed(795)
    q, d_o = (torch.randn(T, heads[0], d, generator=gen, device="cuda").to(torch.bfloat16) for _ in range(2))
    k, v = (torch.randn(T, heads[1], d, generator=gen, device="cuda").to(torch.bfloat16) for _ in range(2))
    o, lse = B.sp_attn_fwd_batched_ex(q, k, v, *pk, d ** -0.5, fl, o=torch.full_like(q, 7.0), lse=torch.full((heads[0], T), 7.0, device="cuda"))
    dq, dk, dv = B.sp_attn_bwd_batched_ex(q, k, v, o, lse, d_o, *pk, d ** -0.5, fl, dq=torch.full_like(q, 7.0))
    torch.cuda.synchronize()
    assert (o[:Lp] == 7).all() and (lse[:, :Lp] == 7).all() and (dq[:Lp] == 7).all()
    starts = torch.repeat_interleave(Lp + torch.tensor([0, *lens[:-1]]).cumsum(0), torch.tensor(lens)).cuda()
    key, row = torch.arange(T, device="cuda"), torch.arange(Lp, T, device="cuda")
    hidden = (key[None] > row[:, None]) | ((key[None] >= Lp) & (key[None] < starts[:, None]))
    K, V = (x[:, kvh].double().contiguous() for x in (k, v))
    rdk, rdv = torch.zeros_like(K), torch.zeros_like(V)
    for h in range(kvh * rep, (kvh + 1) * rep):
        Q, G = q[Lp:, h].double().contiguous(), d_o[Lp:, h].double().contiguous()
        S = (Q @ K.t().contiguous() * d ** -0.5).masked_fill_(hidden, float("-inf"))
        rlse = torch.logsumexp(S, 1)
        P = torch.exp(S - rlse[:, None])
        ro = P @ V
        dS = P * (G @ V.t().contiguous() - (G * ro).sum(1, keepdim=True))
        gate(f"O head {h}", to64(o[Lp:, h]), to64(ro), q.dtype)
        gate_lse(to64(lse[h:h + 1, Lp:]), to64(rlse[None]), q.dtype)
        gate(f"dQ head {h}", to64(dq[Lp:, h]), to64(dS @ K * d ** -0.5), q.dtype)
        rdk += dS.t().contiguous() @ Q * d ** -0.5
        rdv += P.t().contiguous() @ G
    gate("dK", to64(dk[:, kvh]), to64(rdk), q.dtype)
    gate("dV", to64(dv[:, kvh]), to64(rdv), q.dtype)


@pytest.mark.parametrize("name", ["two_prompts", "long_response", "no_prompt"])
def test_sums_stay_in_their_room(name):
    heads = (4, 2)
    w, t, resp, pk = _setup(name, heads, 792)
    q, k, v, fl = t.q.cuda(), t.k.cuda(), t.v.cuda(), B.SP_FLAG_RESPONSE_ROWS
    n, r, T = len(w.groups), len(pk[2]), w.total_tokens
    behind = (B.workspace_bytes(True, T, n, r, *heads, 128, B.SP_BF16) + B.reserve_bytes(T, heads[0], 128, B.SP_BF16)
              + B.row_parts_bytes(T, n, *heads, B.SP_BF16))
    full = B.full_workspace_bytes(T, n, r, *heads, 128, B.SP_BF16)
    ws = torch.full((full + 4096,), 255, dtype=torch.uint8, device="cuda")
    o, lse = B.sp_attn_fwd_batched_ex(q, k, v, *pk, fl, workspace=ws[:full])
    torch.cuda.synchronize()
    assert (ws[behind:full] != 255).any() and (ws[full:] == 255).all()
    ws[:] = 255
    whole, wlse = B.sp_attn_fwd_batched_ex(q, k, v, *pk, fl, workspace=ws[:full - 1])
    torch.cuda.synchronize()
    assert (ws[behind:] == 255).all()
    o, whole, lse, wlse = o[resp], whole[resp], lse[:, resp], wlse[:, resp]
    assert float((o.float() - whole.float()).norm() / whole.float().norm()) < 4e-3      # weights rounded to bf16 against other references
    assert float((lse - wlse).abs().max()) < 2e-5


@pytest.mark.parametrize("heads", [(4, 2), (8, 1)])
@pytest.mark.parametrize("name", list(PACKS))
def test_rows_of_a_full_forward_do_not_depend_on_the_call(name, heads):
    """Several sets in one call, a call of one set on any workspace and one with a residual of its own: the same bits.  (The policy's
    log-probabilities come from one of them, those of the old policy from another, and their ratio is one.)"""
    w, t, _, pk = _setup(name, heads, 794)
    q, k, v = t.q.cuda(), t.k.cuda(), t.v.cuda()
    n, r, T = len(w.groups), len(pk[2]), w.total_tokens
    os, lses = B.sp_attn_fwd_multi([q, q], [k, k], [v, v], *pk)
    one = B.sp_attn_fwd_batched(q, k, v, *pk)
    least = torch.empty(B.workspace_bytes(False, T, n, r, *heads, 128, B.SP_BF16), dtype=torch.uint8, device="cuda")
    small = B.sp_attn_fwd_batched(q, k, v, *pk, workspace=least)
    lo = B.sp_attn_fwd_batched_ex(q, k, v, *pk, 0, o_lo=torch.empty_like(q))
    torch.cuda.synchronize()
    for o, lse in (one, small, lo):
        assert torch.equal(o, os[1]) and torch.equal(lse, lses[1])


@pytest.mark.parametrize("log2_scale", [-118, 100])
@pytest.mark.parametrize("name", ["two_prompts", "no_prompt"])
def test_extreme_scales(name, log2_scale):
    """Rows that see no key of a part start from a reference point that stays finite, times the scale too (as test_gpu_scales.py)."""
    w, t, resp, pk = _setup(name, (4, 2), 793)
    e = -3 - log2_scale
    fq, fk = 2.0 ** (e // 2), 2.0 ** (e - e // 2)
    q, k, v, d_o = (t.q * fq).cuda(), (t.k * fk).cuda(), t.v.cuda(), t.d_o.cuda()
    o, lse = B.sp_attn_fwd_batched(q, k, v, *pk[:3], 2.0 ** log2_scale)
    parts, plse = B.sp_attn_fwd_batched_ex(q, k, v, *pk[:3], 2.0 ** log2_scale, B.SP_FLAG_RESPONSE_ROWS)
    dq, dk, dv = B.sp_attn_bwd_batched(q, k, v, o, lse, d_o, *pk[:3], 2.0 ** log2_scale)
    torch.cuda.synchronize()
    w.scale = 2.0 ** -3
    rdq, rdk, rdv, ro, rlse = oracle_bwd(w, t)
    gate("O", to64(o), ro, w.dtype)
    gate_lse(to64(lse), rlse, w.dtype)
    gate("O of response rows", to64(parts)[resp], ro[resp], w.dtype)
    gate_lse(to64(plse)[:, resp], rlse[:, resp], w.dtype)
    gate("dQ", to64(dq) * fq, rdq, w.dtype)
    gate("dK", to64(dk) * fk, rdk, w.dtype)
    gate("dV", to64(dv), rdv, w.dtype)
