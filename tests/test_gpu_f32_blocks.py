"""float32 kernels in blocks of 16 rows or keys: blocks that span groups, segments around a block and a chunk, head dimensions 64 and
128, several q heads per kv head, response rows added to what the buffers hold; and rows that a block's masked keys must not
reach, whatever those hold."""
import pytest
import torch

from oracle import sp_attn_oracle as orc
from paper_2511_18871_amd import binding as B
from paper_2511_18871_amd import workloads as W
from parity import gate, gate_lse, oracle_bwd, to64

pytestmark = pytest.mark.gpu

GROUPS = [W.Group(5, [3, 0, 9]), W.Group(1, []), W.Group(17, [16, 15, 1]), W.Group(0, [33]), W.Group(70, [64, 65]), W.Group(2, [200])]


@pytest.mark.parametrize("head_dim", [64, 128])
@pytest.mark.parametrize("heads", [(16, 16), (12, 4), (8, 2)])
def test_blocks(heads, head_dim):
    w = W.Workload("blocks", GROUPS, *heads, head_dim, torch.float32, 5200)
    t = W.make_tensors(w)
    pack, sc = (w.prompt_lens(), w.Gs(), w.resp_lens_flat()), w.softmax_scale
    q, k, v, d_o = t.q.cuda(), t.k.cuda(), t.v.cuda(), t.d_o.cuda()
    o, lse = B.sp_attn_fwd_batched(q, k, v, *pack, sc)
    got = B.sp_attn_bwd_batched(q, k, v, o, lse, d_o, *pack, sc)
    torch.cuda.synchronize()
    rdq, rdk, rdv, ro, rlse = oracle_bwd(w, t)
    gate_lse(to64(lse), rlse, w.dtype)
    for name, x, ref in (("O", o, ro), ("dQ", got[0], rdq), ("dK", got[1], rdk), ("dV", got[2], rdv)):
        gate(name, to64(x), ref, w.dtype)
    resp, at = torch.ones(w.total_tokens, dtype=torch.bool), 0
    for g in w.groups:
        resp[at:at + g.prompt_len] = False
        at += g.total
    t.d_o[~resp] = 0
    rdq, rdk, rdv, _, _ = oracle_bwd(w, t)
    fl = B.SP_FLAG_RESPONSE_ROWS
    o2, lse2 = B.sp_attn_fwd_batched_ex(q, k, v, *pack, sc, fl, o=torch.full_like(q, 7.0), lse=torch.full_like(lse, 7.0))
    dq, dk, dv = B.sp_attn_bwd_batched_ex(q, k, v, o, lse, d_o, *pack, sc, fl | B.SP_FLAG_ACCUMULATE_DKDV, dq=torch.full_like(q, 7.0),
                                          dk=torch.ones_like(k), dv=torch.ones_like(v))
    torch.cuda.synchronize()
    idle = ~resp.cuda()
    assert (o2[idle] == 7).all() and (lse2[:, idle] == 7).all() and (dq[idle] == 7).all()
    assert torch.equal(o2[~idle], o[~idle]) and torch.equal(lse2[:, ~idle], lse[:, ~idle])
    gate("dQ of response rows", to64(dq)[resp], rdq[resp], w.dtype)
    gate("dK of response rows", to64(dk), rdk + 1.0, w.dtype)
    gate("dV of response rows", to64(dv), rdv + 1.0, w.dtype)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("T", [65, 97, 131])
def test_an_infinite_last_row_reaches_no_row_ahead(T, d):
    heads, gen = 16, torch.Generator().manual_seed(T)
    q, k, v, d_o = (torch.randn(T, heads, d, generator=gen) for _ in range(4))
    args = (1, [T - 1], d ** -0.5)
    clean, lse0 = B.sp_attn_fwd(q.cuda(), k.cuda(), v.cuda(), *args)
    want = B.sp_attn_bwd(q.cuda(), k.cuda(), v.cuda(), clean, lse0, d_o.cuda(), *args)
    bad_v, bad_do = v.clone(), d_o.clone()
    bad_v[T - 1] = float("inf")                          # seen by the last row alone
    bad_do[T - 1] = float("inf")                         # reaches the dv of every key
    o, _ = B.sp_attn_fwd(q.cuda(), k.cuda(), bad_v.cuda(), *args)
    dq, _, dv = B.sp_attn_bwd(q.cuda(), k.cuda(), v.cuda(), clean, lse0, bad_do.cuda(), *args)
    dq2, _, _ = B.sp_attn_bwd(q.cuda(), k.cuda(), bad_v.cuda(), clean, lse0, d_o.cuda(), *args)
    torch.cuda.synchronize()
    assert torch.all(o[T - 1] == float("inf")) and torch.all(dv == float("inf"))
    for x, ref in ((o, clean), (dq, want[0]), (dq2, want[0])):      # rows ahead: the other way of summing at most
        assert float((x[:T - 1] - ref[:T - 1]).abs().max()) <= 1e-5 * float(ref.abs().max())
