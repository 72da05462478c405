"""All shapes of the float32 kernels (eight waves per row or key, one wave, blocks of 16), head dimensions 64 and 128, several q heads per kv
head: segments around the chunks of 32 and 64 keys, sizes on both sides of the rules; the rowsum within the dq kernel against
its own stage; response rows, added to what the buffers hold."""
import pytest
import torch

from paper_2511_18871_amd import binding as B
from paper_2511_18871_amd import workloads as W
from parity import gate, gate_lse, oracle_bwd, to64

pytestmark = pytest.mark.gpu

EDGES = [W.Group(1, []), W.Group(0, [33, 1]), W.Group(31, [32, 0, 64]), W.Group(65, [31, 63])]
MORE = EDGES + [W.Group(300, [70, 129, 64, 5])]


SHORT = [W.Group(n, [1, n % 3]) for n in range(40)]        # up to 16 groups to a block of 16


# rows (keys) per workgroup of the forward, the dq pass and the dkdv pass: 1 eight waves, 4 a wave each, 16 a block
@pytest.mark.parametrize("groups,heads,head_dim,rows", [
    (EDGES[:3], (2, 2), 64, (1, 1, 1)), (EDGES, (2, 1), 128, (1, 1, 1)), (MORE, (4, 4), 64, (16, 16, 16)), (MORE, (6, 6), 64, (16, 16, 16)),
    (MORE, (12, 3), 64, (16, 16, 16)), (MORE, (2, 2), 128, (16, 16, 16)), (MORE, (4, 1), 128, (16, 16, 1)),
    (SHORT[:16], (12, 6), 64, (4, 4, 1)), (SHORT[:20], (16, 16), 64, (4, 4, 4)), (SHORT[:16], (12, 12), 128, (4, 4, 4)), (SHORT, (12, 3), 128, (4, 16, 16))])
def test_shapes(groups, heads, head_dim, rows):
    w = W.Workload("f32", groups, heads[0], heads[1], head_dim, torch.float32, 5100 + heads[0])
    t = W.make_tensors(w)
    pack, sc = (w.prompt_lens(), w.Gs(), w.resp_lens_flat()), w.softmax_scale
    assert B.sp_attn_f32_rows(*pack, *heads, head_dim) == rows
    q, k, v, d_o = t.q.cuda(), t.k.cuda(), t.v.cuda(), t.d_o.cuda()
    o, lse = B.sp_attn_fwd_batched(q, k, v, *pack, sc)
    one = B.sp_attn_bwd_batched(q, k, v, o, lse, d_o, *pack, sc)
    staged = [torch.full_like(x, float("nan")) for x in (q, k, v)]
    ws = torch.empty(B.workspace_bytes(True, q.shape[0], len(pack[0]), len(pack[2]), *heads, head_dim, B.SP_F32), dtype=torch.uint8, device="cuda")
    for stage in (1, 4, 2):
        B.sp_attn_bwd_batched_stages(q, k, v, o, lse, d_o, *pack, sc, stage, ws, *staged)
    torch.cuda.synchronize()
    for name, a, b in zip(("dQ", "dK", "dV"), one, staged):
        assert torch.equal(a, b), name
    rdq, rdk, rdv, ro, rlse = oracle_bwd(w, t)
    gate_lse(to64(lse), rlse, w.dtype)
    for name, got, ref in (("O", o, ro), ("dQ", one[0], rdq), ("dK", one[1], rdk), ("dV", one[2], rdv)):
        gate(name, to64(got), ref, w.dtype)
    at = 0
    for g in w.groups:                                     # response rows alone: no upstream gradient on the prompt rows
        t.d_o[at:at + g.prompt_len] = 0
        at += g.total
    _, rdk, rdv, _, _ = oracle_bwd(w, t)
    dk, dv = torch.ones_like(k), torch.ones_like(v)
    B.sp_attn_bwd_batched_ex(q, k, v, o, lse, d_o, *pack, sc, B.SP_FLAG_RESPONSE_ROWS | B.SP_FLAG_ACCUMULATE_DKDV,
                             dq=torch.zeros_like(q), dk=dk, dv=dv)
    torch.cuda.synchronize()
    gate("dK of response rows", to64(dk), rdk + 1.0, w.dtype)
    gate("dV of response rows", to64(dv), rdv + 1.0, w.dtype)
