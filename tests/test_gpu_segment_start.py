"""Key tiles of the forward and the dq pass: a response row's own keys are walked from its segment's first key on, or from the
end of the prompt's last tile where that holds it.  Segments that start at, one past and one ahead of multiples of 32 and 64,
prompts that end there, no prompt at all, both workgroup shapes."""
import pytest
import torch

from paper_2511_18871_amd import binding as B
from paper_2511_18871_amd import workloads as W
from parity import gate, gate_lse, oracle_bwd, to64

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [0, 1 << 20])           # eight waves, four
@pytest.mark.parametrize("prompt", [0, 1, 31, 63, 64, 65, 127, 129, 200])
def test_segments_around_tile_edges(prompt, shape):
    resp = [64 - prompt % 64, 1, 63, 64, 65, 130, 2, 31, 97]
    w = W.Workload("starts", [W.Group(prompt, resp), W.Group(prompt + 7, resp[::-1])], 6, 2, 128, torch.bfloat16, 300 + prompt)
    t = W.make_tensors(w)
    pl, Gs, rl, sc = w.prompt_lens(), w.Gs(), w.resp_lens_flat(), w.softmax_scale
    q, k, v, d_o = t.q.cuda(), t.k.cuda(), t.v.cuda(), t.d_o.cuda()
    B.set_small_shape_steps(shape)
    try:
        o, lse = B.sp_attn_fwd_batched(q, k, v, pl, Gs, rl, sc)
        dq, dk, dv = B.sp_attn_bwd_batched(q, k, v, o, lse, d_o, pl, Gs, rl, sc)
        torch.cuda.synchronize()
    finally:
        B.set_small_shape_steps(-1)
    rdq, rdk, rdv, ro, rlse = oracle_bwd(w, t)
    gate_lse(to64(lse), rlse, w.dtype)
    for name, got, ref in (("O", o, ro), ("dQ", dq, rdq), ("dK", dk, rdk), ("dV", dv, rdv)):
        gate(name, to64(got), ref, w.dtype)
