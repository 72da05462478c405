"""Softmax scales at the ends of float32: the scores are ordinary, q and k are not."""
import numpy as np
import pytest
import torch

from paper_2511_18871_amd import binding as B
from paper_2511_18871_amd import workloads as W
from parity import gate, gate_lse, oracle_bwd, to64

pytestmark = pytest.mark.gpu

GROUPS = [W.Group(70, [33, 90, 41]), W.Group(3, [130]), W.Group(200, [])]


@pytest.mark.parametrize("heads,repeats", [((4, 2), 1), ((4, 2), 20), ((8, 8), 1)])
@pytest.mark.parametrize("log2_scale", [-118, -103, -20, 100])
def test_backward_at_extreme_scales(log2_scale, heads, repeats):
    w = W.Workload("scales", GROUPS * repeats, heads[0], heads[1], 128, torch.bfloat16, 40 + heads[0])
    t = W.make_tensors(w)
    # q and k of an ordinary call, times powers of two whose product is ordinary scale / this scale (both exact in bf16)
    e = -3 - log2_scale
    fq, fk = 2.0 ** (e // 2), 2.0 ** (e - e // 2)
    pl, Gs, rl = w.prompt_lens(), w.Gs(), w.resp_lens_flat()
    q, k, v, d_o = (t.q * fq).cuda(), (t.k * fk).cuda(), t.v.cuda(), t.d_o.cuda()
    scale = 2.0 ** log2_scale
    o, lse = B.sp_attn_fwd_batched(q, k, v, pl, Gs, rl, scale)
    dq, dk, dv = B.sp_attn_bwd_batched(q, k, v, o, lse, d_o, pl, Gs, rl, scale)
    torch.cuda.synchronize()
    w.scale = 2.0 ** -3
    rdq, rdk, rdv, ro, rlse = oracle_bwd(w, t)
    gate("O", to64(o), ro, w.dtype)
    gate_lse(to64(lse), rlse, w.dtype)
    # the chain rule undoes the factors: dq carries 1 / fq, dk 1 / fk (powers of two, and no value of either is subnormal
    # but those too small to count)
    gate("dQ", to64(dq) * fq, rdq, w.dtype)
    gate("dK", to64(dk) * fk, rdk, w.dtype)
    gate("dV", to64(dv), rdv, w.dtype)
