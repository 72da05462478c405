"""Calls whose attention kernels look their tiles and segments up themselves, and the ones just beyond (prepared by a launch):
64 groups, 63 responses, and one more of each; tables at the argument limit; groups of one token, without responses, with
empty ones; forward (both shapes), backward with and without per-head partial sums, four dkdv waves, several tensor sets."""
import numpy as np
import pytest
import torch

from paper_2511_18871_amd import binding as B
from paper_2511_18871_amd import workloads as W
from parity import gate, gate_lse, oracle_bwd, to64

pytestmark = pytest.mark.gpu


def lengths(seed, n, hi):
    return [int(x) for x in np.random.default_rng(seed).integers(0, hi, n)]


PACKS = {
    "one_token": ([W.Group(1, [])], (4, 2)),
    "no_responses": ([W.Group(130, [])], (4, 2)),
    "only_empty_responses": ([W.Group(5, [0, 0, 0]), W.Group(0, [0, 3, 0])], (4, 2)),
    "63_responses": ([W.Group(70, lengths(1, 63, 9)), W.Group(3, [40, 0, 90])], (6, 2)),
    "64_responses": ([W.Group(70, lengths(2, 64, 9)), W.Group(3, [40, 0, 90])], (6, 2)),
    "64_groups": ([W.Group(1 + n, [n]) for n in lengths(3, 64, 30)], (4, 2)),
    "65_groups": ([W.Group(1 + n, [n]) for n in lengths(4, 65, 30)], (4, 2)),
    "768_words": ([W.Group(2, lengths(5, 23, 7)) for _ in range(23)] + [W.Group(9, lengths(6, 19, 7))], (2, 1)),
    "769_words": ([W.Group(2, lengths(5, 23, 7)) for _ in range(23)] + [W.Group(9, lengths(6, 20, 7))], (2, 1)),
}


@pytest.mark.parametrize("shape", [0, 1 << 20])           # eight waves, four
@pytest.mark.parametrize("name", list(PACKS))
def test_lookups(name, shape):
    groups, heads = PACKS[name]
    w = W.Workload(name, groups, heads[0], heads[1], 128, torch.bfloat16, 7300 + len(name))
    t = W.make_tensors(w)
    pl, Gs, rl, sc = w.prompt_lens(), w.Gs(), w.resp_lens_flat(), w.softmax_scale
    if name.endswith("_words"):
        assert len(B.sp_attn_segment_table(pl, Gs, rl)) == int(name[:3])
    q, k, v, d_o = t.q.cuda(), t.k.cuda(), t.v.cuda(), t.d_o.cuda()
    B.set_small_shape_steps(shape)
    try:
        o, lse = B.sp_attn_fwd_batched(q, k, v, pl, Gs, rl, sc)
        os, lses = B.sp_attn_fwd_multi([q, q], [k, k], [v, v], pl, Gs, rl, sc)      # prepared by a launch
        dq, dk, dv = B.sp_attn_bwd_batched(q, k, v, o, lse, d_o, pl, Gs, rl, sc)
        torch.cuda.synchronize()
    finally:
        B.set_small_shape_steps(-1)
    assert torch.equal(o, os[1]) and torch.equal(lse, lses[1])
    rdq, rdk, rdv, ro, rlse = oracle_bwd(w, t)
    gate_lse(to64(lse), rlse, w.dtype)
    for what, got, ref in (("O", o, ro), ("dQ", dq, rdq), ("dK", dk, rdk), ("dV", dv, rdv)):
        gate(what, to64(got), ref, w.dtype)


def test_four_dkdv_waves_against_the_prepared_stages():
    # a backward in stages is prepared by a launch and runs the same kernels on the same numbers
    w = W.Workload("four_waves", [W.Group(1450, [725, 725])], 32, 32, 128, torch.bfloat16, 7400)
    t = W.make_tensors(w)
    pack, sc = (w.prompt_lens(), w.Gs(), w.resp_lens_flat()), w.softmax_scale
    assert B.sp_attn_dkdv_waves(*pack, 32, 32) == 4
    q, k, v, d_o = t.q.cuda(), t.k.cuda(), t.v.cuda(), t.d_o.cuda()
    o, lse = B.sp_attn_fwd_batched(q, k, v, *pack, sc)
    one = B.sp_attn_bwd_batched(q, k, v, o, lse, d_o, *pack, sc)
    staged = [torch.full_like(x, float("nan")) for x in (q, k, v)]
    for stage in (1, 4, 2):
        B.sp_attn_bwd_batched_stages(q, k, v, o, lse, d_o, *pack, sc, stage, o._sp_workspace, *staged)
    torch.cuda.synchronize()
    for name, a, b in zip(("dQ", "dK", "dV"), one, staged):
        assert torch.equal(a, b), name
