"""The order in which the dkdv pass takes its key tiles: prompt tiles first, by rows or group by group, in one preparation
launch and in the separate kernels, within one and across several blocks of the schedule.  A place that is given twice or
never leaves a tile of dk / dv unwritten (the outputs start as NaN)."""
import pytest
import torch

from paper_2511_18871_amd import binding as B
from paper_2511_18871_amd import workloads as W
from parity import gate, oracle_bwd, to64
from test_gpu_dkdv_shapes import EDGES

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("repeats,heads,order", [
    (6, (4, 4), "by rows, one launch"),
    (6, (32, 32), "by group, one launch"),
    (20, (4, 4), "by rows, two blocks of tiles"),
    (20, (8, 8), "by group, two blocks of tiles"),
    (26, (4, 4), "by group: more than 256 groups"),
    (6, (28, 4), "by rows, with per-head partial sums where they apply"),
])
def test_every_key_tile_is_taken_once(repeats, heads, order):
    w = W.Workload("order", EDGES * repeats, heads[0], heads[1], 128, torch.bfloat16, 920 + repeats)
    t = W.make_tensors(w)
    pl, Gs, rl, sc = w.prompt_lens(), w.Gs(), w.resp_lens_flat(), w.softmax_scale
    q, k, v, d_o = t.q.cuda(), t.k.cuda(), t.v.cuda(), t.d_o.cuda()
    o, lse = B.sp_attn_fwd_batched(q, k, v, pl, Gs, rl, sc)
    _, dk, dv = B.sp_attn_bwd_batched(q, k, v, o, lse, d_o, pl, Gs, rl, sc, dk=torch.full_like(k, float("nan")),
                                      dv=torch.full_like(v, float("nan")))
    torch.cuda.synchronize()
    _, rdk, rdv, _, _ = oracle_bwd(w, t)
    gate(f"dK ({order})", to64(dk), rdk, w.dtype)
    gate(f"dV ({order})", to64(dv), rdv, w.dtype)
